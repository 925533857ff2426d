// bf_batch_impl.h -- the persistent batch kernels and their launches,
// instantiated per operand type in bf_batch_f16.hip and bf_batch_bf16.hip.
#pragma once
#include "bf_common.h"
#include "bf_workers.h"

namespace lbf {

struct BatchArgs {
    BlockDesc blk[kMaxBatch];
    int item_start[kMaxBatch + 1];   // prefix sums of items per block
    ItemGrid grid[kMaxBatch];
    int n;
};
static_assert(sizeof(BatchArgs) <= 4096, "kernel argument block");

// one persistent launch of batch variant v (batch_variant) over the entries of
// a; *counter is zero when it starts
hipError_t launch_batch_f16(int v, const BatchArgs& a, int* counter, hipStream_t st);
hipError_t launch_batch_bf16(int v, const BatchArgs& a, int* counter, hipStream_t st);

template <int XT, int CT, int PR, int NK, int NS>
__global__ __launch_bounds__(kThreadsH) void bf_batch_kernel(BatchArgs a, int* counter) {
    __shared__ __attribute__((aligned(16))) uint32_t at[h_lds_words(NK, NS)];
    __shared__ int next;
    const int total = a.item_start[a.n];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) next = atomicAdd(counter, 1);
        __syncthreads();
        const int it = next;
        if (it >= total) break;     // every work group leaves once the list is exhausted
        int j = 0;
        while (j + 1 < a.n && a.item_start[j + 1] <= it) ++j;
        item_h_fast<XT, CT, PR, 16, NK, NS>(a.blk[j], it - a.item_start[j], a.grid[j], at);
    }
}

// One persistent launch of variant <XT, CT, PR, NK, NS>: one resident work
// group per slot the hardware offers; the queue, not the grid, spreads the
// uneven items.
template <int XT, int CT, int PR, int NK, int NS>
hipError_t launch_batch_k(const BatchArgs& a, int* counter, hipStream_t st) {
    int dev = 0, cus = 256, per_cu = 1;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, bf_batch_kernel<XT, CT, PR, NK, NS>, kThreadsH, 0);
    if (per_cu < 1) per_cu = 1;
    const int total = a.item_start[a.n];
    const int slots = cus * per_cu;
    hipLaunchKernelGGL((bf_batch_kernel<XT, CT, PR, NK, NS>), dim3(total < slots ? total : slots), dim3(kThreadsH), 0,
                       st, a, counter);
    return hipGetLastError();
}

template <int XT, int CT, int PR, int NK>
hipError_t launch_batch_nk(int v, const BatchArgs& a, int* counter, hipStream_t st) {
    switch (v % 3) {
        case 0: return launch_batch_k<XT, CT, PR, NK, 1>(a, counter, st);
        case 1: return launch_batch_k<XT, CT, PR, NK, 2>(a, counter, st);
        default: return launch_batch_k<XT, CT, PR, NK, 4>(a, counter, st);
    }
}

template <int XT, int CT, int PR>
hipError_t launch_batch_pr(int v, const BatchArgs& a, int* counter, hipStream_t st) {
    switch (v % 15 / 3) {
        case 0: return launch_batch_nk<XT, CT, PR, 4>(v, a, counter, st);
        case 1: return launch_batch_nk<XT, CT, PR, 5>(v, a, counter, st);
        case 2: return launch_batch_nk<XT, CT, PR, 6>(v, a, counter, st);
        case 3: return launch_batch_nk<XT, CT, PR, 7>(v, a, counter, st);
        default: return launch_batch_nk<XT, CT, PR, 8>(v, a, counter, st);
    }
}

template <int CT>
hipError_t launch_batch_variant(int v, const BatchArgs& a, int* counter, hipStream_t st) {
    switch (v / 15) {
        case 0: return launch_batch_pr<XT_CI8, CT, PR_I>(v, a, counter, st);
        case 1: return launch_batch_pr<XT_CI8, CT, PR_IQUV>(v, a, counter, st);
        case 2: return launch_batch_pr<XT_CI16, CT, PR_I>(v, a, counter, st);
        default: return launch_batch_pr<XT_CI16, CT, PR_IQUV>(v, a, counter, st);
    }
}

}  // namespace lbf
