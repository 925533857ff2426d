// bf_fast_impl.h -- kernels and launchers of the fast contraction workers,
// instantiated per operand and sample type in bf_fast_*.hip.
#pragma once
#include "bf_common.h"
#include "bf_workers.h"

namespace lbf {

// 8 waves, two per SIMD; LDS: the three weight planes of 128 beams
template <int PR, int TI, bool FINAL>
__global__ __launch_bounds__(kThreadsH) void bf_f32_fast_kernel(BlockDesc d, ItemGrid grid, int nitems) {
    __shared__ __attribute__((aligned(16))) float pl[3 * kPlaneWords];
    item_f32_fast<PR, TI, FINAL>(d, xcd_remap(blockIdx.x, nitems), grid, pl);
}

// 8 waves, two per SIMD; LDS: NS streams x 2 buffers of one A tile (and the
// incoherent beam's partial sums in the INC form)
template <int XT, int CT, int PR, int TI, int NK, int NS, bool INC>
__global__ __launch_bounds__(kThreadsH) void bf_h_fast_kernel(BlockDesc d, ItemGrid grid, int nitems) {
    __shared__ __attribute__((aligned(16))) uint32_t at[h_lds_words(NK, NS) + (INC ? kIncLdsFloats : 0) +
                                                       (PR == PR_VOLT && NS <= 2 ? 8 * kVoltWords : 0)];
    item_h_fast<XT, CT, PR, TI, NK, NS, INC>(d, xcd_remap(blockIdx.x, nitems), grid, at);
}

// launch one instantiation; PR/TI/NK chosen from the block by the callers
template <int PR, int TI>
inline hipError_t launch_f32_k(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if constexpr (PR != PR_VOLT) {
        if (d.order == 0) {
            hipLaunchKernelGGL((bf_f32_fast_kernel<PR, TI, true>), dim3(n), dim3(kThreadsH), 0, st, d, grid, n);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((bf_f32_fast_kernel<PR, TI, false>), dim3(n), dim3(kThreadsH), 0, st, d, grid, n);
    return hipGetLastError();
}

template <int PR>
inline hipError_t launch_f32_pr(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if constexpr (PR == PR_VOLT) return launch_f32_k<PR, 1>(d, grid, n, st);
    else switch (d.t_int) {
        case 1: return launch_f32_k<PR, 1>(d, grid, n, st);
        case 2: return launch_f32_k<PR, 2>(d, grid, n, st);
        case 4: return launch_f32_k<PR, 4>(d, grid, n, st);
        case 8: return launch_f32_k<PR, 8>(d, grid, n, st);
        default: return launch_f32_k<PR, 16>(d, grid, n, st);
    }
}

inline hipError_t launch_f32(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if (d.product == PR_VOLT) return launch_f32_pr<PR_VOLT>(d, grid, n, st);
    if (d.product == PR_I) return launch_f32_pr<PR_I>(d, grid, n, st);
    return launch_f32_pr<PR_IQUV>(d, grid, n, st);
}

template <int XT, int CT, int PR, int TI, int NS, bool INC>
inline void launch_h_nsi(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    const dim3 g(n), b(kThreadsH);
    switch (fast_h_ksteps(d.S)) {
        case 4: hipLaunchKernelGGL((bf_h_fast_kernel<XT, CT, PR, TI, 4, NS, INC>), g, b, 0, st, d, grid, n); break;
        case 5: hipLaunchKernelGGL((bf_h_fast_kernel<XT, CT, PR, TI, 5, NS, INC>), g, b, 0, st, d, grid, n); break;
        case 6: hipLaunchKernelGGL((bf_h_fast_kernel<XT, CT, PR, TI, 6, NS, INC>), g, b, 0, st, d, grid, n); break;
        case 7: hipLaunchKernelGGL((bf_h_fast_kernel<XT, CT, PR, TI, 7, NS, INC>), g, b, 0, st, d, grid, n); break;
        default: hipLaunchKernelGGL((bf_h_fast_kernel<XT, CT, PR, TI, 8, NS, INC>), g, b, 0, st, d, grid, n); break;
    }
}

// the INC form (incoherent beam beside the Stokes products) only for Stokes
// with several sample streams (fuses_incoherent)
template <int XT, int CT, int PR, int TI, int NS>
inline void launch_h_ns(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if constexpr (PR != PR_VOLT && NS >= 2) {
        if (d.inc != nullptr) {
            launch_h_nsi<XT, CT, PR, TI, NS, true>(d, grid, n, st);
            return;
        }
    }
    launch_h_nsi<XT, CT, PR, TI, NS, false>(d, grid, n, st);
}

template <int XT, int CT, int PR, int TI>
inline hipError_t launch_h_k(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if constexpr (XT == XT_CF32) {
        launch_h_ns<XT, CT, PR, TI, 1>(d, grid, n, st);      // complex f32: one stream (fast_h_streams)
    } else {
        const int ns = fast_h_streams(d);
        if (ns == 1) launch_h_ns<XT, CT, PR, TI, 1>(d, grid, n, st);
        else if (ns == 2) launch_h_ns<XT, CT, PR, TI, 2>(d, grid, n, st);
        else launch_h_ns<XT, CT, PR, TI, 4>(d, grid, n, st);
    }
    return hipGetLastError();
}

template <int XT, int CT, int PR>
inline hipError_t launch_h_pr(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if constexpr (PR == PR_VOLT) return launch_h_k<XT, CT, PR, 1>(d, grid, n, st);
    else switch (d.order == 0 ? (d.t_int == 16 ? -16 : 0) : d.t_int) {
        case -16: return launch_h_k<XT, CT, PR, -16>(d, grid, n, st);     // the final order
        case 0: return launch_h_k<XT, CT, PR, 0>(d, grid, n, st);
        case 1: return launch_h_k<XT, CT, PR, 1>(d, grid, n, st);
        case 2: return launch_h_k<XT, CT, PR, 2>(d, grid, n, st);
        case 4: return launch_h_k<XT, CT, PR, 4>(d, grid, n, st);
        case 8: return launch_h_k<XT, CT, PR, 8>(d, grid, n, st);
        default: return launch_h_k<XT, CT, PR, 16>(d, grid, n, st);
    }
}

template <int XT, int CT>
inline hipError_t launch_h_xt(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    if (d.product == PR_VOLT) return launch_h_pr<XT, CT, PR_VOLT>(d, grid, n, st);
    if (d.product == PR_I) return launch_h_pr<XT, CT, PR_I>(d, grid, n, st);
    return launch_h_pr<XT, CT, PR_IQUV>(d, grid, n, st);
}

// the launch of one part, by sample type (bf_fast_f16_*.hip, bf_fast_bf16_*.hip)
template <int CT> hipError_t launch_fast_h_part(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st);
template <>
inline hipError_t launch_fast_h_part<CT_F16>(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    return d.xtype == XT_CI8    ? launch_f16_ci8(d, grid, n, st)
           : d.xtype == XT_CI16 ? launch_f16_ci16(d, grid, n, st)
                                : launch_f16_cf32(d, grid, n, st);
}
template <>
inline hipError_t launch_fast_h_part<CT_BF16>(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    return d.xtype == XT_CI8    ? launch_bf16_ci8(d, grid, n, st)
           : d.xtype == XT_CI16 ? launch_bf16_ci16(d, grid, n, st)
                                : launch_bf16_cf32(d, grid, n, st);
}

template <int CT>
inline hipError_t launch_fast_h(const BlockDesc& d, hipStream_t st) {
    BlockDesc part[2];
    const int np = split_fast_h(d, part);
    for (int p = 0; p < np; ++p) {
        ItemGrid grid;
        const int n = block_items_fast_h(part[p], &grid);
        const hipError_t e = launch_fast_h_part<CT>(part[p], grid, n, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lbf
