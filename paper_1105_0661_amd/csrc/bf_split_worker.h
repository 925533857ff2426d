// bf_split_worker.h -- the FP32 contraction worker of integer samples: FP32
// results from FP16 matrix instructions.
//
// The FP32 matrix instruction runs at 1/16 of the FP16 rate.  The operands
// of this contraction split without loss into FP16 pieces, and FP16 products
// are exact in the FP32 accumulators:
//  - int8 samples are FP16 numbers; an int16 sample is h + r with h its
//    FP16 rounding and |r| <= 8, and r = 0 for every |x| <= 2048;
//  - a weight is scaled by a power of two per beam (largest component of the
//    beam to [2^14, 2^15)) and cut into three pieces w1 = f16(w), w2 =
//    f16(w - w1), w3 = w - w1 - w2, together its 24 bits.  (A component below
//    2^-15 of the beam's largest is held to 2^-39 of that.)  The scale leaves
//    with the epilogue (2^-s for voltages, 2^-2s for Stokes).
// Two pieces hold 22 bits and two signs, and drop the last bit of a weight in
// four: the block named below took 405 us with two (ci8 360), 590 (540) with
// three, 1655 on FP32 instructions.
//
// A tile is summed small terms first: over all K-steps the products with w3
// and w2, sums 2^-11 of the result whose roundings vanish beside its own, then
// over all K-steps those with w1.  So a result is rounded at its full size
// once or twice per 8 stations, whichever stations are live; a chain of FP32
// instructions rounds it twice per live station.
// Relative rms error of the voltages against 64 bits, weights of modulus one,
// Gaussian int16 samples of sigma 64 (FP32 matrix instructions -> this
// worker): 5.4e-8 -> 2.9e-8 at 4 stations, 1.03e-7 -> 3.5e-8 at 16, 1.44e-7 ->
// 4.1e-8 at 32, 2.02e-7 -> 5.1e-8 at 64 (7.5e-8 over the whole int16 range).
// Of 64 stations with 3, 4 or 8 live, in one K-step or one in each, with
// random, equal, real and uneven weights: 0.43 to 0.97 of the chain's error.
//
// Complex float samples stay on the FP32 instructions: as many bits in both
// operands take six products of three pieces each at the least, and a third
// plane of samples that LDS has no room for.
//
// What the pieces cannot hold takes the exact path, FP32 matrix instructions
// over the same samples (one station each, in station order): a work item one
// of whose beams has a weight that is not finite, stations whose weights
// differ in magnitude by more than 2^14 (the smallest would lose bits to the
// FP16 range), or fewer than kSplitLive stations with a weight.  Such an item
// does nothing else, and has the samples in flight a group of 8 stations ahead
// and the weights in LDS: 2048 channels of 64 stations, 768 samples, 128
// beams, one station at 2^-16 of the others take 1660 us, 1650 on an FP32
// kernel of their own (item_f32_fast's schedule); one load and one product at
// a time, behind the loop of the other waves, took 3061.
// Sample residuals r, where a tile holds any, are summed before the rest,
// straight from HBM.
//
// Work split as in item_h_fast: a work group of 8 waves takes one channel and
// 8/NS beam tiles of 32, its 32-sample tiles dealt to NS streams; samples are
// staged once per work group in LDS, a wave keeps its beam tile's weight
// pieces in registers, one accumulator set, the two waves of a SIMD staggered
// so that one's epilogue meets the other's MFMAs.  With a piece as words (re,
// -im), Re y = (x_re, x_im) . w and Im y = (x_im, -x_re) . w: a piece takes 4 NK
// registers and the sample operand is turned, one packed multiplication a
// word.  w1 is kept as (im, re) too where that fits without spills: 2048
// channels of ci16, 48 stations, 300 beams 1236 -> 1183 us.
#pragma once
#include "bf_common.h"
#include "bf_workers.h"

namespace lbf {

// K-steps of 8 stations of the split worker
__host__ __device__ constexpr int split_ksteps(int S) { return S <= 16 ? 2 : S <= 32 ? 4 : (S + 7) / 8; }

// Sample streams: 4 (items of 64 beams) for at most 64 beams, where an item of
// 128 would leave half its waves idle, else 2; complex int16 from 6 K-steps up
// always 2 (the loaders of 4 streams beside the weight pieces would spill);
// voltages by volt_straight_beams.
inline int split_streams(const BlockDesc& d) {
    if (d.b1 - d.b0 > (d.product == PR_VOLT ? volt_straight_beams(d) : 64)) return 2;
    return d.xtype == XT_CI16 && split_ksteps(d.S) >= 6 ? 2 : 4;
}

// Work items: (channel of [c0, c0 + nc), group of 256/NS beams, segment)
inline int block_items_split(const BlockDesc& d, ItemGrid* grid) {
    return item_grid(d, 8 / split_streams(d) * kTile, grid);
}

// Smallest ratio of a beam's station weights (larger component of each) to
// its largest one that the pieces hold to 24 bits
constexpr float kSplitRange = 16384.0f;

// Fewest stations with a weight, in a beam that has any: a result of one or
// two stations is rounded once or twice by the FP32 chain, and the FP16
// instruction's sum of 8 stations and the accumulator is not the nearest FP32
// number in every case.  rms error against 64 bits, FP32 chain / pieces: one
// station of any weight 3.09e-8 / 3.24e-8, of real weight 2.5e-8 / 3.4e-8,
// two 3.1e-8 / 3.4e-8, three 3.57e-8 / 3.4e-8 and from there on lower.
constexpr int kSplitLive = 3;

LBF_INLINE uint32_t pack_h(_Float16 lo, _Float16 hi) {
    const halfx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, v);
}

// (x_re, x_im) -> (x_im, -x_re), four stations
LBF_INLINE u32x4 turn(const u32x4& v) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = v[i];
        const halfx2 x = __builtin_bit_cast(halfx2, w), sign = {(_Float16)1.0f, (_Float16)-1.0f};
        r[i] = __builtin_bit_cast(uint32_t, (halfx2)(__builtin_shufflevector(x, x, 1, 0) * sign));
    }
    return r;
}

// The residuals x - f16(x) of a complex int16 value, as a packed f16 word
LBF_INLINE uint32_t residual_i16x2(uint32_t w) {
    const int re = (int)(int16_t)w, im = (int)(int16_t)(w >> 16);
    return pack_h((_Float16)(float)(re - (int)(float)(_Float16)(float)re),
                  (_Float16)(float)(im - (int)(float)(_Float16)(float)im));
}

// Stokes or voltages of one tile out of scaled accumulators (weights times
// 2^sc): as stokes_store_tile / volt_store_cm, with the scale taken out exactly
template <int PR, int TI>
LBF_INLINE void split_stokes_store(const floatx16 (&acc)[4], __amdgpu_buffer_rsrc_t rs, const BlockDesc& d, int c,
                                   int beam, int t0, int h, bool ok, int sc) {
    constexpr int NOUT = 16 / TI;
    const int T2 = d.T / TI;
    const int tq0 = (t0 + 16 * h) / TI;
#pragma unroll
    for (int o = 0; o < NOUT; ++o) {
        float sm[4], v[4];
        stokes_sums<PR, TI>(acc, o * TI, sm);
        stokes_from_sums<PR>(sm, v);
#pragma unroll
        for (int q = 0; q < (PR == PR_IQUV ? 4 : 1); ++q) v[q] = __builtin_amdgcn_ldexpf(v[q], -2 * sc);
        const int tq = tq0 + o;
        if (d.order == 0) stokes_store_row<PR, true>(v, rs, d, c, T2, tq, beam, ok && tq < T2);      // uniform
        else stokes_store_row<PR, false>(v, rs, d, c, T2, tq, beam, ok && tq < T2);
        __builtin_amdgcn_sched_barrier(0);                     // one period's temporaries at a time
    }
}

template <int PR>
LBF_INLINE void split_epilogue(const floatx16 (&acc)[4], __amdgpu_buffer_rsrc_t rs, const BlockDesc& d, int c, int beam,
                               int t0, int h, bool ok, int sc) {
    const int T = d.T;
    if constexpr (PR == PR_VOLT) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int t = t0 + 16 * h + k;
            const uint32_t off = store_off(ok && t < T, volt_off(beam, T, t));
            floatx4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_ldexpf(acc[q][k], -sc);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, (int)off, 0, 0);
            if (k & 1) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        switch (d.t_int) {                                       // uniform
            case 1: split_stokes_store<PR, 1>(acc, rs, d, c, beam, t0, h, ok, sc); break;
            case 2: split_stokes_store<PR, 2>(acc, rs, d, c, beam, t0, h, ok, sc); break;
            case 4: split_stokes_store<PR, 4>(acc, rs, d, c, beam, t0, h, ok, sc); break;
            case 8: split_stokes_store<PR, 8>(acc, rs, d, c, beam, t0, h, ok, sc); break;
            default: split_stokes_store<PR, 16>(acc, rs, d, c, beam, t0, h, ok, sc); break;
        }
    }
}

// vbuf: kVoltWords floats per wave for voltages in two streams (four leave no
// room)
template <int XT, int PR, int NK, int NS>
LBF_INLINE void item_f32_split(const BlockDesc& d, int item, const ItemGrid& grid, uint32_t* at, int* flags, float* vbuf) {
    typedef MfmaH<CT_F16> M;
    typedef M::vec V;
    typedef float float2v __attribute__((ext_vector_type(2)));
    constexpr int BYTES = sample_bytes(XT);
    constexpr int NBT = 8 / NS;                            // beam tiles per item
    typedef TileLoader<XT, CT_F16, NK, NS> Loader;
    constexpr int CPT = Loader::CPT;                       // chunks per thread per step
    const int T = d.T, S = d.S;
    const ItemPos ip = item_pos(d, grid, item, NBT * kTile);
    const int c = ip.c, bg = ip.bg, tile_lo = ip.tile_lo, ntiles = ip.ntiles;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int r = lane & 31, h = lane >> 5;
    const int bt = wave % NBT, sigma = wave / NBT;         // beam tile, sample stream
    const int beam = d.b0 + (bg * NBT + bt) * kTile + r;
    const bool beam_ok = beam < d.b1;
    const int nsteps = (ntiles + NS - 1) / NS;
    const uint32_t stride_bytes = (uint32_t)((size_t)d.C * T * BYTES);
    const int T2 = PR == PR_VOLT ? T : T / d.t_int;
    const __amdgpu_buffer_rsrc_t ors =
        PR == PR_VOLT ? channel_rsrc(d, c, out_channel_bytes(d, PR, T2)) : stokes_rsrc(d, c, PR, T2);
    const __amdgpu_buffer_rsrc_t wrs = weight_rsrc(d, c, 8);

    Loader ld;
    ld.init(d, ip);
    u32x4 raw[CPT];
    auto load_chunks = [&](int k) { ld.load(k, raw); };
    auto store_chunk = [&](int k, int i) {
        if (!ld.staged(i)) return;
        ld.store(at, k, i, raw);
        if constexpr (XT == XT_CI16) {
            // any component outside [-2048, 2047]: x + 2048 has one of its top four bits set
            typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
            const u16x2 bias = {2048, 2048};
            uint32_t big = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t v = raw[i][e];             // a value: a bit cast of the element itself reads element 0
                big |= __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, v) + bias));
            }
            if (big & 0xf000f000u) flags[(k & 1) * NS + ld.stream(i)] = k;
        }
    };
    auto store_chunks = [&](int k) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) store_chunk(k, i);
    };
    load_chunks(0);

    // The item's weights, through LDS: a lane's own are 32-byte pieces of rows
    // a whole beam apart, a cache line per lane and load.  Whole rows instead:
    // 8192 channels of ci16, 64 stations, 128 beams 2100 -> 1930 us.
    // Stations >= S and beams >= B as zeros.
    constexpr int NBEAM = NBT * kTile, WROW = 16 * NK + 4;  // words per row: 4 mod 64 banks
    static_assert(NBEAM * WROW <= NS * 2 * kATileWords, "the weights fit the tiles' LDS");
    float* wl = reinterpret_cast<float*>(at);
    {
        float2v w[NBEAM / 8];
#pragma unroll
        for (int j = 0; j < NBEAM / 8; ++j) {
            const int bw = d.b0 + bg * NBEAM + wave + 8 * j;
            w[j] = __builtin_bit_cast(float2v, __builtin_amdgcn_raw_buffer_load_b64(
                wrs, (int)select_off(bw < d.b1 && lane < S, weight_off(bw, S, lane, 8), kNoAccess), 0, 0));
        }
        if (lane < 8 * NK) {
#pragma unroll
            for (int j = 0; j < NBEAM / 8; ++j) *reinterpret_cast<float2v*>(wl + (wave + 8 * j) * WROW + 2 * lane) = w[j];
        }
    }
    int* any_exact = flags + 2 * NS;
    if (tid == 0) *any_exact = 0;
    __syncthreads();
    // this wave's weight pieces, all K-steps.  Magnitudes are compared as
    // integers, which orders NaN above infinity above the numbers.
    constexpr bool BOTH = NK <= (XT == XT_CI8 ? 7 : 6);    // w1 as (im, re) too, where it fits without spills
    u32x4 wr[3][NK], wi[BOTH ? NK : 1];
    int sc;
    {
        // read twice, the magnitudes, then the pieces, so that the raw
        // weights never sit beside all the pieces
        auto load_w = [&](int kk, floatx4 (&w)[2]) {
            const floatx4* p = reinterpret_cast<const floatx4*>(wl + (bt * kTile + r) * WROW + 2 * (8 * kk + 4 * h));
            w[0] = p[0];
            w[1] = p[1];
        };
        uint32_t wmax = 0u, wmin = 0xffffffffu;               // wmin: the smallest non-zero magnitude minus one
        int live = 0;                                         // stations with a weight
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            floatx4 w[2];
            load_w(kk, w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float re = w[i / 2][i % 2 * 2], im = w[i / 2][i % 2 * 2 + 1];
                const uint32_t m = max(__float_as_uint(re) & 0x7fffffffu, __float_as_uint(im) & 0x7fffffffu);
                wmax = max(wmax, m);
                wmin = min(wmin, m - 1u);
                live += m != 0u;
            }
        }
        wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, 32, kWave));
        wmin = min(wmin, (uint32_t)__shfl_xor((int)wmin, 32, kWave));
        live += __shfl_xor(live, 32, kWave);
        const float fmx = __uint_as_float(wmax), fmn = __uint_as_float(wmin + 1u);
        const bool bad = wmax >= 0x7f800000u || (wmax != 0u && (fmn * kSplitRange < fmx || live < kSplitLive));
        if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) *any_exact = 1;
        sc = wmax != 0u && wmax < 0x7f800000u ? 15 - __builtin_amdgcn_frexp_expf(fmx) : 0;
        __asm__ volatile("" : "+v"(sc) : : "memory");           // the second reading stays a second one
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            floatx4 w[2];
            load_w(kk, w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float re = __builtin_amdgcn_ldexpf(w[i / 2][i % 2 * 2], sc);
                float im = __builtin_amdgcn_ldexpf(w[i / 2][i % 2 * 2 + 1], sc);
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const _Float16 pr = (_Float16)re, pi = (_Float16)im;
                    re -= (float)pr;                       // exact
                    im -= (float)pi;
                    wr[p][kk][i] = pack_h(pr, -pi);
                    if (BOTH && p == 0) wi[kk][i] = pack_h(pi, pr);
                }
            }
            if (kk & 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();
    const bool exact = __builtin_amdgcn_readfirstlane(*any_exact) != 0;
    // a wave whose beam tile lies wholly past the block's beams only loads,
    // stages and meets the barriers
    const bool idle = d.b0 + (bg * NBT + bt) * kTile >= d.b1;
    const int trow = tile_row_sample(r);
    const int sw = a_swz(trow);

    floatx16 acc[4];
    int esc = sc;                                          // scale of the accumulators
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = zero16();
    // one operand pair (both polarisations) with a piece kept once, and with w1
    auto mfma_turned = [&](const u32x4& x, const u32x4& y, const u32x4& tx, const u32x4& ty, const u32x4& w4) {
        const V w = __builtin_bit_cast(V, w4);
        acc[0] = M::mfma(__builtin_bit_cast(V, x), w, acc[0]);
        acc[1] = M::mfma(__builtin_bit_cast(V, tx), w, acc[1]);
        acc[2] = M::mfma(__builtin_bit_cast(V, y), w, acc[2]);
        acc[3] = M::mfma(__builtin_bit_cast(V, ty), w, acc[3]);
    };
    auto mfma_first = [&](const u32x4& x, const u32x4& y, int kk) {
        const V a = __builtin_bit_cast(V, x), b = __builtin_bit_cast(V, y);
        const V br = __builtin_bit_cast(V, wr[0][kk]), bi = __builtin_bit_cast(V, wi[BOTH ? kk : 0]);
        acc[0] = M::mfma(a, br, acc[0]);
        acc[1] = M::mfma(a, bi, acc[1]);
        acc[2] = M::mfma(b, br, acc[2]);
        acc[3] = M::mfma(b, bi, acc[3]);
    };
    auto epilogue = [&](int k) {
        const int tile = tile_lo + sigma + NS * k;
        const bool ok = k >= 0 && tile < tile_lo + ntiles && beam_ok;
        int bm = beam, hh = h;
        __asm__ volatile("" : "+v"(bm), "+v"(hh));          // offsets formed anew for each tile
        if constexpr (PR == PR_VOLT && NS <= 2) {
            // the scale is the beam's: taken out before the lanes exchange
            volt_store_rows(acc, vbuf + wave * kVoltWords, ors, T, beam - r, d.b1, tile * kTile, k >= 0 && tile < tile_lo + ntiles,
                            esc);
            return;
        }
        split_epilogue<PR>(acc, ors, d, c, bm, tile * kTile, hh, ok, esc);
    };
    if (exact) {
        // FP32 matrix instructions, lane half h holding the re (0) or im (1)
        // component of station s as K index h of a 32x32x2 MFMA; samples
        // straight from HBM, a group of 8 stations ahead of their use,
        // weights from LDS
        const int nmine = ntiles > sigma ? (ntiles - sigma + NS - 1) / NS : 0;   // this wave's tiles
        if (idle || nmine == 0) return;
        uint32_t hsh = (uint32_t)h * (XT == XT_CI8 ? 8u : 16u);
        int wrow = (bt * kTile + r) * WROW;
        __asm__ volatile("" : "+v"(hsh), "+v"(wrow));
        typedef Raw<XT> R;
        typename R::type ring[8];
        auto load_quad = [&](int q4, int k, int g) {           // stations 8 g + 4 q4 .. + 3 of the wave's tile k
            const int t = min((tile_lo + sigma + NS * min(k, nmine - 1)) * kTile + trow, T - 1);
            const __amdgpu_buffer_rsrc_t rs = group_rsrc(d.x, 8 * g, S, stride_bytes);
#pragma unroll
            for (int i = 4 * q4; i < 4 * q4 + 4; ++i)
                ring[i] = buffer_sample<XT>(rs, sample_off(i, stride_bytes, c, T, t, BYTES));
        };
        esc = 0;
        load_quad(0, 0, 0);
        load_quad(1, 0, 0);
        for (int k = 0; k < nmine; ++k) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = zero16();
            for (int g = 0; g < NK; ++g) {
                const bool last = g == NK - 1;
#pragma unroll
                for (int q4 = 0; q4 < 2; ++q4) {
                    float ax[4], ay[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) R::half(ring[4 * q4 + i], hsh, ax[i], ay[i]);
                    load_quad(q4, last ? k + 1 : k, last ? 0 : g + 1);
                    const floatx4* p = reinterpret_cast<const floatx4*>(wl + wrow + 2 * (8 * g + 4 * q4));
                    const floatx4 w[2] = {p[0], p[1]};
                    __builtin_amdgcn_sched_barrier(0);         // the refill issues before the MFMAs
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float re = w[i / 2][i % 2 * 2], im = w[i / 2][i % 2 * 2 + 1];
                        const float br = h ? -im : re, bi = h ? re : im;
                        acc[0] = mfma_f32(ax[i], br, acc[0]);
                        acc[1] = mfma_f32(ax[i], bi, acc[1]);
                        acc[2] = mfma_f32(ay[i], br, acc[2]);
                        acc[3] = mfma_f32(ay[i], bi, acc[3]);
                    }
                }
            }
            epilogue(k);
        }
        return;
    }

    const bool late = wave >= 4;                           // the second wave of each SIMD
    if constexpr (XT == XT_CI16) {
        if (tid < 2 * NS) flags[tid] = -1;
        __syncthreads();
    }
    store_chunks(0);
    __syncthreads();
    for (int k = 0; k < nsteps; ++k) {
        load_chunks(k + 1);
        if (!idle) {
            if (late && k > 0) epilogue(k - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = zero16();
            if (XT == XT_CI16 && __builtin_amdgcn_readfirstlane(flags[(k & 1) * NS + sigma]) == k) {
                // residuals of this tile's samples, straight from HBM (rows past T: its last sample)
                const int t = min((min(tile_lo + sigma + NS * k, tile_lo + ntiles - 1)) * kTile + trow, T - 1);
#pragma unroll
                for (int kk = 0; kk < NK; ++kk) {
                    const __amdgpu_buffer_rsrc_t rs = group_rsrc(d.x, 8 * kk, S, stride_bytes);
                    u32x4 ux, uy;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                            rs, (int)sample_off(4 * h + i, stride_bytes, c, T, t, BYTES), 0, 0));
                        ux[i] = residual_i16x2(v[0]);
                        uy[i] = residual_i16x2(v[1]);
                    }
                    const u32x4 tx = turn(ux), ty = turn(uy);
#pragma unroll
                    for (int p = 2; p >= 0; --p) mfma_turned(ux, uy, tx, ty, wr[p][kk]);
                    __builtin_amdgcn_sched_barrier(0);         // one K-step's loads at a time
                }
            }
            int rowx = (sigma * 2 + (k & 1)) * kATileWords + 2 * trow * kARow, swx = 4 * (h ^ sw);
            __asm__ volatile("" : "+v"(rowx), "+v"(swx));
            const uint32_t* ax0 = at + rowx;
            __builtin_amdgcn_sched_barrier(0);
            // operands one K-step ahead from LDS, K-steps 0 .. NK - 1 with the
            // small pieces, then again with w1; the next step's samples staged
            // under the later MFMAs
            u32x4 ax[2], ay[2];
            ax[0] = *reinterpret_cast<const u32x4*>(ax0 + swx);
            ay[0] = *reinterpret_cast<const u32x4*>(ax0 + kARow + swx);
#pragma unroll
            for (int j = 0; j < 2 * NK; ++j) {
                const int kk = j % NK;
                if (j + 1 < 2 * NK) {
                    const int off = swx ^ (8 * ((j + 1) % NK));    // 4 ((2 kk + h) ^ sw)
                    ax[(j + 1) & 1] = *reinterpret_cast<const u32x4*>(ax0 + off);
                    ay[(j + 1) & 1] = *reinterpret_cast<const u32x4*>(ax0 + kARow + off);
                }
                const u32x4 &a = ax[j & 1], &b = ay[j & 1];
                if (BOTH && j >= NK) {
                    mfma_first(a, b, kk);
                } else {
                    const u32x4 ta = turn(a), tb = turn(b);
                    if (j < NK) {
                        mfma_turned(a, b, ta, tb, wr[2][kk]);
                        mfma_turned(a, b, ta, tb, wr[1][kk]);
                    } else {
                        mfma_turned(a, b, ta, tb, wr[0][kk]);
                    }
                }
#pragma unroll
                for (int i = 0; i < CPT; ++i)
                    if (j == NK + i * NK / CPT) store_chunk(k + 1, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!late) epilogue(k);
        } else {
            store_chunks(k + 1);
        }
        __syncthreads();
    }
    if (!idle && late) epilogue(nsteps - 1);
}

// 8 waves, two per SIMD; LDS: NS streams x 2 buffers of one A tile
template <int XT, int PR, int NK, int NS>
__global__ __launch_bounds__(kThreadsH) void bf_f32_split_kernel(BlockDesc d, ItemGrid grid, int nitems) {
    __shared__ __attribute__((aligned(16))) uint32_t at[NS * 2 * kATileWords];
    __shared__ __attribute__((aligned(16))) int flags[2 * NS + 1];
    constexpr bool rows = PR == PR_VOLT && NS <= 2;
    __shared__ __attribute__((aligned(16))) float vbuf[rows ? 8 * kVoltWords : 1];
    item_f32_split<XT, PR, NK, NS>(d, xcd_remap(blockIdx.x, nitems), grid, at, flags, vbuf);
}

template <int XT, int PR, int NK>
inline void launch_split_nk(const BlockDesc& d, int ns, const ItemGrid& grid, int n, hipStream_t st) {
    const dim3 g(n), b(kThreadsH);
    if constexpr (XT == XT_CI8 || (XT == XT_CI16 && NK < 6)) {
        if (ns == 4) {
            hipLaunchKernelGGL((bf_f32_split_kernel<XT, PR, NK, 4>), g, b, 0, st, d, grid, n);
            return;
        }
    }
    hipLaunchKernelGGL((bf_f32_split_kernel<XT, PR, NK, 2>), g, b, 0, st, d, grid, n);
}

template <int XT, int PR>
inline void launch_split_pr(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    const int ns = split_streams(d);
    switch (split_ksteps(d.S)) {
        case 2: launch_split_nk<XT, PR, 2>(d, ns, grid, n, st); break;
        case 4: launch_split_nk<XT, PR, 4>(d, ns, grid, n, st); break;
        case 5: launch_split_nk<XT, PR, 5>(d, ns, grid, n, st); break;
        case 6: launch_split_nk<XT, PR, 6>(d, ns, grid, n, st); break;
        case 7: launch_split_nk<XT, PR, 7>(d, ns, grid, n, st); break;
        default: launch_split_nk<XT, PR, 8>(d, ns, grid, n, st); break;
    }
}

template <int XT>
inline hipError_t launch_split_xt(const BlockDesc& d, hipStream_t st) {
    ItemGrid grid;
    const int n = block_items_split(d, &grid);
    if (d.product == PR_VOLT) launch_split_pr<XT, PR_VOLT>(d, grid, n, st);
    else if (d.product == PR_I) launch_split_pr<XT, PR_I>(d, grid, n, st);
    else launch_split_pr<XT, PR_IQUV>(d, grid, n, st);
    return hipGetLastError();
}

}  // namespace lbf
