// bf_addr.h -- the buffer addressing of the fast contraction workers as plain
// integer arithmetic, shared by the kernels and by a host-side walk
// (bf_addr_check.cpp) that checks every access of a block against its
// buffers before anything runs on a device.
//
// The workers address HBM through buffer descriptors: a base address, a range
// in bytes (accesses at or beyond it read zeros or store nothing) and 32-bit
// byte offsets.  What must hold: every descriptor lies inside its buffer, and
// no 32-bit offset wraps.  fast_path() bounds the sizes so that the offsets
// below stay under 2^31.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbf_device.h"

#define LBF_HD __host__ __device__ inline

namespace lbf {

// Work items cut a block's samples into segments of kSegTiles 32-sample
// tiles, or of 2, 4 or 8 times as many while the block keeps at least
// kMinItems items that way: a longer item spreads its prologue (weights into
// registers, the first loads) and its last step over more steps, and enough
// items remain to keep every compute unit busy to the end.  A block too small
// to give every compute unit an item takes shorter segments, down to the 4
// tiles that 4 sample streams work on at once: 16 channels of 1024 samples
// (8 stations, 4 beams, FP32) took 15.2 us in 32 items of 24 tiles, 6.6 us
// in 128 of 4.
constexpr int kSegTiles = 24, kSegTilesMax = 192, kMinItems = 2048;
constexpr int kSegTilesMin = 4, kComputeUnits = kXcds * kCusPerXcd;

inline int seg_tiles(const BlockDesc& d, int nbg) {
    const int ntiles = (d.T + kTile - 1) / kTile;
    int seg = kSegTiles;
    while (seg > kSegTilesMin && (int64_t)d.nc * nbg * ((ntiles + seg - 1) / seg) < kComputeUnits) seg /= 2;   // 24, 12, 6, 3
    if (seg < kSegTilesMin) seg = kSegTilesMin;
    while (seg >= kSegTiles && seg < kSegTilesMax && seg < ntiles &&
           (int64_t)d.nc * nbg * ((ntiles + 2 * seg - 1) / (2 * seg)) >= kMinItems)
        seg *= 2;
    return seg;
}

// "no access": an offset past every output and weight descriptor (fast_path
// bounds both), where the hardware drops a store and a load reads zeros.
// 2^31, not an offset next to 2^32: the range check adds the access size to
// the offset, and such a sum could wrap around to an in-range value.
constexpr uint32_t kNoAccess = 0x80000000u;

// A work item of the fast workers: channel c (of [c0, c0 + nc)), beam group
// bg of `per` beams (a power of two), sample tiles [tile_lo, tile_lo + ntiles).
struct ItemPos {
    int c, bg, tile_lo, ntiles;
};

// How a launch's items are numbered, chosen once on the host: the work groups
// take a number apart with multiplications.  Their prologue is a chain of
// scalar instructions that nothing overlaps in an item of one or two steps;
// the segment rule and four divisions in it cost 16384 channels of ci8, 19
// stations, 64 samples, 3 beams 15 us of 226.
struct ItemGrid {
    uint32_t nseg;                 // segments of the block's samples
    uint32_t mseg, mbg;            // n / nseg = n mseg >> (31 + shift) for n < 2^31, n / beam groups likewise
    uint8_t seg, sseg, sbg, pad;   // tiles per segment, the shifts
};

// m, s with n / d = n m >> (31 + s) for every n < 2^31: m = floor(2^(31 + s) /
// d) + 1 with 2^s >= d fits 32 bits and is too large by at most d / 2^(31 + s)
// of itself, less than 1 / n
inline uint32_t div_magic(uint32_t d, uint8_t* s) {
    *s = 0;
    while ((1ull << *s) < d) ++*s;
    return (uint32_t)((1ull << (31 + *s)) / d) + 1u;
}
LBF_HD uint32_t div_by(uint32_t n, uint32_t m, uint32_t s) { return (uint32_t)(((uint64_t)n * m) >> (31 + s)); }

// The items of a block part; returns their number
inline int item_grid(const BlockDesc& d, int per, ItemGrid* g) {
    const int nbg = (d.b1 - d.b0 + per - 1) / per, seg = seg_tiles(d, nbg);
    const int ntiles = (d.T + kTile - 1) / kTile, nseg = (ntiles + seg - 1) / seg;
    g->nseg = (uint32_t)nseg;
    g->seg = (uint8_t)seg;
    g->mseg = div_magic((uint32_t)nseg, &g->sseg);
    g->mbg = div_magic((uint32_t)nbg, &g->sbg);
    g->pad = 0;
    return d.nc * nbg * nseg;
}

LBF_HD ItemPos item_pos(const BlockDesc& d, const ItemGrid& g, int item, int per) {
    const uint32_t nbg = (uint32_t)(d.b1 - d.b0 + per - 1) / (uint32_t)per;
    const uint32_t cb = div_by((uint32_t)item, g.mseg, g.sseg), c = div_by(cb, g.mbg, g.sbg);
    ItemPos p;
    p.c = d.c0 + (int)c;
    p.bg = (int)(cb - c * nbg);
    p.tile_lo = (int)(((uint32_t)item - cb * g.nseg) * g.seg);
    const int left = (int)((uint32_t)(d.T + kTile - 1) / kTile) - p.tile_lo;
    p.ntiles = left < g.seg ? left : g.seg;
    return p;
}

// Station samples x[s][c][t] (sample_bytes each, station planes stride_bytes
// = C T sample_bytes apart).  A descriptor covers the whole planes of the
// valid stations of one group of 8, [s0, min(s0 + 8, S)); the channel and
// time go into the offset, so a ragged last tile reads past its channel into
// the next one (rows the epilogue never stores) but never past the array.
LBF_HD uint64_t group_base(int s0, uint32_t stride_bytes) { return (uint64_t)s0 * stride_bytes; }

LBF_HD uint32_t group_range(int s0, int S, uint32_t stride_bytes) {
    const int n = S - s0;                                  // (selects, not a clamp: scalar instructions)
    return n >= 8 ? 8u * stride_bytes : n <= 0 ? 0u : (uint32_t)n * stride_bytes;
}

// station s0 + i of a group, channel c, sample t
LBF_HD uint32_t sample_off(int i, uint32_t stride_bytes, int c, int T, int t, int bytes) {
    return (uint32_t)i * stride_bytes + (uint32_t)(c * T + t) * (uint32_t)bytes;
}

// Weights w[c][b][s] (bytes per complex weight): one descriptor per channel.
LBF_HD uint64_t weight_base(const BlockDesc& d, int c, int bytes) { return (uint64_t)c * d.B * d.S * bytes; }
LBF_HD uint32_t weight_range(const BlockDesc& d, int bytes) { return (uint32_t)d.B * (uint32_t)d.S * (uint32_t)bytes; }
LBF_HD uint32_t weight_off(int beam, int S, int s, int bytes) { return ((uint32_t)beam * S + s) * (uint32_t)bytes; }

// Station planes of a tile: the descriptor of group_base / group_range moved
// to channel c (channel_off bytes into each plane) and to sample t of it
// (tile_off further), so that a thread's offset, station and sample within the
// tile, is the same for every tile and channel.  What remains of the range is
// kept signed: past the stations it is negative, and a range of none.
LBF_HD uint32_t channel_off(int c, int T, int bytes) { return (uint32_t)(c * T) * (uint32_t)bytes; }
LBF_HD uint32_t tile_off(int t, int bytes) { return (uint32_t)t * (uint32_t)bytes; }
LBF_HD int channel_limit(int s0, int S, uint32_t stride_bytes, uint32_t coff) {
    return (int)group_range(s0, S, stride_bytes) - (int)coff;
}
LBF_HD uint32_t tile_range(int limit, uint32_t toff) {
    const int r = limit - (int)toff;
    return r > 0 ? (uint32_t)r : 0u;
}

// The sample loaders of the workers that stage tiles in LDS: a tile's 16-byte
// chunks (cps of them per station, 8, 16 or 32), stations padded to the 8 nk
// of the K-steps, are dealt to the work group's waves 64 at a time: 8, 4 or 2
// stations of one group of 8, so wave_loads of them to a group.  Load i of a
// wave is number wave + kLoaderWaves i of the step's ns tiles; its group and
// stream are uniform, and the station within the group does not depend on i.
// (Stations padded to 32 or 64 instead, for divisors that are powers of two,
// cost a step up to 24 stations' loads: 16384 channels of ci8, 38 stations, 192
// samples, 3 beams 396 -> 470 us.  Waves of 8 chunks of 8 stations store to
// LDS with 60 % fewer bank conflicts, which changed no time, and read 128-byte
// runs instead of 256 or 512: an HBM-bound block, 64 stations and 10 beams as
// voltages, took 1041 instead of 1006 us.)
constexpr int kLoaderWaves = 8;

LBF_HD constexpr int wave_loads(int cps) { return cps / 8; }
LBF_HD constexpr int chunks_per_thread(int ns, int nk, int cps) {
    return (ns * nk * wave_loads(cps) + kLoaderWaves - 1) / kLoaderWaves;
}
// number of the wave's load i among the groups of the step's tiles: group n % nk of stream n / nk
LBF_HD constexpr uint32_t chunk_group(uint32_t wave, uint32_t i, uint32_t cps) {
    return wave / (cps / 8) + kLoaderWaves / (cps / 8) * i;
}
// station within the group, chunk of the station
LBF_HD constexpr uint32_t chunk_station(uint32_t wave, uint32_t lane, uint32_t cps) {
    return wave % (cps / 8) * (kWave / cps) + lane / cps;
}
LBF_HD constexpr uint32_t chunk_q(uint32_t lane, uint32_t cps) { return lane % cps; }
// bytes of a thread's offset into the descriptor: station of the group, chunk of the tile
LBF_HD uint32_t chunk_off(int s, int q, uint32_t stride_bytes) { return (uint32_t)s * stride_bytes + 16u * (uint32_t)q; }
// the stream's tile of step k, or the item's last tile once it has run out
LBF_HD int stream_tile(int sg, int k, int ns, int tile_lo, int ntiles) {
    const int i = sg + ns * k;
    return tile_lo + (i < ntiles - 1 ? i : ntiles - 1);
}

// The FP16/BF16 worker's weight rows on their way into LDS, where nk and the
// streams ask for them, in items of at least kRowSteps steps: 16 lanes to a
// beam's row, 4 stations each; pass j is 32 beams further
LBF_HD constexpr bool h_weight_rows(int nk, int ns) { return nk == 8 && ns <= 2; }
constexpr int kRowSteps = 8;
LBF_HD constexpr int h_weight_row(int tid, int j) { return tid / 16 + 32 * j; }
LBF_HD constexpr int h_weight_station(int tid) { return tid % 16 * 4; }

// Output of one channel (order 1 staging, or voltages): one descriptor per
// channel of the item's block, output index c - c0.
LBF_HD uint32_t out_channel_bytes(const BlockDesc& d, int product, int T2) {
    return product == PR_VOLT ? (uint32_t)d.B * d.T * 16u : (uint32_t)T2 * d.ld_row * 4u;
}

LBF_HD uint64_t out_base(const BlockDesc& d, int c, uint32_t channel_bytes) {
    return (uint64_t)(c - d.c0) * channel_bytes;
}

// voltages y[b][t][p] of the channel, 16 bytes per sample
LBF_HD uint32_t volt_off(int beam, int T, int t) { return ((uint32_t)beam * T + t) * 16u; }

// Stokes straight into the final order [b][k][t'][c] (order 0): parameter 0;
// the others follow in planes of stokes_plane bytes.  One descriptor over the
// whole output, which direct_store keeps small.
LBF_HD uint32_t stokes_plane(const BlockDesc& d, int T2) { return (uint32_t)T2 * (uint32_t)d.C * 4u; }
LBF_HD uint32_t stokes_off_final(const BlockDesc& d, int c, int T2, int tq, int beam, int K) {
    return (uint32_t)beam * (uint32_t)K * stokes_plane(d, T2) + ((uint32_t)tq * (uint32_t)d.C + (uint32_t)c) * 4u;
}

// Stokes s[t'][b][k] of the channel, rows of ld floats: 16 bytes (IQUV) or 4 (I)
LBF_HD uint32_t stokes_off(int tq, int ld, int beam, int K) {
    return ((uint32_t)tq * (uint32_t)ld + (uint32_t)beam * (uint32_t)K) * 4u;
}

}  // namespace lbf
