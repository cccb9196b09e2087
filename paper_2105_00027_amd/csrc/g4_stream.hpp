// Geometry of the streamed update kernel (g4_update_stream.hip), host and
// device.
#pragma once

#include "g4_internal.hpp"

namespace g4 {

// LDS layout of one staging buffer in 16-byte chunks.  A chunk is one element of
// one spin (FP64) or two neighbouring columns of one spin (FP32).  Each part
// starts on a multiple of 64 chunks, so that one wave's copy instruction has one
// source.  Exchange rows have an odd pitch (lanes one row apart fall in distinct
// banks).
struct StreamGeom {
    int yn, yp;         // chunks a row of the exchange block needs, and its pitch
    int zn;             // chunks (and pitch) of a row of the PP block
    int nY, nZ;         // rows of the exchange and PP blocks
    int cY, cZ, cA, cB; // chunks of each part (exchange and PP: per spin)
    int oYd, oZu, oZd, oA, oB, total;   // first chunk of each part (exchange up at 0), all parts
};
__host__ __device__ constexpr StreamGeom stream_geom(int epc, int nw, int T2, int M, int channels) {
    StreamGeom g{};
    const int nph = ((channels & CH_MAG) ? 1 : 0) + ((channels & CH_CHG) ? 1 : 0);
    const bool pp = (channels & CH_PP) != 0;
    const int yc = T2 + M - 1, zc = nw + M - 1;
    // FP32: the pairs start on an even column, one before the first when that is odd
    g.yn = epc == 2 ? (yc + 2) / 2 : yc;
    g.yp = g.yn | 1;
    g.zn = epc == 2 ? (zc + 2) / 2 : zc;
    g.nY = nph ? nw + M - 1 : 0;
    g.nZ = pp ? T2 + M - 1 : 0;
    g.cY = g.nY * g.yp;
    g.cZ = g.nZ * g.zn;
    g.cA = nph * M * nw / epc;
    g.cB = nph * M * (epc == 2 ? (T2 + 1) / 2 : T2);
    g.oYd = (g.cY + 63) / 64 * 64;
    g.oZu = 2 * g.oYd;
    g.oZd = g.oZu + (g.cZ + 63) / 64 * 64;
    g.oA = 2 * g.oZd - g.oZu;
    g.oB = g.oA + (g.cA + 63) / 64 * 64;
    g.total = g.oB + (g.cB + 63) / 64 * 64;
    return g;
}
// Copy instructions per wave and measurement of one part (64 chunks each, dealt
// to the four waves in turn), and their bounds where nw is not compiled in.
__host__ __device__ constexpr int stream_copies(int chunks) { return (chunks + 255) / 256; }
constexpr int kStreamY = 6, kStreamZ = 6, kStreamA = 8, kStreamB = 2;
constexpr size_t kLdsBytes = 160 * 1024;   // of a CU, and a block's limit
__host__ __device__ constexpr bool stream_fits(const StreamGeom &g) {
    return stream_copies(g.cY) <= kStreamY && stream_copies(g.cZ) <= kStreamZ && stream_copies(g.cA) <= kStreamA &&
           stream_copies(g.cB) <= kStreamB;
}
// A launch of one measurement (every launch of a plain handle) fills one buffer
// only and has no other: with two the 6x6, 128 frequencies, one-channel plain
// pass fitted one block a CU (16.4 ms a measurement; 12.4 on update_kernel, which
// fits two).
__host__ __device__ constexpr int stream_buffers(int batch) { return batch > 1 ? 2 : 1; }
inline size_t stream_lds_bytes(const StreamGeom &g, int batch) {
    return (size_t)stream_buffers(batch) * g.total * 16 + kMaxPassBatch * 8;
}
inline StreamGeom stream_geom_of(int kind, int channels, int mgroup, int tile, const Dims &d) {
    return stream_geom(kind == 2 ? 2 : 1, d.nw, tile < d.nw ? tile : d.nw, mgroup, channels);
}

// Whether the streamed kernel can run a launch of `batch` measurements: magnetic,
// charge and PP, plane groups of 4 and 8, the rows per thread that are compiled;
// FP32 rows of G have to hold whole pairs of columns; copy offsets are 32-bit
// within a matrix and within a measurement's direct vectors; its buffers fit the
// LDS.
inline bool stream_runs(int kind, int channels, int ept, int mgroup, int tile, const Dims &d, int64_t dir_slot_stride,
                        int batch) {
    if ((channels & ~7) || (mgroup != 4 && mgroup != 8)) return false;
    if (ept != 1 && ept != 2 && !(kind == 2 && ept == 4 && mgroup == 4)) return false;
    if (kind == 2 && d.ng % 2) return false;
    const uint64_t el = kind == 2 ? 8 : 16, lim = 1ull << 32;
    const int nph = __builtin_popcount((unsigned)channels & 3u);
    if ((uint64_t)d.ng * d.ng * el >= lim) return false;
    if (((uint64_t)nph * dir_slot_stride + (uint64_t)d.planes * d.n) * el >= lim) return false;
    const StreamGeom g = stream_geom_of(kind, channels, mgroup, tile, d);
    return stream_fits(g) && stream_lds_bytes(g, batch) <= kLdsBytes;
}

// Blocks a CU holds of either kernel.  The waves per SIMD that their registers
// leave, by complex accumulators a thread (as compiled, or one less):
inline int update_waves(int kind, int channels, int ept, int mgroup) {
    const int accs = __builtin_popcount((unsigned)channels) * ept * mgroup;
    const bool pp = channels == CH_PP;           // no exchange and direct operands
    if (kind == 2) return (accs <= 4 ? 4 : accs <= 8 ? 3 : accs <= 32 ? 2 : 1) + (pp && accs <= 16 ? 1 : 0);
    if (accs <= 8) return pp && (kind == 0 || (mgroup == 4 && ept == 1)) ? 3 : 2;
    return accs <= (kind == 0 && ept == 1 ? 16 : 12) || (pp && accs <= 16) ? 2 : 1;
}
inline int stream_waves_of(int kind, int channels, int ept, int mgroup, bool nw64) {
    const int accs = __builtin_popcount((unsigned)channels) * ept * mgroup;
    const bool pp = channels == CH_PP, mixed = (channels & CH_PP) && !pp;
    int w;
    if (kind == 2) {
        w = accs <= 4 ? 5 : accs <= 8 ? 3 : accs <= 16 || (accs <= 24 && ept == 1) ? 2 : 1;
        if (nw64 && accs <= 16 && ept <= 2 && !mixed && w < 3) w = 3;
        return w + (pp && accs <= 16 && ept < 4 ? 1 : 0);
    }
    w = accs <= 4 ? 3 : accs <= 12 ? 2 : 1;
    if (nw64 && ept == 1 && accs <= 16) w = accs <= 8 ? 3 : 2;
    return w + (pp && accs <= 16 ? 1 : 0);
}
inline int stream_blocks(int kind, int channels, int ept, int mgroup, int tile, const Dims &d, int batch) {
    const size_t lds = stream_lds_bytes(stream_geom_of(kind, channels, mgroup, tile, d), batch);
    const int w = stream_waves_of(kind, channels, ept, mgroup, d.nw == 64 && tile == ept * 4), l = (int)(kLdsBytes / lds);
    return w < l ? w : l;
}
inline int update_blocks(int kind, int channels, int ept, int mgroup, int tile, const Dims &d) {
    const size_t lds = update_lds_bytes(kind, channels, tile, mgroup, d, 0);
    const int w = update_waves(kind, channels, ept, mgroup), l = (int)(kLdsBytes / (lds ? lds : 1));
    return w < l ? w : l;
}

// Whether the streamed kernel is the faster one of a default plan's launch of
// `batch` measurements (`groups` plane groups, `items` work tiles).  Both kernels
// were timed on 5125 random shapes (2x2 to 8x8, 8 to 256 frequencies, 2 to 16
// transfers, every channel set); update_kernel's time over this one's, median (5%
// lowest, 5% highest), in the order of the tests below:
//   fewer blocks a CU than update_kernel, nothing covers the copies' latency: plain
//     0.78 (0.52, 1.05), batched FP64 0.68 (0.55, 1.00), FP32 0.74 (0.49, 1.15);
//   as many or more and 64 frequencies, the geometry compiled in: 1.16 (1.00, 1.43);
//   more in a batched pass of over 512 tiles, two a CU: 1.20 (0.98, 1.50);
//   8 to 12 frequencies, runs of a line or two: 0.97 (0.79, 1.11);
//   plain: 1.04 (0.96, 1.17), but where plane groups are mostly empty, whose LDS is
//     a full one's, 0.96 (0.83, 1.05);
//   batched, three channels: 0.92 (0.73, 1.06);
//   one channel in FP64, or in FP32 with plane groups of 4: 1.05 (0.96, 1.24);
//   else groups that are mostly empty: 0.99 (0.88, 1.07); two channels in FP64: 1.05
//     (0.95, 1.34); FP32 passes of 8 measurements on: 1.07 (0.98, 1.31), of fewer, or
//     of PP beside a PH channel: 0.95 (0.87, 1.10).
inline bool stream_pays(int kind, int channels, int ept, int mgroup, int tile, const Dims &d, int batch, int groups,
                        int items) {
    const int mine = stream_blocks(kind, channels, ept, mgroup, tile, d, batch);
    const int theirs = update_blocks(kind, channels, ept, mgroup, tile, d);
    if (mine < theirs) return false;
    if (d.nw == 64 && tile == ept * 4) return true;
    if (kind != 0 && mine > theirs && items > 512) return true;
    const int nch = __builtin_popcount((unsigned)channels);
    const int64_t full = (int64_t)groups * mgroup;         // planes of full groups
    if (d.nw <= 12) return false;
    if (kind == 0) return (int64_t)d.planes * 100 > full * 27;
    if (nch == 3) return false;
    if (nch == 1 && (kind == 1 || mgroup == 4)) return true;
    if ((int64_t)d.planes * 100 <= full * 40) return false;
    return kind == 1 || (batch >= 8 && !((channels & CH_PP) && nch > 1));
}
// The streamed kernel among launch_update's variants (plans have G4_VARIANT_*).
constexpr int kVariantStreamed = 5;
hipError_t launch_update_stream(int kind, int channels, int ept, int mgroup, int nitems, const UpdateArgs &a,
                                hipStream_t s);

// Whether a G4_F_PACKED plan of passes of `batch` measurements leaves the packing
// out and runs the streamed kernel: packing G costs the same whatever the slice
// holds, and each element then serves few entries.  Both were timed on 7269 random
// shapes; packed time over streamed, median (5% lowest), of those below that stream
// and of those that pack:
//   PP alone                                        1.37 (0.97)   1.15 (0.98)
//   one PH channel, plane groups of 4               1.28 (1.03)   1.07 (0.80)
//     groups of 8, 64 frequencies (compiled in)     1.36 (1.04)   1.07 (0.77)
//     groups of 8, others                           1.34 (0.98)   0.92 (0.73)
//   several channels, 64 frequencies                1.46 (1.17)   1.21 (0.97)
//   magnetic and charge, others                     1.21 (0.91)   0.87 (0.62)
//   PH and PP, others                               1.17 (0.84)   0.90 (0.61)
//   three, others                                   1.15 (0.88)   0.91 (0.55)
// (the first lines pack above the plane counts to which streaming was tried), and
// long passes over less than 1 MB of G pack: few tiles, each waiting for its own
// copies (0.93, 0.72).  Streaming wants few plane groups (each reads its blocks of G
// again), two blocks a CU, and long passes, as more copies then hide behind sums.
inline bool stream_packed(int channels, int ept, int mgroup, int tile, const Dims &d, int batch, int groups) {
    if (batch >= 16 && 2.0 * d.ng * d.ng * 8 < 1e6) return false;
    const int nch = __builtin_popcount((unsigned)channels), p = d.planes;
    const int blocks = stream_blocks(2, channels, ept, mgroup, tile, d, batch);
    const bool pp = (channels & CH_PP) != 0, nw64 = d.nw == 64 && tile == ept * 4, two = blocks >= 2;
    if (nch == 1) {
        if (pp) return p < 32;
        if (mgroup == 4) return p < (batch <= 24 ? 32 : d.nc >= 16 ? 17 : 13);
        if (nw64) return p < (batch <= 24 ? 32 : 20);
        if (d.nw < 20 && blocks >= 3) return p < 24;
        return p < 4 || (two && groups <= 2 && (batch > 2 || d.nw < 20));
    }
    if (p * nch >= 24) return false;
    if (nw64) return true;
    if (!pp) {                                   // magnetic and charge
        if (p <= 2) return true;
        if (!two) return false;
        if (p <= 5) return batch >= 8 || d.nw >= 48;
        return groups == 1 || (groups == 2 && (d.nc < 16 || batch >= 32)) || d.nw >= 128 || (d.nw < 20 && blocks >= 3);
    }
    if (!two) return nch == 2 ? p <= 1 : mgroup == 8 && p <= 3;
    if (nch == 2) return p <= 5 || (groups == 1 && batch >= 8);
    return groups <= 2 && (p <= 4 || (mgroup == 8 && groups == 1 && (batch >= 8 || tile <= 7)));
}

}  // namespace g4
