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
__host__ __device__ constexpr bool stream_fits(const StreamGeom &g) {
    return stream_copies(g.cY) <= kStreamY && stream_copies(g.cZ) <= kStreamZ && stream_copies(g.cA) <= kStreamA &&
           stream_copies(g.cB) <= kStreamB;
}
inline size_t stream_lds_bytes(const StreamGeom &g) { return (size_t)2 * g.total * 16 + kMaxPassBatch * 8; }

// Whether the streamed kernel runs an update of the register-staged plans (its
// old kernel otherwise): magnetic, charge and PP, plane groups of 4 and 8, the
// rows per thread that are compiled; FP32 rows of G have to hold whole pairs of
// columns; copy offsets are 32-bit within a matrix and within a measurement's
// direct vectors; both buffers fit the LDS.  In FP64 two blocks per CU have to
// fit where plane groups are of 4: with one, three channels at 64 frequencies
// took 355 us against the old kernel's 271 (6 momenta of 3 planes, 16
// measurements); groups of 8 gain with one as well (691 against 990).
inline bool stream_runs(int kind, int channels, int ept, int mgroup, int tile, const Dims &d, int64_t dir_slot_stride) {
    if ((channels & ~7) || (mgroup != 4 && mgroup != 8)) return false;
    if (ept != 1 && ept != 2 && !(kind == 2 && ept == 4 && mgroup == 4)) return false;
    if (kind == 2 && d.ng % 2) return false;
    const uint64_t el = kind == 2 ? 8 : 16, lim = 1ull << 32;
    const int nph = __builtin_popcount((unsigned)channels & 3u);
    if ((uint64_t)d.ng * d.ng * el >= lim) return false;
    if (((uint64_t)nph * dir_slot_stride + (uint64_t)d.planes * d.n) * el >= lim) return false;
    const StreamGeom g = stream_geom(kind == 2 ? 2 : 1, d.nw, tile < d.nw ? tile : d.nw, mgroup, channels);
    return stream_fits(g) && stream_lds_bytes(g) <= (kind != 2 && mgroup == 4 ? 80 : 160) * 1024;
}
hipError_t launch_update_stream(int kind, int channels, int ept, int mgroup, int nitems, const UpdateArgs &a,
                                hipStream_t s);

// Small slices run their G4_F_PACKED plan on the streamed kernel: packing G costs
// the same whatever the slice holds, and each element then serves few entries.
// Packed against streamed, us per pass of 32 measurements (4x4, 64 frequencies):
// one channel of 8 planes 555 : 310, 16 planes 696 : 576, 24 planes 838 : 806,
// 30 planes equal; two channels of 8 planes 661 : 553, 16 planes 1023 : 1138;
// three channels of 4 planes 632 : 387, and of 8 planes at 6x6 and 32
// frequencies 1143 : 1480.
constexpr int kStreamPlanes = 32, kStreamPlaneChannels = 24;
inline bool stream_packed(int planes, int channels) {
    const int nch = __builtin_popcount((unsigned)channels);
    return nch == 1 ? planes < kStreamPlanes : planes * nch < kStreamPlaneChannels;
}

}  // namespace g4
