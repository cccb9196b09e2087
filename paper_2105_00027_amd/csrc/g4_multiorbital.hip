// Multi-orbital G4 accumulation for gfx950: every single-particle index
// carries an orbital label, so a G4 entry is (Q; K1, b1, b2; K2, b3, b4) and
// the array grows as nb^4 (the paper's motivating case for distributing G_t:
// Background section, "Memory-Bound Issue in DCA++").
//
// Per measurement b with weight s_b:
//   PH magnetic/charge  s_b [ (Gu -/+ Gd)(K1+Q b1, K1 b2) (Gu -/+ Gd)(K2 b3, K2+Q b4)
//                             - sum_s G_s(K2 b3, K1 b2) G_s(K1+Q b1, K2+Q b4) ]
//   PP up-down          s_b sum_s G_s(Q-K2 b4, Q-K1 b2) G_{-s}(K2 b3, K1 b1)
// G_sigma is (Ng nb) x (Ng nb), index (k*Nwg + n + Nw/2)*nb + b.  The slice is
// stored as documented: entry ((p*N + K2)*nb^2 + b3*nb + b4)*(N nb^2) +
// (K1*nb + b1)*nb + b2, complex128.
//
// Four orbitals in FP32 run on the matrix cores (mo_mfma_kernel), and magnetic
// and charge of two orbitals in one pass (mo_two_kernel); the rest as follows.
// A launch covers up to 32 measurements of one channel over up to 256 planes
// and keeps the sums over the measurements in registers, then reads, adds and
// writes each entry once.  For nb <= 8 (mo_rows_kernel) a thread owns one
// column (K1, b1, b2) of one (plane, K2) and all nb^2 rows (b3, b4): per
// measurement it loads the column's a = G(K1+Q b1, K1 b2) once and the nb
// exchange operands of each side (G(K2 b3, K1 b2) and G(K1+Q b1, K2+Q b4):
// one per b3, one per b4), both spins: 2 + 4 nb vector loads for nb^2 entry
// updates (18 for 16 at nb = 4) instead of eight per entry update; the nb^2
// values b = G(K2 b3, K2+Q b4) are
// the same for the whole block (a block covers one (plane, K2) row), which
// forms them once per launch into LDS.  Lanes run along the column, so each
// of the nb^2 output rows is written as one contiguous run.  Larger nb takes the
// one-thread-per-entry kernel (mo_kernel).  G elements come straight from
// global memory (L2-resident across a plane's rows).  Momenta are added on
// the lattice coordinates in the kernel (no tables).
#include "../../include/g4.h"
#include "g4_internal.hpp"

#include <algorithm>
#include <cstdio>
#include <type_traits>
#include <vector>

namespace g4 {
namespace {

constexpr int kMoPlanes = 256;   // planes per launch
// measurements per launch: 32 keeps a launch's G (2 x 32 x 2.5 MB for the
// 2x2 cluster with 4 orbitals) in the last-level cache; 64 per launch took
// 3.27 ms per 64 measurements there, 32 3.18 ms
constexpr int kMoBatch = 32;
// measurements per launch of mo_mfma_kernel, which sums kMoBatch at a time and
// those sums in a second set of registers, their roundings kept (in LDS): one trip
// of the accumulator to memory and back per 128 measurements
constexpr int kMoLong = 128;

struct MoArgs {
    const void *gu, *gd;
    int64_t g_stride;            // elements between matrices
    double2 *acc;                // slice of this launch's first plane
    double2 *acc2;               // mo_two_kernel with both PH channels: the charge slice
    int64_t total;               // entries of this launch
    int64_t side;                // N nb^2
    int lx, ly, nw, nwg, nb, ngb, channel, batch, planes;
    int matrix;                  // mo_mfma_kernel runs (mo_uses_mfma)
    int2 qm[kMoPlanes];          // (q, m) per plane of the launch
    double sign[kMoLong];
};

template <typename R> struct MoCx;
template <> struct MoCx<double> { using V = double2; };
template <> struct MoCx<float> { using V = float2; };

template <typename V>
__device__ __forceinline__ V mo_ld(const V *g, int64_t i) { return g[i]; }

template <typename R>
__global__ __launch_bounds__(256) void mo_kernel(MoArgs a) {
    using V = typename MoCx<R>::V;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= a.total) return;
    const int nb = a.nb, nw = a.nw, nwg = a.nwg, lx = a.lx, ly = a.ly;
    const int64_t side = a.side, ngb = a.ngb;
    const int64_t col = e % side, rr = e / side;
    const int p = (int)(rr / side);
    const int64_t row = rr % side;
    const int K1 = (int)(col / (nb * nb)), b1 = (int)((col / nb) % nb), b2 = (int)(col % nb);
    const int K2 = (int)(row / (nb * nb)), b3 = (int)((row / nb) % nb), b4 = (int)(row % nb);
    const int q = a.qm[p].x, m = a.qm[p].y;
    const int k1 = K1 / nw, i1 = K1 % nw, k2 = K2 / nw, i2 = K2 % nw;
    const int qx = q % lx, qy = q / lx;
    auto kadd = [&](int k) { return (k % lx + qx) % lx + lx * ((k / lx + qy) % ly); };
    auto ksub = [&](int k) { return (qx - k % lx + lx) % lx + lx * ((qy - k / lx + ly) % ly); };
    // G row/column of (window index, orbital)
    auto gi = [&](int w, int b) { return (int64_t)w * nb + b; };
    const V *gu = static_cast<const V *>(a.gu);
    const V *gd = static_cast<const V *>(a.gd);
    R sr = 0, si = 0;
    if (a.channel == CH_PP) {
        const int w_qk1 = ksub(k1) * nwg + (m + nw - 1 - i1), w_qk2 = ksub(k2) * nwg + (m + nw - 1 - i2);
        const int64_t iz = gi(w_qk2, b4) * ngb + gi(w_qk1, b2);          // G(Q-K2 b4, Q-K1 b2)
        const int64_t ix = gi(k2 * nwg + i2, b3) * ngb + gi(k1 * nwg + i1, b1);   // G(K2 b3, K1 b1)
        for (int b = 0; b < a.batch; ++b) {
            const int64_t o = (int64_t)b * a.g_stride;
            const V zu = mo_ld(gu, o + iz), zd = mo_ld(gd, o + iz), xu = mo_ld(gu, o + ix), xd = mo_ld(gd, o + ix);
            const R s = (R)a.sign[b];
            const R tr = zu.x * xd.x - zu.y * xd.y + zd.x * xu.x - zd.y * xu.y;
            const R ti = zu.x * xd.y + zu.y * xd.x + zd.x * xu.y + zd.y * xu.x;
            sr += s * tr;
            si += s * ti;
        }
    } else {
        const R sg = a.channel == CH_MAG ? (R)-1 : (R)1;
        const int w_k1 = k1 * nwg + i1, w_k2 = k2 * nwg + i2;
        const int w_k1q = kadd(k1) * nwg + i1 + m, w_k2q = kadd(k2) * nwg + i2 + m;
        const int64_t i_a = gi(w_k1q, b1) * ngb + gi(w_k1, b2);    // G(K1+Q b1, K1 b2)
        const int64_t i_b = gi(w_k2, b3) * ngb + gi(w_k2q, b4);    // G(K2 b3, K2+Q b4)
        const int64_t i_x = gi(w_k2, b3) * ngb + gi(w_k1, b2);     // G(K2 b3, K1 b2)
        const int64_t i_y = gi(w_k1q, b1) * ngb + gi(w_k2q, b4);   // G(K1+Q b1, K2+Q b4)
        for (int b = 0; b < a.batch; ++b) {
            const int64_t o = (int64_t)b * a.g_stride;
            const V au = mo_ld(gu, o + i_a), ad = mo_ld(gd, o + i_a);
            const V bu = mo_ld(gu, o + i_b), bd = mo_ld(gd, o + i_b);
            const V xu = mo_ld(gu, o + i_x), xd = mo_ld(gd, o + i_x);
            const V yu = mo_ld(gu, o + i_y), yd = mo_ld(gd, o + i_y);
            const R ar = au.x + sg * ad.x, ai = au.y + sg * ad.y;
            const R br = bu.x + sg * bd.x, bi = bu.y + sg * bd.y;
            const R tr = ar * br - ai * bi - (xu.x * yu.x - xu.y * yu.y) - (xd.x * yd.x - xd.y * yd.y);
            const R ti = ar * bi + ai * br - (xu.x * yu.y + xu.y * yu.x) - (xd.x * yd.y + xd.y * yd.x);
            const R s = (R)a.sign[b];
            sr += s * tr;
            si += s * ti;
        }
    }
    double2 *pa = a.acc + e;
    double2 v = *pa;
    v.x += (double)sr;
    v.y += (double)si;
    *pa = v;
}

// Thread (plane p, K2, column (K1, b1, b2)) for all (b3, b4); NB = nb.  A
// block covers up to 256 columns of one (plane, K2) row, so the row-side
// direct operand b(Q; K2 b3, K2+Q b4) of every measurement is the same for
// the whole block: the block forms it once per launch, weight and spin
// combination folded in, into LDS, and the loop reads it from there.  The
// weight of the exchange term is folded into G(K2 b3, K1 b2) as it arrives,
// so each entry update is the twelve FMAs of its three complex products.
template <typename R, int NB>
__global__ __launch_bounds__(256) void mo_rows_kernel(MoArgs a) {
    using V = typename MoCx<R>::V;
    __shared__ V bsh[kMoBatch][NB * NB];
    const int64_t side = a.side;                       // N NB^2
    const int64_t n = side / (NB * NB);
    const int64_t bpr = (side + 255) / 256;            // blocks per (plane, K2) row
    const int64_t rowi = blockIdx.x / bpr;
    const int64_t col = (blockIdx.x % bpr) * 256 + threadIdx.x;
    const bool act = col < side;
    const int K2 = (int)(rowi % n), p = (int)(rowi / n);
    const int nw = a.nw, nwg = a.nwg, lx = a.lx, ly = a.ly;
    const int64_t ngb = a.ngb;
    const int64_t cl = act ? col : 0;
    const int K1 = (int)(cl / (NB * NB)), b1 = (int)((cl / NB) % NB), b2 = (int)(cl % NB);
    const int q = a.qm[p].x, m = a.qm[p].y;
    const int k1 = K1 / nw, i1 = K1 % nw, k2 = K2 / nw, i2 = K2 % nw;
    const int qx = q % lx, qy = q / lx;
    auto kadd = [&](int k) { return (k % lx + qx) % lx + lx * ((k / lx + qy) % ly); };
    auto ksub = [&](int k) { return (qx - k % lx + lx) % lx + lx * ((qy - k / lx + ly) % ly); };
    auto gi = [&](int w, int b) { return (int64_t)w * NB + b; };
    const V *gu = static_cast<const V *>(a.gu);
    const V *gd = static_cast<const V *>(a.gd);
    R sr[NB][NB], si[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) sr[i][j] = si[i][j] = 0;
    // Operands of one measurement, loaded one measurement ahead into the other
    // of two register sets (the loop alternates them, so nothing is copied).
    // Every product is added by a plain FMA: imaginary parts that enter with a
    // minus sign are negated once per measurement.
    struct Ops {
        V au, ad;
        V xu[NB], xd[NB], yu[NB], yd[NB];
    };
    auto run = [&](auto load, auto compute) __attribute__((always_inline)) {
        if (!act || a.batch == 0) return;
        Ops o0, o1;
        load(0, o0);
        int b = 0;
        for (; b + 1 < a.batch; b += 2) {
            load(b + 1, o1);
            compute(b, o0);
            load(min(b + 2, a.batch - 1), o0);
            compute(b + 1, o1);
        }
        if (b < a.batch) compute(b, o0);
    };
    if (a.channel == CH_PP) {
        const int w_qk1 = ksub(k1) * nwg + (m + nw - 1 - i1), w_qk2 = ksub(k2) * nwg + (m + nw - 1 - i2);
        const int w_k1 = k1 * nwg + i1, w_k2 = k2 * nwg + i2;
        const int64_t iz0 = gi(w_qk2, 0) * ngb + gi(w_qk1, b2);   // G(Q-K2 b4, Q-K1 b2) at b4 = 0 (yu, yd)
        const int64_t ix0 = gi(w_k2, 0) * ngb + gi(w_k1, b1);     // G(K2 b3, K1 b1) at b3 = 0 (xu, xd)
        auto load = [&](int b, Ops &o) __attribute__((always_inline)) {
            const V *pu = gu + (int64_t)b * a.g_stride, *pd = gd + (int64_t)b * a.g_stride;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                o.yu[j] = pu[iz0 + j * ngb];
                o.yd[j] = pd[iz0 + j * ngb];
                o.xu[j] = pu[ix0 + j * ngb];
                o.xd[j] = pd[ix0 + j * ngb];
            }
        };
        auto compute = [&](int b, const Ops &o) __attribute__((always_inline)) {
            const R s = (R)a.sign[b];
            // s G(Q-K2 b4, Q-K1 b2) and its negated imaginary part
            R zur[NB], zui[NB], zun[NB], zdr[NB], zdi[NB], zdn[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                zur[j] = s * o.yu[j].x;
                zui[j] = s * o.yu[j].y;
                zun[j] = -zui[j];
                zdr[j] = s * o.yd[j].x;
                zdi[j] = s * o.yd[j].y;
                zdn[j] = -zdi[j];
            }
#pragma unroll
            for (int b3 = 0; b3 < NB; ++b3)
#pragma unroll
                for (int b4 = 0; b4 < NB; ++b4) {
                    R r = sr[b3][b4], i = si[b3][b4];
                    r += zur[b4] * o.xd[b3].x;
                    r += zun[b4] * o.xd[b3].y;
                    r += zdr[b4] * o.xu[b3].x;
                    r += zdn[b4] * o.xu[b3].y;
                    i += zur[b4] * o.xd[b3].y;
                    i += zui[b4] * o.xd[b3].x;
                    i += zdr[b4] * o.xu[b3].y;
                    i += zdi[b4] * o.xu[b3].x;
                    sr[b3][b4] = r;
                    si[b3][b4] = i;
                }
        };
        run(load, compute);
    } else {
        const R sg = a.channel == CH_MAG ? (R)-1 : (R)1;
        const int w_k1 = k1 * nwg + i1, w_k2 = k2 * nwg + i2;
        const int w_k1q = kadd(k1) * nwg + i1 + m, w_k2q = kadd(k2) * nwg + i2 + m;
        // s_b (Gu -/+ Gd)(K2 b3, K2+Q b4) of every measurement of the launch
        for (int t = threadIdx.x; t < a.batch * NB * NB; t += 256) {
            const int b = t / (NB * NB), j = t % (NB * NB);
            const int64_t ib = (int64_t)b * a.g_stride + gi(w_k2, j / NB) * ngb + gi(w_k2q, j % NB);
            const V u = gu[ib], d = gd[ib];
            const R s = (R)a.sign[b];
            bsh[b][j] = V{s * (u.x + sg * d.x), s * (u.y + sg * d.y)};
        }
        __syncthreads();
        const int64_t ia = gi(w_k1q, b1) * ngb + gi(w_k1, b2);    // G(K1+Q b1, K1 b2)
        const int64_t ix0 = gi(w_k2, 0) * ngb + gi(w_k1, b2);     // G(K2 b3, K1 b2) at b3 = 0
        const int64_t iy0 = gi(w_k1q, b1) * ngb + gi(w_k2q, 0);   // G(K1+Q b1, K2+Q b4) at b4 = 0
        auto load = [&](int b, Ops &o) __attribute__((always_inline)) {
            const V *pu = gu + (int64_t)b * a.g_stride, *pd = gd + (int64_t)b * a.g_stride;
            o.au = pu[ia];
            o.ad = pd[ia];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                o.xu[j] = pu[ix0 + j * ngb];
                o.xd[j] = pd[ix0 + j * ngb];
                o.yu[j] = pu[iy0 + j];
                o.yd[j] = pd[iy0 + j];
            }
        };
        auto compute = [&](int b, const Ops &o) __attribute__((always_inline)) {
            const R s = (R)a.sign[b];
            const R ar = o.au.x + sg * o.ad.x, ai = o.au.y + sg * o.ad.y, an = -ai;
            // -s G(K2 b3, K1 b2) (the exchange's minus and weight), and G(K1+Q b1,
            // K2+Q b4) with its negated imaginary part
            R xur[NB], xui[NB], xdr[NB], xdi[NB], yun[NB], ydn[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                xur[j] = -s * o.xu[j].x;
                xui[j] = -s * o.xu[j].y;
                xdr[j] = -s * o.xd[j].x;
                xdi[j] = -s * o.xd[j].y;
                yun[j] = -o.yu[j].y;
                ydn[j] = -o.yd[j].y;
            }
#pragma unroll
            for (int b3 = 0; b3 < NB; ++b3)
#pragma unroll
                for (int b4 = 0; b4 < NB; ++b4) {
                    const V bb = bsh[b][b3 * NB + b4];
                    R r = sr[b3][b4], i = si[b3][b4];
                    r += ar * bb.x;
                    r += an * bb.y;
                    r += xur[b3] * o.yu[b4].x;
                    r += xui[b3] * yun[b4];
                    r += xdr[b3] * o.yd[b4].x;
                    r += xdi[b3] * ydn[b4];
                    i += ar * bb.y;
                    i += ai * bb.x;
                    i += xur[b3] * o.yu[b4].y;
                    i += xui[b3] * o.yu[b4].x;
                    i += xdr[b3] * o.yd[b4].y;
                    i += xdi[b3] * o.yd[b4].x;
                    sr[b3][b4] = r;
                    si[b3][b4] = i;
                }
        };
        run(load, compute);
    }
    if (!act) return;
    // entry ((p*N + K2)*NB^2 + b3*NB + b4)*side + col
#pragma unroll
    for (int b3 = 0; b3 < NB; ++b3)
#pragma unroll
        for (int b4 = 0; b4 < NB; ++b4) {
            double2 *pa = a.acc + (((int64_t)p * n + K2) * (NB * NB) + b3 * NB + b4) * side + col;
            double2 v = *pa;
            v.x += (double)sr[b3][b4];
            v.y += (double)si[b3][b4];
            *pa = v;
        }
}

// Two orbitals, PH: magnetic, charge, or both from one pass over the operands (MASK
// of CH_MAG | CH_CHG), for two neighbouring K2.  The rows kernel is bound by the
// cache lines its loads touch: lanes run along (K1, b1, b2), and the operands with
// K1+Q in their row index lie one row of G apart (the a and y loads, 192 of 224
// line accesses of a wave, measurement and channel).  Here both channels use the
// same operands, the lanes of b2 = 0 and 1 load one b4 of y each and swap, and a
// serves two K2: 256 line accesses per 16 entries of a thread instead of 896.
// 3x2 cluster, 2 orbitals, Nw = 26, 15 planes, 48 measurements, FP64, all three
// channels: 4.80 -> 2.23 ms a call.
template <typename R, int MASK>
__global__ __launch_bounds__(256) void mo_two_kernel(MoArgs a) {
    using V = typename MoCx<R>::V;
    constexpr int NC = MASK == 3 ? 2 : 1;
    constexpr int LB = sizeof(R) == 8 ? kMoLong : kMoBatch;
    __shared__ V bsh[LB][2][NC][4];
    const int64_t side = a.side;                       // 4 N
    const int n = (int)(side / 4), n2 = n / 2;
    const int bpr = (int)((side + 255) / 256);         // blocks per (plane, pair of K2)
    const int64_t rowi = blockIdx.x / bpr;
    const int64_t col = (int64_t)(blockIdx.x % bpr) * 256 + threadIdx.x;
    const bool act = col < side;
    const int K2 = (int)(rowi % n2) * 2, p = (int)(rowi / n2);
    const int nw = a.nw, nwg = a.nwg, lx = a.lx, ly = a.ly;
    const int64_t ngb = a.ngb;
    const int cl = act ? (int)col : 0;
    const int K1 = cl >> 2, b1 = (cl >> 1) & 1, b2 = cl & 1;
    const int q = a.qm[p].x, m = a.qm[p].y;
    const int k1 = K1 / nw, i1 = K1 % nw, k2 = K2 / nw, i2 = K2 % nw;   // K2 + 1 has the same momentum (nw even)
    const int qx = q % lx, qy = q / lx;
    auto kadd = [&](int k) { return (k % lx + qx) % lx + lx * ((k / lx + qy) % ly); };
    const int w_k1 = k1 * nwg + i1, w_k2 = k2 * nwg + i2;
    const int w_k1q = kadd(k1) * nwg + i1 + m, w_k2q = kadd(k2) * nwg + i2 + m;
    const V *gu = static_cast<const V *>(a.gu), *gd = static_cast<const V *>(a.gd);
    // s_b (Gu -/+ Gd)(K2 b3, K2+Q b4) of every measurement, both K2
    for (int t = threadIdx.x; t < a.batch * 8; t += 256) {
        const int b = t >> 3, j = (t >> 2) & 1, e = t & 3;
        const int64_t ib = (int64_t)b * a.g_stride + ((int64_t)(w_k2 + j) * 2 + (e >> 1)) * ngb + (w_k2q + j) * 2 + (e & 1);
        const V u = gu[ib], d = gd[ib];
        const R s = (R)a.sign[b];
        if (MASK & 1) bsh[b][j][0][e] = V{s * (u.x - d.x), s * (u.y - d.y)};
        if (MASK & 2) bsh[b][j][NC - 1][e] = V{s * (u.x + d.x), s * (u.y + d.y)};
    }
    __syncthreads();
    const int64_t ia = ((int64_t)w_k1q * 2 + b1) * ngb + w_k1 * 2 + b2;   // G(K1+Q b1, K1 b2)
    const int64_t ix = ((int64_t)w_k2 * 2) * ngb + w_k1 * 2 + b2;         // G(K2 b3, K1 b2) at b3 = 0
    const int64_t iy = ((int64_t)w_k1q * 2 + b1) * ngb + w_k2q * 2 + b2;  // G(K1+Q b1, K2+Q b4) at b4 = b2
    R sr[NC][2][2][2], si[NC][2][2][2];                // [channel][K2][b3][b4]
#pragma unroll
    for (int e = 0; e < NC * 8; ++e) (&sr[0][0][0][0])[e] = (&si[0][0][0][0])[e] = 0;
    struct Ops {
        V au, ad, xu[2][2], xd[2][2], yu[2], yd[2];    // x [K2][b3], y [K2]: this lane's b4
    };
    auto load = [&](int b, Ops &o) __attribute__((always_inline)) {
        const V *pu = gu + (int64_t)b * a.g_stride, *pd = gd + (int64_t)b * a.g_stride;
        o.au = pu[ia];
        o.ad = pd[ia];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            o.yu[j] = pu[iy + 2 * j];
            o.yd[j] = pd[iy + 2 * j];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                o.xu[j][c] = pu[ix + (2 * j + c) * ngb];
                o.xd[j][c] = pd[ix + (2 * j + c) * ngb];
            }
        }
    };
    // the neighbour lane's value (lanes 2i and 2i + 1 trade)
    auto other = [](R v) __attribute__((always_inline)) {
        if constexpr (sizeof(R) == 4) {
            return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
        } else {
            return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0xB1, 0xF, 0xF, true),
                                    __builtin_amdgcn_mov_dpp(__double2loint(v), 0xB1, 0xF, 0xF, true));
        }
    };
    auto compute = [&](int b, const Ops &o) __attribute__((always_inline)) {
        const R s = (R)a.sign[b];
        V av[NC];
        if (MASK & 1) av[0] = V{o.au.x - o.ad.x, o.au.y - o.ad.y};
        if (MASK & 2) av[NC - 1] = V{o.au.x + o.ad.x, o.au.y + o.ad.y};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const V ou{other(o.yu[j].x), other(o.yu[j].y)}, od{other(o.yd[j].x), other(o.yd[j].y)};
            // b4 = 0, 1
            const V yu[2] = {b2 ? ou : o.yu[j], b2 ? o.yu[j] : ou}, yd[2] = {b2 ? od : o.yd[j], b2 ? o.yd[j] : od};
#pragma unroll
            for (int b3 = 0; b3 < 2; ++b3) {
                const R xur = -s * o.xu[j][b3].x, xui = -s * o.xu[j][b3].y, xdr = -s * o.xd[j][b3].x, xdi = -s * o.xd[j][b3].y;
#pragma unroll
                for (int b4 = 0; b4 < 2; ++b4) {
                    // the exchange sum, shared by the channels
                    R er = xur * yu[b4].x, ei = xur * yu[b4].y;
                    er = fma(-xui, yu[b4].y, er);
                    ei = fma(xui, yu[b4].x, ei);
                    er = fma(xdr, yd[b4].x, er);
                    ei = fma(xdr, yd[b4].y, ei);
                    er = fma(-xdi, yd[b4].y, er);
                    ei = fma(xdi, yd[b4].x, ei);
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const V bb = bsh[b][j][c][b3 * 2 + b4];
                        R r = sr[c][j][b3][b4], i = si[c][j][b3][b4];
                        r = fma(av[c].x, bb.x, r);
                        r = fma(-av[c].y, bb.y, r);
                        i = fma(av[c].x, bb.y, i);
                        i = fma(av[c].y, bb.x, i);
                        sr[c][j][b3][b4] = r + er;
                        si[c][j][b3][b4] = i + ei;
                    }
                }
            }
        }
    };
    if (a.batch > 0) {
        Ops o0, o1;                                    // one measurement ahead, in turn
        load(0, o0);
        int b = 0;
        for (; b + 1 < a.batch; b += 2) {
            load(b + 1, o1);
            compute(b, o0);
            load(min(b + 2, a.batch - 1), o0);
            compute(b + 1, o1);
        }
        if (b < a.batch) compute(b, o0);
    }
    if (!act) return;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double2 *pa = (c == NC - 1 && MASK == 3 ? a.acc2 : a.acc) + (((int64_t)p * n + K2 + j) * 4 + e) * side + col;
                double2 v = *pa;
                v.x += (double)sr[c][j][e >> 1][e & 1];
                v.y += (double)si[c][j][e >> 1][e & 1];
                *pa = v;
            }
}

constexpr int kMoTk = 4;         // K2 of a wave of mo_mfma_kernel
// its dynamic LDS: the low parts of the sums, only where a launch has more than one part
size_t mo_mfma_lds(int batch, int tq) { return batch > kMoBatch ? (size_t)256 * kMoTk * tq * 2 * 16 : 0; }

// Four orbitals, FP32: the orbital labels of one (Q, K1, K2) make the exchange
// (and PP) term a 16 x 16 outer product summed over measurements and spins,
//   PH  [(b1, b4), (b3, b2)] += G_s(K1+Q b1, K2+Q b4) (-s_b G_s(K2 b3, K1 b2)),
//   PP  [(b2, b4), (b3, b1)] += G_s(Q-K2 b4, Q-K1 b2) ( s_b G_{-s}(K2 b3, K1 b1)),
// so it runs on v_mfma_f32_16x16x4f32, whose four k slots are four measurements
// of one spin: four instructions (Re Re, Im Re, Im Im, Re Im) a spin.
// Result register r of lane l is row 4(l/16) + r, column l % 16: the lane holds
// (h = b1 or b2; b3, c = b2 or b1) of all four b4.  The PH direct term
// a(b1, b2) b(b3, b4) is sixteen 4 x 4 outer products (b1, b3) and lands in the
// same registers through v_mfma_f32_4x4x1_16b_f32, whose block l/4 is (b1, b3),
// column l % 4 = b2 and register row b4.  Both run at the full FP32 matrix rate
// (twice the vector one): 96 matrix cycles per 256 entries and measurement.
// A wave takes TQ planes x 4 K2 of one K1 (8 accumulator registers a tile, and 8
// for the sums of every 32 measurements; what adding those rounds away is kept as
// a second float in LDS, 64 KB a block of two planes and still two blocks a CU,
// and joins the sum in the FP64 accumulator: a launch of 128 measurements gives
// what four of 32 give): the column operand G(K2, K1) is loaded
// once for its planes, the row operand once a tile, straight into the lanes that
// multiply it; each is replaced by the next step's (four measurements, one spin)
// as soon as it has been used, a whole step ahead.
// The block's four waves are four neighbouring K1; the direct operands of its
// 4 K1, 4 K2 and TQ planes are formed once in LDS, four measurements at a time.
// The 2x2 cluster, Nw = 32, 16 planes, 256 measurements: 13.0 ms on the vector
// units (eight launches, 30 TFLOP/s), here 7.2 ms (57 TFLOP/s; 2.7 ms at the rate
// of a large FP32 product).  What is left is the operands' way from L2: runs of
// four elements (32 bytes); with the row operand always in L1 5.1 ms.
template <int TQ, bool PP>
__global__ __launch_bounds__(256, 2) void mo_mfma_kernel(MoArgs a) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int NB = 4, TK = kMoTk;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    f4 *const low = reinterpret_cast<f4 *>(smem_raw) + threadIdx.x;   // [K2][plane][re, im], 256 threads apart
    __shared__ int win1[4], win2[TK], pl1[4][TQ], pl2[TK][TQ];      // window indices of K and of K+Q (PP: Q-K)
    __shared__ float wt[kMoLong];                                   // weights, zeros past the batch
    __shared__ float2 Ash[4][64 * TQ], Bsh[4][64 * TQ];            // [measurement][K of four][plane][orbitals]
    const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ngb = a.ngb;
    const int n = (int)(a.side / (NB * NB));
    // Each XCD takes a contiguous run of squares of 8 x 8 blocks (32 K1 x 32 K2,
    // what its CUs hold at once), a square's plane groups one after another: the
    // squares share rows and columns of G in its L2 (runs of all K1 at 8 K2 read
    // 2.3 times the lines).  Squares past the last K are cut, so that every XCD
    // has the same number of blocks (40 K, 16 planes, 4 measurements: 137 -> 104 us).
    const int t4 = (n + 3) / 4, gq = (a.planes + TQ - 1) / TQ;
    int wk = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    if (wk >= t4 * t4 * gq) return;
    const int band = wk / (8 * t4 * gq), bh = min(8, t4 - 8 * band);
    wk -= band * 8 * t4 * gq;
    const int sq = wk / (8 * bh * gq), bw = min(8, t4 - 8 * sq);
    wk -= sq * 8 * bh * gq;
    const int pb = wk / (bh * bw) * TQ, in = wk % (bh * bw);
    const int k1b = (sq * 8 + in % bw) * 4, k2b = (band * 8 + in / bw) * 4;
    // past the end the last K, plane and measurement repeat: loaded, never used
    if (tid < kMoLong) wt[tid] = tid < a.batch ? (float)a.sign[tid] : 0.f;
    if (tid < 4 * (TQ + 1) * 2) {
        const int side2 = tid >= 4 * (TQ + 1), e = tid - side2 * 4 * (TQ + 1), j = e / (TQ + 1), t = e % (TQ + 1);
        const int nw = a.nw, nwg = a.nwg, lx = a.lx, ly = a.ly;
        const int K = min((side2 ? k2b : k1b) + j, n - 1), k = K / nw, i = K % nw;
        if (t == TQ) {
            (side2 ? win2 : win1)[j] = k * nwg + i;
        } else {
            const int2 qm = a.qm[min(pb + t, a.planes - 1)];
            const int kx = k % lx, ky = k / lx, qx = qm.x % lx, qy = qm.x / lx;
            (side2 ? pl2 : pl1)[j][t] =
                PP ? ((qx - kx + lx) % lx + lx * ((qy - ky + ly) % ly)) * nwg + qm.y + nw - 1 - i
                   : ((kx + qx) % lx + lx * ((ky + qy) % ly)) * nwg + i + qm.y;
        }
    }
    __syncthreads();
    const int hi = (l >> 2) & 3, lo = l & 3;          // row operand (h, b4) and column operand (b3, c) of lane l % 16
    const unsigned gs = (unsigned)(a.g_stride * 8);   // four matrices below 2^32 bytes (launch_mo)
    // byte offsets from a step's first matrix: this lane's measurement, its element
    unsigned xo[TK], yo[TK][TQ];
#pragma unroll
    for (int j = 0; j < TK; ++j) {
        xo[j] = (unsigned)((win2[j] * NB + hi) * ngb + win1[w] * NB + lo) * 8;
#pragma unroll
        for (int t = 0; t < TQ; ++t)
            yo[j][t] = (unsigned)(PP ? (pl2[j][t] * NB + lo) * ngb + pl1[w][t] * NB + hi
                                     : (pl1[w][t] * NB + hi) * ngb + pl2[j][t] * NB + lo) * 8;
    }
    const int par = l >> 4;
    f4 re[TK][TQ], im[TK][TQ], rs[TK][TQ], is[TK][TQ];   // sums of up to 32 measurements, and of those sums
#pragma unroll
    for (int j = 0; j < TK; ++j)
#pragma unroll
        for (int t = 0; t < TQ; ++t) re[j][t] = im[j][t] = rs[j][t] = is[j][t] = f4{0.f, 0.f, 0.f, 0.f};

    // direct operands: a thread forms one (K of four, plane, orbital pair) of each side; threads past them repeat
    const int sid = tid % (64 * TQ);
    const int sk = sid / (TQ * 16), st = (sid / 16) % TQ, se = sid & 15;
    unsigned ao = 0, bo = 0;
    if (!PP) {
        ao = (unsigned)((pl1[sk][st] * NB + (se >> 2)) * ngb + win1[sk] * NB + (se & 3)) * 8;
        bo = (unsigned)((win2[sk] * NB + (se >> 2)) * ngb + pl2[sk][st] * NB + (se & 3)) * 8;
    }
    const float sg = a.channel == CH_MAG ? -1.f : 1.f;
    const char *const gu = static_cast<const char *>(a.gu), *const gd = static_cast<const char *>(a.gd);
    auto at = [](const char *b, unsigned o) __attribute__((always_inline)) { return *reinterpret_cast<const float2 *>(b + o); };
    float2 x[2][TK], y[2][TK][TQ], du[4], dd[4];      // [spin]
    // a step's operands: uniform base, this lane's measurement (the last one past the batch)
    auto lane_off = [&](int b) { return (unsigned)min(par, a.batch - 1 - b) * gs; };
    // this thread's element of one side's direct operands, four measurements
    auto load_direct = [&](int b, unsigned o) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const char *const u = gu + (int64_t)min(b + v, a.batch - 1) * gs;
            du[v] = at(u, o);
            dd[v] = at(u + (gd - gu), o);
        }
    };
    auto keep_direct = [&](int b, bool first) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool live = b + v < a.batch;
            const float f = first ? wt[b + v] : 1.f;  // the weight goes into a
            const float2 d{f * (du[v].x + sg * dd[v].x), f * (du[v].y + sg * dd[v].y)};
            (first ? Ash : Bsh)[v][sid] = live ? d : float2{0.f, 0.f};
        }
    };
    unsigned mine = lane_off(0);                      // folded into the offsets; changes for the last step only
#pragma unroll
    for (int j = 0; j < TK; ++j) {
        xo[j] += mine;
#pragma unroll
        for (int t = 0; t < TQ; ++t) yo[j][t] += mine;
    }
    // in the order in which the loop waits for them
#pragma unroll
    for (int spin = 0; spin < 2; ++spin) {
#pragma unroll
        for (int j = 0; j < TK; ++j) x[spin][j] = at((spin != 0) != PP ? gd : gu, xo[j]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
#pragma unroll
            for (int j = 0; j < TK; ++j) y[spin][j][t] = at(spin ? gd : gu, yo[j][t]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    for (int b = 0; b < a.batch; b += 4) {
        // an absent measurement multiplies zeros by zeros
        const bool live = b + par < a.batch;
        const float f = PP ? wt[b + par] : -wt[b + par];
#pragma unroll
        for (int spin = 0; spin < 2; ++spin) {
            if (!PP) load_direct(b, spin ? bo : ao);
            // the step after this one (the last loads its own again)
            const int nb = b + 4 < a.batch ? b + 4 : b;
            const char *const nu = gu + (int64_t)nb * gs, *const nd = gd + (int64_t)nb * gs;
            const char *const ny = spin ? nd : nu, *const nx = (spin != 0) != PP ? nd : nu;
            const unsigned move = spin == 0 ? lane_off(nb) - mine : 0u;
            mine += move;
            float xr[TK], xi[TK], xn[TK];
#pragma unroll
            for (int j = 0; j < TK; ++j) {
                xr[j] = live ? f * x[spin][j].x : 0.f;
                xi[j] = live ? f * x[spin][j].y : 0.f;
                xn[j] = -xi[j];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < TK; ++j) x[spin][j] = at(nx, xo[j] += move);
            // a plane's four K2 lie side by side in the rows of G: they are loaded
            // one right after another, so that the first brings the line for all
#pragma unroll
            for (int t = 0; t < TQ; ++t) {
                float yr[TK], yi[TK];
#pragma unroll
                for (int j = 0; j < TK; ++j) {
                    yr[j] = live ? y[spin][j][t].x : 0.f;
                    yi[j] = live ? y[spin][j][t].y : 0.f;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < TK; ++j) y[spin][j][t] = at(ny, yo[j][t] += move);
#pragma unroll
                for (int j = 0; j < TK; ++j) re[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(yr[j], xr[j], re[j][t], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < TK; ++j) im[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(yi[j], xr[j], im[j][t], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < TK; ++j) re[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(yi[j], xn[j], re[j][t], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < TK; ++j) im[j][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(yr[j], xi[j], im[j][t], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!PP) keep_direct(b, spin == 0);
        }
        if (!PP) {
            __syncthreads();                          // the four measurements' direct operands are in LDS
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int t = 0; t < TQ; ++t) {
                    const float2 av = Ash[v][(w * TQ + t) * 16 + (l >> 4) * 4 + lo];
                    float2 bv[TK];
#pragma unroll
                    for (int j = 0; j < TK; ++j) bv[j] = Bsh[v][(j * TQ + t) * 16 + (l & 15)];
#pragma unroll
                    for (int j = 0; j < TK; ++j) re[j][t] = __builtin_amdgcn_mfma_f32_4x4x1f32(bv[j].x, av.x, re[j][t], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < TK; ++j) im[j][t] = __builtin_amdgcn_mfma_f32_4x4x1f32(bv[j].x, av.y, im[j][t], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < TK; ++j) re[j][t] = __builtin_amdgcn_mfma_f32_4x4x1f32(-bv[j].y, av.y, re[j][t], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < TK; ++j) im[j][t] = __builtin_amdgcn_mfma_f32_4x4x1f32(bv[j].y, av.x, im[j][t], 0, 0, 0);
                }
            __syncthreads();                          // read: the next four's may follow
        }
        if ((b + 4) % kMoBatch == 0 || b + 4 >= a.batch) {
            const int part = b / kMoBatch;
            // sum + x, its rounding error added to the low part (Knuth's two-sum)
            auto add = [&](f4 &sum, f4 x, int slot) __attribute__((always_inline)) {
                if (part == 0) {
                    sum = x;
                    return;
                }
                const f4 both = sum + x, v = both - sum, err = (sum - (both - v)) + (x - v);
                low[slot * 256] = part == 1 ? err : low[slot * 256] + err;
                sum = both;
            };
#pragma unroll
            for (int j = 0; j < TK; ++j)
#pragma unroll
                for (int t = 0; t < TQ; ++t) {
                    add(rs[j][t], re[j][t], (j * TQ + t) * 2);
                    add(is[j][t], im[j][t], (j * TQ + t) * 2 + 1);
                    re[j][t] = im[j][t] = f4{0.f, 0.f, 0.f, 0.f};
                }
        }
    }
    if (k1b + w >= n) return;
    // entry ((p*N + K2)*16 + b3*4 + b4)*side + (K1*4 + b1)*4 + b2; a K2's entries are read together
    const int h = l >> 4;
    const int64_t col = (int64_t)(k1b + w) * 16 + (PP ? lo * 4 + h : h * 4 + lo);
#pragma unroll
    for (int j = 0; j < TK; ++j) {
        if (k2b + j >= n) continue;
        double2 v[TQ][4];
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            const double2 *row = a.acc + ((((int64_t)min(pb + t, a.planes - 1) * n + k2b + j) * 16 + hi * 4) * a.side + col);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[t][r] = row[r * a.side];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            if (pb + t >= a.planes) continue;
            double2 *row = a.acc + ((((int64_t)(pb + t) * n + k2b + j) * 16 + hi * 4) * a.side + col);
            f4 lr{0.f, 0.f, 0.f, 0.f}, li = lr;
            if (a.batch > kMoBatch) {
                lr = low[((j * TQ + t) * 2) * 256];
                li = low[((j * TQ + t) * 2 + 1) * 256];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[t][r].x += (double)rs[j][t][r] + (double)lr[r];
                v[t][r].y += (double)is[j][t][r] + (double)li[r];
                row[r * a.side] = v[t][r];
            }
        }
    }
}

// The blocks of a launch of mo_mfma_kernel, a multiple of 8 (one run per XCD).
int64_t mo_mfma_blocks(const MoArgs &a, int tq) {
    const int64_t n = a.side / 16;
    const int64_t t4 = (n + 3) / 4;
    return ((a.planes + tq - 1) / tq * t4 * t4 + 7) / 8 * 8;
}

// The blocks of a launch of mo_two_kernel, and whether it runs: one channel of two
// orbitals from a block per CU on (2x2, 32 measurements, rows kernel against this
// one: 60 blocks 28 : 39 us, 96 36 : 45, 256 69 : 54, 512 114 : 79), both channels
// where they share a launch.
int64_t mo_two_blocks(const MoArgs &a) { return (int64_t)a.planes * (a.side / 8) * ((a.side + 255) / 256); }
bool mo_uses_two(const MoArgs &a) {
    return a.nb == 2 && a.channel != CH_PP && (a.channel == (CH_MAG | CH_CHG) || mo_two_blocks(a) >= 256);
}

// Whether the `planes` planes of a call's magnetic and charge slices share launches.
// Small slices sum their measurements in a chain that two launches of the rows
// kernel shorten: its time over this kernel's, median (5% lowest, 5% highest) on
// 1465 random shapes, shared 1.45 (1.17, 3.0), not shared 0.98 (0.84, 1.12).
bool mo_both(int64_t planes, int64_t side, bool f32, int batch) {
    const int64_t n = side / 4, rows = planes * n * ((side + 255) / 256);
    return !(rows <= 284 && n <= 42 && batch > 12 && (f32 || batch <= 40));
}

// Four orbitals in FP32 fill the 16 x 16 matrix instruction (three use 81 of its
// 256 products and stay on the vector units); the kernel takes 32-bit byte
// offsets within four matrices.  Each of its steps takes four measurements, and a
// block all of a plane pair's orbitals of 16 momentum-frequency pairs: calls of
// fewer measurements, and few blocks of few measurements, are quicker on the rows
// kernel (2561 random shapes, its time over this kernel's, median, 5% lowest and
// highest: taken here 1.39 (0.98, 2.29), left 0.97 (0.78, 1.12)).  `batch` counts the whole call's: what
// a launch may hold follows from the choice, made once for all of a call.
bool mo_uses_mfma(const MoArgs &a, bool f32, int batch) {
    if (!f32 || a.nb != 4 || a.g_stride * 8 >= ((int64_t)1 << 30) || batch < 4) return false;
    return a.planes == 1 || mo_mfma_blocks(a, 2) > 128 || batch > 40;
}

template <typename R>
hipError_t launch_mo(const MoArgs &a, hipStream_t st) {
    const int64_t n = a.side / ((int64_t)a.nb * a.nb);
    // rows kernel: whole blocks per (plane, K2) row; entry kernel: one thread per entry
    const int64_t blocks = a.nb <= 8 ? (int64_t)a.planes * n * ((a.side + 255) / 256) : (a.total + 255) / 256;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
    const dim3 g((unsigned)blocks), b(256);
    if constexpr (std::is_same<R, float>::value)
        if (a.matrix) {
            const int tq = a.planes > 1 ? 2 : 1;
            const int64_t mb = mo_mfma_blocks(a, tq);
            if (mb >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
            const dim3 gm((unsigned)mb);
            const bool pp = a.channel == CH_PP;
            const void *const fn = tq == 2 ? (pp ? reinterpret_cast<const void *>(&mo_mfma_kernel<2, true>)
                                                 : reinterpret_cast<const void *>(&mo_mfma_kernel<2, false>))
                                           : (pp ? reinterpret_cast<const void *>(&mo_mfma_kernel<1, true>)
                                                 : reinterpret_cast<const void *>(&mo_mfma_kernel<1, false>));
            const size_t lds = mo_mfma_lds(a.batch, tq);
            // beside the kernel's own 9 KB
            if (lds)
                if (hipError_t e = ensure_lds_limit(fn, lds + 16 * 1024); e != hipSuccess) return e;
            MoArgs arg = a;
            void *params[] = {&arg};
            return hipLaunchKernel(fn, gm, b, params, lds, st);
        }
    if (mo_uses_two(a)) {
        const int64_t tb = mo_two_blocks(a);
        if (tb >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
        const dim3 gt((unsigned)tb);
        switch (a.channel) {
            case 1: hipLaunchKernelGGL((mo_two_kernel<R, 1>), gt, b, 0, st, a); break;
            case 2: hipLaunchKernelGGL((mo_two_kernel<R, 2>), gt, b, 0, st, a); break;
            default: hipLaunchKernelGGL((mo_two_kernel<R, 3>), gt, b, 0, st, a); break;
        }
        return hipGetLastError();
    }
    switch (a.nb) {
        case 1: hipLaunchKernelGGL((mo_rows_kernel<R, 1>), g, b, 0, st, a); break;
        case 2: hipLaunchKernelGGL((mo_rows_kernel<R, 2>), g, b, 0, st, a); break;
        case 3: hipLaunchKernelGGL((mo_rows_kernel<R, 3>), g, b, 0, st, a); break;
        case 4: hipLaunchKernelGGL((mo_rows_kernel<R, 4>), g, b, 0, st, a); break;
        case 5: hipLaunchKernelGGL((mo_rows_kernel<R, 5>), g, b, 0, st, a); break;
        case 6: hipLaunchKernelGGL((mo_rows_kernel<R, 6>), g, b, 0, st, a); break;
        case 7: hipLaunchKernelGGL((mo_rows_kernel<R, 7>), g, b, 0, st, a); break;
        case 8: hipLaunchKernelGGL((mo_rows_kernel<R, 8>), g, b, 0, st, a); break;
        default: hipLaunchKernelGGL(mo_kernel<R>, g, b, 0, st, a); break;
    }
    return hipGetLastError();
}

}  // namespace

int set_error(int code, const char *msg);

}  // namespace g4

extern "C" int g4_accumulate_mo(int32_t lx, int32_t ly, int32_t nw, int32_t nwex, int32_t nb, int32_t nq,
                                const int32_t *q_list, int64_t q_begin, int64_t q_end, uint32_t channels,
                                int32_t prod, const void *G_up, const void *G_dn, const double *sign,
                                int32_t batch, void *acc_mag, void *acc_chg, void *acc_pp, void *stream) {
    using namespace g4;
    if (lx < 1 || ly < 1 || (int64_t)lx * ly > 4096 || nw < 2 || (nw & 1) || nw > 4096 || nwex < 1 ||
        nwex > 4096 || nb < 1 || nb > 64)
        return set_error(G4_E_ARG, "multi-orbital: bad cluster, frequency or orbital count");
    const int nc = lx * ly;
    if (nq < 1 || nq > nc) return set_error(G4_E_ARG, "multi-orbital: nq outside [1, Nc]");
    std::vector<int> ql(nq), seen(nc, 0);
    for (int i = 0; i < nq; ++i) {
        ql[i] = q_list ? q_list[i] : i;
        if (ql[i] < 0 || ql[i] >= nc || seen[ql[i]]) return set_error(G4_E_ARG, "multi-orbital: bad q_list");
        seen[ql[i]] = 1;
    }
    if (q_begin < 0 || q_end > (int64_t)nq * nwex || q_begin >= q_end)
        return set_error(G4_E_ARG, "multi-orbital: slice planes outside [0, nq*nwex)");
    if (channels == 0 || (channels & ~7u)) return set_error(G4_E_ARG, "multi-orbital: channels of 1|2|4 only");
    if (prod != G4_PROD_F64 && prod != G4_PROD_F32)
        return set_error(G4_E_ARG, "multi-orbital: prod must be G4_PROD_F64 or G4_PROD_F32");
    if (batch < 0) return set_error(G4_E_ARG, "multi-orbital: batch < 0");
    void *acc[3] = {acc_mag, acc_chg, acc_pp};
    for (int c = 0; c < 3; ++c)
        if (((channels >> c) & 1u) != (acc[c] != nullptr))
            return set_error(G4_E_ARG, "multi-orbital: one accumulator per channel, NULL for the others");
    const int64_t nwg = nw + nwex - 1;
    const int64_t ngb = (int64_t)nc * nwg * nb;
    const int64_t side = (int64_t)nc * nw * nb * nb;
    if (ngb * ngb >= ((int64_t)1 << 40) || side > ((int64_t)1 << 30))
        return set_error(G4_E_UNSUPPORTED, "multi-orbital: matrices too large");
    if (batch == 0) return G4_OK;
    if (!G_up || !G_dn || !sign) return set_error(G4_E_ARG, "multi-orbital: NULL G or sign");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t planes = q_end - q_begin;
    for (int c = 0; c < 3; ++c) {
        if (!acc[c]) continue;
        // two orbitals: magnetic and charge in the same launches
        const bool pair = nb == 2 && c < 2 && acc[0] && acc[1] && mo_both(planes, side, prod == G4_PROD_F32, batch);
        const bool both = pair && c == 0;
        if (pair && c == 1) continue;
        for (int64_t p0 = 0; p0 < planes; p0 += kMoPlanes) {
            const int np = (int)std::min<int64_t>(kMoPlanes, planes - p0);
            MoArgs shape{};
            shape.nb = nb; shape.planes = np; shape.side = side; shape.g_stride = ngb * ngb;
            shape.channel = both ? CH_MAG | CH_CHG : 1 << c;
            const bool matrix = mo_uses_mfma(shape, prod == G4_PROD_F32, batch);
            const int most = matrix || (prod == G4_PROD_F64 && mo_uses_two(shape)) ? kMoLong : kMoBatch;
            for (int b0 = 0; b0 < batch; b0 += most) {
                MoArgs a{};
                a.g_stride = ngb * ngb;
                const size_t el = prod == G4_PROD_F64 ? 16 : 8;
                a.gu = static_cast<const char *>(G_up) + (size_t)b0 * a.g_stride * el;
                a.gd = static_cast<const char *>(G_dn) + (size_t)b0 * a.g_stride * el;
                a.acc = static_cast<double2 *>(acc[c]) + p0 * side * side;
                a.total = (int64_t)np * side * side;
                a.side = side;
                a.lx = lx; a.ly = ly; a.nw = nw; a.nwg = (int)nwg; a.nb = nb; a.ngb = (int)ngb;
                a.acc2 = both ? static_cast<double2 *>(acc[1]) + p0 * side * side : nullptr;
                a.channel = both ? CH_MAG | CH_CHG : 1 << c;
                a.batch = std::min(most, batch - b0);
                a.planes = np;
                a.matrix = matrix;
                for (int i = 0; i < np; ++i) {
                    const int64_t iQ = q_begin + p0 + i;
                    a.qm[i] = int2{ql[(size_t)(iQ / nwex)], (int)(iQ % nwex)};
                }
                for (int j = 0; j < a.batch; ++j) a.sign[j] = sign[b0 + j];
                if ((a.total + 255) / 256 >= ((int64_t)1 << 31))
                    return set_error(G4_E_UNSUPPORTED, "multi-orbital: grid too large");
                const hipError_t e = prod == G4_PROD_F64 ? launch_mo<double>(a, st) : launch_mo<float>(a, st);
                if (e != hipSuccess) {
                    char msg[160];
                    std::snprintf(msg, sizeof(msg), "multi-orbital launch: %s", hipGetErrorString(e));
                    return set_error(G4_E_HIP, msg);
                }
            }
        }
    }
    return G4_OK;
}
