// G_sigma of a batch of measurements from their expansion configurations:
// the walker's nonuniform Fourier transform written as matrix products
// (Background section, the solver workflow), for gfx950.
//
// For measurement b with n vertices (imaginary times tau_i, cluster sites
// r_i) and the walker's n x n matrix M_b:
//   E_b[K][i] = exp(i (w_n tau_i + k . r_i))                 (Ng x n)
//   G_b       = diag(g0) - diag(g0) (E_b M_b E_b^H) diag(g0) / (beta Nc)
// Launches per call (few vertices or sites; the others transform site by site,
// further down):
//   g0_kernel             g0 over the window, FP64, into the workspace;
//   phase_kernel          E_b, phases in FP64 (k . r as an exact fraction
//                         of 2 pi), stored in the output precision;
//   cgemm_kernel<N>       T_b = E_b M_b;
//   cgemm_kernel<H, G>    G_b from T_b E_b^H with the g0 scaling and the
//                         diagonal fused into the store.
// The complex GEMM runs on v_mfma_{f32,f64}_16x16x4: per step of two complex
// k, the four k slots hold (Re, Im) of both (Re C: A slots (Re a, -Im a),
// Im C: (Im a, Re a), B slots (Re b, Im b)).  A 256-thread block owns a
// 64 x 64 output tile (each wave 32 x 32: 2 x 2 MFMA tiles, Re and Im),
// staged through LDS in k chunks of 16, the next chunk held in registers
// while the current one is multiplied; LDS holds the operands in the form
// each lane hands to the MFMA, so the inner loop is LDS reads and MFMAs.
#include "../../include/g4.h"
#include "g4_internal.hpp"

#include <algorithm>
#include <cstdio>

namespace g4 {
namespace {

template <typename T> struct Cx2;
template <> struct Cx2<float> { using V = float2; using V4 = float __attribute__((ext_vector_type(4))); };
template <> struct Cx2<double> { using V = double2; using V4 = double __attribute__((ext_vector_type(4))); };

__device__ __forceinline__ Cx2<float>::V4 mfma16(float a, float b, Cx2<float>::V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Cx2<double>::V4 mfma16(double a, double b, Cx2<double>::V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr double kPi = 3.14159265358979323846;

struct GsShape {
    int lx, ly, nc, nw, nwg, ng, n, count, spin;
    double beta, mu, h, t;
};

// g0(K) = 1 / (i w_n + mu + s h - eps_k) for every K of the window, in FP64
__global__ __launch_bounds__(256) void g0_kernel(GsShape s, double2 *g0) {
    const int K = blockIdx.x * blockDim.x + threadIdx.x;
    if (K >= s.ng) return;
    const int k = K / s.nwg, nn = K % s.nwg - s.nw / 2;
    const double w = (2.0 * nn + 1.0) * kPi / s.beta;
    const double eps = -2.0 * s.t * (cos(2.0 * kPi * (k % s.lx) / s.lx) + cos(2.0 * kPi * (k / s.lx) / s.ly));
    const double r = s.mu + (s.spin == 0 ? s.h : -s.h) - eps;
    const double d = r * r + w * w;
    g0[K] = double2{r / d, -w / d};
}

template <typename T>
__global__ __launch_bounds__(256) void phase_kernel(GsShape s, const double *tau, const int32_t *site,
                                                    typename Cx2<T>::V *E) {
    using V = typename Cx2<T>::V;
    const int64_t total = (int64_t)s.count * s.ng * s.n;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx % s.n);
        const int64_t rest = idx / s.n;
        const int K = (int)(rest % s.ng);
        const int64_t b = rest / s.ng;
        const int k = K / s.nwg, nn = K % s.nwg - s.nw / 2;
        const double w = (2.0 * nn + 1.0) * kPi / s.beta;
        const int st = site[b * s.n + i];
        const int kx = k % s.lx, ky = k / s.lx, rx = st % s.lx, ry = st / s.lx;
        const double th = w * tau[b * s.n + i] +
                          2.0 * kPi * ((double)((kx * rx) % s.lx) / s.lx + (double)((ky * ry) % s.ly) / s.ly);
        double sn, cs;
        sincos(th, &sn, &cs);
        E[idx] = V{(T)cs, (T)sn};
    }
}

// Batched complex GEMM C_b = A_b op(B_b): A_b M x K (lda), op(B_b) = B_b
// (K x N, ldb) or, with BH, the conjugate transpose of B_b (N x K, ldb).
// With GEPI the store is G = (K1 == K2 ? g0(K1) : 0) - g0(K1) C g0(K2) * scale.
struct CgArgs {
    const void *A, *B;
    void *C;
    const double2 *g0;           // GEPI: g0 of every K
    int64_t sA, sB, sC;          // elements between batches
    int lda, ldb, ldc;
    int M, N, K;
    double scale;
};

constexpr int BN = 64, BK = 16;

// TM: 16-row MFMA tiles per wave along M; the block is (32 TM) x 64.
template <typename T, bool BH, bool GEPI, int TM>
__global__ __launch_bounds__(256) void cgemm_kernel(CgArgs a) {
    using V = typename Cx2<T>::V;
    using V4 = typename Cx2<T>::V4;
    constexpr int BM = 32 * TM;
    // Operands in LDS in the form each lane feeds the MFMA: A twice, as
    // (Re, Im) for the real-part slots and (-Im, Re) for the imaginary-part
    // slots; B split into its real and imaginary planes.
    __shared__ V Ap[2][BM][BK + 1];
    __shared__ T Bp[2][BK][BN + 4];
    constexpr int PA = BM * BK / 256, PB = BK * BN / 256;   // elements a thread stages per chunk
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
    const int b = blockIdx.z;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const V *A = static_cast<const V *>(a.A) + (int64_t)b * a.sA;
    const V *B = static_cast<const V *>(a.B) + (int64_t)b * a.sB;
    const int wr = (w >> 1) * 16 * TM, wc = (w & 1) * 32;
    const int slot = l >> 4, comp = slot & 1, kh = slot >> 1, lr = l & 15;
    V4 re[TM][2], im[TM][2];
    for (int i = 0; i < TM; ++i)
        for (int j = 0; j < 2; ++j) {
            re[i][j] = V4{0, 0, 0, 0};
            im[i][j] = V4{0, 0, 0, 0};
        }
    // the next chunk's operands are loaded into registers while the current one is multiplied
    V ra[PA], rb[PB];
    auto load = [&](int k0) {
        for (int u = 0; u < PA; ++u) {
            const int e = tid + 256 * u;
            const int r = e / BK, c = e % BK;
            const int gr = m0 + r, gc = k0 + c;
            ra[u] = (gr < a.M && gc < a.K) ? A[(int64_t)gr * a.lda + gc] : V{0, 0};
        }
        for (int u = 0; u < PB; ++u) {
            const int e = tid + 256 * u;
            const int r = e / BK, c = e % BK;
            if (BH) {
                const int gj = n0 + r, gk = k0 + c;          // B_b row n0 + r, column k0 + c
                rb[u] = (gj < a.N && gk < a.K) ? B[(int64_t)gj * a.ldb + gk] : V{0, 0};
            } else {
                const int rr = e / BN, cc = e % BN;
                const int gk = k0 + rr, gj = n0 + cc;
                rb[u] = (gk < a.K && gj < a.N) ? B[(int64_t)gk * a.ldb + gj] : V{0, 0};
            }
        }
    };
    auto store = [&]() {
        for (int u = 0; u < PA; ++u) {
            const int e = tid + 256 * u;
            const int r = e / BK, c = e % BK;
            const V v = ra[u];
            Ap[0][r][c] = v;
            Ap[1][r][c] = V{-v.y, v.x};
        }
        for (int u = 0; u < PB; ++u) {
            const int e = tid + 256 * u;
            const int r = e / BK, c = e % BK;
            if (BH) {                 // conj(B_b(n0 + r, k0 + c)) at k = c, column r
                Bp[0][c][r] = rb[u].x;
                Bp[1][c][r] = -rb[u].y;
            } else {
                const int rr = e / BN, cc = e % BN;
                Bp[0][rr][cc] = rb[u].x;
                Bp[1][rr][cc] = rb[u].y;
            }
        }
    };
    if (a.K > 0) load(0);
    for (int k0 = 0; k0 < a.K; k0 += BK) {
        __syncthreads();      // the previous chunk's reads are done
        store();
        __syncthreads();
        if (k0 + BK < a.K) load(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            const int kc = kk + kh;
            T are[TM], aim[TM], bv[2];
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const V av = Ap[comp][wr + 16 * t + lr][kc];
                are[t] = av.x;
                aim[t] = av.y;
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) bv[t] = Bp[comp][kc][wc + 16 * t + lr];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    re[i][j] = mfma16(are[i], bv[j], re[i][j]);
                    im[i][j] = mfma16(aim[i], bv[j], im[i][j]);
                }
        }
    }
    // result register r of lane l holds column l % 16 of each 16 x 16 tile, row
    // 4(l/16) + r (FP32) or 4r + l/16 (FP64)
    V *C = static_cast<V *>(a.C) + (int64_t)b * a.sC;
    for (int j = 0; j < 2; ++j) {
        const int col = n0 + wc + 16 * j + lr;
        if (col >= a.N) continue;
        double2 gc{0.0, 0.0};
        if (GEPI) gc = a.g0[col];
        for (int i = 0; i < TM; ++i)
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wr + 16 * i + (sizeof(T) == 4 ? 4 * slot + r : 4 * r + slot);
                if (row >= a.M) continue;
                double cr = (double)re[i][j][r], ci = (double)im[i][j][r];
                if (GEPI) {
                    const double2 gr = a.g0[row];
                    // g0(row) c g0(col) * scale, subtracted from the diagonal g0
                    const double tr = gr.x * cr - gr.y * ci, ti = gr.x * ci + gr.y * cr;
                    double vr = -(tr * gc.x - ti * gc.y) * a.scale;
                    double vi = -(tr * gc.y + ti * gc.x) * a.scale;
                    if (row == col) {
                        vr += gr.x;
                        vi += gr.y;
                    }
                    cr = vr;
                    ci = vi;
                }
                C[(int64_t)row * a.ldc + col] = V{(T)cr, (T)ci};
            }
    }
}

// ---- the transform by sites --------------------------------------------------
// The phase of a vertex factorises, e^{i th_i(k,n)} = e^{i w_n tau_i} e^{i k.r_i},
// and only Nc sites occur.  With the vertices of a measurement sorted by site,
//   T(r, n1; j)    = sum_{i at r} P(n1, i) M(i, j),      P(n, i) = e^{i w_n tau_i}
//   T(k1, n1; j)   = sum_r e^{i k1.r} T(r, n1; j)        (equal to E M)
//   U(K1; r', n2)  = sum_{j at r'} T(K1; j) conj(P(n2, j))
//   G(K1; k2, n2)  = g0 - g0 g0 / (beta Nc) sum_r' e^{-i k2.r'} U(K1; r', n2)
// takes Nwg n^2 + Ng Nwg n products in the two matrix steps instead of Ng n^2 +
// Ng^2 n, and two small Fourier sums over the lattice, done along its two
// directions.  On the 4x4 window at n = 512 that is a ninth of the products.
// 64 measurements, Ng = 1136, n = 512, complex64: 4.51 -> 1.03 ms a call;
// complex128, Ng = 2288, n = 317, 8 measurements: 2.33 -> 0.67 ms.  U lives in G's place.

constexpr int kSiteVertices = 8192;   // vertices per measurement at most (sort keys of 25 bits, 32 KB of them)

// position in site order of every vertex of a measurement (by site, then by
// index), and the first position of each site: one block per measurement.
// Sites outside the lattice stand for the site that they wrap to.
__global__ __launch_bounds__(256) void site_sort_kernel(GsShape s, const int32_t *site, int32_t *perm, int32_t *first) {
    extern __shared__ __align__(16) int32_t sh[];      // site * kSiteVertices + index, four at a time
    const int b = blockIdx.x, n4 = (s.n + 3) / 4;
    for (int i = threadIdx.x; i < 4 * n4; i += 256) {
        const int st = i < s.n ? site[(int64_t)b * s.n + i] : 0;
        const int r = (st % s.lx + s.lx) % s.lx + s.lx * ((st / s.lx % s.ly + s.ly) % s.ly);
        sh[i] = i < s.n ? r * kSiteVertices + i : 0x7fffffff;
    }
    __syncthreads();
    auto below = [&](int key) {
        int c = 0;
        for (int j = 0; j < n4; ++j) {
            const int4 v = reinterpret_cast<const int4 *>(sh)[j];
            c += (v.x < key) + (v.y < key) + (v.z < key) + (v.w < key);
        }
        return c;
    };
    for (int i = threadIdx.x; i < s.n; i += 256) perm[(int64_t)b * s.n + below(sh[i])] = i;
    for (int r = threadIdx.x; r <= s.nc; r += 256) first[(int64_t)b * (s.nc + 1) + r] = below(r * kSiteVertices);
}

// P(n, i) of the sorted vertices, and M with rows and columns in that order
template <typename T>
__global__ __launch_bounds__(256) void site_phase_kernel(GsShape s, const double *tau, const int32_t *perm,
                                                         typename Cx2<T>::V *P) {
    using V = typename Cx2<T>::V;
    const int64_t total = (int64_t)s.count * s.nwg * s.n;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx % s.n);
        const int64_t rest = idx / s.n;
        const int64_t b = rest / s.nwg;
        const int nn = (int)(rest % s.nwg) - s.nw / 2;
        double sn, cs;
        sincos((2.0 * nn + 1.0) * kPi / s.beta * tau[b * s.n + perm[b * s.n + i]], &sn, &cs);
        P[idx] = V{(T)cs, (T)sn};
    }
}
template <typename V>
__global__ __launch_bounds__(256) void site_order_kernel(int n, const int32_t *perm, const V *M, V *out) {
    const int64_t b = blockIdx.y;
    const int i = blockIdx.x;
    perm += b * n;
    const V *row = M + (b * n + perm[i]) * (int64_t)n;
    V *dst = out + (b * n + i) * (int64_t)n;
    for (int j = threadIdx.x; j < n; j += 256) dst[j] = row[perm[j]];
}

// C = A op(B) over the k range [first[z], first[z+1]) of one measurement and one
// site: A M x K (lda), B K x N or, with BH, the conjugate transpose of N x K
// (ldb).  Blocks of (64 TM) x (16 TN), a wave 16 TM rows of all columns; operands
// in LDS and on the matrix cores as in cgemm_kernel.
struct SgArgs {
    const void *A, *B;
    void *C;
    const int32_t *first;
    int64_t sA, sB, sC, siteC;   // elements between measurements; between a measurement's sites in C
    int lda, ldb, ldc, M, N, nc;
};
template <typename T, bool BH, int TM, int TN>
__global__ __launch_bounds__(256) void site_gemm_kernel(SgArgs a) {
    using V = typename Cx2<T>::V;
    using V4 = typename Cx2<T>::V4;
    constexpr int BM = 64 * TM, BNS = 16 * TN, BKS = 8;
    constexpr int PA = BM * BKS / 256, PB = (BKS * BNS + 255) / 256;
    __shared__ V Ap[2][BM][BKS + 1];
    __shared__ T Bp[2][BKS][BNS + 4];
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
    const int b = blockIdx.z / a.nc, r = blockIdx.z % a.nc;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BNS;
    const int kb = a.first[(int64_t)b * (a.nc + 1) + r], ke = a.first[(int64_t)b * (a.nc + 1) + r + 1];
    const V *A = static_cast<const V *>(a.A) + (int64_t)b * a.sA;
    const V *B = static_cast<const V *>(a.B) + (int64_t)b * a.sB;
    const int slot = l >> 4, comp = slot & 1, kh = slot >> 1, lr = l & 15;
    V4 re[TM][TN], im[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) re[i][j] = im[i][j] = V4{0, 0, 0, 0};
    V ra[PA], rb[PB];
    auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PA; ++u) {
            const int e = tid + 256 * u, gr = m0 + e / BKS, gc = k0 + e % BKS;
            ra[u] = (gr < a.M && gc < ke) ? A[(int64_t)gr * a.lda + gc] : V{0, 0};
        }
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int e = tid + 256 * u;
            const int gk = k0 + (BH ? e % BKS : e / BNS), gj = n0 + (BH ? e / BKS : e % BNS);
            rb[u] = (e < BKS * BNS && gk < ke && gj < a.N) ? B[BH ? (int64_t)gj * a.ldb + gk : (int64_t)gk * a.ldb + gj] : V{0, 0};
        }
    };
    if (kb < ke) load(kb);
    for (int k0 = kb; k0 < ke; k0 += BKS) {
        __syncthreads();      // the previous chunk's reads are done
#pragma unroll
        for (int u = 0; u < PA; ++u) {
            const int e = tid + 256 * u;
            Ap[0][e / BKS][e % BKS] = ra[u];
            Ap[1][e / BKS][e % BKS] = V{-ra[u].y, ra[u].x};
        }
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int e = tid + 256 * u;
            if (e < BKS * BNS) {
                const int kk = BH ? e % BKS : e / BNS, jj = BH ? e / BKS : e % BNS;
                Bp[0][kk][jj] = rb[u].x;
                Bp[1][kk][jj] = BH ? -rb[u].y : rb[u].y;
            }
        }
        __syncthreads();
        if (k0 + BKS < ke) load(k0 + BKS);
#pragma unroll
        for (int kk = 0; kk < BKS; kk += 2) {
            const int kc = kk + kh;
            T are[TM], aim[TM];
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                const V av = Ap[comp][(w * TM + t) * 16 + lr][kc];
                are[t] = av.x;
                aim[t] = av.y;
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const T bv = Bp[comp][kc][16 * j + lr];
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    re[i][j] = mfma16(are[i], bv, re[i][j]);
                    im[i][j] = mfma16(aim[i], bv, im[i][j]);
                }
            }
        }
    }
    V *C = static_cast<V *>(a.C) + (int64_t)b * a.sC + r * a.siteC;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = n0 + 16 * j + lr;
        if (col >= a.N) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = m0 + (w * TM + i) * 16 + (sizeof(T) == 4 ? 4 * slot + q : 4 * q + slot);
                if (row < a.M) C[(int64_t)row * a.ldc + col] = V{re[i][j][q], im[i][j][q]};
            }
    }
}

// Fourier sum over the sites, in place: out(k) = sum_r e^{+-i k.r} in(r), k and r
// as x + lx y: column e has its Nc values at base(e) + r * stride.  x direction,
// then y.  With GEPI the sign is minus and the store is G (see cgemm_kernel's),
// columns (row K1, frequency n2).
struct DftArgs {
    void *data;
    const double2 *g0;
    int64_t columns, run, jump, stride;   // column e at (e / run) * jump + e % run
    int lx, ly, nwg, ng;
    double scale;
};
template <typename T, bool GEPI>
__device__ __forceinline__ void site_twiddles(const DftArgs &a, typename Cx2<T>::V *wx, typename Cx2<T>::V *wy) {
    for (int i = threadIdx.x; i < a.lx + a.ly; i += 256) {
        const int j = i < a.lx ? i : i - a.lx, len = i < a.lx ? a.lx : a.ly;
        double sn, cs;
        sincos(2.0 * kPi * j / len, &sn, &cs);
        (i < a.lx ? wx + j : wy + j)[0] = typename Cx2<T>::V{(T)cs, (T)(GEPI ? -sn : sn)};
    }
}
// what a column's value of momentum o becomes: g0 - g0 v g0 scale at (row, o nwg + n2)
template <typename T>
__device__ __forceinline__ typename Cx2<T>::V site_g(const DftArgs &a, typename Cx2<T>::V v, int row, double2 gr, int col) {
    const double2 gc = a.g0[col];
    const double cr = (double)v.x, ci = (double)v.y;
    const double tr = gr.x * cr - gr.y * ci, ti = gr.x * ci + gr.y * cr;
    double vr = -(tr * gc.x - ti * gc.y) * a.scale, vi = -(tr * gc.y + ti * gc.x) * a.scale;
    if (row == col) {
        vr += gr.x;
        vi += gr.y;
    }
    return typename Cx2<T>::V{(T)vr, (T)vi};
}

// a column per thread, its values in registers: the lattices below
template <typename T, bool GEPI, int LX, int LY>
__global__ __launch_bounds__(256) void site_dft_reg_kernel(DftArgs a) {
    using V = typename Cx2<T>::V;
    __shared__ V wx[LX], wy[LY];
    site_twiddles<T, GEPI>(a, wx, wy);
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool act = e < a.columns;
    const int64_t er = act ? e / a.run : 0;
    const int in = act ? (int)(e - er * a.run) : 0;
    V *base = static_cast<V *>(a.data) + er * a.jump + in;
    V v[LY][LX];
#pragma unroll
    for (int y = 0; y < LY; ++y)
#pragma unroll
        for (int x = 0; x < LX; ++x) v[y][x] = base[(x + LX * y) * a.stride];
    __syncthreads();
    // one direction: out(k) = sum_j w(k j mod L) in(j), w(0) = 1
    auto sum = [](auto get, const V *w, int k, int L) __attribute__((always_inline)) {
        V s = get(0);
#pragma unroll
        for (int j = 1; j < L; ++j) {
            const V u = get(j);
            const int ph = k * j % L;
            if (ph == 0) {
                s.x += u.x;
                s.y += u.y;
            } else {
                const V t = w[ph];
                s.x = fma(t.x, u.x, s.x);
                s.x = fma(-t.y, u.y, s.x);
                s.y = fma(t.x, u.y, s.y);
                s.y = fma(t.y, u.x, s.y);
            }
        }
        return s;
    };
#pragma unroll
    for (int y = 0; y < LY; ++y) {
        V t[LX];
#pragma unroll
        for (int k = 0; k < LX; ++k) t[k] = sum([&](int j) __attribute__((always_inline)) { return v[y][j]; }, wx, k, LX);
#pragma unroll
        for (int k = 0; k < LX; ++k) v[y][k] = t[k];
    }
    const int row = GEPI ? (int)(er % a.ng) : 0;
    const double2 gr = GEPI ? a.g0[row] : double2{0.0, 0.0};
#pragma unroll
    for (int k = 0; k < LX; ++k)
#pragma unroll
        for (int ky = 0; ky < LY; ++ky) {
            V s = sum([&](int j) __attribute__((always_inline)) { return v[j][k]; }, wy, ky, LY);
            const int o = k + LX * ky;
            if (GEPI) s = site_g<T>(a, s, row, gr, o * a.nwg + in);
            if (act) base[o * a.stride] = s;
        }
}

// any lattice: 64 columns per block, through two buffers in LDS
template <typename T, bool GEPI>
__global__ __launch_bounds__(256) void site_dft_kernel(DftArgs a) {
    using V = typename Cx2<T>::V;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nc = a.lx * a.ly, tid = threadIdx.x, c = tid & 63, g = tid >> 6;
    V *in = reinterpret_cast<V *>(smem_raw), *mid = in + nc * 64, *wx = mid + nc * 64, *wy = wx + a.lx;
    site_twiddles<T, GEPI>(a, wx, wy);
    const int64_t e = (int64_t)blockIdx.x * 64 + c;
    const bool act = e < a.columns;
    const int64_t er = act ? e / a.run : 0;
    const int ei = act ? (int)(e - er * a.run) : 0;
    V *base = static_cast<V *>(a.data) + er * a.jump + ei;
    for (int r = g; r < nc; r += 4) in[r * 64 + c] = base[r * a.stride];
    __syncthreads();
    for (int o = g; o < nc; o += 4) {                 // o = kx + lx y
        const int kx = o % a.lx, y = o / a.lx;
        V s{0, 0};
        int ph = 0;
        for (int x = 0; x < a.lx; ++x) {
            const V v = in[(x + a.lx * y) * 64 + c], t = wx[ph];
            s.x += t.x * v.x - t.y * v.y;
            s.y += t.x * v.y + t.y * v.x;
            ph += kx;
            if (ph >= a.lx) ph -= a.lx;
        }
        mid[o * 64 + c] = s;
    }
    __syncthreads();
    const int row = GEPI ? (int)(er % a.ng) : 0;
    const double2 gr = GEPI ? a.g0[row] : double2{0.0, 0.0};
    for (int o = g; o < nc; o += 4) {                 // o = kx + lx ky
        const int kx = o % a.lx, ky = o / a.lx;
        V s{0, 0};
        int ph = 0;
        for (int y = 0; y < a.ly; ++y) {
            const V v = mid[(kx + a.lx * y) * 64 + c], t = wy[ph];
            s.x += t.x * v.x - t.y * v.y;
            s.y += t.x * v.y + t.y * v.x;
            ph += ky;
            if (ph >= a.ly) ph -= a.ly;
        }
        if (GEPI) s = site_g<T>(a, s, row, gr, o * a.nwg + ei);
        if (act) base[o * a.stride] = s;
    }
}

template <typename T, bool GEPI>
hipError_t launch_site_dft(const DftArgs &a, hipStream_t st) {
    const auto blocks = [&](int per) { return (a.columns + per - 1) / per; };
    if (blocks(64) >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
    const dim3 g((unsigned)blocks(256));
#define G4_DFT(X, Y)                                                                                        \
    if (a.lx == X && a.ly == Y) {                                                                           \
        hipLaunchKernelGGL((site_dft_reg_kernel<T, GEPI, X, Y>), g, dim3(256), 0, st, a);                   \
        return hipGetLastError();                                                                           \
    }
    G4_DFT(2, 2) G4_DFT(3, 2) G4_DFT(3, 3) G4_DFT(4, 2) G4_DFT(4, 4) G4_DFT(5, 5) G4_DFT(6, 6)
#undef G4_DFT
    const size_t lds = (size_t)(2 * a.lx * a.ly * 64 + a.lx + a.ly) * 2 * sizeof(T);
    if (hipError_t e = ensure_lds_limit(reinterpret_cast<const void *>(&site_dft_kernel<T, GEPI>), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL((site_dft_kernel<T, GEPI>), dim3((unsigned)blocks(64)), dim3(256), lds, st, a);
    return hipGetLastError();
}

// Workspace: g0 of the window (Ng complex128), then E and T (count x Ng x n each)
uint64_t workspace_bytes(int64_t ng, int64_t n, int64_t count, int esize) {
    return count == 0 ? 0 : (uint64_t)ng * 16 + 2ull * (uint64_t)count * ng * n * esize;
}

// Whether the transform by sites runs.  It trades matrix products for three more
// trips of T and G through memory and pads each site's vertices to 8: with the
// column of a Fourier sum in registers it is ahead from about 64 vertices on (4x4,
// complex64, 64 measurements: n = 64 547 : 554 us, n = 128 984 : 587 us; 6x6, 8
// measurements: n = 64 161 : 146, n = 200 436 : 167), through LDS from about 4 a
// site (8x8: n = 128 783 : 1215 us; complex128 n = 256 3.01 : 2.56 ms).  Its
// arrays have to fit the workspace, whose size the other path sets.
bool dft_in_registers(int lx, int ly) {
    return (lx == 2 && ly == 2) || (lx == 3 && (ly == 2 || ly == 3)) || (lx == 4 && (ly == 2 || ly == 4)) ||
           (lx == 5 && ly == 5) || (lx == 6 && ly == 6);
}
template <typename T>
bool gsigma_by_sites(const GsShape &s) {
    const uint64_t esize = 2 * sizeof(T), n = (uint64_t)s.n;
    const uint64_t extra = (n * n + (uint64_t)s.nwg * n) * esize + (n + s.nc + 1) * 4 + 64;
    const uint64_t lds = (uint64_t)(2 * s.nc * 64 + s.lx + s.ly) * esize;
    return s.nc >= 4 && s.n >= 72 && (dft_in_registers(s.lx, s.ly) || s.n >= 4 * s.nc) && s.n <= kSiteVertices &&
           lds <= 140 * 1024 && extra <= (uint64_t)s.ng * n * esize && (int64_t)s.count * s.nc <= 65535;
}

template <typename T, bool BH, int TM>
hipError_t launch_site_gemm(const SgArgs &a, int count, hipStream_t st) {
    // the column tile (48, 64 or 80) that covers N with the least padding, the widest of equals
    int best = 5;
    for (int tn : {4, 3})
        if ((a.N + 16 * tn - 1) / (16 * tn) * tn < (a.N + 16 * best - 1) / (16 * best) * best) best = tn;
    const dim3 g((a.N + 16 * best - 1) / (16 * best), (a.M + 64 * TM - 1) / (64 * TM), count * a.nc);
    if (best == 5) hipLaunchKernelGGL((site_gemm_kernel<T, BH, TM, 5>), g, dim3(256), 0, st, a);
    else if (best == 4) hipLaunchKernelGGL((site_gemm_kernel<T, BH, TM, 4>), g, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((site_gemm_kernel<T, BH, TM, 3>), g, dim3(256), 0, st, a);
    return hipGetLastError();
}

template <typename T>
hipError_t run_gsigma_by_sites(const GsShape &s, const double *tau, const int32_t *site, const void *M, void *G,
                               double2 *g0, void *ws, hipStream_t st) {
    using V = typename Cx2<T>::V;
    const int64_t n = s.n, per_t = (int64_t)s.ng * n;
    V *Tm = static_cast<V *>(ws), *Ms = Tm + s.count * per_t, *P = Ms + s.count * n * n;
    int32_t *perm = reinterpret_cast<int32_t *>(P + s.count * s.nwg * n), *first = perm + s.count * n;
    hipLaunchKernelGGL(site_sort_kernel, dim3(s.count), dim3(256), (n + 3) / 4 * 16, st, s, site, perm, first);
    const int64_t np = s.count * s.nwg * n;
    hipLaunchKernelGGL(site_phase_kernel<T>, dim3((unsigned)std::min<int64_t>((np + 255) / 256, 65536)), dim3(256), 0, st, s,
                       tau, perm, P);
    hipLaunchKernelGGL(site_order_kernel<V>, dim3(s.n, s.count), dim3(256), 0, st, s.n, perm, static_cast<const V *>(M), Ms);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    // T(r, n1; j)
    SgArgs a{};
    a.A = P; a.B = Ms; a.C = Tm; a.first = first;
    a.sA = s.nwg * n; a.sB = n * n; a.sC = per_t; a.siteC = s.nwg * n;
    a.lda = a.ldb = a.ldc = s.n; a.M = s.nwg; a.N = s.n; a.nc = s.nc;
    if (hipError_t e = launch_site_gemm<T, false, 1>(a, s.count, st); e != hipSuccess) return e;
    // over r: T(k1, n1; j)
    DftArgs d{};
    d.data = Tm; d.run = s.nwg * n; d.jump = per_t; d.stride = s.nwg * n; d.columns = s.count * d.run;
    d.lx = s.lx; d.ly = s.ly; d.nwg = s.nwg; d.ng = s.ng; d.g0 = g0;
    if (hipError_t e = launch_site_dft<T, false>(d, st); e != hipSuccess) return e;
    // U(K1; r', n2), in G's place
    a.A = Tm; a.B = P; a.C = G;
    a.sA = per_t; a.sB = s.nwg * n; a.sC = (int64_t)s.ng * s.ng; a.siteC = s.nwg;
    a.lda = a.ldb = s.n; a.ldc = s.ng; a.M = s.ng; a.N = s.nwg;
    if (hipError_t e = launch_site_gemm<T, true, 1>(a, s.count, st); e != hipSuccess) return e;
    // over r', scaled: G(K1; k2, n2)
    d.data = G; d.run = s.nwg; d.jump = s.ng; d.stride = s.nwg; d.columns = (int64_t)s.count * s.ng * s.nwg;
    d.scale = 1.0 / (s.beta * s.nc);
    return launch_site_dft<T, true>(d, st);
}

template <typename T>
hipError_t run_gsigma(const GsShape &s, const double *tau, const int32_t *site, const void *M, void *G, void *ws,
                      hipStream_t st) {
    using V = typename Cx2<T>::V;
    constexpr int kTM = sizeof(T) == 4 ? 4 : 2, kBM = 32 * kTM;   // FP64: registers and LDS allow 64-row blocks
    const int64_t per_e = (int64_t)s.ng * s.n;
    double2 *g0 = static_cast<double2 *>(ws);
    V *E = reinterpret_cast<V *>(g0 + s.ng);
    V *Tm = E + (int64_t)s.count * per_e;
    hipLaunchKernelGGL(g0_kernel, dim3((s.ng + 255) / 256), dim3(256), 0, st, s, g0);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (gsigma_by_sites<T>(s)) return run_gsigma_by_sites<T>(s, tau, site, M, G, g0, E, st);
    const int64_t total = (int64_t)s.count * per_e;
    if (total > 0) {
        int64_t grid = (total + 255) / 256;
        if (grid > 65536) grid = 65536;
        hipLaunchKernelGGL(phase_kernel<T>, dim3((unsigned)grid), dim3(256), 0, st, s, tau, site, E);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        CgArgs a1{};
        a1.A = E; a1.B = M; a1.C = Tm;
        a1.sA = per_e; a1.sB = (int64_t)s.n * s.n; a1.sC = per_e;
        a1.lda = s.n; a1.ldb = s.n; a1.ldc = s.n;
        a1.M = s.ng; a1.N = s.n; a1.K = s.n; a1.scale = 1.0;
        hipLaunchKernelGGL((cgemm_kernel<T, false, false, kTM>), dim3((s.n + BN - 1) / BN, (s.ng + kBM - 1) / kBM, s.count),
                           dim3(256), 0, st, a1);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    CgArgs a2{};
    a2.A = Tm; a2.B = E; a2.C = G; a2.g0 = g0;
    a2.sA = per_e; a2.sB = per_e; a2.sC = (int64_t)s.ng * s.ng;
    a2.lda = s.n; a2.ldb = s.n; a2.ldc = s.ng;
    a2.M = s.ng; a2.N = s.ng; a2.K = s.n; a2.scale = 1.0 / (s.beta * s.nc);
    // n = 0 still writes G = diag(g0) (the k loop is empty)
    hipLaunchKernelGGL((cgemm_kernel<T, true, true, kTM>), dim3((s.ng + BN - 1) / BN, (s.ng + kBM - 1) / kBM, s.count),
                       dim3(256), 0, st, a2);
    return hipGetLastError();
}

}  // namespace

int set_error(int code, const char *msg);

}  // namespace g4

extern "C" {

int g4_gsigma_workspace(int32_t lx, int32_t ly, int32_t nw, int32_t nwex, int32_t n, int32_t count, int32_t dtype,
                        uint64_t *bytes) {
    if (!bytes) return g4::set_error(G4_E_ARG, "bytes is NULL");
    if (lx < 1 || ly < 1 || (int64_t)lx * ly > 4096 || nw < 2 || (nw & 1) || nw > 4096 || nwex < 1 ||
        nwex > 4096 || n < 0 || count < 0 || (dtype != G4_IN_C128 && dtype != G4_IN_C64))
        return g4::set_error(G4_E_ARG, "bad G_sigma shape");
    *bytes = g4::workspace_bytes((int64_t)lx * ly * (nw + nwex - 1), n, count, dtype == G4_IN_C128 ? 16 : 8);
    return G4_OK;
}

int g4_gsigma(int32_t lx, int32_t ly, int32_t nw, int32_t nwex, double beta, double mu, double h, double t,
              int32_t spin, int32_t n, int32_t count, const double *tau, const int32_t *site, const void *M,
              int32_t dtype, void *G, void *workspace, uint64_t workspace_bytes, void *stream) {
    uint64_t need = 0;
    if (int rc = g4_gsigma_workspace(lx, ly, nw, nwex, n, count, dtype, &need); rc) return rc;
    if (!(beta > 0) || (spin != 0 && spin != 1)) return g4::set_error(G4_E_ARG, "beta must be positive, spin 0 or 1");
    const int64_t ng = (int64_t)lx * ly * (nw + nwex - 1);
    if (ng * ng >= ((int64_t)1 << 31)) return g4::set_error(G4_E_UNSUPPORTED, "G side above 46340");
    if (count > 65535) return g4::set_error(G4_E_UNSUPPORTED, "more than 65535 measurements per call");
    if (count == 0) return G4_OK;
    if (!G || (n > 0 && (!tau || !site || !M))) return g4::set_error(G4_E_ARG, "NULL pointer");
    if (!workspace || workspace_bytes < need)
        return g4::set_error(G4_E_ARG, "workspace too small (g4_gsigma_workspace gives the size)");
    g4::GsShape s;
    s.lx = lx; s.ly = ly; s.nc = lx * ly; s.nw = nw; s.nwg = nw + nwex - 1; s.ng = (int)ng; s.n = n;
    s.count = count; s.spin = spin; s.beta = beta; s.mu = mu; s.h = h; s.t = t;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const hipError_t e = dtype == G4_IN_C128 ? g4::run_gsigma<double>(s, tau, site, M, G, workspace, st)
                                             : g4::run_gsigma<float>(s, tau, site, M, G, workspace, st);
    if (e != hipSuccess) {
        char msg[160];
        std::snprintf(msg, sizeof(msg), "G_sigma launch: %s", hipGetErrorString(e));
        return g4::set_error(G4_E_HIP, msg);
    }
    return G4_OK;
}

}  // extern "C"
