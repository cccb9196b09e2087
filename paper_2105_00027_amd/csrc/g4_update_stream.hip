// Slice-update kernel that streams its operands from G straight into LDS, for
// gfx950: every kind (plain FP64, batched FP64, batched FP32) of the magnetic,
// charge and PP channels.  Compiled once per kind G4_KIND.
//
// Same tiles, thread mapping, arithmetic (operation by operation) and epilogue
// as update_kernel in g4_update.hpp.  There a measurement's operands passed
// through registers into LDS, two barriers a measurement, the direct vectors and
// the G(K2,K1) rows with them.  Here global_load_lds_dwordx4 copies 16-byte
// chunks (an FP64 element, or two neighbouring FP32 columns of one spin) from G
// and from the direct vectors into one of two buffers while the other is read,
// G(K2,K1) goes from G into the registers of the threads that multiply it, one
// measurement ahead, and a measurement has one barrier.
//
// FP32 columns come in pairs that start on an even column of G, so that a copy
// stays inside its row (Ng even; other slices keep update_kernel).  An
// exchange operand is then two 8-byte reads, one per spin, whose lanes (one row
// apart, odd row pitch) would use every other pair of banks: lanes in which
// bits 3 and 4 differ take the planes of a pair in the other order (plane m ^ 1
// at step m, kept in accumulator m until the epilogue), which is the other half of
// a chunk, and the reads spread over all banks.
// Whole 4x4 array, PH magnetic: FP32 passes of 16 measurements 2.80 -> 2.10 ms
// (5.5 TB/s beyond L2: what bounds it now), FP64 passes of 13 4.1 -> 3.3 ms (the
// LDS reads: 64 bytes per entry and measurement).
#include "g4_update.hpp"
#include "g4_dma.hpp"
#include "g4_stream.hpp"

#if !defined(G4_KIND)
#error "G4_KIND must be defined"
#endif

namespace g4 {
namespace upd {
namespace {

// Division of small numbers (e * d < 2^32) by one divisor: a product where the
// divisor is not known at compile time.  The generic copies do up to 22 of them per
// thread before the first measurement (54 frequencies, one channel, two
// measurements a pass: 51.6 -> 49.0 us).
template <bool CONST>
struct Div {
    int d;
    unsigned m;
    __device__ __forceinline__ explicit Div(int d_) : d(d_), m(0) {
        if (!CONST) m = __builtin_amdgcn_readfirstlane(0xffffffffu / (unsigned)d_ + 1);   // 0 for d = 1
    }
    __device__ __forceinline__ int operator()(int e) const {
        return CONST ? e / d : m ? (int)__umulhi((unsigned)e, m) : e;
    }
};

// Waves per SIMD the registers are held to: what the LDS allows where that fits
// without spilling.
template <int KIND, int EPT, int MG, int CH, int NWC>
constexpr int stream_waves() {
    constexpr int accs = ChanInfo<CH>::count * EPT * MG;
    constexpr bool mixed = ChanInfo<CH>::ph && ChanInfo<CH>::pp;
    if (KIND == 2) return NWC && accs <= 16 && EPT <= 2 && !mixed ? 3 : accs <= 16 || (NWC && accs <= 24 && EPT <= 2) ? 2 : 1;
    return accs <= 8 || (EPT == 1 && accs <= (NWC ? 16 : 12)) ? 2 : 1;
}

// NWC: nw fixed at compile time (0: taken from the arguments); the tile is then
// EPT * 256 / NWC rows and the LDS addresses are one base plus constants.
template <int KIND, int EPT, int MG, int CH, int NWC>
__global__ __launch_bounds__(NT, (stream_waves<KIND, EPT, MG, CH, NWC>())) void update_stream_kernel(UpdateArgs a) {
    using R = typename KindInfo<KIND>::R;
    using V = typename Cx<R>::V;
    using CI = ChanInfo<CH>;
    constexpr int EPC = sizeof(R) == 4 ? 2 : 1, SV = sizeof(V);
    constexpr bool PF = KindInfo<KIND>::prefetch;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x, l = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = NWC ? NWC : a.d.nw, nwg = a.d.nwg, nc = a.d.nc, n = a.d.n, ng = a.d.ng;
    const int tile = NWC ? EPT * (NT / NWC) : a.tile;
    const StreamGeom g = stream_geom(EPC, nw, min(tile, nw), MG, CH);   // a full tile's, for all tiles
    const int bufb = g.total * 16;
    R *sg = reinterpret_cast<R *>(smem_raw + stream_buffers(a.batch) * bufb);
    if (tid < a.batch) sg[tid] = (R)a.sign[tid];

    const int4 it = a.t.items[blockIdx.x];
    const int4 gr = a.t.groups[it.x];
    const int q = gr.x, m_lo = gr.y, M = gr.z, p0 = gr.w;
    const int k1 = it.y, k2 = it.z, c0 = it.w;
    const int T2 = min(tile, nw - c0);
    const int rowY = CI::ph ? a.t.kadd[k1 * nc + q] * nwg + m_lo : 0;
    const int colY = CI::ph ? a.t.kadd[k2 * nc + q] * nwg + c0 + m_lo : 0;
    const int rowZ = CI::pp ? a.t.ksub[q * nc + k2] * nwg + m_lo + nw - c0 - T2 : 0;
    const int colZ = CI::pp ? a.t.ksub[q * nc + k1] * nwg + m_lo : 0;
    const int sY = EPC == 2 ? colY & 1 : 0, sZ = EPC == 2 ? colZ & 1 : 0;

    // ---- copies: a part's chunks go in runs of 64, dealt to the waves in turn;
    // rows, columns and planes past the tile's or the group's end repeat its last
    // one (in bounds, never used), and runs of nothing else are left out.  Both spins have the same offsets.
    constexpr StreamGeom gc = stream_geom(EPC, NWC ? NWC : 2, NWC ? EPT * (NT / (NWC ? NWC : 1)) : 2, MG, CH);
    constexpr int KY = !CI::ph ? 0 : NWC ? stream_copies(gc.cY) : kStreamY, KZ = !CI::pp ? 0 : NWC ? stream_copies(gc.cZ) : kStreamZ;
    constexpr int KA = !CI::ph ? 0 : NWC ? stream_copies(gc.cA) : kStreamA, KB = !CI::ph ? 0 : NWC ? stream_copies(gc.cB) : kStreamB;
    const int hp = EPC == 2 ? (min(tile, nw) + 1) / 2 : min(tile, nw);   // chunks of b per plane
    unsigned offY[KY + 1], offZ[KZ + 1], offA[KA + 1], offB[KB + 1];
    const Div<NWC != 0> divY(g.yp), divZ(g.zn), divA(nw / EPC), divB(hp);
    static_for<0, KY>([&](auto k) {
        if (!NWC && (k * 4 + wave) * 64 >= g.cY) return;
        const int e = min((k * 4 + wave) * 64 + l, g.cY - 1);
        const int r = divY(e), c = e - r * g.yp;
        offY[k] = (unsigned)((rowY + min(r, nw + M - 2)) * ng + colY - sY + min(c, (T2 + M - 2 + sY) / EPC) * EPC) * SV;
    });
    static_for<0, KZ>([&](auto k) {
        if (!NWC && (k * 4 + wave) * 64 >= g.cZ) return;
        const int e = min((k * 4 + wave) * 64 + l, g.cZ - 1);
        const int r = divZ(e), c = e - r * g.zn;
        offZ[k] = (unsigned)((rowZ + min(r, T2 + M - 2)) * ng + colZ - sZ + min(c, (nw + M - 2 + sZ) / EPC) * EPC) * SV;
    });
    static_for<0, KA>([&](auto k) {
        if (!NWC && (k * 4 + wave) * 64 >= g.cA) return;
        const int e = min((k * 4 + wave) * 64 + l, g.cA - 1), w = nw / EPC;
        const int sm = divA(e), c = e - sm * w, sl = sm / MG, m = min(sm - sl * MG, M - 1);
        offA[k] = (unsigned)(sl * a.dir_slot_stride + (int64_t)(p0 + m) * n + k1 * nw + c * EPC) * SV;
    });
    static_for<0, KB>([&](auto k) {
        if (!NWC && (k * 4 + 3 - wave) * 64 >= g.cB) return;
        const int e = min((k * 4 + 3 - wave) * 64 + l, g.cB - 1);
        const int sm = divB(e), c = e - sm * hp, sl = sm / MG, m = min(sm - sl * MG, M - 1);
        offB[k] = (unsigned)(sl * a.dir_slot_stride + (int64_t)(p0 + m) * n + k2 * nw + min(c0 + c * EPC, nw - EPC)) * SV;
    });
    // ends of the parts: their last row or plane that the group reads
    const int wA = nw / EPC;
    const int eY = (nw + M - 1) * g.yp, eZ = (T2 + M - 1) * g.zn;
    const int eA = ((CI::nph - 1) * MG + M) * wA, eB = ((CI::nph - 1) * MG + M) * hp;
    const unsigned lds_base = (unsigned)(uintptr_t)(lds_t *)smem_raw;
    auto issue = [&](int b) __attribute__((always_inline)) {
        const unsigned buf = lds_base + (b & 1) * bufb;
        // part of `chunks` chunks from chunk o on, run s by wave w, without the runs
        // inside [lo, hi): a partial group's planes past the end
        auto part = [&](auto K, const unsigned *off, const char *base, int o, int chunks, int w, int lo, int hi) __attribute__((always_inline)) {
            static_for<0, decltype(K)::value>([&](auto k) {
                const int s = k * 4 + w;
                if (s * 64 < chunks && !(s * 64 >= lo && s * 64 + 64 <= hi)) dma16(base, off[k], buf + (o + s * 64) * 16);
            });
        };
        const int64_t go = (int64_t)b * a.g_stride * SV, vo = (int64_t)b * a.dir_b_stride * SV;
        const char *const pu = static_cast<const char *>(a.gu) + go, *const pd = static_cast<const char *>(a.gd) + go;
        if constexpr (CI::ph) {
            part(std::integral_constant<int, KY>{}, offY, pu, 0, eY, wave, eY, eY);
            part(std::integral_constant<int, KY>{}, offY, pd, g.oYd, eY, wave, eY, eY);
        }
        if constexpr (CI::pp) {
            part(std::integral_constant<int, KZ>{}, offZ, pu, g.oZu, eZ, wave, eZ, eZ);
            part(std::integral_constant<int, KZ>{}, offZ, pd, g.oZd, eZ, wave, eZ, eZ);
        }
        if constexpr (CI::ph) {
            part(std::integral_constant<int, KA>{}, offA, static_cast<const char *>(a.dir_a) + vo, g.oA, eA, wave, M * wA, MG * wA);
            part(std::integral_constant<int, KB>{}, offB, static_cast<const char *>(a.dir_b) + vo, g.oB, eB, 3 - wave, M * hp, MG * hp);
        }
    };

    // ---- this thread's entries
    const int RP = NT / nw;
    const bool act = tid < RP * nw;
    const int i1 = tid % nw, r0 = tid / nw;
    constexpr bool SWAP = EPC == 2 && CI::ph && MG > 1;
    const int gx = SWAP ? ((l >> 3) ^ (l >> 4)) & 1 : 0;     // PH planes in the other order within a pair
    const int64_t nn = (int64_t)n * n;
    const int64_t ebase = (((int64_t)p0 * nc + k2) * nc + k1) * nw * nw + (int64_t)(c0 + r0) * nw + i1;
    V acc[CI::count][EPT][MG];
    static_for<0, CI::count>([&](auto c) {
        static_for<0, EPT>([&](auto j) { static_for<0, MG>([&](auto m) { acc[c][j][m] = V{0, 0}; }); });
    });
    if constexpr (PF) {
        if (act)
            static_for<0, EPT>([&](auto j) {
                static_for<0, MG>([&](auto m) {
                    if (r0 + j * RP < T2 && m < M) {
                        const int64_t e = ebase + m * nn + (int64_t)j * RP * nw;
                        if (CI::mag) acc[0][j][m] = acc_ld(static_cast<const V *>(a.acc[0]) + e);
                        if (CI::chg) acc[CI::slot_chg][j][m] = acc_ld(static_cast<const V *>(a.acc[1]) + e);
                        if (CI::pp) acc[CI::slot_pp][j][m] = acc_ld(static_cast<const V *>(a.acc[2]) + e);
                    }
                });
            });
    }
    // G(K2,K1) of this thread's rows
    unsigned xoff[EPT];
    V xu[EPT], xd[EPT], nxu[EPT], nxd[EPT];
    static_for<0, EPT>([&](auto j) {
        xoff[j] = (unsigned)((k2 * nwg + c0 + min(r0 + j * RP, T2 - 1)) * ng + k1 * nwg + i1) * SV;
    });
    auto load_x = [&](int b) __attribute__((always_inline)) {
        const char *const pu = static_cast<const char *>(a.gu) + (int64_t)b * a.g_stride * SV;
        const char *const pd = static_cast<const char *>(a.gd) + (int64_t)b * a.g_stride * SV;
        static_for<0, EPT>([&](auto j) {
            nxu[j] = ld(reinterpret_cast<const V *>(pu + xoff[j]));
            nxd[j] = ld(reinterpret_cast<const V *>(pd + xoff[j]));
        });
    };
    // byte addresses within a buffer: plane m adds m steps (and gx one more or less), row j its own
    const int stepY = g.yp * 16 + SV, stepZ = g.zn * 16 + SV;
    const int fy = i1 * g.yp * 16 + (r0 + sY) * SV;
    const int fy2[2] = {fy + gx * stepY, fy - gx * stepY};
    const int fa = g.oA * 16 + i1 * SV;
    const int fa2[2] = {fa + gx * nw * SV, fa - gx * nw * SV};
    int fb[EPT], fz[EPT];
    static_for<0, EPT>([&](auto j) {
        const int r = min(r0 + j * RP, T2 - 1);
        const int half = EPC == 2 ? c0 + r - min(c0 + (r & ~1), nw - 2) : 0;
        fb[j] = (g.oB + r / EPC) * 16 + half * SV;
        fz[j] = g.oZu * 16 + (T2 - 1 - r) * g.zn * 16 + (nw - 1 - i1 + sZ) * SV;
    });
    const int fbx[2] = {gx * hp * 16, -gx * hp * 16};

    if (a.batch > 0) {
        issue(0);
        load_x(0);
    }
    const bool full = T2 == tile && M == MG;
    for (int b = 0; b < a.batch; ++b) {
        wait_vm(0);
        __syncthreads();                 // b's copies landed everywhere; the other buffer is free
        if (b + 1 < a.batch) issue(b + 1);
        if (!act) continue;
        const R s = sg[b];
        // G(K2,K1) times -s_b for the PH exchange (its minus folded in), +s_b for PP
        static_for<0, EPT>([&](auto j) {
            xu[j] = cscale(nxu[j], CI::ph ? -s : s);
            xd[j] = cscale(nxd[j], CI::ph ? -s : s);
        });
        __builtin_amdgcn_sched_barrier(0);
        load_x(min(b + 1, a.batch - 1));
        const unsigned char *const L = smem_raw + (b & 1) * bufb;
        auto at = [&](int o) __attribute__((always_inline)) { return ld(reinterpret_cast<const V *>(L + o)); };
        struct Ops {
            V yu[EPT], yd[EPT], zu[EPT], zd[EPT];
            V av[CI::nph > 0 ? CI::nph : 1], bv[CI::nph > 0 ? CI::nph : 1][EPT];
        };
        auto load = [&](auto m, Ops &o) __attribute__((always_inline)) {
            static_for<0, EPT>([&](auto j) {
                const int rj = j * (NWC ? NT / (NWC ? NWC : 1) : RP);
                if (CI::ph) {
                    o.yu[j] = at(fy2[m & 1] + m * stepY + rj * SV);
                    o.yd[j] = at(fy2[m & 1] + m * stepY + rj * SV + g.oYd * 16);
                }
                if (CI::pp) {
                    o.zu[j] = at(fz[j] + m * stepZ);
                    o.zd[j] = at(fz[j] + m * stepZ + (g.oZd - g.oZu) * 16);
                }
                static_for<0, CI::nph>([&](auto c) { o.bv[c][j] = at(fb[j] + fbx[m & 1] + (c * MG + m) * hp * 16); });
            });
            static_for<0, CI::nph>([&](auto c) { o.av[c] = at(fa2[m & 1] + (c * MG + m) * nw * SV); });
        };
        auto compute = [&](auto m, const Ops &o) __attribute__((always_inline)) {
            static_for<0, EPT>([&](auto j) {
                if constexpr (CI::nph == 2) {
                    // both PH channels share the exchange sum: computed once
                    V ex = cmul(xu[j], o.yu[j]);
                    cmac(ex, xd[j], o.yd[j]);
                    static_for<0, 2>([&](auto c) {
                        V &r = acc[c][j][m];
                        cmac(r, o.av[c], o.bv[c][j]);
                        r.x += ex.x;
                        r.y += ex.y;
                    });
                } else if constexpr (CI::nph == 1) {
                    V &r = acc[0][j][m];
                    cmac(r, o.av[0], o.bv[0][j]);
                    cmac(r, xu[j], o.yu[j]);
                    cmac(r, xd[j], o.yd[j]);
                }
                if constexpr (CI::pp) {
                    V &r = acc[CI::slot_pp][j][m];
                    if (CI::ph) {
                        // the PP term takes +s_b: undo the PH negation folded into x
                        V w = cmul(o.zu[j], xd[j]);
                        cmac(w, o.zd[j], xu[j]);
                        r.x -= w.x;
                        r.y -= w.y;
                    } else {
                        cmac(r, o.zu[j], xd[j]);
                        cmac(r, o.zd[j], xu[j]);
                    }
                }
            });
        };
        // plane m + 1's operands are read before plane m's arithmetic; a partial
        // group skips the pairs of planes it does not have
        auto run = [&](auto FULL) __attribute__((always_inline)) {
            constexpr bool F = decltype(FULL)::value;
            Ops o[2];
            load(std::integral_constant<int, 0>{}, o[0]);
            static_for<0, MG>([&](auto m) {
                if constexpr (m + 1 < MG)
                    if (F || ((m + 1) & ~1) < M) load(std::integral_constant<int, m + 1>{}, o[(m + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                if (F || (m & ~1) < M) compute(m, o[m & 1]);
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        if (full) run(std::true_type{});
        else run(std::false_type{});
    }
    if (!act) return;
    // planes back in their places, so that a store instruction's lanes write one
    // run (4x4, 54 frequencies, 10 planes, magnetic and charge, two measurements a
    // pass: 262 -> 211 us)
    if constexpr (SWAP)
        static_for<0, CI::nph>([&](auto c) {
            static_for<0, EPT>([&](auto j) {
                static_for<0, MG / 2>([&](auto h) {
                    V &p = acc[c][j][2 * h], &q = acc[c][j][2 * h + 1];
                    const V t = p;
                    p.x = gx ? q.x : p.x;
                    p.y = gx ? q.y : p.y;
                    q.x = gx ? t.x : q.x;
                    q.y = gx ? t.y : q.y;
                });
            });
        });
    static_for<0, EPT>([&](auto j) {
        static_for<0, MG>([&](auto m) {
            if (r0 + j * RP >= T2) return;
            const int64_t ej = ebase + (int64_t)j * RP * nw;
            if constexpr (PF) {
                if (m < M) {
                    const int64_t e = ej + m * nn;
                    if (CI::mag) acc_st(static_cast<V *>(a.acc[0]) + e, acc[0][j][m]);
                    if (CI::chg) acc_st(static_cast<V *>(a.acc[1]) + e, acc[CI::slot_chg][j][m]);
                    if (CI::pp) acc_st(static_cast<V *>(a.acc[2]) + e, acc[CI::slot_pp][j][m]);
                }
            } else {
                if (CI::ph && m < M) {
                    if (CI::mag) acc_update(a.acc[0], a.acc_kind, ej + m * nn, acc[0][j][m]);
                    if (CI::chg) acc_update(a.acc[1], a.acc_kind, ej + m * nn, acc[CI::slot_chg][j][m]);
                }
                if (CI::pp && m < M) acc_update(a.acc[2], a.acc_kind, ej + m * nn, acc[CI::slot_pp][j][m]);
            }
        });
    });
}

template <int EPT, int MG, int NWC>
hipError_t launch_stream_ch(int channels, int nitems, size_t lds, const UpdateArgs &a, hipStream_t s) {
    const void *fn = nullptr;
    switch (channels) {
#define G4_CASE(CHV)                                                                                   \
    case CHV:                                                                                          \
        fn = reinterpret_cast<const void *>(&update_stream_kernel<G4_KIND, EPT, MG, CHV, NWC>);        \
        break;
        G4_CASE(1) G4_CASE(2) G4_CASE(3) G4_CASE(4) G4_CASE(5) G4_CASE(6) G4_CASE(7)
#undef G4_CASE
        default: return hipErrorInvalidValue;
    }
    if (hipError_t e = ensure_lds_limit(fn, lds); e != hipSuccess) return e;
    UpdateArgs arg = a;
    void *params[] = {&arg};
    return hipLaunchKernel(fn, dim3(nitems), dim3(NT), params, lds, s);
}

}  // namespace
}  // namespace upd

#define G4_SNAME2(k) launch_update_stream_k##k
#define G4_SNAME(k) G4_SNAME2(k)

hipError_t G4_SNAME(G4_KIND)(int channels, int ept, int mgroup, int nitems, size_t lds, const UpdateArgs &a,
                             hipStream_t s) {
    using namespace upd;
    // nw = 64: the copies with the sizes compiled in
#define G4_E(e, mg)                                                                                          \
    if (ept == e && mgroup == mg)                                                                            \
        return a.d.nw == 64 && a.tile == e * 4 ? launch_stream_ch<e, mg, 64>(channels, nitems, lds, a, s)     \
                                               : launch_stream_ch<e, mg, 0>(channels, nitems, lds, a, s);
    G4_E(1, 8) G4_E(1, 4) G4_E(2, 8) G4_E(2, 4)
#if G4_KIND == 2
    G4_E(4, 4)
#endif
#undef G4_E
    return hipErrorInvalidValue;
}

}  // namespace g4
