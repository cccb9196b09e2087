// C ABI of the G4 slice library: validation, index tables, device memory,
// the per-call pass schedule and the synchronous copies.  See include/g4.h
// for the contract of each entry point.
#include "../../include/g4.h"

#include <hip/hip_runtime.h>

#include <dlfcn.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <new>
#include <sstream>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include "g4_internal.hpp"
#include "g4_stream.hpp"

using namespace g4;

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

// Named ranges for rocprofv3 --marker-trace: the roctx library is opened at
// the first pass (dlopen, so the library does not depend on it); absent, or
// with G4_ROCTX=0, the ranges cost nothing.
struct RoctxApi {
    int (*push)(const char *);
    int (*pop)();
};
const RoctxApi &roctx_api() {
    static const RoctxApi api = [] {
        RoctxApi a{nullptr, nullptr};
        const char *e = std::getenv("G4_ROCTX");
        if (e && e[0] == '0') return a;
        if (void *lib = dlopen("librocprofiler-sdk-roctx.so.1", RTLD_NOW | RTLD_LOCAL)) {
            a.push = reinterpret_cast<int (*)(const char *)>(dlsym(lib, "roctxRangePushA"));
            a.pop = reinterpret_cast<int (*)()>(dlsym(lib, "roctxRangePop"));
            if (!a.push || !a.pop) a = RoctxApi{nullptr, nullptr};
        }
        return a;
    }();
    return api;
}
struct RoctxRange {
    bool on;
    explicit RoctxRange(const char *name) : on(roctx_api().push != nullptr) {
        if (on) roctx_api().push(name);
    }
    ~RoctxRange() {
        if (on) roctx_api().pop();
    }
};

constexpr int kMaxNw = 256;      // one K1 row per lane group of a 256-thread block
constexpr int kMaxBatch = kMaxPassBatch;
constexpr int kSignSlots = 8;
constexpr uint64_t kScratchEntries = 4u << 20;   // readback/load staging, complex128
constexpr int kReadbackLanes = 8;                // threads of a large readback, one pinned slot each
constexpr uint64_t kLaneEntries = kScratchEntries / kReadbackLanes;   // 8 MiB per slot

int acc_entry_bytes(int acc) { return acc == G4_ACC_C64 ? 8 : 16; }

int popcount3(uint32_t c) { return (c & 1) + ((c >> 1) & 1) + ((c >> 2) & 1); }

// Everything derived from a configuration, computed without touching HIP.
struct Plan {
    Dims d;
    int prec;          // 0 FP64 products, 1 FP32
    int kind;          // update kernel: 0 plain FP64, 1 batched FP64, 2 batched FP32
    int variant;       // 0 VALU kernel, 1 MFMA direct term, 2 packed operands, 3 deep packed,
                       // 4 packed with the direct term on MFMA (G4_VARIANT_*)
    int split;         // direct term from split operands on MFMA: 0 no, 1 bf16 hi+lo, 2 fp16 hi+lo
    int persistent;    // packed variants under G4_F_PERSISTENT: a persistent grid
    int batch;         // measurements per pass
    int mgroup;        // transfer planes per work tile (compile-time bound)
    int tile;          // K2 rows per work tile
    int ept;           // K2 rows per thread
    int slots;         // direct-vector slots (bit 0 magnetic, bit 1 charge)
    int nslots;
    uint64_t entries;  // per channel
    int ldp;           // packed variant: row pitch of a packed G matrix (16-byte elements)
    int pcb;           // packed variant: column pitch of one momentum block (Nwg rounded up to 8)
    uint64_t pack_stride;   // bytes per measurement of the packed buffer (G + direct vectors)
    uint64_t acc_bytes, dir_bytes, stage_bytes, sign_bytes, scratch_bytes, table_bytes, pack_bytes;
    uint64_t total_bytes;
    std::vector<int32_t> qlist;
};

// Variants whose pass packs G first (and need the packed buffer).
bool uses_pack(int variant) {
    return variant == G4_VARIANT_PACKED || variant == G4_VARIANT_PACKED_DEEP || variant == G4_VARIANT_PACKED_MFMA;
}

// Plane groups of a slice (see build_work)
int plane_groups(const Plan &P) {
    int n = 0;
    const int64_t nwex = P.d.nwex, end = P.d.q_begin + P.d.planes;
    for (int64_t iQ = P.d.q_begin; iQ < end; ++n) iQ = std::min({end, (iQ / nwex + 1) * nwex, iQ + P.mgroup});
    return n;
}

// A packed plan whose slice has too few planes to repay the packing of G: the
// streamed kernel takes the operands from G itself.
bool streams(const Plan &P, uint32_t channels) {
    return P.variant == G4_VARIANT_PACKED && !P.split && !P.persistent &&
           stream_packed((int)channels, P.ept, P.mgroup, P.tile, P.d, P.batch, plane_groups(P)) &&
           stream_runs(P.kind, (int)channels, P.ept, P.mgroup, P.tile, P.d, (int64_t)P.batch * P.d.planes * P.d.n,
                       P.batch);
}

// Bytes of the packed buffer that a plan needs, for passes of max_batch: none
// where it streams.
uint64_t pack_need(const Plan &P, const g4_config &c) {
    return uses_pack(P.variant) && !streams(P, c.channels) ? (uint64_t)c.max_batch * P.pack_stride : 0;
}

// Transfer planes per work tile: 8 when Nwex allows, else 4, else 1.
// G4_PLANE_GROUP=1|4|8 in the environment sets it instead, for measurements
// (a group larger than Nwex is always partial; the packed MFMA plans, which
// need plane pairs, reject 1).
int choose_mgroup(int nwex) {
    if (const char *e = std::getenv("G4_PLANE_GROUP")) {
        const int g = std::atoi(e);
        if (g == 1 || g == 4 || g == 8) return g;
    }
    return nwex == 1 ? 1 : (nwex <= 4 ? 4 : 8);
}

// Largest K2-rows-per-thread count keeping the register accumulators and the
// LDS tiles modest; tile = ept * (256 / nw).
int choose_ept(int prec, int nch, int mgroup, int nw) {
    const int rp = 256 / nw;
    const int budget = prec == 0 ? 8 : 16;    // complex accumulators per thread
    int ept = 8;
    while (ept > 1 && (nch * ept * mgroup > budget || ept * rp > nw)) ept >>= 1;
    return ept;
}

int validate(const g4_config *c, Plan *p) {
    if (!c) return fail(G4_E_ARG, "config is NULL");
    if (c->abi_version != G4_ABI_VERSION)
        return fail(G4_E_ARG, "abi_version %u, library speaks %u", c->abi_version, G4_ABI_VERSION);
    if (c->lx < 1 || c->ly < 1 || (int64_t)c->lx * c->ly > 4096)
        return fail(G4_E_ARG, "cluster %d x %d out of range", c->lx, c->ly);
    const int nc = c->lx * c->ly;
    if (c->nw < 2 || (c->nw & 1)) return fail(G4_E_ARG, "nw=%d must be even and >= 2", c->nw);
    if (c->nwex < 1) return fail(G4_E_ARG, "nwex=%d must be >= 1", c->nwex);
    if (c->nq < 1 || c->nq > nc) return fail(G4_E_ARG, "nq=%d outside [1, %d]", c->nq, nc);
    std::vector<int32_t> ql(c->nq);
    std::vector<char> seen(nc, 0);
    for (int i = 0; i < c->nq; ++i) {
        const int32_t q = c->q_list ? c->q_list[i] : i;
        if (q < 0 || q >= nc) return fail(G4_E_ARG, "q_list[%d]=%d outside [0, %d)", i, q, nc);
        if (seen[q]) return fail(G4_E_ARG, "q_list repeats momentum %d", q);
        seen[q] = 1;
        ql[i] = q;
    }
    const int64_t nQ = (int64_t)c->nq * c->nwex;
    if (c->q_begin < 0 || c->q_end > nQ || c->q_begin >= c->q_end)
        return fail(G4_E_ARG, "slice [%lld, %lld) not inside [0, %lld)", (long long)c->q_begin,
                    (long long)c->q_end, (long long)nQ);
    // channel families: {1, 2, 4}, {8, 16, 32} (spin-resolved PH), {64, 128} (PP singlet / triplet)
    const bool spin_set = (c->channels & ~7u) != 0;
    const int families = ((c->channels & 7u) ? 1 : 0) + ((c->channels & 56u) ? 1 : 0) + ((c->channels & 192u) ? 1 : 0);
    if (c->channels == 0 || (c->channels & ~255u) || families != 1)
        return fail(G4_E_ARG, "channels bitmask 0x%x invalid (one family: bits of 1|2|4, 8|16|32 or 64|128)",
                    c->channels);
    if (c->g_in != G4_IN_C128 && c->g_in != G4_IN_C64) return fail(G4_E_ARG, "g_in=%d", c->g_in);
    if (c->prod < G4_PROD_F64 || c->prod > G4_PROD_F16X2) return fail(G4_E_ARG, "prod=%d", c->prod);
    if (c->acc < G4_ACC_C128 || c->acc > G4_ACC_C64) return fail(G4_E_ARG, "acc=%d", c->acc);
    if (c->mode != G4_MODE_PLAIN && c->mode != G4_MODE_BATCHED) return fail(G4_E_ARG, "mode=%d", c->mode);
    if (c->flags & ~(uint32_t)(G4_F_CHECK_FINITE | G4_F_KERNEL_TIMING | G4_F_GRAPH | G4_F_MFMA | G4_F_PACKED |
                               G4_F_PACKED_DEEP | G4_F_PERSISTENT))
        return fail(G4_E_ARG, "unknown flags 0x%x", c->flags);
    if (c->device < 0) return fail(G4_E_ARG, "device=%d", c->device);
    if (c->mode == G4_MODE_PLAIN) {
        if (c->prod != G4_PROD_F64 || c->g_in != G4_IN_C128 || c->acc != G4_ACC_C128)
            return fail(G4_E_ARG, "plain mode is FP64 throughout: g_in C128, prod F64, acc C128");
    } else if (c->max_batch < 1 || c->max_batch > kMaxBatch) {
        return fail(G4_E_ARG, "max_batch=%d outside [1, %d]", c->max_batch, kMaxBatch);
    }
    if (c->prod == G4_PROD_F64 && c->g_in != G4_IN_C128)
        return fail(G4_E_ARG, "FP64 products need complex128 G");
    if (c->tile < 0) return fail(G4_E_ARG, "tile=%d", c->tile);

    Plan &P = *p;
    Dims &d = P.d;
    d.lx = c->lx;
    d.ly = c->ly;
    d.nc = nc;
    d.nw = c->nw;
    d.nwex = c->nwex;
    d.nwg = c->nw + c->nwex - 1;
    const int64_t ng = (int64_t)nc * d.nwg;
    const int64_t n = (int64_t)nc * c->nw;
    if (ng > (1 << 20) || n > (1 << 20)) return fail(G4_E_ARG, "G side %lld too large", (long long)ng);
    if (ng * ng >= (int64_t)1 << 31)
        return fail(G4_E_UNSUPPORTED, "G side %lld: matrices above 2^31 elements", (long long)ng);
    d.ng = (int)ng;
    d.n = (int)n;
    d.planes = (int)(c->q_end - c->q_begin);
    d.q_begin = c->q_begin;
    P.entries = (uint64_t)d.planes * (uint64_t)n * (uint64_t)n;
    P.qlist = ql;

    // --- what this build runs
    if (c->nw > kMaxNw) return fail(G4_E_UNSUPPORTED, "nw=%d above %d", c->nw, kMaxNw);
    P.split = c->prod == G4_PROD_BF16X2 ? 1 : (c->prod == G4_PROD_F16X2 ? 2 : 0);
    P.prec = c->prod == G4_PROD_F64 ? 0 : 1;
    P.kind = c->mode == G4_MODE_PLAIN ? 0 : (P.prec == 0 ? 1 : 2);
    P.batch = c->mode == G4_MODE_PLAIN ? 1 : c->max_batch;
    P.mgroup = choose_mgroup(c->nwex);
    const int nch = popcount3((uint32_t)acc_slots((int)c->channels));
    const int rp = 256 / c->nw;
    const uint32_t vf = c->flags & (G4_F_MFMA | G4_F_PACKED | G4_F_PACKED_DEEP);
    if (popcount3(vf >> 3) > 1 && vf != (G4_F_MFMA | G4_F_PACKED))
        return fail(G4_E_ARG, "G4_F_MFMA, G4_F_PACKED and G4_F_PACKED_DEEP are exclusive "
                              "(except G4_F_PACKED | G4_F_MFMA)");
    P.variant = vf == (G4_F_MFMA | G4_F_PACKED) ? G4_VARIANT_PACKED_MFMA
              : (c->flags & G4_F_MFMA) ? G4_VARIANT_MFMA
              : (c->flags & G4_F_PACKED) ? G4_VARIANT_PACKED
              : (c->flags & G4_F_PACKED_DEEP) ? G4_VARIANT_PACKED_DEEP : G4_VARIANT_VALU;
    if (spin_set && (P.variant != G4_VARIANT_VALU || P.split))
        return fail(G4_E_UNSUPPORTED, "spin-resolved and PP singlet / triplet channels run on the VALU kernels "
                                      "only (no G4_F_MFMA, G4_F_PACKED, G4_F_PACKED_DEEP or split products)");
    // split-precision plans run the packed kernels (their direct vectors can be
    // read as zeros there, with no test in the arithmetic loop)
    if (P.split && P.variant == G4_VARIANT_VALU) P.variant = G4_VARIANT_PACKED;
    const bool packed = uses_pack(P.variant);
    P.persistent = packed && (c->flags & G4_F_PERSISTENT) ? 1 : 0;
    if (packed && P.kind != 2) return fail(G4_E_UNSUPPORTED, "packed operands need batched FP32 products");
    if (P.variant == G4_VARIANT_PACKED_MFMA) {
        // MFMA accumulator layout: per plane pair, 8 K2 rows x 2 planes x 64 columns
        if (P.split) return fail(G4_E_UNSUPPORTED, "packed MFMA kernel: the split direct term runs separately");
        if (c->nw != 64) return fail(G4_E_UNSUPPORTED, "packed MFMA kernel needs nw = 64");
        if (c->channels & G4_PP_UPDOWN) return fail(G4_E_UNSUPPORTED, "packed MFMA kernel: PH channels only");
        if (c->tile && c->tile != 8) return fail(G4_E_UNSUPPORTED, "packed MFMA kernel uses 8-row tiles");
        if (P.mgroup < 4) return fail(G4_E_UNSUPPORTED, "packed MFMA kernel needs plane pairs (nwex >= 2)");
    }
    // K2 rows covered by one sweep of the block's threads
    const int rp_v = P.variant == G4_VARIANT_PACKED_DEEP ? 512 / c->nw : rp;
    if (P.variant == 1) {
        // MFMA kernel: 16-row tiles, 64-column slabs per wave, register budget
        if (P.kind != 2 || P.split) return fail(G4_E_UNSUPPORTED, "MFMA direct term needs batched FP32 products");
        if (c->nw % 64 || c->nw > 128) return fail(G4_E_UNSUPPORTED, "MFMA direct term needs nw = 64 or 128");
        if (nch * (c->nw / 64) * P.mgroup > 16)
            return fail(G4_E_UNSUPPORTED, "MFMA direct term: %d channels x %d slabs x %d planes exceed the register budget",
                        nch, c->nw / 64, P.mgroup);
        if (c->tile && c->tile != 16) return fail(G4_E_UNSUPPORTED, "MFMA direct term uses 16-row tiles");
    }
    if (P.variant == 1) {
        P.ept = 0;
        P.tile = 16;
    } else if (P.variant == G4_VARIANT_PACKED_MFMA) {
        P.ept = 2;                    // tile 8: the copies of the packed kernel with 2 rows per thread
    } else if (c->tile) {
        if (c->tile % rp_v || c->tile >= c->nw + rp_v)
            return fail(G4_E_UNSUPPORTED, "tile=%d: must be a multiple of %d below nw + %d", c->tile, rp_v, rp_v);
        const int e = c->tile / rp_v;
        if (e != 1 && e != 2 && e != 4 && e != 8) return fail(G4_E_UNSUPPORTED, "tile=%d: tile/%d must be 1, 2, 4 or 8", c->tile, rp_v);
        P.ept = e;
    } else {
        P.ept = choose_ept(P.prec, nch, P.mgroup, c->nw);
        // packed FP32 with three channels on plane groups of 4 (the 8x8
        // three-channel slice): two K2 rows per thread stage a fifth fewer
        // bytes per entry update than the register budget's one, and ran 8%
        // faster there (75.7 against 82.3 ms per 32-measurement pass)
        if (P.variant == G4_VARIANT_PACKED && nch == 3 && P.mgroup == 4 && P.ept == 1 && 2 * rp_v <= c->nw)
            P.ept = 2;
        if (P.variant == G4_VARIANT_PACKED_DEEP) P.ept = std::min(P.ept, 2);
        // packed operands move direct vectors in pairs: the default tile is even
        const int emax = P.variant == G4_VARIANT_PACKED_DEEP ? 2 : 8;
        while (packed && P.ept < emax && ((P.ept * rp_v) % 2 || std::min(P.ept * rp_v, c->nw) % 2)) P.ept *= 2;
    }
    if (P.variant == G4_VARIANT_PACKED_DEEP && P.ept > 2)
        return fail(G4_E_UNSUPPORTED, "deep packed blocks take one or two K2 rows per thread (tile=%d)", P.ept * rp_v);
    if (P.variant != 1) P.tile = P.ept * rp_v;
    if (update_lds_bytes(P.kind, (int)c->channels, P.tile, P.mgroup, d, P.variant) > 160 * 1024)
        return fail(G4_E_UNSUPPORTED, "LDS tile above 160 KiB");
    P.slots = direct_recipes((int)c->channels);
    P.nslots = __builtin_popcount((unsigned)P.slots);
    // packed operands: one block per measurement, [G rows of ldp 16-byte
    // elements | direct vectors a | b]; every copy offset inside it is 32-bit.
    // Momentum blocks of columns start on 128-byte boundaries; one zero
    // column at least follows the last.
    P.pcb = (d.nwg + 7) / 8 * 8;
    P.ldp = (int)((d.nc * P.pcb + 1 + 7) / 8 * 8);
    P.pack_stride = ((uint64_t)ng * P.ldp * 16 + 2ull * P.nslots * d.planes * n * 8 + 255) / 256 * 256;
    P.pack_bytes = 0;
    if (packed) {
        const bool deep = P.variant == G4_VARIANT_PACKED_DEEP;
        const int T2 = std::min(P.tile, c->nw);
        const bool areg = P.variant == G4_VARIANT_PACKED &&
                          packed_a_in_regs(c->nw, P.tile, P.mgroup, (int)c->channels, deep);
        const PackedGeom g = packed_geom(c->nw, T2, P.mgroup, (int)c->channels, deep, areg);
        if (P.tile % 2 || T2 % 2) return fail(G4_E_UNSUPPORTED, "packed operands need an even tile (tile=%d)", P.tile);
        if (packed_slots(g, deep) > (areg ? kPackedSlotsAReg : kPackedSlots))
            return fail(G4_E_UNSUPPORTED, "packed operands: %d staging chunks per tile above %d", g.nbuf,
                        kPackedSlots * packed_threads(deep));
        if (P.pack_stride >= (1ull << 31))
            return fail(G4_E_UNSUPPORTED, "packed operands: %llu bytes per measurement above 2^31",
                        (unsigned long long)P.pack_stride);
        P.pack_bytes = pack_need(P, *c);
    }

    // --- device memory
    const uint64_t el = P.prec == 0 ? 16 : 8;
    P.acc_bytes = P.entries * (uint64_t)acc_entry_bytes(c->acc);
    P.dir_bytes = 2ull * P.nslots * P.batch * (uint64_t)d.planes * n * el;
    if ((uint64_t)P.nslots * P.batch * d.planes * n >= (1ull << 31))
        return fail(G4_E_UNSUPPORTED, "direct-term vectors above 2^31 elements; lower max_batch");
    P.stage_bytes = (P.prec == 1 && c->g_in == G4_IN_C128) ? 2ull * P.batch * ng * ng * 8 : 0;
    P.sign_bytes = (uint64_t)kSignSlots * kMaxBatch * sizeof(double);
    P.scratch_bytes = std::min<uint64_t>(P.entries, kScratchEntries) * 16;
    // work tiles of the smallest tile any plan may install later (one K2 row):
    // the kernels take the tile count as a 32-bit grid size
    const uint64_t nitems_max = (uint64_t)d.planes * nc * nc * (uint64_t)c->nw;
    if (nitems_max >= (1ull << 31))
        return fail(G4_E_UNSUPPORTED, "%llu work tiles at one K2 row per tile: above 2^31",
                    (unsigned long long)nitems_max);
    P.table_bytes = 2ull * nc * nc * 4 + (uint64_t)d.planes * 16 + nitems_max * 16 + (uint64_t)d.planes * 8;
    P.total_bytes = P.acc_bytes * nch + P.dir_bytes + P.stage_bytes + P.sign_bytes +
                    P.scratch_bytes + P.table_bytes + P.pack_bytes;
    return G4_OK;
}

// Host-built integer index maps: momentum addition/subtraction on cluster
// coordinates with wraparound; plane decode iQ -> (q, m).
void build_momentum_maps(const Dims &d, std::vector<int32_t> &kadd, std::vector<int32_t> &ksub) {
    kadd.assign((size_t)d.nc * d.nc, 0);
    ksub.assign((size_t)d.nc * d.nc, 0);
    for (int k = 0; k < d.nc; ++k) {
        const int kx = k % d.lx, ky = k / d.lx;
        for (int q = 0; q < d.nc; ++q) {
            const int qx = q % d.lx, qy = q / d.lx;
            kadd[(size_t)k * d.nc + q] = (kx + qx) % d.lx + d.lx * ((ky + qy) % d.ly);
            ksub[(size_t)q * d.nc + k] = (qx - kx + d.lx) % d.lx + d.lx * ((qy - ky + d.ly) % d.ly);
        }
    }
}

void build_planes(const Plan &P, int nwex, std::vector<int2> &plane_qm) {
    plane_qm.resize(P.d.planes);
    for (int p = 0; p < P.d.planes; ++p) {
        const int64_t iQ = P.d.q_begin + p;
        plane_qm[p] = int2{P.qlist[(size_t)(iQ / nwex)], (int)(iQ % nwex)};
    }
}

// The variant of launch_update that a pass of nb measurements runs: the plan's,
// or the streamed kernel.  `slot_stride`: elements between direct-vector slots.
int pass_variant(const Plan &P, uint32_t channels, int groups, int items, int nb, int64_t slot_stride) {
    if (P.variant == G4_VARIANT_PACKED) return streams(P, channels) ? kVariantStreamed : P.variant;
    if (P.variant != G4_VARIANT_VALU) return P.variant;
    return stream_runs(P.kind, (int)channels, P.ept, P.mgroup, P.tile, P.d, slot_stride, nb) &&
                   stream_pays(P.kind, (int)channels, P.ept, P.mgroup, P.tile, P.d, nb, groups, items)
               ? kVariantStreamed : P.variant;
}

// Its name (G4_LOG, ranges)
const char *kernel_name(int variant) {
    static const char *names[] = {"registers", "mfma-direct", "packed", "packed-deep", "packed-mfma-direct", "streamed"};
    return variant >= 0 && variant <= kVariantStreamed ? names[variant] : "?";
}

// work tiles of a list that leaves none out
int64_t whole_tiles(const Plan &P) {
    return (int64_t)plane_groups(P) * P.d.nc * P.d.nc * ((P.d.nw + P.tile - 1) / P.tile);
}

double pair_bytes(const Plan &P) { return 2.0 * P.d.ng * P.d.ng * (P.kind == 2 ? 8 : 16); }   // both spins' matrices

// PP singlet and triplet, batched: rows K2 and Q - K2 may be summed once (kTileMirror)
bool takes_pair_rows(const Plan &P, uint32_t channels) {
    return P.kind != 0 && (channels & (G4_PP_SINGLET | G4_PP_TRIPLET)) != 0;
}

// ... and are where the sums saved outweigh the partner row's read and write of the
// accumulators, which nothing overlaps: single planes, and longer passes over more
// frequencies.  Time of whole tiles over this, median (5% lowest, 5% highest), on
// 4544 random shapes:
//   matrices beyond an XCD's L2: taken 1.38 (0.98, 2.11), left 0.99 (0.78, 1.30)
//   smaller ones, which need two tiles a CU besides: 1.22 (0.97, 1.79), left 0.96
//     (0.76, 1.07)
bool pair_rows_once(const Plan &P, uint32_t channels) {
    if (!takes_pair_rows(P, channels)) return false;
    const int nw = P.d.nw;
    const double pair = pair_bytes(P);
    const bool single = P.mgroup == 1 || P.d.planes == 1;
    if (pair <= 4e6) return whole_tiles(P) > 512 && (single || (nw >= 28 && P.batch > 10));
    if (single) return true;
    return nw >= 42 ? P.batch >= 4 || pair > 26e6 : nw >= 28 ? P.batch >= 8 || pair > 78e6 : P.batch >= 8 && P.mgroup < 8;
}

// The tile order of a plan (see build_work): runs of constant k1 + q for packed
// operands, windows for register-staged and streamed ones; or orbits (on 6996
// random shapes, windows over orbits with the streamed kernel, or runs over orbits
// with the packed one, median, 5% lowest and highest)
//   packed operands of fewer than 32 planes: 1.01 (0.96, 1.13), but for several
//     groups of single planes: 0.99 (0.88, 1.03);
//   one plane group, whose matrices exceed an XCD's L2: plain 1.02 (0.98, 1.10);
//     batched passes, where tiles of three rows or more are at most 6000 frequencies
//     times measurements long, or clusters of 16 sites take up to 8 measurements:
//     1.03 (0.95, 1.21), the 8x8 three-channel share 1.6 (not PP of 4 sites: 0.98
//     (0.66, 1.12)).  In longer passes the tiles that share a block drift apart: 0.99
//     (0.78, 1.07) on 3686 shapes of 80 to 256 frequencies;
//   several groups, whose transfers spread an orbit wider than an L2, in long FP32
//     passes of PH channels on large clusters and matrices: 1.03 (0.91, 1.17), the
//     6x6 share of 14 planes 1.05.
// Several groups otherwise lose: 0.99 (0.88, 1.06), three channels of 128
// frequencies at 6x6 0.70, and so do long FP32 passes of groups of single planes:
// 0.99 (0.63, 1.13).
int default_order(const Plan &P, uint32_t channels) {
    if (channels & (G4_PP_SINGLET | G4_PP_TRIPLET)) return pair_rows_once(P, channels) && P.mgroup < 8 ? 4 : 2;
    const Dims &d = P.d;
    const bool streamed = streams(P, channels);
    const bool singles = P.mgroup == 1 && d.planes > 1;   // several groups of a plane
    if (uses_pack(P.variant) && !streamed) return d.planes < 32 && !singles ? 4 : 3;
    const double pair = pair_bytes(P);
    if (plane_groups(P) == 1)
        return pair > 4e6 && (P.kind == 0 || (P.batch <= 8 && d.nc >= 16) ||
                              (P.tile >= 3 && (int64_t)d.nw * P.batch <= 6000 &&
                               !((channels & G4_PP_UPDOWN) && d.nc <= 4))) ? 4 : 2;
    const bool ph = channels == G4_PH_MAGNETIC || channels == G4_PH_CHARGE ||
                    (streamed && channels == (G4_PH_MAGNETIC | G4_PH_CHARGE));
    return ph && P.kind == 2 && !singles && d.nc >= 32 && d.planes < 32 &&
           (P.batch >= 32 ? pair > 16e6 : P.batch >= 8 && pair > 32e6) ? 4 : 2;
}

// The order of a list made for one call of `batch` measurements (g4_accumulate_into).
// Orbits take a few microseconds longer to make than windows, which the reuse of
// seven measurements does not earn back: one plane of an 8x8 cluster, 22
// frequencies, 13 measurements 303 us in windows and 260 in orbits, one measurement
// 100 and 111.
int call_order(const Plan &P, uint32_t channels, int batch) {
    if (!(channels & (G4_PP_SINGLET | G4_PP_TRIPLET)) && batch < 8) return 2;
    return default_order(P, channels);
}

// Work decomposition: plane groups (one q, at most mgroup consecutive m) and
// tiles (group, k1, k2, c0).
//
// Tile order.  A tile (k1, k2, q) reads the G block (k2, k1) and the G block
// (k1+q, k2+q); both lie on the block diagonal of momentum difference
// d = k1 - k2 (and -d).  Tiles are sorted by the difference class {d, -d};
// inside a class (order 2) by windows of up to 4 momenta k1 that
// are neighbours along a lattice row x 4 consecutive plane groups x half the
// K2 tiles: k1 + q then stays on one lattice row, so the ~64 tiles an XCD
// holds at once share about 4 G(K2,K1) blocks and 4 exchange blocks (order 1:
// one k1 at a time).  The sorted list is cut into 8 equal contiguous parts,
// one per XCD, and interleaved so that tile i lands on XCD i mod 8 under
// round-robin workgroup dispatch: each XCD's L2 serves a narrow band of G
// blocks.  order 0 keeps the plain (group, k2, k1, rows) order.
// Cut the sorted list into 8 contiguous parts, one per XCD, and interleave
// them so that tile i lands on XCD i mod 8 under round-robin dispatch.
void spread_over_xcds(const std::vector<int4> &sorted, std::vector<int4> &items) {
    const size_t total = sorted.size(), parts = 8;
    const size_t per = (total + parts - 1) / parts;
    items.reserve(total);
    for (size_t i = 0; i < per; ++i)
        for (size_t x = 0; x < parts; ++x) {
            const size_t src = x * per + i;
            if (src < total) items.push_back(sorted[src]);
        }
}

// PP singlet and triplet: the tiles left of a whole list where rows K2 and Q - K2
// are summed once (kTileMirror).  Row i2 of plane m is column i2 of the mirrored
// list at m + nw - 1 - i2: rows below m have no partner, and a mirrored tile that
// holds such rows stays, for them alone (kTileEdge).
void mirror_pairs(const Plan &P, const std::vector<int4> &groups, std::vector<int4> &items) {
    const Dims &d = P.d;
    size_t kept = 0;
    for (int4 it : items) {
        const int4 g = groups[(size_t)it.x];
        const int qx = g.x % d.lx, qy = g.x / d.lx, kx = it.z % d.lx, ky = it.z / d.lx;
        const int k2m = (qx - kx + d.lx) % d.lx + d.lx * ((qy - ky + d.ly) % d.ly);
        if (it.z < k2m) it.w |= kTileMirror;
        if (it.z > k2m) {
            if (it.w >= g.y + g.z - 1) continue;
            it.w |= kTileEdge;
        }
        items[kept++] = it;
    }
    items.resize(kept);
}

void build_work(const Plan &P, int nwex, int order, uint32_t channels, bool pair, std::vector<int4> &groups,
                std::vector<int4> &items) {
    const bool pp = (channels & G4_PP_UPDOWN) != 0;
    groups.clear();
    items.clear();
    const Dims &d = P.d;
    int64_t iQ = d.q_begin;
    const int64_t end = d.q_begin + d.planes;
    while (iQ < end) {
        const int iq = (int)(iQ / nwex), m = (int)(iQ % nwex);
        const int64_t qend = std::min<int64_t>(end, (int64_t)(iq + 1) * nwex);
        const int cnt = (int)std::min<int64_t>(qend - iQ, P.mgroup);
        groups.push_back(int4{P.qlist[(size_t)iq], m, cnt, (int)(iQ - d.q_begin)});
        iQ += cnt;
    }
    const int ng = (int)groups.size();
    if (order == 0) {
        for (int g = 0; g < ng; ++g)
            for (int k2 = 0; k2 < d.nc; ++k2)
                for (int k1 = 0; k1 < d.nc; ++k1)
                    for (int c0 = 0; c0 < d.nw; c0 += P.tile) items.push_back(int4{g, k1, k2, c0});
        if (pair) mirror_pairs(P, groups, items);
        return;
    }
    // difference classes: d and -d together
    auto sub = [&](int a, int b) {   // momentum a - b
        const int ax = a % d.lx, ay = a / d.lx, bx = b % d.lx, by = b / d.lx;
        return (ax - bx + d.lx) % d.lx + d.lx * ((ay - by + d.ly) % d.ly);
    };
    const int ntile = (d.nw + P.tile - 1) / P.tile;
    if (order == 4 && pair) {
        // Tiles of the same rows K2 side by side: their G(K2,K1) and G(K2,Q-K1)
        // are one band of rows of G for every transfer, and the rows Q-K2 of one
        // transfer one band for every K1 (4x4, 3 planes a transfer, FP64: 5.67 ms
        // in windows, 4.60 so; plane groups of 8 read more of each band and are
        // the faster in windows: 12.6 against 13.1 ms)
        std::vector<int4> sorted;
        sorted.reserve((size_t)ng * d.nc * d.nc * ntile);
        for (int k2 = 0; k2 < d.nc; ++k2)
            for (int c = 0; c < ntile; ++c)
                for (int g = 0; g < ng; ++g)
                    for (int k1 = 0; k1 < d.nc; ++k1) sorted.push_back(int4{g, k1, k2, c * P.tile});
        mirror_pairs(P, groups, sorted);
        spread_over_xcds(sorted, items);
        return;
    }
    if (order == 3) {
        // Inside a class, runs of constant k1 + q: the tiles of a run read the
        // same exchange block (rows k1+q, columns k2+q = k1+q-d), and tiles
        // that start one after another on an XCD run about one measurement
        // apart, so each reuses the lines its predecessor just brought into
        // L2.  Two K2 tiles side by side share the direct vector a(q, k1)
        // and half of the exchange block's halo.
        std::vector<std::vector<int>> groups_of(d.nc);
        for (int g = 0; g < ng; ++g) groups_of[(size_t)groups[(size_t)g].x].push_back(g);
        std::vector<int> done(d.nc, 0);
        std::vector<int4> sorted;
        sorted.reserve((size_t)ng * d.nc * d.nc * ntile);
        for (int dd = 0; dd < d.nc; ++dd) {
            if (done[dd]) continue;
            const int neg = sub(0, dd);
            done[dd] = done[neg] = 1;
            const int members[2] = {dd, neg};
            for (int mi = 0; mi < (neg == dd ? 1 : 2); ++mi)
                for (int cb = 0; cb < ntile; cb += 2)
                    for (int K = 0; K < d.nc; ++K)
                        for (int k1 = 0; k1 < d.nc; ++k1)
                            for (int g : groups_of[(size_t)sub(K, k1)])
                                for (int c = cb; c < std::min(ntile, cb + 2); ++c)
                                    sorted.push_back(int4{g, k1, sub(k1, members[mi]), c * P.tile});
        }
        if (pair) mirror_pairs(P, groups, sorted);
        spread_over_xcds(sorted, items);
        return;
    }
    if (order == 4) {
        // Orbits of (k1, k2) under the slice's momentum transfers: the exchange
        // block of a tile is the G(K2,K1) block of the tile (k2+q, k1+q), its PP
        // block that of (q-k1, q-k2), so tiles of one orbit that run together on
        // an XCD read each block of G once for all three uses.  Inside an orbit
        // pairs of K2 tiles, then runs of constant k1 + q.
        // The list is made on every call of g4_accumulate_into: momenta come from
        // tables and the runs from a count per target, with no sort of tiles (8x8,
        // 30 momenta, 8 frequencies: 7.6 -> 1.1 ms a list; the windows take 0.7).
        std::vector<int> by_q(ng), qs, first;                    // groups by momentum; the momenta; each one's first group
        for (int g = 0; g < ng; ++g) by_q[(size_t)g] = g;
        std::stable_sort(by_q.begin(), by_q.end(), [&](int x, int y) { return groups[(size_t)x].x < groups[(size_t)y].x; });
        for (int i = 0; i < ng; ++i)
            if (const int q = groups[(size_t)by_q[(size_t)i]].x; qs.empty() || qs.back() != q) {
                qs.push_back(q);
                first.push_back(i);
            }
        first.push_back(ng);
        const size_t nq = qs.size();
        std::vector<int> plus(nq * d.nc), minus(nq * d.nc);      // k + q and q - k, [k][q of qs]
        for (int k = 0; k < d.nc; ++k)
            for (size_t i = 0; i < nq; ++i) {
                minus[k * nq + i] = sub(qs[i], k);
                plus[k * nq + i] = sub(qs[i], sub(0, k));
            }
        std::vector<char> seen((size_t)d.nc * d.nc, 0);
        std::vector<int> at(d.nc, 0);                            // per target k1 + q: tiles, then the next one's place
        std::vector<int> with_k1(d.nc, 0), k1s;                  // the orbit's pairs by k1, and its k1
        std::vector<int2> orbit;                                 // {k1, k2}
        std::vector<int> targets;
        std::vector<int4> sorted((size_t)ng * d.nc * d.nc * ntile);
        size_t base = 0, left = (size_t)d.nc * d.nc;             // the orbit's first tile; pairs not seen yet
        for (int seed = 0; seed < d.nc * d.nc; ++seed) {
            if (seen[(size_t)seed]) continue;
            seen[(size_t)seed] = 1;
            --left;
            orbit.assign(1, int2{seed % d.nc, seed / d.nc});
            targets.clear();
            k1s.clear();
            for (size_t i = 0; i < orbit.size(); ++i) {
                const int2 o = orbit[i];
                if (!with_k1[(size_t)o.x]++) k1s.push_back(o.x);
                if (!left) continue;
                const int *const p1 = &plus[o.x * nq], *const p2 = &plus[o.y * nq];
                const int *const m1 = &minus[o.x * nq], *const m2 = &minus[o.y * nq];
                auto visit = [&](int a1, int a2) {
                    char &s = seen[(size_t)a2 * d.nc + a1];
                    if (s) return;
                    s = 1;
                    --left;
                    orbit.push_back(int2{a1, a2});
                };
                for (size_t j = 0; j < nq; ++j) visit(p2[j], p1[j]);
                if (pp) for (size_t j = 0; j < nq; ++j) visit(m1[j], m2[j]);
            }
            const size_t tiles = orbit.size() * (size_t)ng;
            for (int k1 : k1s) {
                const int pairs = with_k1[(size_t)k1];
                with_k1[(size_t)k1] = 0;
                for (size_t j = 0; j < nq; ++j) {
                    int &count = at[(size_t)plus[k1 * nq + j]];
                    if (!count) targets.push_back(plus[k1 * nq + j]);
                    count += pairs * (first[j + 1] - first[j]);
                }
            }
            std::sort(targets.begin(), targets.end());
            int place = 0;
            for (int t : targets) {
                const int here = at[(size_t)t];
                at[(size_t)t] = place;
                place += here;
            }
            for (const int2 &o : orbit)
                for (size_t j = 0; j < nq; ++j) {
                    size_t pl = (size_t)at[(size_t)plus[o.x * nq + j]];
                    at[(size_t)plus[o.x * nq + j]] += first[j + 1] - first[j];
                    for (int i = first[j]; i < first[j + 1]; ++i, ++pl)
                        if (ntile == 1) sorted[base + pl] = int4{by_q[(size_t)i], o.x, o.y, 0};
                        else for (int c = 0; c < ntile; ++c) {
                            const size_t before = base + (size_t)(c & ~1) * tiles, w = (c | 1) < ntile ? 2 : 1;
                            sorted[before + pl * w + (c & 1)] = int4{by_q[(size_t)i], o.x, o.y, c * P.tile};
                        }
                }
            base += tiles * ntile;
            for (int t : targets) at[(size_t)t] = 0;
        }
        if (pair) mirror_pairs(P, groups, sorted);
        spread_over_xcds(sorted, items);
        return;
    }
    // order 2: inside a class, windows of bk momenta k1 (neighbours along a
    // lattice row) x bg consecutive plane groups x half the K2 tiles, so that
    // the tiles resident together read few G(K2,K1) and exchange blocks
    const int bk = order == 2 ? std::min(d.lx, 4) : 1;
    const int bg = order == 2 ? std::min(ng, 4) : ng;
    const int bc = order == 2 ? std::max(1, (ntile + 1) / 2) : ntile;
    std::vector<int> cls_done(d.nc, 0);
    std::vector<int4> sorted;
    sorted.reserve((size_t)ng * d.nc * d.nc * ntile);
    for (int dd = 0; dd < d.nc; ++dd) {
        if (cls_done[dd]) continue;
        const int neg = sub(0, dd);
        cls_done[dd] = cls_done[neg] = 1;
        const int members[2] = {dd, neg};
        for (int mi = 0; mi < (neg == dd ? 1 : 2); ++mi)
            for (int kb = 0; kb < d.nc; kb += bk)
                for (int gb = 0; gb < ng; gb += bg)
                    for (int cb = 0; cb < ntile; cb += bc)
                        for (int k1 = kb; k1 < std::min(d.nc, kb + bk); ++k1) {
                            const int k2 = sub(k1, members[mi]);
                            for (int g = gb; g < std::min(ng, gb + bg); ++g)
                                for (int c = cb; c < std::min(ntile, cb + bc); ++c)
                                    sorted.push_back(int4{g, k1, k2, c * P.tile});
                        }
    }
    if (pair) mirror_pairs(P, groups, sorted);
    spread_over_xcds(sorted, items);
}

}  // namespace

struct g4_slice {
    g4_config cfg;
    Plan P;
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    bool poisoned = false;
    void *acc[3] = {nullptr, nullptr, nullptr};
    int32_t *kadd = nullptr, *ksub = nullptr;
    int4 *groups = nullptr, *items = nullptr;
    int2 *plane_qm = nullptr;
    int32_t *qpos = nullptr;
    int ngroups = 0, nitems = 0;
    bool pair_rows = false;   // the tile list sums rows once (kTileMirror)
    size_t items_cap = 0;
    int order = -1;         // tile order (see build_work), -1 = by variant; G4_TILE_ORDER overrides
    void *dir = nullptr;
    void *stage = nullptr;
    void *pack = nullptr;        // packed variant, max_batch blocks of P.pack_stride bytes
    double *sign_dev = nullptr;
    double *sign_host = nullptr;     // pinned
    hipEvent_t sign_ev[kSignSlots] = {};
    bool sign_ev_used[kSignSlots] = {};
    int sign_next = 0;
    double *scratch = nullptr;
    void *readback_host = nullptr;   // pinned, kReadbackLanes slots; allocated by the first large readback
    int *finite_dev = nullptr;       // G4_F_CHECK_FINITE: set by the check kernel
    int *finite_host = nullptr;      // pinned copy of it
    uint64_t measurements = 0;
    double sign_sum = 0.0;
    uint64_t launches = 0;
    double kernel_ms = 0.0;
    uint64_t timed = 0;
    std::vector<hipEvent_t> ev_free;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_pending;
    // G4_F_GRAPH: one recorded pass per (inputs, pass size) under the current plan
    struct GraphEntry {
        const void *gu, *gd;
        int nb;
        double *dsign;            // the pass's weights, uploaded before each launch
        hipGraphExec_t exec;      // null until recorded (second use)
        int uses;
        uint64_t last;
    };
    std::vector<GraphEntry> graphs;
    uint64_t graph_clock = 0;
};

namespace {

int hip_fail(g4_slice *h, hipError_t e, const char *what) {
    if (h) h->poisoned = true;
    return fail(G4_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define G4_HIP(h, call)                                     \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return hip_fail(h, e_, #call); \
    } while (0)

int usable(g4_slice *h) {
    if (!h) return fail(G4_E_ARG, "handle is NULL");
    if (h->poisoned) return fail(G4_E_STATE, "handle poisoned by an earlier HIP error");
    return G4_OK;
}

int channel_slot(uint32_t channel) {
    switch (channel) {
        case G4_PH_MAGNETIC: case G4_PH_LONG_UPUP: case G4_PP_SINGLET: return 0;
        case G4_PH_CHARGE: case G4_PH_LONG_UPDOWN: case G4_PP_TRIPLET: return 1;
        case G4_PP_UPDOWN: case G4_PH_TRANSVERSE: return 2;
        default: return -1;
    }
}

// The kernel of a pass of nb measurements on a slice (see pass_variant)
int kernel_of(const g4_slice *h, int nb) {
    return pass_variant(h->P, h->cfg.channels, h->ngroups, h->nitems, nb, (int64_t)h->P.batch * h->P.d.planes * h->P.d.n);
}

// G4_LOG=1: one line on stderr whenever a plan is installed.
void log_plan(const g4_slice *h, const char *why) {
    const char *e = std::getenv("G4_LOG");
    if (!e || !e[0] || e[0] == '0') return;
    const Plan &P = h->P;
    static const char *names[] = {"valu", "mfma-direct", "packed", "packed-deep", "packed-mfma-direct"};
    std::fprintf(stderr,
                 "g4: %s: channels 0x%x, %llu entries per channel, kind %d, variant %s, kernel %s, tile %d, pass %d, "
                 "rows/thread %d, plane group %d, %d work tiles%s, %llu device bytes\n",
                 why, h->cfg.channels, (unsigned long long)P.entries, P.kind,
                 P.variant >= 0 && P.variant <= 4 ? names[P.variant] : "?", kernel_name(kernel_of(h, P.batch)),
                 P.tile, P.batch, P.ept, P.mgroup,
                 h->nitems, P.persistent ? " (persistent grid)" : "", (unsigned long long)P.total_bytes);
}

void drop_graphs(g4_slice *h) {
    for (auto &g : h->graphs) {
        if (g.exec) (void)hipGraphExecDestroy(g.exec);
        if (g.dsign) (void)hipFree(g.dsign);
    }
    h->graphs.clear();
}

void release(g4_slice *h) {
    if (!h) return;
    (void)hipSetDevice(h->device);
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    drop_graphs(h);
    for (auto &pr : h->ev_pending) {
        (void)hipEventDestroy(pr.first);
        (void)hipEventDestroy(pr.second);
    }
    for (auto e : h->ev_free) (void)hipEventDestroy(e);
    for (int i = 0; i < kSignSlots; ++i)
        if (h->sign_ev[i]) (void)hipEventDestroy(h->sign_ev[i]);
    for (void *p : {(void *)h->acc[0], (void *)h->acc[1], (void *)h->acc[2], (void *)h->kadd,
                    (void *)h->ksub, (void *)h->groups, (void *)h->items, (void *)h->plane_qm, (void *)h->qpos,
                    h->dir, h->stage, h->pack, (void *)h->sign_dev, (void *)h->scratch, (void *)h->finite_dev})
        if (p) (void)hipFree(p);
    if (h->sign_host) (void)hipHostFree(h->sign_host);
    if (h->finite_host) (void)hipHostFree(h->finite_host);
    if (h->readback_host) (void)hipHostFree(h->readback_host);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
}

uint32_t with_variant(uint32_t flags, int variant) {
    flags &= ~(uint32_t)(G4_F_MFMA | G4_F_PACKED | G4_F_PACKED_DEEP);
    if (variant == G4_VARIANT_MFMA) flags |= G4_F_MFMA;
    if (variant == G4_VARIANT_PACKED) flags |= G4_F_PACKED;
    if (variant == G4_VARIANT_PACKED_DEEP) flags |= G4_F_PACKED_DEEP;
    if (variant == G4_VARIANT_PACKED_MFMA) flags |= G4_F_PACKED | G4_F_MFMA;
    return flags;
}

// The packed buffer is allocated when a plan that uses it is first installed.
int ensure_pack(g4_slice *h, const Plan &P) {
    if (P.pack_bytes == 0 || h->pack) return G4_OK;
    hipError_t e = hipMalloc(&h->pack, P.pack_bytes);
    if (e != hipSuccess) {
        h->pack = nullptr;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? G4_E_OOM : G4_E_HIP, "packed buffer of %llu bytes: %s",
                    (unsigned long long)P.pack_bytes, hipGetErrorString(e));
    }
    h->P.ldp = P.ldp;
    h->P.pcb = P.pcb;
    h->P.pack_stride = P.pack_stride;
    h->P.pack_bytes = P.pack_bytes;
    return G4_OK;
}

int fold_timings(g4_slice *h) {
    for (auto &pr : h->ev_pending) {
        G4_HIP(h, hipEventSynchronize(pr.second));
        float ms = 0.f;
        G4_HIP(h, hipEventElapsedTime(&ms, pr.first, pr.second));
        h->kernel_ms += ms;
        h->timed += 1;
        h->ev_free.push_back(pr.first);
        h->ev_free.push_back(pr.second);
    }
    h->ev_pending.clear();
    return G4_OK;
}

int take_event(g4_slice *h, hipEvent_t *out) {
    if (!h->ev_free.empty()) {
        *out = h->ev_free.back();
        h->ev_free.pop_back();
        return G4_OK;
    }
    G4_HIP(h, hipEventCreate(out));
    return G4_OK;
}

Tables tables_of(const g4_slice *h) {
    Tables t;
    t.kadd = h->kadd;
    t.ksub = h->ksub;
    t.groups = h->groups;
    t.items = h->items;
    t.plane_qm = h->plane_qm;
    t.qpos = h->qpos;
    return t;
}

int rebuild_work(g4_slice *h) {
    if (!h->graphs.empty()) {
        G4_HIP(h, hipStreamSynchronize(h->stream));
        drop_graphs(h);
    }
    std::vector<int4> groups, items;
    const int order = h->order >= 0 ? h->order : default_order(h->P, h->cfg.channels);
    const bool pair = pair_rows_once(h->P, h->cfg.channels);
    build_work(h->P, h->cfg.nwex, order, h->cfg.channels, pair, groups, items);
    if (items.size() > (size_t)INT32_MAX) return fail(G4_E_UNSUPPORTED, "more than 2^31 work tiles");
    if (items.size() > h->items_cap) {
        G4_HIP(h, hipStreamSynchronize(h->stream));
        if (h->items) G4_HIP(h, hipFree(h->items));
        h->items = nullptr;
        h->items_cap = 0;
        G4_HIP(h, hipMalloc(&h->items, items.size() * sizeof(int4)));
        h->items_cap = items.size();
    }
    G4_HIP(h, hipMemcpyAsync(h->groups, groups.data(), groups.size() * sizeof(int4), hipMemcpyHostToDevice, h->stream));
    G4_HIP(h, hipMemcpyAsync(h->items, items.data(), items.size() * sizeof(int4), hipMemcpyHostToDevice, h->stream));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    h->ngroups = (int)groups.size();
    h->nitems = (int)items.size();
    h->pair_rows = pair;
    return G4_OK;
}

// The weights of a pass go to its first kernel by value, which stores them at
// `ds` for the update kernel.
void weights_by_value(GatherArgs &ga, const double *sign, int nb, double *ds) {
    std::memcpy(ga.sgn, sign, (size_t)nb * sizeof(double));
    ga.sign_out = ds;
}

// The update (and split direct term) of the measurements that `ga` describes,
// whose direct vectors and packed blocks are in place and whose weights are at
// ds: one slice-update kernel launch, counted and, if asked, timed.
int enqueue_update(g4_slice *h, const GatherArgs &ga, const double *ds, bool timing) {
    const Plan &P = h->P;
    const bool packed = uses_pack(P.variant) && !streams(P, h->cfg.channels);
    UpdateArgs ua;
    ua.gu = ga.gu;
    ua.gd = ga.gd;
    ua.g_stride = ga.g_stride;
    ua.dir_a = ga.dir_a;
    ua.dir_b = ga.dir_b;
    ua.dir_slot_stride = ga.dir_slot_stride;
    ua.dir_b_stride = ga.dir_b_stride;
    ua.pack = packed ? h->pack : nullptr;
    ua.pack_stride = (int64_t)P.pack_stride;
    ua.ldp = P.ldp;
    ua.pcb = P.pcb;
    ua.nitems = h->nitems;
    ua.skip_direct = P.split && P.slots ? 1 : 0;
    ua.sign = ds;
    ua.batch = ga.batch;
    ua.acc[0] = h->acc[0];
    ua.acc[1] = h->acc[1];
    ua.acc[2] = h->acc[2];
    ua.acc_kind = h->cfg.acc;
    ua.tile = P.tile;
    ua.pair_rows = h->pair_rows;
    ua.persistent = P.persistent;
    ua.d = P.d;
    ua.t = ga.t;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (timing) {
        int rc = take_event(h, &e0);
        if (rc) return rc;
        rc = take_event(h, &e1);
        if (rc) return rc;
        G4_HIP(h, hipEventRecord(e0, h->stream));
    }
    const int variant = pass_variant(P, h->cfg.channels, h->ngroups, h->nitems, ga.batch, ua.dir_slot_stride);
    G4_HIP(h, launch_update(P.kind, (int)h->cfg.channels, P.ept, P.mgroup, h->nitems, variant, ua, h->stream));
    if (timing) {
        G4_HIP(h, hipEventRecord(e1, h->stream));
        h->ev_pending.emplace_back(e0, e1);
    }
    if (ua.skip_direct) {
        // split-precision direct term: GEMM over the pass on MFMA, its own read-modify-write
        DirectArgs da;
        da.dir_a = ga.dir_a;
        da.dir_b = ga.dir_b;
        da.dir_slot_stride = ga.dir_slot_stride;
        da.dir_b_stride = ga.dir_b_stride;
        da.batch = ga.batch;
        da.nslots = P.nslots;
        da.acc[0] = (P.slots & 1) ? h->acc[0] : h->acc[1];
        da.acc[1] = h->acc[1];
        da.acc_kind = h->cfg.acc;
        da.p0 = 0;
        da.d = P.d;
        G4_HIP(h, launch_direct_split(P.split, da, h->stream));
    }
    h->launches += 1;
    return G4_OK;
}

// The device work of one pass (conversion, packing or gather, update, split
// direct term) on inputs pu, pd.  hs: the pass's weights, handed over by value
// and kept at device address ds; NULL when they are at ds already (a recording,
// which may hold no host values).
int enqueue_pass(g4_slice *h, const void *pu, const void *pd, double *ds, const double *hs, int nb, bool timing) {
    const Plan &P = h->P;
    const int64_t per = (int64_t)P.d.ng * P.d.ng;
    if (P.prec == 1 && h->cfg.g_in == G4_IN_C128) {
        float2 *su = static_cast<float2 *>(h->stage);
        float2 *sd = su + (size_t)P.batch * per;
        G4_HIP(h, launch_convert_c128_to_c64(pu, su, (int64_t)nb * per, h->stream));
        G4_HIP(h, launch_convert_c128_to_c64(pd, sd, (int64_t)nb * per, h->stream));
        pu = su;
        pd = sd;
    }
    const size_t el = P.prec == 0 ? 16 : 8;
    const int64_t pn = (int64_t)P.d.planes * P.d.n;
    // direct vectors: [slot][b][p][K] in their own buffer, or, for packed
    // operands, inside each measurement's packed block after its G rows
    const bool packed = uses_pack(P.variant) && !streams(P, h->cfg.channels);
    int64_t dir_slot = (int64_t)P.batch * pn, dir_bstride = pn;
    void *dir_a = h->dir;
    if (packed) {
        if (!h->pack) return fail(G4_E_STATE, "packed operands selected without a packed buffer");
        dir_slot = pn;
        dir_bstride = (int64_t)(P.pack_stride / 8);
        dir_a = static_cast<char *>(h->pack) + (size_t)P.d.ng * P.ldp * 16;
    }
    void *dir_b = static_cast<char *>(dir_a) + (size_t)P.nslots * dir_slot * el;
    GatherArgs ga;
    ga.gu = pu;
    ga.gd = pd;
    ga.g_stride = per;
    ga.dir_a = dir_a;
    ga.dir_b = dir_b;
    ga.dir_slot_stride = dir_slot;
    ga.dir_b_stride = dir_bstride;
    ga.sign = ds;
    ga.batch = nb;
    ga.slots = P.slots;
    ga.d = P.d;
    ga.t = tables_of(h);
    if (hs) weights_by_value(ga, hs, nb, ds);
    if (packed) {
        // one pass over G: packed copy plus the direct vectors
        PackArgs pa;
        pa.g = ga;
        pa.pack = h->pack;
        pa.pack_stride16 = (int64_t)(P.pack_stride / 16);
        pa.ldp = P.ldp;
        pa.pcb = P.pcb;
        G4_HIP(h, launch_pack_gather(pa, h->stream));
    } else {
        G4_HIP(h, launch_gather(P.prec, ga, h->stream));
    }
    return enqueue_update(h, ga, ds, timing);
}

// The recorded pass for these inputs, created (without a recording) if new;
// the least recently used of 64 is dropped to make room.
int graph_entry(g4_slice *h, const void *pu, const void *pd, int nb, g4_slice::GraphEntry **out) {
    for (auto &g : h->graphs)
        if (g.gu == pu && g.gd == pd && g.nb == nb) {
            *out = &g;
            return G4_OK;
        }
    if (h->graphs.size() >= 64) {
        size_t lru = 0;
        for (size_t i = 1; i < h->graphs.size(); ++i)
            if (h->graphs[i].last < h->graphs[lru].last) lru = i;
        G4_HIP(h, hipStreamSynchronize(h->stream));
        if (h->graphs[lru].exec) G4_HIP(h, hipGraphExecDestroy(h->graphs[lru].exec));
        G4_HIP(h, hipFree(h->graphs[lru].dsign));
        h->graphs.erase(h->graphs.begin() + (std::ptrdiff_t)lru);
    }
    g4_slice::GraphEntry g{pu, pd, nb, nullptr, nullptr, 0, 0};
    G4_HIP(h, hipMalloc(&g.dsign, kMaxBatch * sizeof(double)));
    h->graphs.push_back(g);
    *out = &h->graphs.back();
    return G4_OK;
}

// One pass: up to P.batch measurements starting at b0.  With G4_F_GRAPH a pass
// on inputs seen before replays its recorded graph (the first use runs
// directly, the second records); the weights are uploaded before the launch.
int run_pass(g4_slice *h, const char *gu, const char *gd, const double *sign, int b0, int nb) {
    const Plan &P = h->P;
    char range[96];
    std::snprintf(range, sizeof(range), "g4 pass: %d measurements, variant %d, kernel %s, tile %d", nb, P.variant,
                  kernel_name(kernel_of(h, nb)), P.tile);
    const RoctxRange rr(range);
    const size_t in_el = h->cfg.g_in == G4_IN_C128 ? 16 : 8;
    const int64_t per = (int64_t)P.d.ng * P.d.ng;
    const void *pu = gu + (size_t)b0 * per * in_el;
    const void *pd = gd + (size_t)b0 * per * in_el;
    const bool graph = (h->cfg.flags & G4_F_GRAPH) && h->cfg.mode == G4_MODE_BATCHED;
    const bool timing = (h->cfg.flags & G4_F_KERNEL_TIMING) != 0;
    g4_slice::GraphEntry *ge = nullptr;
    if (graph) {
        int rc = graph_entry(h, pu, pd, nb, &ge);
        if (rc) return rc;
    }

    if (!graph) return enqueue_pass(h, pu, pd, h->sign_dev, sign + b0, nb, timing);
    // a recording reads its weights from its own buffer: pinned slot -> device
    const int slot = h->sign_next;
    h->sign_next = (h->sign_next + 1) % kSignSlots;
    if (h->sign_ev_used[slot]) G4_HIP(h, hipEventSynchronize(h->sign_ev[slot]));
    double *hs = h->sign_host + (size_t)slot * kMaxBatch;
    double *ds = ge->dsign;
    std::memcpy(hs, sign + b0, (size_t)nb * sizeof(double));
    G4_HIP(h, hipMemcpyAsync(ds, hs, (size_t)nb * sizeof(double), hipMemcpyHostToDevice, h->stream));
    G4_HIP(h, hipEventRecord(h->sign_ev[slot], h->stream));
    h->sign_ev_used[slot] = true;

    ge->last = ++h->graph_clock;
    if (!ge->exec && ge->uses++ == 0) return enqueue_pass(h, pu, pd, ds, nullptr, nb, timing);
    if (!ge->exec) {
        hipGraph_t g = nullptr;
        G4_HIP(h, hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal));
        const int rc = enqueue_pass(h, pu, pd, ds, nullptr, nb, false);
        const hipError_t e = hipStreamEndCapture(h->stream, &g);
        if (rc) {
            if (g) (void)hipGraphDestroy(g);
            return rc;
        }
        if (e != hipSuccess) return hip_fail(h, e, "hipStreamEndCapture");
        h->launches -= 1;                     // counted below, when the graph runs
        const hipError_t ei = hipGraphInstantiate(&ge->exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (ei != hipSuccess) {
            ge->exec = nullptr;
            return hip_fail(h, ei, "hipGraphInstantiate");
        }
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (timing) {
        int rc = take_event(h, &e0);
        if (rc) return rc;
        rc = take_event(h, &e1);
        if (rc) return rc;
        G4_HIP(h, hipEventRecord(e0, h->stream));
    }
    G4_HIP(h, hipGraphLaunch(ge->exec, h->stream));
    if (timing) {
        G4_HIP(h, hipEventRecord(e1, h->stream));
        h->ev_pending.emplace_back(e0, e1);
    }
    h->launches += 1;
    return G4_OK;
}

// Plain mode: one update launch per measurement.  The direct vectors of as many
// measurements as the readback scratch holds are gathered in one launch (the
// scratch is otherwise used only inside calls that wait for the stream); a
// slice too large for that gathers one measurement at a time.
int run_plain(g4_slice *h, const char *gu, const char *gd, const double *sign, int batch) {
    const Plan &P = h->P;
    const int64_t per = (int64_t)P.d.ng * P.d.ng, pn = (int64_t)P.d.planes * P.d.n;
    const bool timing = (h->cfg.flags & G4_F_KERNEL_TIMING) != 0;
    const uint64_t each = 2ull * P.nslots * pn * 16;
    const uint64_t fit = each ? P.scratch_bytes / each : (uint64_t)kMaxBatch;
    const int group = (int)std::max<uint64_t>(1, std::min<uint64_t>(kMaxBatch, fit));
    char range[96];
    std::snprintf(range, sizeof(range), "g4 pass: 1 measurements, variant %d, kernel %s, tile %d", P.variant,
                  kernel_name(kernel_of(h, 1)), P.tile);
    for (int b0 = 0; b0 < batch; b0 += group) {
        const int nb = std::min(group, batch - b0);
        GatherArgs ga;
        ga.gu = gu + (size_t)b0 * per * 16;
        ga.gd = gd + (size_t)b0 * per * 16;
        ga.g_stride = per;
        ga.dir_a = fit ? (void *)h->scratch : h->dir;
        ga.dir_slot_stride = (int64_t)nb * pn;
        ga.dir_b_stride = pn;
        ga.dir_b = static_cast<char *>(ga.dir_a) + (size_t)P.nslots * ga.dir_slot_stride * 16;
        ga.sign = h->sign_dev;
        ga.batch = nb;
        ga.slots = P.slots;
        ga.d = P.d;
        ga.t = tables_of(h);
        weights_by_value(ga, sign + b0, nb, h->sign_dev);
        G4_HIP(h, launch_gather(P.prec, ga, h->stream));
        GatherArgs one = ga;
        one.batch = 1;
        for (int b = 0; b < nb; ++b) {
            const RoctxRange rr(range);
            one.gu = static_cast<const char *>(ga.gu) + (size_t)b * per * 16;
            one.gd = static_cast<const char *>(ga.gd) + (size_t)b * per * 16;
            one.dir_a = static_cast<char *>(ga.dir_a) + (size_t)b * pn * 16;
            one.dir_b = static_cast<char *>(ga.dir_b) + (size_t)b * pn * 16;
            if (int rc = enqueue_update(h, one, h->sign_dev + b, timing); rc) return rc;
        }
    }
    return G4_OK;
}

// A readback of several slots' worth of entries: kReadbackLanes threads take
// slot-sized ranges in turn, each converting into its own part of the scratch,
// copying that to its own pinned slot and from there to the caller's memory, so
// that the device copies follow one another (57 GB/s) while the other threads
// move what has arrived.  One thread through the runtime's staging of pageable
// memory took 202 ms for the 2.15 GB of the 4x4 slice, this 46 ms (47 GB/s).
// *ran = false (nothing done) where the pinned slots or the threads cannot be had.
int readback_lanes(g4_slice *h, int c, uint64_t first, uint64_t count, double *out, bool *ran) {
    *ran = false;
    if (!h->readback_host) {
        if (hipHostMalloc(&h->readback_host, kScratchEntries * 16, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            h->readback_host = nullptr;
            return G4_OK;
        }
    }
    std::atomic<uint64_t> next{0};
    std::atomic<int> bad{(int)hipSuccess};
    const uint64_t ranges = (count + kLaneEntries - 1) / kLaneEntries;
    auto lane = [&](int i) {
        double *dev = h->scratch + 2 * i * kLaneEntries;
        double *host = static_cast<double *>(h->readback_host) + 2 * i * kLaneEntries;
        hipEvent_t ev = nullptr;
        hipError_t e = hipSetDevice(h->device);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        for (uint64_t r; e == hipSuccess && bad.load() == (int)hipSuccess && (r = next.fetch_add(1)) < ranges;) {
            const uint64_t off = r * kLaneEntries, cnt = std::min(kLaneEntries, count - off);
            e = launch_acc_to_c128(h->cfg.acc, h->acc[c], first + off, cnt, dev, h->P.d.nc, h->P.d.nw, h->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(host, dev, cnt * 16, hipMemcpyDeviceToHost, h->stream);
            if (e == hipSuccess) e = hipEventRecord(ev, h->stream);
            if (e == hipSuccess) e = hipEventSynchronize(ev);
            if (e == hipSuccess) std::memcpy(out + 2 * off, host, cnt * 16);
        }
        if (ev) (void)hipEventDestroy(ev);
        if (e != hipSuccess) bad.store((int)e);
    };
    std::vector<std::thread> threads;
    try {
        threads.reserve(kReadbackLanes - 1);
        for (int i = 1; i < kReadbackLanes; ++i) threads.emplace_back(lane, i);
    } catch (const std::exception &) {
        // fewer threads: the ones there, and this one, take every range
    }
    lane(0);
    for (auto &t : threads) t.join();
    *ran = true;
    const hipError_t e = (hipError_t)bad.load();
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(h->stream);
        return hip_fail(h, e, "readback");
    }
    return G4_OK;
}

}  // namespace

namespace {

// ---- the allocation-free accumulation (g4_accumulate_into) ----------------
// Everything g4_accumulate keeps in a slice's own allocations (index tables,
// work tiles, direct vectors, weights) is laid out in a caller-provided
// device workspace instead; the accumulators are the caller's.  Runs the
// VALU kernels (plain FP64, or batched with FP64 or FP32 products) with the
// pass schedule of g4_accumulate.  Synchronous: host tables stay alive until
// their copies are done.
int noalloc_accumulate(const g4_config *cfg, void *const acc[3], const void *G_up, const void *G_dn,
                       const double *sign, int32_t batch, void *ws, uint64_t ws_bytes) {
    Plan P;
    int rc = validate(cfg, &P);
    if (rc) return rc;
    if (P.variant != G4_VARIANT_VALU || P.split)
        return fail(G4_E_UNSUPPORTED, "g4_accumulate_into runs the VALU kernels only (no G4_F_MFMA, "
                                      "G4_F_PACKED, G4_F_PACKED_DEEP or split products)");
    if (cfg->flags & (G4_F_GRAPH | G4_F_KERNEL_TIMING | G4_F_CHECK_FINITE))
        return fail(G4_E_UNSUPPORTED, "g4_accumulate_into takes no G4_F_GRAPH, G4_F_KERNEL_TIMING or "
                                      "G4_F_CHECK_FINITE");
    if (P.prec == 1 && cfg->g_in == G4_IN_C128)
        return fail(G4_E_UNSUPPORTED, "g4_accumulate_into: FP32 products need complex64 G");
    if (batch < 0) return fail(G4_E_ARG, "batch=%d", batch);
    for (int c = 0; c < 3; ++c) {
        const bool want = (acc_slots((int)cfg->channels) >> c) & 1;
        if (want != (acc[c] != nullptr))
            return fail(G4_E_ARG, "accumulator %d must be %s", c, want ? "given" : "NULL for an absent channel");
    }
    if (batch == 0) return G4_OK;
    if (!G_up || !G_dn || !sign) return fail(G4_E_ARG, "NULL G or sign pointer");
    // host tables
    std::vector<int32_t> kadd, ksub;
    build_momentum_maps(P.d, kadd, ksub);
    std::vector<int2> pq;
    build_planes(P, cfg->nwex, pq);
    std::vector<int32_t> qpos(P.d.nc, -1);
    for (size_t i = 0; i < P.qlist.size(); ++i) qpos[(size_t)P.qlist[i]] = (int32_t)i;
    // workspace layout, 256-byte aligned parts
    auto up = [](uint64_t b) { return (b + 255) / 256 * 256; };
    const uint64_t el = P.prec == 0 ? 16 : 8;
    const int64_t pn = (int64_t)P.d.planes * P.d.n;
    // A batched pass has at most this call's measurements.  A workspace too small for
    // the list of whole tiles gets the shorter one of rows summed once.
    Plan call = P;
    if (P.kind != 0) call.batch = std::min(P.batch, batch);
    const uint64_t whole = up(kadd.size() * 4) + up(ksub.size() * 4) + up(pq.size() * sizeof(int2)) +
                           up(qpos.size() * 4) + up(plane_groups(P) * sizeof(int4)) +
                           up(whole_tiles(P) * sizeof(int4)) + 2 * up((uint64_t)P.nslots * P.batch * pn * el) +
                           up((uint64_t)P.batch * sizeof(double));
    const bool pair = pair_rows_once(call, cfg->channels) || (takes_pair_rows(P, cfg->channels) && whole > ws_bytes);
    std::vector<int4> groups, items;
    build_work(P, cfg->nwex, call_order(call, cfg->channels, batch), cfg->channels, pair, groups, items);
    if (items.size() > (size_t)INT32_MAX) return fail(G4_E_UNSUPPORTED, "more than 2^31 work tiles");
    if (P.kind == 0) {
        // The plain kernel adds a launch's measurements one after another to the
        // entry it holds in registers, the same operations in the same order as
        // launches of one: as many per launch as the workspace holds the direct
        // vectors of save the accumulator's trip to memory and back (the whole
        // 4x4 array, 64 measurements: 61.3 ms one at a time, 20.7 ms in groups of 13).
        const uint64_t tables = up(kadd.size() * 4) + up(ksub.size() * 4) + up(pq.size() * sizeof(int2)) +
                                up(qpos.size() * 4) + up(groups.size() * sizeof(int4)) +
                                up(items.size() * sizeof(int4)) + up(kMaxBatch * sizeof(double)) + 512;
        const uint64_t each = 2ull * P.nslots * pn * el;
        const int64_t fit = tables >= ws_bytes ? 1 : each ? (int64_t)((ws_bytes - tables) / each) : kMaxBatch;
        const int most = (int)std::max<int64_t>(1, std::min<int64_t>({fit, kMaxBatch, batch}));
        const int passes = (batch + most - 1) / most;
        P.batch = (batch + passes - 1) / passes;
    }
    const uint64_t dir_half = (uint64_t)P.nslots * P.batch * pn * el;
    uint64_t o = 0;
    const uint64_t o_kadd = o; o += up(kadd.size() * 4);
    const uint64_t o_ksub = o; o += up(ksub.size() * 4);
    const uint64_t o_pq = o; o += up(pq.size() * sizeof(int2));
    const uint64_t o_qpos = o; o += up(qpos.size() * 4);
    const uint64_t o_groups = o; o += up(groups.size() * sizeof(int4));
    const uint64_t o_items = o; o += up(items.size() * sizeof(int4));
    const uint64_t o_dir = o; o += 2 * up(dir_half);
    const uint64_t o_sign = o; o += up((uint64_t)P.batch * sizeof(double));
    if (o > ws_bytes)
        return fail(G4_E_UNSUPPORTED, "g4_accumulate_into needs %llu bytes of workspace, the static one holds %llu "
                                      "(fewer planes or a smaller max_batch)",
                    (unsigned long long)o, (unsigned long long)ws_bytes);
    char *w = static_cast<char *>(ws);
    hipStream_t st = static_cast<hipStream_t>(cfg->stream);
    hipError_t e = hipSetDevice(cfg->device);
#define G4_NA(call)                                                           \
    do {                                                                      \
        e = (call);                                                           \
        if (e != hipSuccess) return fail(G4_E_HIP, "%s: %s", #call, hipGetErrorString(e)); \
    } while (0)
    G4_NA(e);
    G4_NA(hipMemcpyAsync(w + o_kadd, kadd.data(), kadd.size() * 4, hipMemcpyHostToDevice, st));
    G4_NA(hipMemcpyAsync(w + o_ksub, ksub.data(), ksub.size() * 4, hipMemcpyHostToDevice, st));
    G4_NA(hipMemcpyAsync(w + o_pq, pq.data(), pq.size() * sizeof(int2), hipMemcpyHostToDevice, st));
    G4_NA(hipMemcpyAsync(w + o_qpos, qpos.data(), qpos.size() * 4, hipMemcpyHostToDevice, st));
    G4_NA(hipMemcpyAsync(w + o_groups, groups.data(), groups.size() * sizeof(int4), hipMemcpyHostToDevice, st));
    G4_NA(hipMemcpyAsync(w + o_items, items.data(), items.size() * sizeof(int4), hipMemcpyHostToDevice, st));
    Tables t;
    t.kadd = reinterpret_cast<const int32_t *>(w + o_kadd);
    t.ksub = reinterpret_cast<const int32_t *>(w + o_ksub);
    t.plane_qm = reinterpret_cast<const int2 *>(w + o_pq);
    t.qpos = reinterpret_cast<const int32_t *>(w + o_qpos);
    t.groups = reinterpret_cast<const int4 *>(w + o_groups);
    t.items = reinterpret_cast<const int4 *>(w + o_items);
    double *ds = reinterpret_cast<double *>(w + o_sign);
    void *dir_a = w + o_dir, *dir_b = w + o_dir + up(dir_half);
    const size_t in_el = cfg->g_in == G4_IN_C128 ? 16 : 8;
    const int64_t per = (int64_t)P.d.ng * P.d.ng;
    for (int b0 = 0; b0 < batch; b0 += P.batch) {
        const int nb = std::min(P.batch, batch - b0);
        const void *pu = static_cast<const char *>(G_up) + (size_t)b0 * per * in_el;
        const void *pd = static_cast<const char *>(G_dn) + (size_t)b0 * per * in_el;
        GatherArgs ga;
        ga.gu = pu;
        ga.gd = pd;
        ga.g_stride = per;
        ga.dir_a = dir_a;
        ga.dir_b = dir_b;
        ga.dir_slot_stride = (int64_t)P.batch * pn;
        ga.dir_b_stride = pn;
        ga.sign = ds;
        ga.batch = nb;
        ga.slots = P.slots;
        ga.d = P.d;
        ga.t = t;
        // the previous pass has read the weights (stream order) before they are replaced
        weights_by_value(ga, sign + b0, nb, ds);
        G4_NA(launch_gather(P.prec, ga, st));
        UpdateArgs ua;
        ua.gu = pu;
        ua.gd = pd;
        ua.g_stride = per;
        ua.dir_a = dir_a;
        ua.dir_b = dir_b;
        ua.dir_slot_stride = ga.dir_slot_stride;
        ua.dir_b_stride = pn;
        ua.pack = nullptr;
        ua.pack_stride = 0;
        ua.ldp = 0;
        ua.pcb = 0;
        ua.nitems = (int)items.size();
        ua.skip_direct = 0;
        ua.sign = ds;
        ua.batch = nb;
        ua.acc[0] = acc[0];
        ua.acc[1] = acc[1];
        ua.acc[2] = acc[2];
        ua.acc_kind = cfg->acc;
        ua.tile = P.tile;
        ua.pair_rows = pair;
        ua.persistent = P.persistent;
        ua.d = P.d;
        ua.t = t;
        const int variant = pass_variant(P, cfg->channels, (int)groups.size(), (int)items.size(), nb, ua.dir_slot_stride);
        G4_NA(launch_update(P.kind, (int)cfg->channels, P.ept, P.mgroup, (int)items.size(), variant, ua, st));
    }
    G4_NA(hipStreamSynchronize(st));
#undef G4_NA
    g_err[0] = 0;
    return G4_OK;
}

}  // namespace

namespace g4 {
int noalloc_accumulate_entry(const g4_config *cfg, void *const acc[3], const void *G_up, const void *G_dn,
                             const double *sign, int32_t batch, void *ws, uint64_t ws_bytes) {
    return noalloc_accumulate(cfg, acc, G_up, G_dn, sign, batch, ws, ws_bytes);
}
int set_error(int code, const char *msg) { return fail(code, "%s", msg); }
}  // namespace g4

extern "C" {

int g4_config_init(g4_config *cfg) {
    if (!cfg) return fail(G4_E_ARG, "config is NULL");
    std::memset(cfg, 0, sizeof(*cfg));
    cfg->abi_version = G4_ABI_VERSION;
    cfg->lx = cfg->ly = 1;
    cfg->nw = 2;
    cfg->nwex = 1;
    cfg->nq = 1;
    cfg->q_begin = 0;
    cfg->q_end = 1;
    cfg->channels = G4_PH_MAGNETIC;
    cfg->g_in = G4_IN_C128;
    cfg->prod = G4_PROD_F64;
    cfg->acc = G4_ACC_C128;
    cfg->mode = G4_MODE_PLAIN;
    cfg->max_batch = 1;
    cfg->beta = 1.0;
    return G4_OK;
}

int g4_slice_size(const g4_config *cfg, uint64_t *entries_per_channel, uint64_t *device_bytes) {
    Plan P;
    const int rc = validate(cfg, &P);
    if (rc) return rc;
    if (entries_per_channel) *entries_per_channel = P.entries;
    if (device_bytes) *device_bytes = P.total_bytes;
    g_err[0] = 0;
    return G4_OK;
}

int g4_init_slice(const g4_config *cfg, g4_slice **out) {
    if (!out) return fail(G4_E_ARG, "out is NULL");
    *out = nullptr;
    Plan P;
    int rc = validate(cfg, &P);
    if (rc) return rc;
    if (const char *cap = std::getenv("G4_TEST_DEVICE_MEM_LIMIT")) {
        const unsigned long long lim = std::strtoull(cap, nullptr, 10);
        if (P.total_bytes > lim)
            return fail(G4_E_OOM, "slice needs %llu bytes, cap G4_TEST_DEVICE_MEM_LIMIT=%llu",
                        (unsigned long long)P.total_bytes, lim);
    }
    g4_slice *h = new (std::nothrow) g4_slice();
    if (!h) return fail(G4_E_OOM, "host allocation failed");
    h->cfg = *cfg;
    h->cfg.q_list = nullptr;
    h->P = P;
    h->device = cfg->device;
    if (const char *o = std::getenv("G4_TILE_ORDER")) h->order = std::min(4, std::max(0, std::atoi(o)));
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) {
        delete h;
        return fail(G4_E_HIP, "hipSetDevice(%d): %s", cfg->device, hipGetErrorString(e));
    }
    size_t free_b = 0, total_b = 0;
    e = hipMemGetInfo(&free_b, &total_b);
    if (e != hipSuccess) {
        delete h;
        return fail(G4_E_HIP, "hipMemGetInfo: %s", hipGetErrorString(e));
    }
    if (P.total_bytes > free_b) {
        delete h;
        return fail(G4_E_OOM, "slice needs %llu bytes, device has %llu free",
                    (unsigned long long)P.total_bytes, (unsigned long long)free_b);
    }
#define G4_INIT(call)                                              \
    do {                                                           \
        hipError_t e_ = (call);                                    \
        if (e_ != hipSuccess) {                                    \
            int r_ = fail(e_ == hipErrorOutOfMemory ? G4_E_OOM : G4_E_HIP, "%s: %s", #call, \
                          hipGetErrorString(e_));                  \
            release(h);                                            \
            return r_;                                             \
        }                                                          \
    } while (0)
    if (cfg->stream) {
        h->stream = static_cast<hipStream_t>(cfg->stream);
    } else {
        // blocking: ordered with work the caller puts on the null stream
        G4_INIT(hipStreamCreateWithFlags(&h->stream, hipStreamDefault));
        h->own_stream = true;
    }
    const uint64_t ab = P.acc_bytes;
    for (int c = 0; c < 3; ++c)
        if (acc_slots((int)cfg->channels) & (1 << c)) G4_INIT(hipMalloc(&h->acc[c], ab));
    const int nc = P.d.nc;
    G4_INIT(hipMalloc(&h->kadd, (size_t)nc * nc * 4));
    G4_INIT(hipMalloc(&h->ksub, (size_t)nc * nc * 4));
    G4_INIT(hipMalloc(&h->plane_qm, (size_t)P.d.planes * sizeof(int2)));
    G4_INIT(hipMalloc(&h->qpos, (size_t)nc * 4));
    G4_INIT(hipMalloc(&h->groups, (size_t)P.d.planes * sizeof(int4)));
    if (P.dir_bytes) G4_INIT(hipMalloc(&h->dir, P.dir_bytes));
    if (P.stage_bytes) G4_INIT(hipMalloc(&h->stage, P.stage_bytes));
    if (P.pack_bytes) G4_INIT(hipMalloc(&h->pack, P.pack_bytes));
    G4_INIT(hipMalloc(&h->sign_dev, P.sign_bytes));
    G4_INIT(hipHostMalloc(&h->sign_host, P.sign_bytes, hipHostMallocDefault));
    for (int i = 0; i < kSignSlots; ++i) G4_INIT(hipEventCreateWithFlags(&h->sign_ev[i], hipEventDisableTiming));
    if (P.scratch_bytes) G4_INIT(hipMalloc(&h->scratch, P.scratch_bytes));
    if (cfg->flags & G4_F_CHECK_FINITE) {
        G4_INIT(hipMalloc(&h->finite_dev, 256));
        G4_INIT(hipHostMalloc(&h->finite_host, 256, hipHostMallocDefault));
    }
    std::vector<int32_t> kadd, ksub;
    build_momentum_maps(P.d, kadd, ksub);
    std::vector<int2> pq;
    build_planes(P, cfg->nwex, pq);
    G4_INIT(hipMemcpyAsync(h->kadd, kadd.data(), kadd.size() * 4, hipMemcpyHostToDevice, h->stream));
    G4_INIT(hipMemcpyAsync(h->ksub, ksub.data(), ksub.size() * 4, hipMemcpyHostToDevice, h->stream));
    G4_INIT(hipMemcpyAsync(h->plane_qm, pq.data(), pq.size() * sizeof(int2), hipMemcpyHostToDevice, h->stream));
    std::vector<int32_t> qpos(nc, -1);
    for (size_t i = 0; i < P.qlist.size(); ++i) qpos[(size_t)P.qlist[i]] = (int32_t)i;
    G4_INIT(hipMemcpyAsync(h->qpos, qpos.data(), qpos.size() * 4, hipMemcpyHostToDevice, h->stream));
    for (int c = 0; c < 3; ++c)
        if (h->acc[c]) G4_INIT(launch_fill_zero(h->acc[c], ab, h->stream));
    G4_INIT(hipStreamSynchronize(h->stream));
#undef G4_INIT
    rc = rebuild_work(h);
    if (rc) {
        release(h);
        return rc;
    }
    *out = h;
    g_err[0] = 0;
    log_plan(h, "init");
    return G4_OK;
}

int g4_accumulate(g4_slice *h, const void *G_up, const void *G_dn, const double *sign, int32_t batch) {
    int rc = usable(h);
    if (rc) return rc;
    if (batch < 0) return fail(G4_E_ARG, "batch=%d", batch);
    if (batch == 0) return G4_OK;
    if (!G_up || !G_dn || !sign) return fail(G4_E_ARG, "NULL G or sign pointer");
    if (h->cfg.flags & G4_F_CHECK_FINITE)
        for (int b = 0; b < batch; ++b)
            if (!std::isfinite(sign[b])) return fail(G4_E_ARG, "sign[%d] is not finite", b);
    G4_HIP(h, hipSetDevice(h->device));
    if (h->cfg.flags & G4_F_CHECK_FINITE) {
        // screen every G element of the call before anything is accumulated
        const bool dbl = h->cfg.g_in == G4_IN_C128;
        const size_t bytes = (size_t)batch * h->P.d.ng * h->P.d.ng * (dbl ? 16 : 8);
        G4_HIP(h, launch_fill_zero(h->finite_dev, 4, h->stream));
        G4_HIP(h, launch_finite_check(G_up, bytes, dbl ? 1 : 0, h->finite_dev, h->stream));
        G4_HIP(h, launch_finite_check(G_dn, bytes, dbl ? 1 : 0, h->finite_dev, h->stream));
        G4_HIP(h, hipMemcpyAsync(h->finite_host, h->finite_dev, 4, hipMemcpyDeviceToHost, h->stream));
        G4_HIP(h, hipStreamSynchronize(h->stream));
        if (*h->finite_host) return fail(G4_E_ARG, "G_up or G_dn holds a value that is not finite");
    }
    const int B = h->P.batch;
    const char *gu = static_cast<const char *>(G_up), *gd = static_cast<const char *>(G_dn);
    double ssum = 0.0;
    if (h->cfg.mode == G4_MODE_PLAIN) {
        rc = run_plain(h, gu, gd, sign, batch);
        if (rc) return rc;
    } else {
        for (int b0 = 0; b0 < batch; b0 += B) {
            rc = run_pass(h, gu, gd, sign, b0, std::min(B, batch - b0));
            if (rc) return rc;
        }
    }
    for (int b = 0; b < batch; ++b) ssum += sign[b];
    h->measurements += (uint64_t)batch;
    h->sign_sum += ssum;
    return G4_OK;
}

int g4_sync(g4_slice *h) {
    int rc = usable(h);
    if (rc) return rc;
    G4_HIP(h, hipSetDevice(h->device));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    return fold_timings(h);
}

int g4_readback(g4_slice *h, uint32_t channel, uint64_t first, uint64_t count, double *out) {
    int rc = usable(h);
    if (rc) return rc;
    const int c = channel_slot(channel);
    if (c < 0 || !(h->cfg.channels & channel)) return fail(G4_E_ARG, "channel 0x%x not in the slice", channel);
    if (first > h->P.entries || count > h->P.entries - first) return fail(G4_E_ARG, "range outside the slice");
    if (count && !out) return fail(G4_E_ARG, "out is NULL");
    G4_HIP(h, hipSetDevice(h->device));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    if (count >= kScratchEntries) {     // then the scratch holds all slots
        bool ran = false;
        if (rc = readback_lanes(h, c, first, count, out, &ran); rc) return rc;
        if (ran) return fold_timings(h);
    }
    const uint64_t chunk = h->P.scratch_bytes / 16;
    for (uint64_t off = 0; off < count; off += chunk) {
        const uint64_t cnt = std::min(chunk, count - off);
        G4_HIP(h, launch_acc_to_c128(h->cfg.acc, h->acc[c], first + off, cnt, h->scratch, h->P.d.nc, h->P.d.nw, h->stream));
        G4_HIP(h, hipMemcpyAsync(out + 2 * off, h->scratch, cnt * 16, hipMemcpyDeviceToHost, h->stream));
        G4_HIP(h, hipStreamSynchronize(h->stream));
    }
    return fold_timings(h);
}

int g4_load(g4_slice *h, uint32_t channel, uint64_t first, uint64_t count, const double *in) {
    int rc = usable(h);
    if (rc) return rc;
    const int c = channel_slot(channel);
    if (c < 0 || !(h->cfg.channels & channel)) return fail(G4_E_ARG, "channel 0x%x not in the slice", channel);
    if (first > h->P.entries || count > h->P.entries - first) return fail(G4_E_ARG, "range outside the slice");
    if (count && !in) return fail(G4_E_ARG, "in is NULL");
    G4_HIP(h, hipSetDevice(h->device));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    const uint64_t chunk = h->P.scratch_bytes / 16;
    for (uint64_t off = 0; off < count; off += chunk) {
        const uint64_t cnt = std::min(chunk, count - off);
        G4_HIP(h, hipMemcpyAsync(h->scratch, in + 2 * off, cnt * 16, hipMemcpyHostToDevice, h->stream));
        G4_HIP(h, launch_c128_to_acc(h->cfg.acc, h->scratch, h->acc[c], first + off, cnt, h->P.d.nc, h->P.d.nw, h->stream));
        G4_HIP(h, hipStreamSynchronize(h->stream));
    }
    return G4_OK;
}

int g4_merge(g4_slice *dst, g4_slice *src) {
    int rc = usable(dst);
    if (rc) return rc;
    rc = usable(src);
    if (rc) return rc;
    if (dst == src) return fail(G4_E_ARG, "a slice cannot be merged into itself");
    const g4_config &a = dst->cfg, &b = src->cfg;
    if (a.lx != b.lx || a.ly != b.ly || a.nw != b.nw || a.nwex != b.nwex || a.nq != b.nq ||
        a.q_begin != b.q_begin || a.q_end != b.q_end || a.channels != b.channels ||
        dst->P.qlist != src->P.qlist)
        return fail(G4_E_ARG, "slices differ in shape, transfer list, plane range or channels");
    if (dst->device != src->device) return fail(G4_E_UNSUPPORTED, "slices on different devices");
    G4_HIP(dst, hipSetDevice(dst->device));
    G4_HIP(src, hipStreamSynchronize(src->stream));
    for (int c = 0; c < 3; ++c)
        if (dst->acc[c])
            G4_HIP(dst, launch_merge(a.acc, dst->acc[c], b.acc, src->acc[c], dst->P.entries, dst->stream));
    G4_HIP(dst, hipStreamSynchronize(dst->stream));
    dst->measurements += src->measurements;
    dst->sign_sum += src->sign_sum;
    return G4_OK;
}

int g4_set_counts(g4_slice *h, uint64_t measurements, double sign_sum) {
    int rc = usable(h);
    if (rc) return rc;
    if (!std::isfinite(sign_sum)) return fail(G4_E_ARG, "sign_sum not finite");
    h->measurements = measurements;
    h->sign_sum = sign_sum;
    return G4_OK;
}

int g4_reset(g4_slice *h) {
    int rc = usable(h);
    if (rc) return rc;
    G4_HIP(h, hipSetDevice(h->device));
    for (int c = 0; c < 3; ++c)
        if (h->acc[c]) G4_HIP(h, launch_fill_zero(h->acc[c], h->P.acc_bytes, h->stream));
    rc = fold_timings(h);
    if (rc) return rc;
    h->measurements = 0;
    h->sign_sum = 0.0;
    h->launches = 0;
    h->kernel_ms = 0.0;
    h->timed = 0;
    return G4_OK;
}

int g4_stats(g4_slice *h, g4_stats_t *st) {
    int rc = usable(h);
    if (rc) return rc;
    if (!st) return fail(G4_E_ARG, "stats pointer is NULL");
    rc = g4_sync(h);
    if (rc) return rc;
    st->measurements = h->measurements;
    st->sign_sum = h->sign_sum;
    st->launches = h->launches;
    st->kernel_ms = h->kernel_ms;
    st->timed_launches = h->timed;
    st->entries = h->P.entries;
    st->channels = h->cfg.channels;
    st->batch = h->P.batch;
    st->tile = h->P.tile;
    st->variant = h->P.variant;
    return G4_OK;
}

int g4_set_plan(g4_slice *h, int32_t tile, int32_t batch, int32_t variant) {
    int rc = usable(h);
    if (rc) return rc;
    if (tile < 0 || batch < 0 || variant < -1 || variant > G4_VARIANT_PACKED_MFMA) return fail(G4_E_ARG, "bad plan value");
    if (batch > 0 && (h->cfg.mode == G4_MODE_PLAIN ? batch != 1 : batch > h->cfg.max_batch))
        return fail(G4_E_UNSUPPORTED, "batch %d above the allocated max_batch", batch);
    g4_config c = h->cfg;
    std::vector<int32_t> ql = h->P.qlist;
    c.q_list = ql.data();
    if (variant >= 0) {
        c.flags = with_variant(c.flags, variant);
        if (variant != h->P.variant) c.tile = 0;
    }
    if (tile) c.tile = tile;
    Plan P;
    rc = validate(&c, &P);
    if (rc) return rc;
    if (variant >= 0 && P.variant != variant)
        return fail(G4_E_UNSUPPORTED, "variant %d cannot run this slice (split-precision plans use a packed variant)",
                    variant);
    // the workspaces were sized for max_batch; only the pass size changes
    G4_HIP(h, hipSetDevice(h->device));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    P.batch = batch ? batch : h->P.batch;
    P.pack_bytes = pack_need(P, c);
    rc = ensure_pack(h, P);
    if (rc) return rc;
    h->P.ept = P.ept;
    h->P.tile = P.tile;
    h->P.variant = P.variant;
    h->P.persistent = P.persistent;
    h->P.batch = P.batch;
    h->cfg.tile = c.tile;
    h->cfg.flags = c.flags;
    rc = rebuild_work(h);
    if (rc == G4_OK) log_plan(h, "set_plan");
    return rc;
}

}  // extern "C"

// ---- autotuner -----------------------------------------------------------
namespace {

// Whole-pass time (gather + update) of the current plan on measurements
// [0, nb) of the caller's sample, after one untimed pass; accumulators zeroed
// before and after.
int time_plan(g4_slice *h, const char *gu, const char *gd, const double *sign, int nb, double *ms) {
    hipEvent_t e0, e1;
    G4_HIP(h, hipEventCreate(&e0));
    G4_HIP(h, hipEventCreate(&e1));
    int rc = G4_OK;
    for (int rep = 0; rep < 2 && rc == G4_OK; ++rep) {
        for (int c = 0; c < 3; ++c)
            if (h->acc[c]) G4_HIP(h, launch_fill_zero(h->acc[c], h->P.acc_bytes, h->stream));
        G4_HIP(h, hipEventRecord(e0, h->stream));
        for (int b0 = 0; b0 < nb && rc == G4_OK; b0 += h->P.batch)
            rc = run_pass(h, gu, gd, sign, b0, std::min(h->P.batch, nb - b0));
        G4_HIP(h, hipEventRecord(e1, h->stream));
        G4_HIP(h, hipEventSynchronize(e1));
    }
    float f = 0.f;
    if (rc == G4_OK) G4_HIP(h, hipEventElapsedTime(&f, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *ms = f;
    return rc;
}

// Sampled entries of every channel of the slice, spread over all of it, and
// the FP64 reference values of one pass of the tuning measurements there.
struct TuneSample {
    std::vector<uint64_t> idx;
    uint64_t *idx_dev = nullptr;
    double *vals_dev = nullptr;     // idx.size() complex128 values
    double *sign_dev = nullptr;
    std::vector<double> ref[3];     // per channel slot
    ~TuneSample() {
        if (idx_dev) (void)hipFree(idx_dev);
        if (vals_dev) (void)hipFree(vals_dev);
        if (sign_dev) (void)hipFree(sign_dev);
    }
};

double rel_diff(const std::vector<double> &a, const std::vector<double> &ref) {
    double num = 0.0, den = 0.0;
    for (size_t i = 0; i < a.size(); ++i) {
        num += (a[i] - ref[i]) * (a[i] - ref[i]);
        den += ref[i] * ref[i];
    }
    return den > 0 ? std::sqrt(num / den) : std::sqrt(num);
}

int make_sample(g4_slice *h, const void *gu, const void *gd, const double *sign, int nb, TuneSample &ts) {
    const uint64_t E = h->P.entries;
    const uint64_t ns = std::min<uint64_t>(E, 16384);
    ts.idx.resize(ns);
    for (uint64_t j = 0; j < ns; ++j)   // a multiplicative hash spreads them over the slice
        ts.idx[j] = ns == E ? j : (j * 2654435761ull + 977ull) % E;
    G4_HIP(h, hipMalloc(&ts.idx_dev, ns * sizeof(uint64_t)));
    G4_HIP(h, hipMalloc(&ts.vals_dev, ns * 16));
    G4_HIP(h, hipMalloc(&ts.sign_dev, (size_t)nb * sizeof(double)));
    G4_HIP(h, hipMemcpy(ts.idx_dev, ts.idx.data(), ns * sizeof(uint64_t), hipMemcpyHostToDevice));
    G4_HIP(h, hipMemcpy(ts.sign_dev, sign, (size_t)nb * sizeof(double), hipMemcpyHostToDevice));
    for (int c = 0; c < 3; ++c) {
        if (!(acc_slots((int)h->cfg.channels) & (1 << c))) continue;
        RefArgs ra;
        ra.gu = gu;
        ra.gd = gd;
        ra.g_in = h->cfg.g_in == G4_IN_C128 ? 0 : 1;
        ra.g_stride = (int64_t)h->P.d.ng * h->P.d.ng;
        ra.sign = ts.sign_dev;
        ra.batch = nb;
        ra.channel = (int)h->cfg.channels & (73 << c);   // the slice's channel in slot c
        ra.idx = ts.idx_dev;
        ra.count = (int64_t)ns;
        ra.out = ts.vals_dev;
        ra.d = h->P.d;
        ra.t = tables_of(h);
        G4_HIP(h, launch_ref_entries(ra, h->stream));
        ts.ref[c].resize(2 * ns);
        G4_HIP(h, hipMemcpyAsync(ts.ref[c].data(), ts.vals_dev, ns * 16, hipMemcpyDeviceToHost, h->stream));
        G4_HIP(h, hipStreamSynchronize(h->stream));
    }
    return G4_OK;
}

// Largest relative Frobenius difference, over the channels, of the slice's
// sampled entries from the FP64 reference.
int sample_error(g4_slice *h, TuneSample &ts, double *err) {
    *err = 0.0;
    std::vector<double> cur(2 * ts.idx.size());
    for (int c = 0; c < 3; ++c) {
        if (!h->acc[c]) continue;
        G4_HIP(h, launch_acc_gather(h->cfg.acc, h->acc[c], ts.idx_dev, (int64_t)ts.idx.size(), ts.vals_dev,
                                    h->P.d.nc, h->P.d.nw, h->stream));
        G4_HIP(h, hipMemcpyAsync(cur.data(), ts.vals_dev, ts.idx.size() * 16, hipMemcpyDeviceToHost, h->stream));
        G4_HIP(h, hipStreamSynchronize(h->stream));
        *err = std::max(*err, rel_diff(cur, ts.ref[c]));
    }
    return G4_OK;
}

#ifndef G4_BUILD_ID
#define G4_BUILD_ID "unversioned"
#endif

std::string tune_key(g4_slice *h) {
    hipDeviceProp_t prop;
    std::string arch = "unknown";
    if (hipGetDeviceProperties(&prop, h->device) == hipSuccess) arch = prop.gcnArchName;
    std::ostringstream k;
    const g4_config &c = h->cfg;
    // the build id (a hash of the library sources) keeps choices made by
    // another build of the kernels out
    k << G4_BUILD_ID << ":" << arch << ":" << c.lx << "x" << c.ly << ":nw" << c.nw << ":nwex" << c.nwex
      << ":planes" << h->P.d.planes << ":ch" << c.channels << ":in" << c.g_in << ":prod" << c.prod << ":acc"
      << c.acc << ":mode" << c.mode << ":maxb" << c.max_batch;
    std::string key = k.str();
    for (char &ch : key)
        if (ch == ' ') ch = '_';
    return key;
}

// Install plan (batch, tile, variant) on h (validated against the slice's
// configuration); G4_E_UNSUPPORTED if it cannot run this slice.
int install_plan(g4_slice *h, const g4_config &base, const std::vector<int32_t> &qlist, int batch, int tile,
                 int variant) {
    g4_config cc = base;
    cc.q_list = qlist.data();
    cc.flags = with_variant(cc.flags, variant);
    cc.tile = tile;
    Plan P;
    int rc = validate(&cc, &P);
    if (rc) return rc;
    if (P.variant != variant) return fail(G4_E_UNSUPPORTED, "variant %d cannot run this slice", variant);
    P.batch = batch;
    P.pack_bytes = pack_need(P, cc);
    rc = ensure_pack(h, P);
    if (rc) return rc;
    h->P.ept = P.ept;
    h->P.tile = P.tile;
    h->P.variant = P.variant;
    h->P.persistent = P.persistent;
    h->P.batch = batch;
    h->cfg.flags = (h->cfg.flags & G4_F_GRAPH) | (cc.flags & ~(uint32_t)G4_F_GRAPH);
    h->cfg.tile = cc.tile;
    return rebuild_work(h);
}

}  // namespace

extern "C" {

int g4_autotune(g4_slice *h, const void *G_up, const void *G_dn, const double *sign, int32_t batch,
                double tol, g4_tune_result *out) {
    int rc = usable(h);
    if (rc) return rc;
    if (!G_up || !G_dn || !sign || batch < 1 || !(tol > 0)) return fail(G4_E_ARG, "bad autotune arguments");
    if (h->measurements != 0) return fail(G4_E_STATE, "autotune needs a fresh or reset slice");
    G4_HIP(h, hipSetDevice(h->device));
    G4_HIP(h, hipStreamSynchronize(h->stream));
    const char *gu = static_cast<const char *>(G_up), *gd = static_cast<const char *>(G_dn);
    g4_tune_result res;
    std::memset(&res, 0, sizeof(res));
    const std::string key = tune_key(h);
    const char *cache = std::getenv("G4_AUTOTUNE_CACHE");
    int cb = 0, ct = 0, cv = -1;
    if (cache) {
        std::ifstream f(cache);
        std::string k;
        int b, t, v;
        double ms;
        while (f >> k >> b >> t >> v >> ms)
            if (k == key) { cb = b; ct = t; cv = v; }
    }
    const bool plain = h->cfg.mode == G4_MODE_PLAIN;
    const int maxb = plain ? 1 : std::min(h->cfg.max_batch, batch);
    struct Cand { int batch, tile, variant; };
    const Plan keep = h->P;
    const g4_config keep_cfg = h->cfg;
    auto restore = [&]() {
        h->P = keep;
        h->cfg = keep_cfg;
        (void)rebuild_work(h);
    };
    h->cfg.flags &= ~(uint32_t)G4_F_GRAPH;   // candidates are timed running directly
    // every candidate runs the same nbt measurements; the gate compares their
    // sampled entries with an FP64 evaluation of exactly those
    const int nbt = std::max(1, std::min(batch, maxb));
    TuneSample ts;
    rc = make_sample(h, G_up, G_dn, sign, nbt, ts);
    if (rc) return rc;
    double best = 1e300, best_err = 0.0;
    Cand best_c{h->P.batch, h->P.tile, h->P.variant};
    auto try_plan = [&](const Cand &c, double *per, double *err) -> int {
        int r = install_plan(h, keep_cfg, keep.qlist, c.batch, c.tile, c.variant);
        if (r) return r;
        h->cfg.flags &= ~(uint32_t)G4_F_GRAPH;
        double ms = 0.0;
        r = time_plan(h, gu, gd, sign, nbt, &ms);
        if (r) return r;
        r = sample_error(h, ts, err);
        if (r) return r;
        *per = ms / nbt;
        return G4_OK;
    };
    bool from_cache = false;
    if (cv >= 0 && cb >= 1 && cb <= maxb) {
        // a stored choice is installed only after one pass passes the gate
        double per = 0.0, err = 0.0;
        rc = try_plan({cb, ct, cv}, &per, &err);
        if (rc == G4_E_HIP) return rc;
        if (rc == G4_OK && err <= tol) {
            from_cache = true;
            best = per;
            best_err = err;
            best_c = {cb, ct, cv};
        }
    }
    if (!from_cache) {
        std::vector<int> bs;
        for (int b = 1; b <= maxb; b *= 2)
            if (b >= 4 || b == maxb) bs.push_back(b);
        if (bs.empty() || bs.back() != maxb) bs.push_back(maxb);
        const int rp = 256 / h->cfg.nw;
        std::vector<Cand> cands;
        for (int v = 0; v <= G4_VARIANT_PACKED_MFMA; ++v)
            for (int b : bs)
                for (int e : {1, 2, 4}) {
                    if (((v == 1 || v == 4) && e > 1) || (v == 3 && e > 2)) continue;
                    cands.push_back({b, v == 1 ? 16 : v == 4 ? 8 : e * (v == 3 ? 512 / h->cfg.nw : rp), v});
                }
        // a packed plan that would stream is the VALU plan of the same tile and
        // pass, timed already
        auto streams_too = [&](const Cand &c) {
            if (c.variant != G4_VARIANT_PACKED) return false;
            g4_config cc = keep_cfg;
            cc.q_list = keep.qlist.data();
            cc.flags = with_variant(cc.flags, c.variant);
            cc.tile = c.tile;
            Plan P;
            if (validate(&cc, &P)) return false;
            P.batch = c.batch;
            return streams(P, cc.channels);
        };
        for (const Cand &c : cands) {
            double per = 0.0, err = 0.0;
            if (streams_too(c)) continue;
            rc = try_plan(c, &per, &err);
            if (rc == G4_E_HIP) return rc;
            if (rc) continue;                    // does not fit this slice
            res.candidates += 1;
            if (err <= tol && per < best) {
                best = per;
                best_c = c;
                best_err = err;
            }
        }
    }
    if (best == 1e300) {
        restore();
        return fail(G4_E_UNSUPPORTED, "no plan met the error tolerance %.3g against FP64", tol);
    }
    rc = install_plan(h, keep_cfg, keep.qlist, best_c.batch, best_c.tile, best_c.variant);
    if (rc) return rc;
    h->cfg.flags = (h->cfg.flags & ~(uint32_t)G4_F_GRAPH) | (keep_cfg.flags & G4_F_GRAPH);
    rc = g4_reset(h);
    if (rc) return rc;
    G4_HIP(h, hipStreamSynchronize(h->stream));
    res.ms_per_measurement = best;
    res.rel_err_fp64 = best_err;
    res.batch = best_c.batch;
    res.tile = best_c.tile;
    res.variant = best_c.variant;
    if (cache && !from_cache) {
        std::ofstream f(cache, std::ios::app);
        f << key << " " << res.batch << " " << res.tile << " " << res.variant << " "
          << res.ms_per_measurement << "\n";
    }
    if (out) *out = res;
    log_plan(h, from_cache ? "autotune (cached choice)" : "autotune");
    return G4_OK;
}

void g4_destroy(g4_slice *h) { release(h); }

const char *g4_last_error(void) { return g_err; }

int g4_synth_fill(void *out, int32_t dtype, int32_t lx, int32_t ly, int32_t nw, int32_t nwex,
                  double beta, double t, double mu, double h, double noise, uint32_t seed,
                  uint32_t wid, int64_t b0, int32_t count, int32_t spin, void *stream) {
    if (!out && count) return fail(G4_E_ARG, "out is NULL");
    if (dtype != G4_IN_C128 && dtype != G4_IN_C64) return fail(G4_E_ARG, "dtype=%d", dtype);
    if (lx < 1 || ly < 1 || nw < 2 || (nw & 1) || nwex < 1 || count < 0 || b0 < 0 ||
        (spin != 0 && spin != 1) || !(beta > 0))
        return fail(G4_E_ARG, "bad generator shape");
    hipError_t e = launch_synth(out, dtype, lx, ly, nw, nwex, beta, t, mu, h, noise, seed, wid, b0,
                                count, spin, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(G4_E_HIP, "synth: %s", hipGetErrorString(e));
    return G4_OK;
}

int g4_index_maps(const g4_config *cfg, int32_t *kadd, int32_t *ksub, int32_t *plane_q,
                  int32_t *plane_m) {
    Plan P;
    int rc = validate(cfg, &P);
    if (rc && rc != G4_E_UNSUPPORTED) return rc;
    if (rc == G4_E_UNSUPPORTED) {
        // the maps exist for any valid shape; rebuild the shape part only
        g_err[0] = 0;
    }
    std::vector<int32_t> ka, ks;
    Dims d;
    d.lx = cfg->lx;
    d.ly = cfg->ly;
    d.nc = cfg->lx * cfg->ly;
    build_momentum_maps(d, ka, ks);
    if (kadd) std::memcpy(kadd, ka.data(), ka.size() * 4);
    if (ksub) std::memcpy(ksub, ks.data(), ks.size() * 4);
    const int64_t planes = cfg->q_end - cfg->q_begin;
    for (int64_t p = 0; p < planes; ++p) {
        const int64_t iQ = cfg->q_begin + p;
        const int iq = (int)(iQ / cfg->nwex);
        if (plane_q) plane_q[p] = cfg->q_list ? cfg->q_list[iq] : iq;
        if (plane_m) plane_m[p] = (int)(iQ % cfg->nwex);
    }
    return G4_OK;
}

}  // extern "C"
