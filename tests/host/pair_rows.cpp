// Rows K2 and Q - K2 of PP singlet and triplet slices (host code): which plans sum
// them once, and that each list, whole or not, adds every row of every plane once.
#include "../../paper_2105_00027_amd/csrc/g4_abi.cpp"

#include <random>

namespace {

int plan(int lx, int ly, int nw, int nwex, int nq, int64_t q0, int64_t q1, int prod, int batch, uint32_t ch, int mode,
         g4_config *c, Plan *P) {
    g4_config_init(c);
    c->lx = lx; c->ly = ly; c->nw = nw; c->nwex = nwex; c->nq = nq; c->q_begin = q0; c->q_end = q1;
    c->channels = ch; c->mode = mode; c->prod = prod; c->g_in = prod ? G4_IN_C64 : G4_IN_C128; c->max_batch = batch;
    return validate(c, P);
}

// every (plane, k1, k2, row): counts of the additions its tiles make
bool covers(const Plan &P, const std::vector<int4> &groups, const std::vector<int4> &items) {
    const Dims &d = P.d;
    std::vector<int> hits((size_t)d.planes * d.nc * d.nc * d.nw, 0);
    auto at = [&](int p, int k1, int k2, int i) -> int & { return hits[(((size_t)p * d.nc + k1) * d.nc + k2) * d.nw + i]; };
    for (const int4 &t : items) {
        const int4 g = groups[(size_t)t.x];
        const int c0 = t.w & ~(kTileMirror | kTileEdge);
        const int qx = g.x % d.lx, qy = g.x / d.lx, kx = t.z % d.lx, ky = t.z / d.lx;
        const int k2m = (qx - kx + d.lx) % d.lx + d.lx * ((qy - ky + d.ly) % d.ly);
        for (int j = 0; j < g.z; ++j)
            for (int i = c0; i < std::min(c0 + P.tile, d.nw); ++i) {
                const int m = g.y + j, r = m + d.nw - 1 - i;   // the partner's row
                const bool partner = r >= 0 && r < d.nw;
                if ((t.w & kTileEdge) && partner) continue;
                ++at(g.w + j, t.y, t.z, i);
                if ((t.w & kTileMirror) && partner) ++at(g.w + j, t.y, k2m, r);
            }
    }
    for (int h : hits)
        if (h != 1) return false;
    return true;
}

}  // namespace

int main() {
    int bad = 0;
    // few measurements of few frequencies, and small matrices of few measurements or tiles, keep whole tiles
    struct Case { int lx, ly, nw, nwex, nq; int64_t q0, q1; int prod, batch; uint32_t ch; int want; };
    const Case cases[] = {{4, 4, 32, 8, 16, 0, 16, 0, 2, 192, 0},  {4, 4, 32, 8, 16, 0, 16, 0, 8, 192, 1},
                          {8, 8, 16, 8, 64, 0, 16, 1, 8, 64, 0},   {8, 8, 16, 4, 64, 0, 16, 1, 8, 64, 1},
                          {8, 8, 16, 1, 64, 0, 16, 1, 2, 64, 1},   {2, 2, 32, 8, 4, 0, 32, 0, 32, 192, 0},
                          {4, 4, 64, 8, 16, 0, 16, 1, 3, 128, 0},  {4, 4, 64, 8, 16, 0, 16, 1, 4, 128, 1},
                          {4, 4, 64, 8, 16, 0, 16, 0, 1, 128, 1},  {3, 2, 34, 5, 6, 3, 27, 0, 12, 192, 1},
                          {3, 2, 34, 5, 6, 3, 27, 1, 12, 192, 1},  {3, 2, 34, 5, 6, 3, 27, 0, 10, 192, 0},
                          {3, 2, 46, 3, 6, 2, 18, 1, 12, 192, 1},  {3, 2, 46, 3, 6, 2, 18, 0, 3, 192, 0},
                          {3, 2, 70, 1, 6, 0, 6, 0, 3, 192, 1},    {8, 8, 8, 12, 64, 348, 349, 1, 4, 192, 1},
                             {3, 2, 70, 1, 6, 0, 6, 1, 3, 192, 1},  {4, 4, 64, 8, 16, 0, 128, 1, 64, 7, 0}};
    g4_config c;
    Plan P;
    for (const Case &k : cases) {
        const int got = plan(k.lx, k.ly, k.nw, k.nwex, k.nq, k.q0, k.q1, k.prod, k.batch, k.ch, G4_MODE_BATCHED, &c, &P) == G4_OK
                            ? pair_rows_once(P, k.ch) : -1;
        if (got != k.want) {
            std::printf("%dx%d nw %d prod %d batch %d channels %u: %d, not %d\n", k.lx, k.ly, k.nw, k.prod, k.batch, k.ch, got, k.want);
            ++bad;
        }
    }
    std::mt19937 rng(7);
    int once = 0, whole = 0;
    for (int i = 0; i < 600; ++i) {
        const int lx = 1 + (int)(rng() % 4), ly = 1 + (int)(rng() % 4), nwex = 1 + (int)(rng() % 16), nq = 1 + (int)(rng() % (lx * ly));
        const int64_t q0 = rng() % (nq * nwex), q1 = q0 + 1 + rng() % (nq * nwex - q0);
        const int nw = 2 * (int)(1 + rng() % 40), ch = 64 * (int)(1 + rng() % 3);
        if (plan(lx, ly, nw, nwex, nq, q0, q1, (int)(rng() % 2), 1 + (int)(rng() % 32), ch, G4_MODE_BATCHED, &c, &P) != G4_OK) continue;
        (pair_rows_once(P, ch) ? once : whole)++;
        for (bool pair : {false, true})
            for (int order : {0, 2, 4}) {
                std::vector<int4> groups, items;
                build_work(P, nwex, order, ch, pair, groups, items);
                const bool ok = covers(P, groups, items) && (pair || (int64_t)items.size() == whole_tiles(P));
                if (!ok) std::printf("%dx%d nw %d nwex %d order %d pair %d: rows not added once\n", lx, ly, nw, nwex, order, pair);
                bad += !ok;
            }
    }
    // a workspace that holds the list of rows summed once but not that of whole tiles is still taken: the call gets
    // as far as its device, which is none
    plan(4, 4, 32, 8, 16, 0, 128, 0, 2, 192, G4_MODE_BATCHED, &c, &P);
    c.device = 1 << 20;
    double sign[2] = {1.0, 1.0};
    void *acc[3] = {sign, sign, nullptr};
    std::vector<int4> groups, items;
    build_work(P, c.nwex, 2, 192, true, groups, items);
    // small tables and each part's rounding up take less than 16 KB; the lists differ by more
    const uint64_t vectors = 2ull * P.nslots * P.batch * P.d.planes * P.d.n * 16;
    const uint64_t lw = (uint64_t)whole_tiles(P) * sizeof(int4), lo = items.size() * sizeof(int4);
    bad += lw < lo + 32768;
    const int whole_rc = noalloc_accumulate(&c, acc, sign, sign, sign, 2, sign, vectors + lw + 16384);
    const int once_rc = noalloc_accumulate(&c, acc, sign, sign, sign, 2, sign, vectors + lo + 16384);
    const int none_rc = noalloc_accumulate(&c, acc, sign, sign, sign, 2, sign, vectors + lo);
    if (whole_rc != G4_E_HIP || once_rc != G4_E_HIP || none_rc != G4_E_UNSUPPORTED) {
        std::printf("workspaces: %d %d %d\n", whole_rc, once_rc, none_rc);
        ++bad;
    }
    std::printf("%d plans sum rows once, %d do not, %d wrong\n", once, whole, bad);
    return bad || once < 50 || whole < 50;
}
