// The work-tile list in orbits (order 4) against its plain definition, and its
// cost against the list in windows (order 2), which g4_accumulate_into made on
// every call before it.  Exit status 0 when every check holds.
#include "../../paper_2105_00027_amd/csrc/g4_abi.cpp"

#include <chrono>

namespace {

// Orbits of (k1, k2) in the order of their first pair; a pair's neighbours are
// (k2+q, k1+q) and, with PP, (q-k1, q-k2); an orbit's tiles by pairs of K2 tiles,
// then by k1 + q, then as found.
std::vector<int4> orbits(const Plan &P, const std::vector<int4> &groups, bool pp) {
    const Dims &d = P.d;
    auto add = [&](int a, int b) { return (a % d.lx + b % d.lx) % d.lx + d.lx * ((a / d.lx + b / d.lx) % d.ly); };
    auto sub = [&](int a, int b) {
        return (a % d.lx - b % d.lx + d.lx) % d.lx + d.lx * ((a / d.lx - b / d.lx + d.ly) % d.ly);
    };
    std::vector<int> qs;
    for (int q = 0; q < d.nc; ++q)
        for (const int4 &g : groups)
            if (g.x == q) {
                qs.push_back(q);
                break;
            }
    std::vector<char> seen((size_t)d.nc * d.nc, 0);
    std::vector<int4> sorted;
    for (int seed = 0; seed < d.nc * d.nc; ++seed) {
        if (seen[(size_t)seed]) continue;
        std::vector<int> orbit{seed};
        seen[(size_t)seed] = 1;
        for (size_t i = 0; i < orbit.size(); ++i) {
            const int k1 = orbit[i] % d.nc, k2 = orbit[i] / d.nc;
            std::vector<int> next;
            for (int q : qs) next.push_back(add(k1, q) * d.nc + add(k2, q));
            if (pp) for (int q : qs) next.push_back(sub(q, k2) * d.nc + sub(q, k1));
            for (int e : next)
                if (!seen[(size_t)e]) {
                    seen[(size_t)e] = 1;
                    orbit.push_back(e);
                }
        }
        std::vector<int4> run;
        for (int e : orbit)
            for (int q : qs)
                for (int g = 0; g < (int)groups.size(); ++g)
                    if (groups[(size_t)g].x == q) run.push_back(int4{g, e % d.nc, e / d.nc, add(e % d.nc, q)});
        std::stable_sort(run.begin(), run.end(), [](const int4 &x, const int4 &y) { return x.w < y.w; });
        for (int cb = 0; cb < d.nw; cb += 2 * P.tile)
            for (const int4 &t : run)
                for (int c = cb; c < std::min(d.nw, cb + 2 * P.tile); c += P.tile) sorted.push_back(int4{t.x, t.y, t.z, c});
    }
    std::vector<int4> items;
    spread_over_xcds(sorted, items);
    return items;
}

// the quickest of many lists in orders 2 and 4, made in turn
void best_us(const Plan &P, int nwex, uint32_t ch, double *t2, double *t4) {
    *t2 = *t4 = 1e300;
    for (int r = 0; r < 100; ++r)
        for (int order : {2, 4}) {
            double &best = order == 2 ? *t2 : *t4;
            std::vector<int4> groups, items;
            const auto t = std::chrono::steady_clock::now();
            build_work(P, nwex, order, ch, false, groups, items);
            best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t).count());
        }
}

}  // namespace

int main() {
    struct Shape { int lx, ly, nw, nwex, nq; int64_t q0, q1; uint32_t channels; };
    const Shape shapes[] = {{1, 1, 16, 3, 1, 0, 3, 1},    {2, 2, 16, 1, 1, 0, 1, 1},   {3, 2, 50, 5, 4, 3, 17, 7},
                            {4, 4, 8, 2, 16, 0, 30, 4},   {4, 4, 54, 8, 3, 5, 20, 3},  {5, 3, 22, 4, 15, 9, 40, 5},
                            {6, 6, 8, 1, 36, 0, 30, 7},   {8, 8, 22, 1, 16, 14, 15, 1}, {8, 8, 8, 4, 64, 0, 30, 1},
                            {8, 8, 8, 1, 64, 0, 30, 1}};
    int bad = 0;
    for (const Shape &s : shapes) {
        g4_config c;
        g4_config_init(&c);
        c.lx = s.lx; c.ly = s.ly; c.nw = s.nw; c.nwex = s.nwex; c.nq = s.nq; c.q_begin = s.q0; c.q_end = s.q1;
        c.channels = s.channels; c.mode = G4_MODE_BATCHED; c.prod = G4_PROD_F32; c.g_in = G4_IN_C64; c.max_batch = 16;
        Plan P;
        if (validate(&c, &P) != G4_OK) {
            std::printf("refused: %s\n", g4_last_error());
            return 2;
        }
        std::vector<int4> groups, items;
        build_work(P, s.nwex, 4, s.channels, false, groups, items);
        const std::vector<int4> want = orbits(P, groups, (s.channels & G4_PP_UPDOWN) != 0);
        const bool same = items.size() == want.size() && !std::memcmp(items.data(), want.data(), want.size() * sizeof(int4));
        double t2, t4;
        best_us(P, s.nwex, s.channels, &t2, &t4);
        // half as much again as the windows and 10 us for a short list would do; twice that for a busy machine
        const bool quick = t4 <= 3.0 * t2 + 20.0;
        std::printf("%dx%d nw %d planes %lld: %zu tiles, windows %.1f us, orbits %.1f us%s%s\n", s.lx, s.ly, s.nw,
                    (long long)(s.q1 - s.q0), items.size(), t2, t4, same ? "" : "  DIFFERENT", quick ? "" : "  SLOW");
        bad += !same + !quick;
    }
    // the order of a plan: orbits for one plane group beyond an L2, long FP32 passes of PH channels on large clusters
    // and few planes of packed operands; windows (runs for packed operands) otherwise
    struct Order { int l, nw, nwex, nq; int64_t q0, q1; uint32_t channels; int prod, batch; uint32_t flags; int want; };
    const Order orders[] = {{8, 64, 4, 64, 64, 68, 7, 1, 32, G4_F_PACKED, 4}, {6, 64, 8, 5, 13, 27, 1, 1, 16, G4_F_PACKED, 4},
                            {6, 64, 8, 5, 13, 27, 1, 1, 2, 0, 2},             {6, 64, 8, 5, 13, 27, 3, 1, 16, 0, 2},
                            {6, 128, 16, 36, 3, 14, 7, 1, 16, 0, 2},          {6, 54, 16, 36, 3, 14, 1, 0, 4, 0, 2},
                            {4, 64, 8, 16, 0, 16, 1, 1, 64, 0, 2},            {4, 128, 8, 16, 0, 8, 1, 0, 8, 0, 4},
                            {2, 16, 8, 4, 0, 8, 1, 0, 8, 0, 2},               {4, 64, 8, 16, 0, 128, 1, 1, 64, G4_F_PACKED, 3},
                            {4, 64, 8, 16, 0, 31, 1, 1, 64, G4_F_PACKED, 4},  {6, 32, 4, 36, 0, 8, 1, 1, 64, G4_F_PACKED, 4},
                            {6, 64, 8, 5, 13, 27, 24, 1, 16, 0, 2},           {4, 128, 2, 16, 8, 9, 7, 0, 27, 0, 2},
                            {4, 128, 2, 16, 8, 9, 7, 0, 8, 0, 4},             {2, 128, 8, 4, 0, 8, 1, 0, 8, 0, 2},
                            {4, 64, 8, 16, 0, 8, 1, 0, 64, 0, 4},             {4, 160, 4, 16, 4, 6, 7, 1, 64, 0, 2},
                            {6, 50, 1, 36, 2, 12, 1, 1, 30, 0, 2},            {6, 50, 1, 36, 2, 3, 1, 1, 30, 0, 4},
                            {2, 128, 1, 4, 0, 1, 4, 0, 11, 0, 2},             {3, 128, 1, 9, 0, 9, 1, 1, 32, G4_F_PACKED, 3},
                            {3, 128, 1, 9, 0, 1, 1, 1, 32, G4_F_PACKED, 4}};
    for (const Order &o : orders) {
        g4_config c;
        g4_config_init(&c);
        c.lx = c.ly = o.l; c.nw = o.nw; c.nwex = o.nwex; c.nq = o.nq; c.q_begin = o.q0; c.q_end = o.q1;
        c.channels = o.channels; c.mode = G4_MODE_BATCHED; c.prod = o.prod; c.g_in = o.prod ? G4_IN_C64 : G4_IN_C128;
        c.max_batch = o.batch; c.flags = o.flags;
        Plan P;
        const int got = validate(&c, &P) == G4_OK ? default_order(P, c.channels) : -1;
        std::vector<int4> groups, items;
        if (got >= 0) build_work(P, c.nwex, got, c.channels, false, groups, items);
        if (got != o.want || plane_groups(P) != (int)groups.size()) {
            std::printf("%dx%d nw %d planes %lld channels %u: order %d, not %d\n", o.l, o.l, o.nw, (long long)(o.q1 - o.q0),
                        o.channels, got, o.want);
            ++bad;
        }
    }
    // a call of few measurements makes the quicker list
    g4_config c;
    g4_config_init(&c);
    c.lx = c.ly = 8; c.nw = 22; c.nq = 1; c.q_end = 1; c.channels = 1; c.max_batch = 16;
    for (int mode : {G4_MODE_PLAIN, G4_MODE_BATCHED}) {
        c.mode = mode;
        Plan P;
        if (validate(&c, &P) != G4_OK || call_order(P, 1, 7) != 2 || call_order(P, 1, 8) != 4) {
            std::printf("one plane of 8x8, mode %d: orders %d and %d\n", mode, call_order(P, 1, 7), call_order(P, 1, 8));
            ++bad;
        }
    }
    return bad ? 1 : 0;
}
