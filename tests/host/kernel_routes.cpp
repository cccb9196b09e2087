// Which kernel a default plan's launch runs (host code): over many shapes, the
// streamed kernel never where it holds fewer blocks a CU than the register-staged
// one, always within the LDS, and the launch-time check accepts what was routed.
#include "../../paper_2105_00027_amd/csrc/g4_abi.cpp"

#include <random>

int main() {
    std::mt19937 rng(5);
    auto pick = [&](std::initializer_list<int> l) { return *(l.begin() + rng() % l.size()); };
    int bad = 0, streamed = 0, total = 0;
    for (int i = 0; i < 20000; ++i) {
        g4_config c;
        g4_config_init(&c);
        c.lx = pick({1, 2, 3, 4, 6, 8});
        c.ly = pick({1, 2, 3, 4, 6, 8});
        c.nw = 2 * (int)(1 + rng() % 128);
        if (rng() % 4 == 0) c.nw = 64;
        c.nwex = (int)(1 + rng() % 16);
        c.nq = 1 + (int)(rng() % (c.lx * c.ly));
        c.q_begin = rng() % (c.nq * c.nwex);
        c.q_end = c.q_begin + 1 + rng() % (c.nq * c.nwex - c.q_begin);
        c.channels = (uint32_t)pick({1, 2, 3, 4, 5, 6, 7});
        const int kind = (int)(rng() % 3);
        c.mode = kind ? G4_MODE_BATCHED : G4_MODE_PLAIN;
        c.prod = kind == 2 ? G4_PROD_F32 : G4_PROD_F64;
        c.g_in = kind == 2 ? G4_IN_C64 : G4_IN_C128;
        c.max_batch = pick({1, 2, 5, 16, 64});
        Plan P;
        if (validate(&c, &P) != G4_OK) continue;
        std::vector<int4> groups, items;
        if ((int64_t)P.d.planes * P.d.nc * P.d.nc > 200000) continue;
        build_work(P, c.nwex, 2, c.channels, false, groups, items);
        for (int nb : {1, P.batch}) {
            const int64_t slot = (int64_t)P.batch * P.d.planes * P.d.n;
            const int v = pass_variant(P, c.channels, (int)groups.size(), (int)items.size(), nb, slot);
            ++total;
            if (v != kVariantStreamed) continue;
            ++streamed;
            const size_t lds = stream_lds_bytes(stream_geom_of(P.kind, (int)c.channels, P.mgroup, P.tile, P.d), nb);
            const int mine = stream_blocks(P.kind, (int)c.channels, P.ept, P.mgroup, P.tile, P.d, nb);
            const int theirs = update_blocks(P.kind, (int)c.channels, P.ept, P.mgroup, P.tile, P.d);
            if (lds > 160 * 1024 || mine < 1 || mine < theirs ||
                !stream_runs(P.kind, (int)c.channels, P.ept, P.mgroup, P.tile, P.d, slot, nb)) {
                std::printf("%dx%d nw %d nwex %d channels %u kind %d batch %d: %zu bytes, %d blocks, registers %d\n", c.lx,
                            c.ly, c.nw, c.nwex, c.channels, kind, nb, lds, mine, theirs);
                ++bad;
            }
        }
    }
    // the 6x6, 128 frequencies, one-channel plain pass: one buffer, two blocks a CU
    Dims d{};
    d.lx = d.ly = 6; d.nc = 36; d.nw = 128; d.nwex = 16; d.nwg = 143; d.ng = 36 * 143; d.n = 36 * 128; d.planes = 72;
    const StreamGeom g = stream_geom_of(0, 1, 8, 2, d);
    if (stream_lds_bytes(g, 1) > 80 * 1024 || stream_blocks(0, 1, 1, 8, 2, d, 1) < 2) {
        std::printf("one measurement, 128 frequencies: %zu bytes\n", stream_lds_bytes(g, 1));
        ++bad;
    }
    std::printf("%d launches, %d streamed, %d wrong\n", total, streamed, bad);
    return bad || streamed < 1000 || total - streamed < 1000;
}
