"""Device bytes of packed plans: the packed buffer is counted where the plan packs
and only there (no GPU needed)."""
import pytest

from paper_2105_00027_amd import g4


def size(flags, **kw):
    c = dict(lx=8, ly=8, nw=64, nwex=4, nq=64, q_begin=64, q_end=68, channels=7, mode=1, prod=1, g_in=1, max_batch=32)
    c.update(kw)
    return g4.g4_slice_size(g4.Config(flags=flags, **c))[1]


def packed_bytes(lx, ly, nw, nwex, planes, slots, batch):
    nwg, nc = nw + nwex - 1, lx * ly
    ldp = (nc * ((nwg + 7) // 8 * 8) + 1 + 7) // 8 * 8
    return batch * ((nc * nwg * ldp * 16 + 2 * slots * planes * nc * nw * 8 + 255) // 256 * 256)


@pytest.mark.parametrize("kw", [dict(), dict(lx=6, ly=6, nwex=8, nq=5, q_begin=13, q_end=27, channels=1, max_batch=16),
                                dict(q_end=65, channels=1), dict(channels=4, q_begin=0, q_end=31)])
def test_a_plan_that_streams_has_no_packed_buffer(kw):
    """The 8x8 three-channel share would count 10 GB that no kernel touches."""
    P = g4.G4_F_PACKED
    assert size(P, **kw) == size(0, **kw)
    # the persistent form packs, and counts its buffer
    c = dict(dict(lx=8, ly=8, nw=64, nwex=4, q_begin=64, q_end=68, channels=7, max_batch=32), **kw)
    want = packed_bytes(c["lx"], c["ly"], c["nw"], c["nwex"], c["q_end"] - c["q_begin"],
                        bin(c["channels"] & 3).count("1"), c["max_batch"])
    assert size(P | g4.G4_F_PERSISTENT, **kw) - size(P, **kw) == want > 1 << 28


def test_a_plan_that_packs_counts_it():
    P = g4.G4_F_PACKED
    kw = dict(lx=4, ly=4, nwex=8, nq=16, q_begin=0, q_end=128, channels=1, max_batch=64)
    assert size(P, **kw) - size(0, **kw) == packed_bytes(4, 4, 64, 8, 128, 1, 64)
    assert size(P | g4.G4_F_PERSISTENT, **kw) == size(P, **kw)


def test_what_a_packed_plan_refuses_stays_refused():
    for kw in (dict(nw=130, nwex=1, q_begin=0, q_end=4, lx=2, ly=2, nq=4, tile=1), dict(prod=0, g_in=0), dict(mode=0, prod=0, g_in=0)):
        with pytest.raises(g4.G4Error) as e:
            size(g4.G4_F_PACKED, **kw)
        assert e.value.code == g4.G4_E_UNSUPPORTED, kw
