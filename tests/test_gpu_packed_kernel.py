"""The packed update kernel itself: slices of enough planes that the plan packs
G (the plan line has to say so), plane groups cut at both ends of the slice,
ragged last passes, every accumulator kind.  Sampled entries against the FP64
oracle, FP32 bar 1e-6 as elsewhere; runs of one plan agree bit for bit."""
import functools

import numpy as np
import pytest

from gpu_common import config_for, g4mod, run_slice, to_dev
from oracle import ref
from synth import Workload
from test_gpu_plan_kernels import kernels

pytestmark = pytest.mark.gpu

# nw = 128: groups of 4 (from m = 4 on), 8, 8 and 1 planes; nw = 256: of 4 (from m = 2 on), 6, 6 and 5; nw = 64: of 5, 8, 8, 8
# and 5; nw = 24, nwex = 5: of 2, 5 x 6 and 2
W128 = Workload("nw128", lx=2, ly=2, nw=128, nwex=8, nq=4, q_begin=4, q_end=25)
W256 = Workload("nw256", lx=4, ly=1, nw=256, nwex=6, nq=4, q_begin=2, q_end=23)
W64 = Workload("nw64", lx=3, ly=2, nw=64, nwex=8, nq=5, q_begin=3, q_end=37)
W24 = Workload("nw24", lx=4, ly=2, nw=24, nwex=5, nq=8, q_begin=3, q_end=37)
W64X3 = Workload("nw64, nwex 3", lx=4, ly=3, nw=64, nwex=3, nq=12, q_begin=1, q_end=35)


@functools.lru_cache(maxsize=1)
def inputs(w, count):
    rng = np.random.default_rng(w.ng + count)
    g = [(rng.normal(size=(count, w.ng, w.ng)) + 1j * rng.normal(size=(count, w.ng, w.ng))).astype(np.complex64)
         for _ in range(2)]
    return g[0], g[1], np.where(rng.random(count) < 0.8, 1.0, -0.75)


def check_packed(capfd, monkeypatch, w, count, g_in=1, twice=False, **kw):
    g4 = g4mod()
    print(f"\ncase {w.name} channels={w.channels} count={count} g_in={g_in} {kw}", flush=True)
    gu, gd, s = inputs(w.with_(channels=1), count)
    cfg = config_for(w, mode=1, prod=1, g_in=g_in, flags=g4.G4_F_PACKED, **kw)
    assert kernels(capfd, monkeypatch, cfg) == ["packed"]
    du, dd = to_dev(gu, g_in), to_dev(gd, g_in)
    got, st = run_slice(cfg, du, dd, s)
    assert st["variant"] == g4.G4_VARIANT_PACKED and st["launches"] == -(-count // kw["batch"])
    if twice:
        again, _ = run_slice(cfg, du, dd, s)
        assert all(np.array_equal(got[ch], again[ch]) for ch in got)
    idx = np.random.default_rng(5).integers(0, w.planes * w.n * w.n, size=6000)
    idx[:4] = [0, w.planes * w.n * w.n - 1, w.n * w.n - 1, (w.planes - 1) * w.n * w.n]
    for ch, v in got.items():
        want = ref.entries(w, ch, gu.astype(np.complex128), gd.astype(np.complex128), s, idx)
        assert np.linalg.norm(v.reshape(-1)[idx] - want) <= 1e-6 * np.linalg.norm(want), ch


@pytest.mark.parametrize("g_in", [0, 1], ids=["c128-in", "c64-in"])
@pytest.mark.parametrize("acc", [0, 1, 2], ids=["acc-c128", "acc-kahan", "acc-c64"])
@pytest.mark.parametrize("w,channels,count,B,tile", [(W128, 1, 5, 2, 4), (W128, 1, 4, 4, 2), (W128, 2, 3, 2, 0),
                                                     (W256, 1, 3, 2, 0), (W256, 2, 4, 3, 2)],
                         ids=["nw128-mag-t4", "nw128-mag-t2", "nw128-chg", "nw256-mag", "nw256-chg-t2"])
def test_direct_vector_in_registers(capfd, monkeypatch, w, channels, count, B, tile, acc, g_in):
    """One PH channel at 128 frequencies and more: a(Q, K1) is read into registers."""
    check_packed(capfd, monkeypatch, w.with_(channels=channels), count, g_in, acc=acc, batch=B, tile=tile)


@pytest.mark.parametrize("acc", [0, 1, 2], ids=["acc-c128", "acc-kahan", "acc-c64"])
@pytest.mark.parametrize("channels", [1, 2, 3])
def test_nw64_tile8(capfd, monkeypatch, channels, acc):
    check_packed(capfd, monkeypatch, W64.with_(channels=channels), 7, acc=acc, batch=3, tile=8)


@pytest.mark.parametrize("channels", [1, 2, 4, 5])
def test_channel_subsets(capfd, monkeypatch, channels):
    check_packed(capfd, monkeypatch, W24.with_(channels=channels), 5, acc=0, batch=3)


def test_long_pass(capfd, monkeypatch):
    check_packed(capfd, monkeypatch, W64X3, 21, acc=0, batch=16)


def test_runs_agree_bit_for_bit(capfd, monkeypatch):
    check_packed(capfd, monkeypatch, W128, 3, acc=0, batch=2, twice=True)
