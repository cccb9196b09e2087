"""The streamed update kernel, held to itself: every plan listed has to run it (the
plan line says so) or to be refused as listed; sampled entries against the FP64
oracle.  Bars: FP64 1e-12, FP32 products 1e-6, as elsewhere.  G in FP32 may lie on
8 bytes: a copy of 16 bytes takes two columns from wherever they are."""
import functools

import numpy as np
import pytest

from gpu_common import config_for, g4mod, run_slice, to_dev
from oracle import ref
from synth import Workload
from test_gpu_plan_kernels import kernels

pytestmark = pytest.mark.gpu

# 7 rows a sweep and one row in the last tile; plane groups of 3, 8 and 4; odd first columns at 64 frequencies, with the
# geometry compiled in; groups of 4; one and two rows a sweep; the geometry at run time over partial groups
CASES = {
    "36 rows": Workload("36 rows", lx=2, ly=1, nw=36, nwex=8, nq=2, q_begin=0, q_end=14),
    "50 rows, nwex 3": Workload("50 rows, nwex 3", lx=2, ly=2, nw=50, nwex=3, nq=4, q_begin=1, q_end=11),
    "nw 64": Workload("nw 64", lx=3, ly=2, nw=64, nwex=8, nq=2, q_begin=3, q_end=14),
    "nw 64, nwex 4": Workload("nw 64, nwex 4", lx=2, ly=2, nw=64, nwex=4, nq=4, q_begin=2, q_end=9),
    "nw 128, nwex 8": Workload("nw 128, nwex 8", lx=2, ly=1, nw=128, nwex=8, nq=2, q_begin=0, q_end=7),
}
PLAIN, F64, F32 = dict(mode=0), dict(mode=1, batch=3), dict(mode=1, prod=1, g_in=1, batch=8)
PACKED = dict(F32, flags=16)
RUNS = [
    ("36 rows", PLAIN, (1, 2, 4)), ("36 rows", F64, (1, 2, 4, 3)), ("36 rows", F32, (1, 4, 3)), ("36 rows", PACKED, (1, 4)),
    ("50 rows, nwex 3", PLAIN, (1, 4, 3, 7)), ("50 rows, nwex 3", F64, (1, 4, 3)), ("50 rows, nwex 3", F32, (1, 2)),
    ("50 rows, nwex 3", PACKED, (1, 4)),
    ("nw 64", PLAIN, (1, 4, 3, 5, 7)), ("nw 64", F64, (1, 4, 3, 5, 7)), ("nw 64", F32, (1, 4, 3, 5, 7)),
    ("nw 64", dict(F32, acc=1, tile=4), (1, 3, 7)), ("nw 64", PACKED, (1, 4, 3, 5)),
    ("nw 64, nwex 4", PLAIN, (1, 3, 7)), ("nw 64, nwex 4", F64, (1, 3)), ("nw 64, nwex 4", dict(F32, acc=2), (1, 3, 7)),
    ("nw 64, nwex 4", PACKED, (1, 3, 7)),
    ("nw 128, nwex 8", PLAIN, (1, 2, 4)), ("nw 128, nwex 8", dict(F64, batch=1), (1, 4)), ("nw 128, nwex 8", F32, (1, 4)),
]


@functools.lru_cache(maxsize=2)
def inputs(w, count):
    rng = np.random.default_rng(w.ng + count)
    g = [(rng.normal(size=(count, w.ng, w.ng)) + 1j * rng.normal(size=(count, w.ng, w.ng))).astype(np.complex64)
         for _ in range(2)]
    return g[0], g[1], np.where(rng.random(count) < 0.8, 1.0, -0.75)


@pytest.mark.parametrize("name,kw,channels", [(n, kw, ch) for n, kw, chs in RUNS for ch in chs],
                         ids=lambda v: None if isinstance(v, dict) else str(v))
def test_streamed_plans(capfd, monkeypatch, name, kw, channels):
    w = CASES[name].with_(channels=channels)
    print(f"\ncase {name} channels={channels} {kw}", flush=True)
    cfg = config_for(w, **kw)
    assert kernels(capfd, monkeypatch, cfg) == ["streamed"]
    gu, gd, s = inputs(CASES[name], 11)
    g_in = kw.get("g_in", 0)
    got, _ = run_slice(cfg, to_dev(gu, g_in), to_dev(gd, g_in), s)
    size = w.planes * w.n * w.n
    idx = np.random.default_rng(3).integers(0, size, size=5000)
    idx[:4] = [0, size - 1, w.n * w.n - 1, size - w.n * w.n]
    for ch, v in got.items():
        want = ref.entries(w, ch, gu.astype(np.complex128), gd.astype(np.complex128), s, idx)
        err = np.linalg.norm(v.reshape(-1)[idx] - want)
        assert err <= (1e-6 if kw.get("prod") else 1e-12) * np.linalg.norm(want), ch


@pytest.mark.parametrize("kw,code", [(dict(F64, tile=5), "G4_E_UNSUPPORTED"), (dict(PACKED, prod=0, g_in=0), "G4_E_UNSUPPORTED"),
                                     (dict(PLAIN, prod=1, g_in=1), "G4_E_ARG"), (dict(F32, batch=0), "G4_E_ARG")])
def test_refused_plans(kw, code):
    g4 = g4mod()
    with pytest.raises(g4.G4Error) as e:
        g4.g4_slice_size(config_for(CASES["nw 64"], **kw))
    assert e.value.code == getattr(g4, code)


@pytest.mark.parametrize("name,kw", [("nw 64", F32), ("nw 64", PACKED), ("36 rows", F32), ("nw 64, nwex 4", PACKED)],
                         ids=lambda v: None if isinstance(v, dict) else str(v))
@pytest.mark.parametrize("channels", [1, 7])
def test_g_on_eight_bytes(name, kw, channels):
    """Matrices that start on 8 but not on 16 bytes: the same bits."""
    import torch
    w = CASES[name].with_(channels=channels)
    print(f"\ncase offset {name} channels={channels} {kw}", flush=True)
    gu, gd, s = inputs(CASES[name], 11)

    def shifted(a):
        buf = torch.zeros(a.size + 1, dtype=torch.complex64, device="cuda")
        buf[1:] = torch.from_numpy(a.reshape(-1)).cuda()
        t = buf[1:].view(a.shape)
        assert t.data_ptr() % 16 == 8
        return t

    cfg = config_for(w, **kw)
    want, _ = run_slice(cfg, to_dev(gu, 1), to_dev(gd, 1), s)
    got, _ = run_slice(cfg, shifted(gu), shifted(gd), s)
    for ch in want:
        assert np.array_equal(got[ch], want[ch]), ch
