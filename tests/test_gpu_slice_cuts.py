"""Slices cut differently hold the same bits: which update kernel a part runs
depends on its planes, the arithmetic of an entry does not."""
import numpy as np
import pytest

from gpu_common import config_for, g4mod, host_inputs, run_slice, to_dev
from synth import Workload
from test_gpu_plan_kernels import kernels

pytestmark = pytest.mark.gpu

MANY = Workload("2x2, 40 planes", lx=2, ly=2, nw=16, nwex=10, nq=4)
NW64 = Workload("2x1, nw 64, 16 planes", lx=2, ly=1, nw=64, nwex=8, nq=2)
F32 = dict(mode=1, prod=1, g_in=1, batch=3)


def whole_and_parts(w, cuts, kw, count=7):
    gu, gd, s = host_inputs(w, count)
    s = s * np.array([1.0, 0.5, 1.0, 2.0, 1.0, 0.75, 1.0])[:count]
    g_in = kw.get("g_in", 0)
    du, dd = to_dev(gu, g_in), to_dev(gd, g_in)
    full, _ = run_slice(config_for(w, q_begin=0, q_end=w.nQ, **kw), du, dd, s)
    parts = [run_slice(config_for(w, q_begin=a, q_end=b, **kw), du, dd, s)[0] for a, b in zip(cuts[:-1], cuts[1:])]
    return full, {ch: np.concatenate([p[ch] for p in parts]) for ch in full}


@pytest.mark.parametrize("acc", [0, 1], ids=["c128", "kahan"])
@pytest.mark.parametrize("w,channels,cuts", [(MANY, 1, [0, 3, 10, 13, 18, 40]), (MANY, 3, [0, 3, 10, 13, 15, 40]),
                                             (MANY, 5, [0, 3, 5, 40]), (MANY, 7, [0, 3, 5, 40]),
                                             (NW64, 3, [0, 3, 16]), (NW64, 5, [0, 8, 11, 16]), (NW64, 7, [0, 3, 10, 16])],
                         ids=lambda v: v.name if isinstance(v, Workload) else None)
def test_packed_plans(capfd, monkeypatch, w, channels, cuts, acc):
    print(f"\ncase packed {w.name} channels={channels} cuts={cuts} acc={acc}", flush=True)
    g4 = g4mod()
    kw = dict(F32, acc=acc, flags=g4.G4_F_PACKED, channels=channels)
    ran = {kernels(capfd, monkeypatch, config_for(w, q_begin=a, q_end=b, **kw))[0]
           for a, b in zip([0] + cuts[:-1], [w.nQ] + cuts[1:])}
    assert ran == {"packed", "streamed"}
    full, parts = whole_and_parts(w, cuts, kw)
    for ch in full:
        assert np.array_equal(full[ch], parts[ch]), ch


@pytest.mark.parametrize("kw", [dict(mode=0), dict(mode=1, batch=3), F32], ids=["plain", "f64", "f32"])
@pytest.mark.parametrize("w,channels", [(MANY, 3), (MANY, 7), (NW64, 1), (NW64, 5), (NW64, 7)],
                         ids=lambda v: v.name if isinstance(v, Workload) else None)
def test_default_plans(w, channels, kw):
    """Parts of one, two and five planes (partial groups) against whole groups."""
    print(f"\ncase default {w.name} channels={channels} {kw}", flush=True)
    full, parts = whole_and_parts(w, [0, 1, 3, 8, w.nQ], dict(kw, channels=channels))
    for ch in full:
        assert np.array_equal(full[ch], parts[ch]), ch


@pytest.mark.parametrize("channels", [1, 3, 5, 7])
def test_plain_launches_of_one_and_of_many(channels):
    """Plain mode: a handle's launches of one measurement and one launch of all
    of them in g4_accumulate_into."""
    import torch
    g4 = g4mod()
    w = Workload("2x1, nw 36", lx=2, ly=1, nw=36, nwex=8, nq=2, q_begin=2, q_end=13, channels=channels)
    print(f"\ncase plain channels={channels}", flush=True)
    gu, gd, s = host_inputs(w, 6)
    du, dd = to_dev(gu, 0), to_dev(gd, 0)
    handle, _ = run_slice(config_for(w, mode=0), du, dd, s)
    n, nc = w.n, w.lx * w.ly
    accs = [torch.zeros((w.planes, n, n), dtype=torch.complex128, device="cuda") if channels & (1 << c) else None
            for c in range(3)]
    g4.g4_accumulate_into(config_for(w, mode=0), *accs, du, dd, s)
    for c, a in enumerate(accs):
        if a is not None:
            got = a.cpu().numpy().reshape(w.planes, nc, nc, w.nw, w.nw).transpose(0, 1, 3, 2, 4).reshape(w.planes, n, n)
            assert np.array_equal(got, handle[1 << c]), c
