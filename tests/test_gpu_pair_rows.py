"""PP singlet and triplet slices whose rows K2 and Q - K2 are summed once, and
slices of the same shapes whose plans keep whole tiles, against the FP64 oracle:
plane groups of 1, 4 and 8, odd momenta grids, slices cut inside a group, a pass
shorter than the others.  The bars are those of the other channels (1e-12 for
FP64 products, 1e-6 for FP32 ones)."""
import numpy as np
import pytest

from gpu_common import config_for, g4mod, host_inputs, run_slice, to_dev
from metrics import check_entries
from oracle import ref
from synth import Workload

pytestmark = pytest.mark.gpu

PAIR = ref.PP_SINGLET | ref.PP_TRIPLET
G8 = Workload("3x2, groups of 8", lx=3, ly=2, nw=34, nwex=5, nq=6, q_list=(4, 0, 5, 1, 3, 2), q_begin=3, q_end=27,
              seed=51, wid=51, channels=PAIR)
G4 = G8.with_(name="3x2, groups of 4", nwex=3, nq=6, q_begin=2, q_end=18, nw=46)
G1 = G8.with_(name="3x2, single planes", nwex=1, nq=6, q_begin=0, q_end=6, nw=70)
_cache = {}


def want_of(w, count):
    if (w, count) not in _cache:
        gu, gd, s = host_inputs(w, count)
        _cache[(w, count)] = {ch: ref.accumulate(w, ch, gu, gd, s) for ch in (ref.PP_SINGLET, ref.PP_TRIPLET)}
    return _cache[(w, count)]


def check(got, want, tol):
    for ch, v in want.items():
        check_entries(got[ch], v, tol, what="channel %d" % ch)


@pytest.mark.parametrize("kw,tol", [(dict(mode=1), 1e-12), (dict(mode=1, prod=1, g_in=1), 1e-6)], ids=["f64", "f32"])
@pytest.mark.parametrize("w", [G8, G4, G1], ids=lambda w: w.name)
@pytest.mark.parametrize("batch", [12, 3])
def test_slices(w, kw, tol, batch):
    print(f"\ncase {w.name} batch={batch} {kw}", flush=True)
    gu, gd, s = host_inputs(w, 14)
    g_in = kw.get("g_in", 0)
    got, _ = run_slice(config_for(w, batch=batch, **kw), to_dev(gu, g_in), to_dev(gd, g_in), s)
    check(got, want_of(w, 14), tol)


@pytest.mark.parametrize("count", [2, 14])
def test_no_alloc(count):
    """One call of few measurements keeps whole tiles, one of many does not."""
    import torch
    g4 = g4mod()
    w = G8
    print(f"\ncase into count={count}", flush=True)
    gu, gd, s = host_inputs(w, count)
    cfg = config_for(w, mode=1, batch=14)
    slots = (w.channels | (w.channels >> 3) | (w.channels >> 6)) & 7
    accs = [torch.zeros((w.planes, w.n, w.n), dtype=torch.complex128, device="cuda") if slots & (1 << c) else None
            for c in range(3)]
    g4.g4_accumulate_into(cfg, *accs, to_dev(gu, 0), to_dev(gd, 0), s)
    nc = w.lx * w.ly
    want = want_of(w, count)
    for c, ch in ((0, ref.PP_SINGLET), (1, ref.PP_TRIPLET)):
        if accs[c] is not None:
            a = accs[c].cpu().numpy().reshape(w.planes, nc, nc, w.nw, w.nw).transpose(0, 1, 3, 2, 4).reshape(w.planes, w.n, w.n)
            check_entries(a, want[ch], 1e-12, what="channel %d" % ch)
