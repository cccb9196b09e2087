"""Plain FP64 calls of more measurements than one gather (a slice) or one launch
(g4_accumulate_into) takes: the groups' edges, and a slice whose readback scratch
holds no direct vectors (2 x nslots above N).

Bar 1e-12 relative against the oracle (FP64 sums of up to 300 terms: 300 * 2^-53
per entry); the two entry points apply the same operations in the same order, so
they agree bit for bit."""
import numpy as np
import pytest

from gpu_common import config_for, g4mod, host_inputs, run_slice, to_dev
from oracle import ref
from synth import Workload

pytestmark = pytest.mark.gpu

CASES = [   # workload, measurements
    (Workload("gather groups of 32", lx=2, ly=2, nw=16, nwex=1, nq=1, channels=1), 70),
    (Workload("weights by the 256", lx=1, ly=1, nw=4, nwex=2, nq=1, channels=4), 300),
    (Workload("no room in the scratch", lx=1, ly=1, nw=2, nwex=3, nq=1, channels=3), 9),
    (Workload("three channels, odd", lx=3, ly=1, nw=6, nwex=5, nq=2, q_begin=3, q_end=9, channels=7), 33),
]


@pytest.mark.parametrize("w,count", CASES, ids=lambda v: getattr(v, "name", str(v)))
def test_plain_groups(w, count):
    import torch
    print(f"\ncase {w.name} count={count}", flush=True)
    g4 = g4mod()
    gu, gd, s = host_inputs(w, count)
    s = s * np.linspace(0.5, 1.5, count)
    du, dd = to_dev(gu, 0), to_dev(gd, 0)
    out, st = run_slice(config_for(w), du, dd, s)
    assert st["launches"] == count and st["measurements"] == count
    place = {1: 0, 2: 1, 4: 2}
    accs = [None] * 3
    for ch in out:
        accs[place[ch]] = torch.zeros(w.entries, dtype=torch.complex128, device="cuda")
    g4.g4_accumulate_into(config_for(w), *accs, du, dd, s)
    for ch, got in out.items():
        want = ref.accumulate(w, ch, gu, gd, s)
        err = np.linalg.norm(got - want.reshape(got.shape)) / np.linalg.norm(want)
        assert err <= 1e-12, (ch, err)
        into = accs[place[ch]].cpu().numpy().reshape(w.planes, w.nc, w.nc, w.nw, w.nw)
        assert np.array_equal(into.transpose(0, 1, 3, 2, 4).reshape(got.shape), got), ch
