"""Readbacks around the size from which several threads share the copy (4 Mi
entries): below it, at it, one above, a ragged last range, an odd first entry.
What g4_load put there comes back bit for bit (compensated accumulators: the
float sum and its remainder, so values of at most 24 bits are exact)."""
import numpy as np
import pytest

from gpu_common import config_for, g4mod
from synth import Workload

pytestmark = pytest.mark.gpu

W = Workload("large readback", lx=2, ly=1, nw=200, nwex=15, nq=2, channels=2)   # 4,800,000 entries
MI = 1 << 22


@pytest.mark.parametrize("acc", [0, 1, 2], ids=["c128", "kahan", "c64"])
def test_large_readback(acc):
    print(f"\ncase {W.entries} entries acc={acc}", flush=True)
    g4 = g4mod()
    rng = np.random.default_rng(acc)
    v = rng.normal(size=W.entries) + 1j * rng.normal(size=W.entries)
    if acc:
        v = v.astype(np.complex64).astype(np.complex128)
    h = g4.g4_init_slice(config_for(W, mode=1, prod=1, g_in=1, acc=acc, batch=2))
    try:
        g4.g4_load(h, 2, 0, v)
        for first, count in ((0, W.entries), (0, MI - 1), (5, MI), (77, MI + 1), (12345, W.entries - 12345), (3, 1)):
            assert np.array_equal(g4.g4_readback(h, 2, first, count), v[first:first + count]), (first, count)
    finally:
        g4.g4_destroy(h)
