"""The update kernel that streams its operands from G: FP32 columns in pairs, so
odd and even first columns, row counts of a tile that are odd, one row, a last
tile shorter than the others; plane groups cut to odd lengths; every channel
set; the sizes compiled in (nw = 64) and not; the plans it serves (default,
packed with few planes) and the one it leaves to the older kernel (odd Ng).

Bars: FP64 1e-12, FP32 products 1e-6 relative to the oracle, as elsewhere."""
import numpy as np
import pytest

from gpu_common import config_for, g4mod, host_inputs, run_slice, to_dev
from oracle import ref
from synth import Workload

pytestmark = pytest.mark.gpu

CASES = [
    # nw = 36: 7 rows per sweep, the last tile has one row; groups of 3, 8 and 4 planes
    Workload("36 rows, cut groups", lx=2, ly=1, nw=36, nwex=8, nq=2, q_begin=5, q_end=12),
    Workload("50 rows, nwex 3", lx=2, ly=2, nw=50, nwex=3, nq=4, q_begin=1, q_end=11),
    Workload("nw 64, odd first columns", lx=3, ly=2, nw=64, nwex=8, nq=2, q_begin=3, q_end=14),
    Workload("nw 128, nwex 4", lx=2, ly=1, nw=128, nwex=4, nq=2, q_begin=1, q_end=4),
    Workload("nw 256, one row per sweep", lx=1, ly=1, nw=256, nwex=6, nq=1, q_begin=2, q_end=5),
    Workload("nw 10, nwex 12", lx=4, ly=1, nw=10, nwex=12, nq=3, q_begin=7, q_end=30),
    Workload("odd Ng", lx=3, ly=1, nw=12, nwex=4, nq=3, q_begin=0, q_end=12),
]


@pytest.mark.parametrize("channels", [1, 2, 4, 3, 5, 7])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_streamed_update(w, channels):
    w = w.with_(channels=channels)
    print(f"\ncase {w.name} channels={channels}", flush=True)
    g4 = g4mod()
    count = 5
    gu, gd, s = host_inputs(w, count)
    s = s * np.array([1.0, 0.5, 1.0, 2.0, 1.0])
    ru, rd = (x.astype(np.complex64).astype(np.complex128) for x in (gu, gd))
    plans = [("f64", dict(mode=1, batch=3), 0, 1e-12), ("f32", dict(mode=1, prod=1, g_in=1, batch=4), 1, 1e-6)]
    plans += [("f32 tile x2", dict(mode=1, prod=1, g_in=1, acc=1, batch=2, tile=2 * (256 // w.nw)), 1, 1e-6),
              ("packed", dict(mode=1, prod=1, g_in=1, batch=3, flags=g4.G4_F_PACKED), 1, 1e-6)]
    for name, kw, g_in, bar in plans:
        try:
            cfg = config_for(w, **kw)
            g4.g4_slice_size(cfg)
        except g4.G4Error:
            continue                                 # this plan does not run this shape
        a, b = (gu, gd) if g_in == 0 else (ru, rd)
        out, _ = run_slice(cfg, to_dev(a, g_in), to_dev(b, g_in), s)
        for ch, got in out.items():
            want = ref.accumulate(w, ch, a, b, s).reshape(got.shape)
            err = np.linalg.norm(got - want) / np.linalg.norm(want)
            assert err <= bar, (name, ch, err)
