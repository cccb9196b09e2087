"""Which update kernel a plan runs: the G4_LOG line names it, so that a test of
one kernel can hold it to that kernel, and the autotuner times each once."""
import re

import pytest

from gpu_common import config_for, g4mod, host_inputs, to_dev
from synth import Workload

pytestmark = pytest.mark.gpu

W = Workload("kernels", lx=2, ly=1, nw=16, nwex=8, nq=2, q_begin=1, q_end=12)
MANY = Workload("kernels, 40 planes", lx=4, ly=1, nw=16, nwex=10, nq=4, q_begin=0, q_end=40)
F32 = dict(mode=1, prod=1, g_in=1, batch=4)


def kernels(capfd, monkeypatch, cfg, act=lambda h: None):
    """The kernels named by the plan lines of a slice's creation and of act()."""
    monkeypatch.setenv("G4_LOG", "1")
    g4 = g4mod()
    capfd.readouterr()
    h = g4.g4_init_slice(cfg)
    try:
        act(h)
    finally:
        g4.g4_destroy(h)
    lines = [ln for ln in capfd.readouterr().err.splitlines() if ln.startswith("g4: ")]
    return [re.search(r"kernel ([a-z-]+),", ln).group(1) for ln in lines]


@pytest.mark.parametrize("w,kw,want", [
    (W, dict(mode=1, batch=4), "streamed"), (W, dict(F32, batch=8), "streamed"),
    (W.with_(channels=8), dict(F32, batch=8), "registers"), (W.with_(nwex=7, lx=3), dict(F32, batch=8), "streamed"),
    (W.with_(nwex=8, lx=3), dict(F32, batch=8), "registers"),                # odd Ng
    (W, dict(F32, flags=16), "streamed"), (MANY, dict(F32, flags=16), "packed"),
    (W.with_(channels=3), dict(F32, flags=16), "streamed"), (W.with_(channels=3, nw=64), dict(F32, flags=16), "streamed"),
    (W.with_(channels=3, q_end=3), dict(F32, flags=16), "streamed"), (W.with_(channels=7), dict(F32, flags=16), "packed"),
    (MANY.with_(q_end=31, channels=4), dict(F32, flags=16), "streamed"),
    (MANY.with_(nw=24, q_end=10), dict(F32, flags=16), "streamed"), (MANY.with_(nw=24, q_end=11), dict(F32, flags=16), "packed"),
    (MANY.with_(nw=64, q_end=31), dict(F32, flags=16), "streamed"),
    (MANY.with_(nw=64, q_end=20), dict(F32, batch=32, flags=16), "packed"),
    (MANY.with_(nw=24, nwex=4, q_end=16), dict(F32, flags=16), "streamed"),
    (MANY.with_(nw=24, lx=5, nq=5, channels=3, q_end=11), dict(F32, flags=16), "packed"),   # three groups
    (MANY.with_(nw=24, nwex=4, q_end=13), dict(F32, batch=32, flags=16), "packed"),
    (W, dict(F32, batch=64, flags=16), "packed"),                            # a long pass over little of G
    (W, dict(F32, flags=16 | 64), "packed"), (W, dict(F32, prod=2, flags=16), "packed"),
    (W, dict(F32, flags=32), "packed-deep"), (W.with_(nw=64), dict(F32, flags=8), "mfma-direct"),
    (W.with_(nw=64), dict(F32, flags=24), "packed-mfma-direct")])
def test_plan_line_names_the_kernel(capfd, monkeypatch, w, kw, want):
    print(f"\ncase {w} {kw}", flush=True)
    assert kernels(capfd, monkeypatch, config_for(w, **kw)) == [want]


G128 = Workload("nw 128", lx=2, ly=1, nw=128, nwex=8, nq=2, q_begin=0, q_end=8)


# Fewer blocks a CU than the register-staged kernel: two buffers of a batched pass at 128 frequencies (a launch of one
# measurement has one buffer), three channels there; plane groups that are mostly empty; 8 frequencies.
@pytest.mark.parametrize("w,kw,want", [
    (G128, dict(mode=0), "streamed"), (G128, dict(mode=1, batch=1), "streamed"), (G128, dict(mode=1, batch=4), "registers"),
    (G128.with_(channels=7), F32, "registers"), (G128.with_(channels=7), dict(F32, batch=1), "registers"),
    (G128.with_(channels=7, nw=64), F32, "streamed"), (G128.with_(nw=64, q_end=1), dict(mode=0), "streamed"),
    (G128.with_(nw=54, q_end=2), dict(mode=0), "registers"), (G128.with_(nw=54, q_end=8), dict(mode=0), "streamed"),
    (G128.with_(nw=54, q_end=8), dict(F32, batch=8), "streamed"), (G128.with_(nw=54, q_end=8), F32, "registers"),
    (G128.with_(nw=54, q_end=3), dict(F32, batch=8), "registers"), (G128.with_(nw=8), dict(mode=0), "registers")])
def test_default_plan_kernel(capfd, monkeypatch, w, kw, want):
    print(f"\ncase {w} {kw}", flush=True)
    assert kernels(capfd, monkeypatch, config_for(w, **kw)) == [want]


def test_autotuner_times_the_streamed_kernel_once(capfd, monkeypatch):
    """A packed plan that would stream is no candidate of its own: the tuner
    leaves a VALU plan, or one whose kernel is another."""
    monkeypatch.delenv("G4_AUTOTUNE_CACHE", raising=False)
    g4 = g4mod()
    gu, gd, s = host_inputs(W, 4)
    found = {}

    def tune(h):
        found.update(g4.g4_autotune(h, to_dev(gu, 1), to_dev(gd, 1), s, tol=1e-6))

    names = kernels(capfd, monkeypatch, config_for(W.with_(channels=1), **F32), tune)
    # one pass size (4); tiles of 1, 2 and 4 rows a thread: VALU (16 rows at most), deep packed of 1 and 2
    valu = sum(1 for e in (1, 2, 4) if e * 16 < 16 + 16)
    deep = sum(1 for e in (1, 2) if e * 32 < 16 + 32)
    assert found["candidates"] == valu + deep
    assert (names[-1], found["variant"]) in (("streamed", 0), ("registers", 0), ("packed-deep", 3))


def test_packed_buffer_comes_with_the_plan_that_packs(capfd, monkeypatch):
    """A streaming packed slice allocates its packed buffer when set_plan installs
    a plan that packs: another variant, or one whose passes or tiles pack."""
    import numpy as np
    from gpu_common import run_slice
    g4 = g4mod()
    w = MANY.with_(nw=24, q_end=10)
    gu, gd, s = host_inputs(w, 6)
    du, dd = to_dev(gu, 1), to_dev(gd, 1)
    cfg = config_for(w, **dict(F32, flags=g4.G4_F_PACKED))
    want, _ = run_slice(config_for(w, **dict(F32, flags=0)), du, dd, s)
    out = []

    def change(h):
        g4.g4_accumulate(h, du, dd, s)
        out.append(g4.g4_readback(h, 1))
        for batch, variant in ((4, g4.G4_VARIANT_PACKED_DEEP), (2, g4.G4_VARIANT_PACKED), (4, g4.G4_VARIANT_PACKED)):
            g4.g4_set_plan(h, 0, batch, variant)
            g4.g4_reset(h)
            g4.g4_accumulate(h, du, dd, s)
            out.append(g4.g4_readback(h, 1))

    # passes of two over these plane groups pack
    assert kernels(capfd, monkeypatch, cfg, change) == ["streamed", "packed-deep", "packed", "streamed"]
    for o in out:
        assert np.linalg.norm(o.reshape(want[1].shape) - want[1]) <= 1e-6 * np.linalg.norm(want[1])
