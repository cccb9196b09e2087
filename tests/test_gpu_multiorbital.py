"""Parity of the multi-orbital G4 path (g4_accumulate_mo through the C ABI)
with the FP64 oracle.

Bars: FP64 products 1e-12, FP32 products 1e-6 (relative Frobenius, Eq. (2)/(3)
on real and imaginary parts, and the small half of the entries), per channel.
Shapes: one to nine orbitals (four: rows of 384 columns, a full and a partial
block each; six: rows of 864 columns; nine: the one-thread-per-entry
kernel), a transfer list in a
different order, a slice cut through a transfer momentum, entry counts that
are not multiples of the 256-thread block; 70 measurements (three launches of
at most 32).  Argument
errors are rejected before any launch.
"""
import numpy as np
import pytest

from gpu_common import g4mod
from metrics import check_entries
from oracle import ref
from synth import Workload

pytestmark = pytest.mark.gpu

W2 = Workload("mo-3x1", lx=3, ly=1, nw=4, nwex=3, nq=3, q_list=(2, 0, 1), q_begin=1, q_end=8, beta=6.0)
W3 = Workload("mo-2x2", lx=2, ly=2, nw=6, nwex=2, nq=4, q_begin=0, q_end=5, beta=5.0)


def inputs(w, nb, count, seed):
    rng = np.random.default_rng(seed)
    ngb = w.ng * nb
    g = lambda: (rng.normal(size=(count, ngb, ngb)) + 1j * rng.normal(size=(count, ngb, ngb))) * 0.3
    s = np.where(rng.random(count) < 0.9, 1.0, -1.0)
    return g(), g(), s


def run(w, nb, channels, prod, gu, gd, s):
    import torch
    g4 = g4mod()
    dt = torch.complex128 if prod == 0 else torch.complex64
    du = torch.from_numpy(gu).to(device="cuda", dtype=dt)
    dd = torch.from_numpy(gd).to(device="cuda", dtype=dt)
    side = w.n * nb * nb
    accs = [torch.zeros((w.planes, side, side), dtype=torch.complex128, device="cuda") if channels & (1 << c)
            else None for c in range(3)]
    g4.g4_accumulate_mo(w.lx, w.ly, w.nw, w.nwex, nb, w.nq, w.q_list, w.q0, w.q1, channels, prod, du, dd, s, *accs)
    torch.cuda.synchronize()
    return {1 << c: a.cpu().numpy() for c, a in enumerate(accs) if a is not None}


@pytest.mark.parametrize("prod", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("w,nb,count", [(W2, 2, 5), (W3, 3, 3), (W2, 1, 70), (W3, 4, 3), (W2, 5, 2), (W3, 6, 2),
                                         (W2, 7, 2), (W2, 8, 2), (W2, 9, 1)],
                         ids=["3x1-nb2", "2x2-nb3", "3x1-nb1-70meas", "2x2-nb4", "3x1-nb5", "2x2-nb6",
                              "3x1-nb7", "3x1-nb8", "3x1-nb9-entry-kernel"])
def test_matches_oracle(w, nb, count, prod):
    print("\ncase %s nb=%d count=%d prod=%d" % (w.name, nb, count, prod), flush=True)
    gu, gd, s = inputs(w, nb, count, 10 * nb + count)
    if prod == 1:
        gu = gu.astype(np.complex64).astype(np.complex128)
        gd = gd.astype(np.complex64).astype(np.complex128)
    got = run(w, nb, 7, prod, gu, gd, s)
    tol = 1e-12 if prod == 0 else 1e-6
    for ch in (1, 2, 4):
        want = ref.accumulate_mo(w, nb, ch, gu, gd, s)
        check_entries(got[ch], want, tol, what="channel %d" % ch)


def test_channel_subset_and_accumulation():
    """One channel, two calls: the second adds to the first."""
    w, nb = W3, 2
    gu, gd, s = inputs(w, nb, 4, 3)
    import torch
    g4 = g4mod()
    du = torch.from_numpy(gu).cuda()
    dd = torch.from_numpy(gd).cuda()
    side = w.n * nb * nb
    acc = torch.zeros((w.planes, side, side), dtype=torch.complex128, device="cuda")
    g4.g4_accumulate_mo(w.lx, w.ly, w.nw, w.nwex, nb, w.nq, None, w.q0, w.q1, 4, 0, du[:2], dd[:2], s[:2],
                        None, None, acc)
    g4.g4_accumulate_mo(w.lx, w.ly, w.nw, w.nwex, nb, w.nq, None, w.q0, w.q1, 4, 0, du[2:], dd[2:], s[2:],
                        None, None, acc)
    torch.cuda.synchronize()
    check_entries(acc.cpu().numpy(), ref.accumulate_mo(w, nb, 4, gu, gd, s), 1e-12)


def test_argument_errors():
    import torch
    g4 = g4mod()
    w, nb = W2, 2
    gu, gd, s = inputs(w, nb, 1, 1)
    du = torch.from_numpy(gu).cuda()
    dd = torch.from_numpy(gd).cuda()
    side = w.n * nb * nb
    acc = torch.zeros((w.planes, side, side), dtype=torch.complex128, device="cuda")
    bad = [dict(channels=8), dict(channels=3), dict(prod=2), dict(nb=0), dict(q_end=100)]
    for kw in bad:
        a = dict(channels=1, prod=0, nb=nb, q_end=w.q1)
        a.update(kw)
        with pytest.raises(g4.G4Error) as e:
            g4.g4_accumulate_mo(w.lx, w.ly, w.nw, w.nwex, a["nb"], w.nq, w.q_list, w.q0, a["q_end"], a["channels"],
                                a["prod"], du, dd, s, acc if a["nb"] == nb else 0)
        assert e.value.code == g4.G4_E_ARG, kw
    torch.cuda.synchronize()
    assert float(acc.abs().max()) == 0.0


# The matrix-instruction kernel (four orbitals, FP32): squares of 32 K cut short, K counts that are not multiples of four,
# odd plane counts and one plane, batches around its steps of 4, sums of 32 and launches of 128.
@pytest.mark.parametrize("lx,ly,nw,nwex,q0,q1,count", [(1, 1, 2, 1, 0, 1, 1), (3, 1, 2, 3, 1, 6, 3), (2, 1, 18, 2, 0, 3, 5),
                                                       (1, 1, 34, 1, 0, 1, 32), (2, 1, 6, 3, 1, 5, 35), (1, 1, 4, 2, 0, 2, 131)])
def test_four_orbital_matrix_kernel(lx, ly, nw, nwex, q0, q1, count):
    import torch
    g4 = g4mod()
    nb, nq = 4, lx * ly
    w = Workload("mo4", lx=lx, ly=ly, nw=nw, nwex=nwex, nq=nq, q_begin=q0, q_end=q1)
    print(f"\ncase mo4 {lx}x{ly} nw={nw} nwex={nwex} planes [{q0}, {q1}) count={count}", flush=True)
    rng = np.random.default_rng(100 * nw + count)
    ngb, side = w.ng * nb, w.n * nb * nb
    gu, gd = (((rng.normal(size=(count, ngb, ngb)) + 1j * rng.normal(size=(count, ngb, ngb))) * 0.3).astype(np.complex64)
              for _ in range(2))
    s = np.where(rng.random(count) < 0.8, 1.0, -0.75)
    du, dd = torch.from_numpy(gu).cuda(), torch.from_numpy(gd).cuda()
    acc = [torch.full((q1 - q0, side, side), 0.5 + 0.25j, dtype=torch.complex128, device="cuda") for _ in range(3)]
    g4.g4_accumulate_mo(lx, ly, nw, nwex, nb, nq, None, q0, q1, 7, g4.G4_PROD_F32, du, dd, s, *acc)
    idx = rng.integers(0, (q1 - q0) * side * side, size=400)
    for c, a in enumerate(acc):
        got = a.cpu().numpy().reshape(-1)[idx] - (0.5 + 0.25j)
        want = ref.entries_mo(w, nb, 1 << c, gu.astype(np.complex128), gd.astype(np.complex128), s, idx)
        # the FP32 bar of the other multi-orbital cases
        assert np.linalg.norm(got - want) <= 1e-6 * np.linalg.norm(want), c


# Sizes at which calls of few measurements run the matrix kernel, and either side of them: single planes, blocks beyond
# 128 with K and planes that do not fill their fours and pairs, three and four measurements, 40 and 41.
@pytest.mark.parametrize("lx,ly,nw,nwex,q0,q1,count", [(2, 1, 10, 2, 1, 2, 4), (2, 1, 10, 2, 1, 2, 3), (3, 1, 6, 3, 2, 3, 9),
                                                       (3, 1, 14, 3, 1, 4, 5), (3, 1, 14, 3, 0, 3, 3), (3, 1, 14, 1, 0, 2, 6),
                                                       (1, 1, 6, 4, 0, 3, 40), (1, 1, 6, 4, 0, 3, 41)])
def test_four_orbital_kernel_choice(lx, ly, nw, nwex, q0, q1, count):
    test_four_orbital_matrix_kernel(lx, ly, nw, nwex, q0, q1, count)


# The two-orbital PH kernel: each channel set, batches around its launches (32 in FP32, 128 in FP64), an accumulator that
# is not zero, columns that do not fill a block.
@pytest.mark.parametrize("channels", [1, 2, 3, 7])
@pytest.mark.parametrize("prod,count", [(0, 1), (0, 130), (1, 2), (1, 33)])
def test_two_orbital_kernel(channels, prod, count):
    import torch
    w, nb = W2.with_(nw=6, q_list=None), 2
    print(f"\ncase mo2 channels={channels} prod={prod} count={count}", flush=True)
    gu, gd, s = inputs(w, nb, count, 7 * count + channels)
    if prod == 1:
        gu, gd = (g.astype(np.complex64).astype(np.complex128) for g in (gu, gd))
    got = run(w, nb, channels, prod, gu, gd, s)
    for ch in got:
        check_entries(got[ch], ref.accumulate_mo(w, nb, ch, gu, gd, s), 1e-12 if prod == 0 else 1e-6, what="channel %d" % ch)


# Small slices of two orbitals, either side of the lines at which their PH channels share launches (n 42, 284 rows'
# blocks, 12 and 40 measurements): both channels in one call give what a call each gives, and the oracle's entries.
@pytest.mark.parametrize("lx,nw,planes,prod,count", [(3, 14, 1, 1, 13), (3, 14, 1, 1, 12), (2, 22, 1, 1, 13), (2, 6, 6, 1, 33),
                                                     (2, 20, 8, 1, 14), (2, 20, 7, 1, 14), (2, 6, 4, 0, 40), (2, 6, 4, 0, 41)])
def test_two_orbital_channels_together_and_alone(lx, nw, planes, prod, count):
    import torch
    g4 = g4mod()
    nb = 2
    w = Workload("mo2-both", lx=lx, ly=1, nw=nw, nwex=4, nq=2, q_begin=0, q_end=planes)
    print(f"\ncase mo2 both lx={lx} nw={nw} planes={planes} prod={prod} count={count}", flush=True)
    gu, gd, s = inputs(w, nb, count, 11 * count + planes)
    dtype = np.complex64 if prod else np.complex128
    du, dd = (torch.from_numpy(g.astype(dtype)).cuda() for g in (gu, gd))
    side = w.n * nb * nb

    def call(channels):
        acc = [torch.zeros((planes, side, side), dtype=torch.complex128, device="cuda") if channels >> c & 1 else None
               for c in range(2)]
        g4.g4_accumulate_mo(lx, 1, nw, 4, nb, 2, None, 0, planes, channels, prod, du, dd, s, *acc)
        return acc

    both, alone = call(3), [call(1)[0], call(2)[1]]
    idx = np.random.default_rng(1).integers(0, planes * side * side, size=200)
    gu, gd = (g.astype(dtype).astype(np.complex128) for g in (gu, gd))
    for c in range(2):
        want = ref.entries_mo(w, nb, 1 << c, gu, gd, s, idx)
        for got in (both[c], alone[c]):
            got = got.cpu().numpy().reshape(-1)[idx]
            assert np.linalg.norm(got - want) <= (1e-6 if prod else 1e-12) * np.linalg.norm(want), c


# The parts of a long launch (sums of 32 measurements in FP32) join in more than FP32: a call gives what calls of 32
# give, whose sums meet in the complex128 accumulator.  Each of up to three additions rounds away at most 2^-24 of the
# sum, kept to 2^-24 of itself: 5 * 2^-48 in all, 2^-53 a call on the other side; the bar is 2^-44 of the largest sum.
# The sizes are those where calls of 32 and fewer run the matrix kernel too.
@pytest.mark.parametrize("planes,count", [(5, 133), (1, 128), (6, 64), (5, 37)])
def test_four_orbital_parts_keep_their_width(planes, count):
    import torch
    g4 = g4mod()
    nb, nw = 4, 16
    w = Workload("mo4-parts", lx=2, ly=1, nw=nw, nwex=3, nq=2, q_begin=0, q_end=planes)
    print(f"\ncase mo4 parts planes={planes} count={count}", flush=True)
    rng = np.random.default_rng(7 + count)
    ngb, side = w.ng * nb, w.n * nb * nb
    mean = [rng.normal(size=(1, ngb, ngb)) + 1j * rng.normal(size=(1, ngb, ngb)) for _ in range(2)]
    du, dd = (torch.from_numpy((m + 0.05 * rng.normal(size=(count, ngb, ngb))).astype(np.complex64)).cuda() for m in mean)
    s = np.ones(count)

    def call(acc, lo, hi):
        g4.g4_accumulate_mo(2, 1, nw, 3, nb, 2, None, 0, planes, 7, g4.G4_PROD_F32, du[lo:hi], dd[lo:hi], s[lo:hi], *acc)

    zeros = lambda: [torch.zeros((planes, side, side), dtype=torch.complex128, device="cuda") for _ in range(3)]  # noqa: E731
    whole, parts, largest = zeros(), zeros(), [0.0] * 3
    call(whole, 0, count)
    for lo in range(0, count, 32):
        call(parts, lo, min(lo + 32, count))
        largest = [max(m, float(torch.view_as_real(a).abs().max())) for m, a in zip(largest, parts)]
    for c in range(3):
        assert float(torch.view_as_real(whole[c] - parts[c]).abs().max()) <= 2.0 ** -44 * largest[c], c
