"""Passes that order their rows or columns by natural neighbours, at the sizes
where that order can go wrong: runs that fill a tile or leave a remainder,
steps in either direction, turns that wrap, several signals, the four-step
axis on either side, three axes with a pass each, and the batched launch.

The natural transform is compared with the FP64 oracle and with the same plan
in grid order, which uses none of it.  Tolerance: a power-of-two FFT of m
points adds at most 8 u per radix-2 level to the relative 2-norm error (u =
2^-24: sums, products of twiddle powers and table rounding); the turn and the
four-step twiddle add 8 u each."""
import math
import os
import subprocess
import sys

import numpy as np
import pytest

from oracle import dft, lattice as L
import workloads

torch = pytest.importorskip("torch")

U = 2.0 ** -24
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# name, M, batch, what the plan log says of (forward, inverse)
CASES = [
    ("rows_four_step", ((64, 3), (0, 256)), 3, ("stores", "stores")),
    ("rows_step_of_one", ((1, 0), (0, 16384)), 1, ("stores", "stores")),
    ("rows_with_leading_axis", ((64, 8), (0, 1024)), 2, ("stores", "stores")),
    ("rows_four_of_2048", ((512, 77), (0, 512)), 1, ("stores", "stores")),
    ("columns_step_2", ((256, 128), (0, 256)), 3, ("stores", "loads")),
    ("columns_step_back", ((256, 192), (0, 256)), 1, ("stores", "loads")),
    ("columns_input_first", ((256, 0), (128, 256)), 2, ("loads", "stores")),
    ("columns_register_kernel", ((128, 64), (0, 128)), 5, ("stores", "loads")),
    ("columns_four_step_input", ((2, 1), (0, 8192)), 1, ("stores", "loads")),
    ("three_axes_a_pass_each", ((64, 16, 0), (0, 64, 16), (0, 0, 64)), 1, None),
    ("three_axes_long", ((256, 64, 0), (0, 256, 64), (0, 0, 64)), 1, None),
    ("streaming_columns_2^20", ((1024, 256), (0, 1024)), 2, ("stores", "loads")),
    ("full_tiles_of_spread_lines", ((2048, 16), (0, 2048)), 1, None),
    ("rows_8192_after_short_axis", ((4096, 32), (0, 2048)), 1, None),
]
# M, what the plan log says of the first pass (forward, inverse) and the last
TILES = [
    (((2048, 16), (0, 2048)), "pencil 1024 x 8 ", "pencil 1024 x 16 ", "pencil 4096 x 4 "),
    (((2048, 2), (0, 2048)), "pencil 1024 x 8 ", "pencil 1024 x 8 ", "pencil 4096 x 4 "),
    (((4096, 32), (0, 2048)), "pencil 1024 x 8 ", "pencil 1024 x 16 ", "pencil 8192 x 2 "),
    (((1024, 16), (0, 2048)), "pencil 1024 x 8 ", "pencil 1024 x 8 ", "pencil 2048 x 4 "),
]
LOGGED = [c for c in CASES if c[3]]


@pytest.mark.parametrize("name,M,batch,log", LOGGED, ids=[c[0] for c in LOGGED])
def test_rule_applies(name, M, batch, log):
    """(CPU) The plan takes the order on the sides it is meant for."""
    code = ("import sys; sys.path.insert(0, %r); from paper_1107_5415_amd import lfft; "
            "lfft.LatticePlan(%r, batch=%d, host_only=True)" % (ROOT, M, batch))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True,
                       env=dict(os.environ, LFFT_LOG="1"))
    assert r.returncode == 0, r.stderr
    for side, want in zip(("forward", "inverse"), log):
        lines = [l for l in r.stderr.splitlines() if "  " + side in l]
        assert lines and any(want + " in natural runs" in l for l in lines), r.stderr


@pytest.mark.parametrize("M,fwd,inv,last", TILES)
def test_tiles_of_a_short_axis_and_a_long_one(M, fwd, inv, last):
    """(CPU) Tile width of the first pass and rows of the last."""
    code = ("import sys; sys.path.insert(0, %r); from paper_1107_5415_amd import lfft; "
            "lfft.LatticePlan(%r, host_only=True)" % (ROOT, M))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True,
                       env=dict(os.environ, LFFT_LOG="1"))
    assert r.returncode == 0, r.stderr
    for side, want in (("forward", fwd), ("inverse", inv)):
        lines = [l for l in r.stderr.splitlines() if "  " + side in l]
        assert want in lines[0] and last in lines[1], r.stderr


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _tol(m):
    return U * (8 * math.log2(m) + 32)


@pytest.mark.gpu
@pytest.mark.parametrize("name,M,batch,log", CASES, ids=[c[0] for c in CASES])
def test_against_oracle_and_grid(name, M, batch, log):
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", name, "m", m, "batch", batch, flush=True)
    x = workloads.complex_normal(97, (batch, m))
    plan = lfft.LatticePlan(M, batch=batch)
    xd = torch.from_numpy(x).cuda()
    X, Y = plan.forward(xd), plan.inverse(xd)
    z = x.astype(np.complex128)
    assert _rel(X.cpu().numpy(), dft.lattice_dft_hnf(M, z)) < _tol(m)
    assert _rel(Y.cpu().numpy(), dft.lattice_dft_hnf(M, z, inverse=True)) < _tol(m)
    s = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_SAMPLES)).cuda()
    f = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_FREQS)).cuda()
    xg = torch.empty_like(xd)
    xg[:, s] = xd
    both = plan.forward(xg, layout=lfft.LFFT_IN_GRID | lfft.LFFT_OUT_GRID)
    assert _rel(both[:, f].cpu().numpy(), X.cpu().numpy()) < 2 * _tol(m)
    # one side in grid order at a time
    half = plan.forward(xg, layout=lfft.LFFT_IN_GRID)
    assert _rel(half.cpu().numpy(), X.cpu().numpy()) < 2 * _tol(m)
    half = plan.forward(xd, layout=lfft.LFFT_OUT_GRID)
    assert _rel(half[:, f].cpu().numpy(), X.cpu().numpy()) < 2 * _tol(m)


@pytest.mark.gpu
@pytest.mark.parametrize("tile_lg", [11, 12, 13])
def test_batched(tile_lg):
    """The same lattices in one batched launch, whose tiles have other widths."""
    from paper_1107_5415_amd import lfft
    Ms = [c[1] for c in CASES if len(c[1]) == 2]
    plan = lfft.BatchPlan(Ms)
    plan.configure(tile_lg)
    x = workloads.complex_normal(98, plan.total)
    xd = torch.from_numpy(x).cuda()
    for inverse in (False, True):
        y = plan.execute(xd, inverse=inverse, mode=lfft.LFFT_BATCH_PERSISTENT).cpu().numpy()
        for i, M in enumerate(Ms):
            a, b = plan.offsets[i], plan.offsets[i + 1]
            ref = dft.lattice_dft_hnf(M, x[None, a:b].astype(np.complex128), inverse=inverse)[0]
            assert _rel(y[a:b], ref) < _tol(b - a), (M, inverse)
