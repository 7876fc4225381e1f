"""Rows of a last pass whose natural neighbours come round after fewer rows than
a tile holds, and grid layouts with tiles or a tile order of their own.

Natural results are compared with the FP64 oracle, grid layouts with the
natural transform of the same plan, which shares neither.  Tolerance: 8 u per
radix-2 level (u = 2^-24: sums, products of twiddle powers and table rounding),
16 u for the four-step twiddle and the turn; both sides of the second
comparison may be that far off."""
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

# cycles of 2 rows in tiles of 4 and 8, of 4 in tiles of 8; one and more signals
SHORT = [
    (((512, 2), (0, 512)), 1),
    (((128, 2), (0, 128)), 3),
    (((128, 4), (0, 128)), 2),
    (((64, 2), (0, 512)), 5),
]
# first passes in tiles of 16 columns from natural order, of 8 from grid order
# and columns before a four-step axis in 32 groups of 16 tiles
GRID = [((2048, 8), (0, 4096)), ((4096, 32), (0, 2048)), ((2048, 512), (0, 4096))]


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _tol(m):
    return U * (8 * math.log2(m) + 16)


@pytest.mark.parametrize("M,batch", SHORT)
def test_short_cycles_share_a_tile(M, batch):
    """(CPU) The rows of short cycles are written in runs, too."""
    code = ("import sys; sys.path.insert(0, %r); from paper_1107_5415_amd import lfft; "
            "lfft.LatticePlan(%r, batch=%d, host_only=True)" % (ROOT, M, batch))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True,
                       env=dict(os.environ, LFFT_LOG="1"))
    assert r.returncode == 0, r.stderr
    last = [l for l in r.stderr.splitlines() if " pass 2/2 " in l]
    assert len(last) == 2 and all("stores in natural runs" in l for l in last), r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("M,batch", SHORT)
def test_short_cycles_against_oracle(M, batch):
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", M, batch, flush=True)
    x = workloads.complex_normal(205, (batch, m))
    plan = lfft.LatticePlan(M, batch=batch)
    xd = torch.from_numpy(x).cuda()
    z = x.astype(np.complex128)
    assert _rel(plan.forward(xd).cpu().numpy(), dft.lattice_dft_hnf(M, z)) < _tol(m)
    back = dft.lattice_dft_hnf(M, z, inverse=True)
    assert _rel(plan.inverse(xd).cpu().numpy(), back) < _tol(m)


@pytest.mark.gpu
@pytest.mark.parametrize("M", GRID)
def test_grid_layouts(M):
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", M, flush=True)
    plan = lfft.LatticePlan(M)
    g = torch.Generator(device="cuda").manual_seed(206)
    x = torch.randn(m, dtype=torch.complex64, device="cuda", generator=g)
    s = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_SAMPLES)).cuda()
    f = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_FREQS)).cuda()

    def near(a, b):
        d = torch.linalg.vector_norm((a - b).to(torch.complex128))
        return (d / torch.linalg.vector_norm(b.to(torch.complex128))).item() < 2 * _tol(m)

    for run, src, dst in ((plan.forward, s, f), (plan.inverse, f, s)):
        natural = run(x)
        xg = torch.empty_like(x)
        xg[src] = x
        assert near(run(xg, layout=lfft.LFFT_IN_GRID), natural)
        assert near(run(x, layout=lfft.LFFT_OUT_GRID)[dst], natural)
        assert near(run(xg, layout=lfft.LFFT_IN_GRID | lfft.LFFT_OUT_GRID)[dst], natural)
