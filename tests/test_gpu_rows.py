"""Rows of a last pass whose natural neighbours come round after fewer rows than
a tile holds, against the FP64 oracle.  Tolerance: 8 u per radix-2 level (u =
2^-24: sums, products of twiddle powers and table rounding), 16 u for the
four-step twiddle and the turn."""
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
