"""Lattices of 2^30 points and more (64-bit coordinates) whose cycles are no
powers of two: mixed-radix passes, and a long axis by chirp-z.

Exact bins of a sparse signal at sampled frequencies and samples (its unitary
DFT in closed form, phases reduced in integers).  Tolerance: 8 u per radix-2
level (u = 2^-24), twice that for the two transforms of a convolution of up to
8 m points, 32 u for four-step twiddles, chirps and their tables."""
import math

import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = 2.0 ** -24

# name, sides of the box (M is their diagonal), passes, tolerance
CASES = [
    ("cycle_5x2^28", (5 << 28,), 3, U * (8 * 31 + 32)),
    ("256_by_long_axis_of_prime_16411", (256, 256 * 16411), 2, U * (16 * 34 + 32)),
]


@pytest.mark.parametrize("name,sides,passes,tol", CASES, ids=[c[0] for c in CASES])
def test_sparse_signal(name, sides, passes, tol):
    from paper_1107_5415_amd import lfft
    m = math.prod(sides)
    assert m >= 1 << 30
    M = tuple(tuple(s if i == j else 0 for j in range(len(sides))) for i, s in enumerate(sides))
    print("case", name, m, flush=True)
    plan = lfft.LatticePlan(M)
    assert plan.query()["passes"] == passes
    rng = np.random.default_rng(207)
    k = rng.choice(m, 8, replace=False).astype(np.int64)
    h = np.concatenate([rng.integers(0, m, 4096), [0, 1, m - 1]]).astype(np.int64)
    a = workloads.complex_normal(208, 8)
    x = torch.zeros(m, dtype=torch.complex64, device="cuda")
    x[torch.from_numpy(k).cuda()] = torch.from_numpy(a).cuda()
    turns = np.zeros((len(h), len(k)))
    kk, hh = k, h
    for s in reversed(sides):
        turns += ((hh[:, None] % s) * (kk[None, :] % s)) % s / s
        kk, hh = kk // s, hh // s
    for run, sign in ((plan.forward, -1), (plan.inverse, 1)):
        y = run(x)
        got = y[torch.from_numpy(h).cuda()].cpu().numpy().astype(np.complex128)
        del y
        want = (a.astype(np.complex128)[None, :] * np.exp(sign * 2j * np.pi * turns)).sum(1) / np.sqrt(m)
        assert np.linalg.norm(got - want) / np.linalg.norm(want) < tol
    del x, plan
    torch.cuda.empty_cache()
