"""Mixed-radix passes (pencils with factors other than two, and short ones)
against the FP64 oracle, at the sizes where they can go wrong: every register
radix alone, digits of several stages, pencils of several digits, primes past
the registers, tiles that end inside a signal or span several, both thread
orders and every layout.

Tolerance: a radix-R butterfly sums R products, so it adds at most (R + 6) u
to the relative 2-norm error (u = 2^-24; the products, the table's rounding
and up to four products of twiddle powers), and the stages add up."""
import numpy as np
import pytest

from oracle import dft, lattice as L
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = 2.0 ** -24

CASES = (
    # one register radix (the load and the store share the stage), primes with
    # a pass over LDS on both sides, and one past the registers
    [("radix_%d" % r, ((r,),), 3, (r,)) for r in list(range(2, 17)) + [17, 19, 23, 29, 31, 37]]
    + [
        ("one_signal_two_stages", ((143,),), 1, (13, 11)),
        ("three_stages", ((15 * 14 * 13,),), 2, (15, 14, 13)),
        ("prime_between", ((8 * 31 * 9,),), 2, (9, 31, 8)),
        ("two_large_primes", ((29 * 31,),), 2, (29, 31)),
        # several digits in one pencil
        ("two_axes_small", ((6, 0), (0, 12)), 5, (6, 12)),
        ("three_axes", ((3, 0, 0), (0, 15, 0), (0, 0, 30)), 4, (3, 15, 6, 5)),
        ("prime_sum_in_axes", ((2, 0), (0, 2 * 41)), 3, (2, 2, 41)),
        # many signals per tile, the last tile ragged
        ("tiny_signals", ((5, 2), (0, 3)), 1001, (15,)),
        # the largest pencils of one tile
        ("pencil_8190", ((8190,),), 2, (15, 14, 13, 3)),
        ("pencil_8191_prime_sum", ((2, 0), (0, 2 * 2039)), 1, (2, 2, 2039)),
        # several passes: columns and rows, four-step twiddle, three axes
        ("two_pass_diagonal", ((90, 0), (0, 900)), 3, (15, 6, 10, 10, 9)),
        ("two_pass_sheared", ((90, 7), (0, 1001)), 2, (13, 11, 10, 9, 7)),
        ("cycle_of_100000", ((100000,),), 1, (16, 10, 10, 10, 10)),
        ("cycle_17x31x36", ((17 * 31 * 36,),), 3, (17, 31, 6, 6)),
        ("three_passes", ((50, 0, 0), (0, 150, 0), (0, 0, 300)), 1, (10, 5, 15, 10, 15, 10, 2)),
        ("four_dimensions", ((6, 1, 0, 0), (0, 6, 1, 0), (0, 0, 12, 0), (0, 0, 0, 24)), 2,
         (12, 12, 16, 9)),
        ("negative_lower", ((-45, 0), (31, 77)), 2, (11, 9, 7, 5)),
    ])


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _oracle(M, x, inverse):
    m = abs(L.det(M))
    f = dft.lattice_dft_direct if m <= 1024 else dft.lattice_dft_hnf
    return f(M, x.astype(np.complex128), inverse=inverse)


@pytest.mark.parametrize("name,M,batch,radices", CASES, ids=[c[0] for c in CASES])
def test_against_oracle(name, M, batch, radices):
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", name, "m", m, "batch", batch, flush=True)
    tol = U * (8 + sum(r + 6 for r in radices))
    x = workloads.complex_normal(91, (batch, m))
    plan = lfft.LatticePlan(M, batch=batch)
    xd = torch.from_numpy(x).cuda()
    X = plan.forward(xd)
    Y = plan.inverse(xd)
    some = slice(None) if batch < 100 else slice(batch - 20, batch)
    assert _rel(X.cpu().numpy()[some], _oracle(M, x[some], False)) < tol
    assert _rel(Y.cpu().numpy()[some], _oracle(M, x[some], True)) < tol
    # grid order: the same values, only placed differently
    s, f = plan.index_map(lfft.LFFT_MAP_SAMPLES), plan.index_map(lfft.LFFT_MAP_FREQS)
    xg = torch.empty_like(xd)
    xg[:, torch.from_numpy(s).cuda()] = xd
    both = plan.forward(xg, layout=lfft.LFFT_IN_GRID | lfft.LFFT_OUT_GRID)
    assert _rel(both[:, torch.from_numpy(f).cuda()].cpu().numpy(), X.cpu().numpy()) < 2 * tol
    back = plan.inverse(both, layout=lfft.LFFT_IN_GRID | lfft.LFFT_OUT_GRID)
    assert _rel(back.cpu().numpy(), xg.cpu().numpy()) < 2 * tol
