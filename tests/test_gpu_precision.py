"""How far results are from 64 bits, where an order of evaluation or a rounded
constant can add to the rounding that a transform of the length cannot do
without."""
import numpy as np
import pytest

from oracle import dft, lattice as L
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("M,batch", [
    (((128, 0), (64, 128)), 16),      # register-resident columns
    (((256, 0), (128, 256)), 4),      # streaming columns
    (((1024, 0), (256, 1024)), 1),
])
def test_order_of_loads_adds_no_rounding(M, batch):
    """A first pass over columns of natural input takes them in runs of natural
    neighbours.  That is a matter of order: the transform in grid order has the
    same stages (its passes the other way round), so the errors may differ by
    the scatter of the samples of roundings only (2^18 and more: 2%)."""
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", M, batch, flush=True)
    plan = lfft.LatticePlan(M, batch=batch)
    x = workloads.complex_normal(201, (batch, m))
    xd = torch.from_numpy(x).cuda()
    s = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_SAMPLES)).cuda()
    f = torch.from_numpy(plan.index_map(lfft.LFFT_MAP_FREQS)).cuda()
    xg = torch.empty_like(xd)
    xg[:, s] = xd
    want = dft.lattice_dft_hnf(M, x.astype(np.complex128))
    natural = plan.forward(xd).cpu().numpy()
    grid = plan.forward(xg, layout=lfft.LFFT_IN_GRID | lfft.LFFT_OUT_GRID)[:, f].cpu().numpy()
    assert _rel(natural, want) < 1.02 * _rel(grid, want)


@pytest.mark.parametrize("M,batch", [
    (((1000, 0), (0, 1000)), 1),
    (((100, 3, 0), (0, 100, 3), (0, 0, 100)), 1),
    (((2000,),), 50),
    (((4096,),), 64),
    (((2048, 0), (0, 512)), 1),
])
def test_length_of_the_output(M, batch):
    """The transform is unitary: the result may be off by roundings in every
    direction, but not longer or shorter by what rounding the output scale or
    the few constants of a butterfly adds up to (7e-8 on 64 x 4096 points and
    1.4e-7 on 10^6 with scale and constants in one float each).  What the
    twiddle tables leave is about 1e-8 a stage of short digits."""
    from paper_1107_5415_amd import lfft
    m = abs(L.det(M))
    print("case", M, batch, flush=True)
    plan = lfft.LatticePlan(M, batch=batch)
    x = workloads.complex_normal(202, (batch, m))
    xd = torch.from_numpy(x).cuda()
    for inverse, y in ((False, plan.forward(xd)), (True, plan.inverse(xd))):
        want = dft.lattice_dft_hnf(M, x.astype(np.complex128), inverse=inverse)
        gain = (np.vdot(want, y.cpu().numpy()) / np.vdot(want, want)).real
        assert abs(gain - 1) < 4e-8, (inverse, gain - 1)


# M, batch, error of the forward and the inverse transform (relative 2-norm, on
# the input of the test) with radices 2 .. 16 only, direct sums for every prime
# from 5 to 8191 and every twiddle from a table
FIGURES = [
    (((360,),), 300, 1.066e-7, 1.068e-7),
    (((900,),), 100, 1.210e-7, 1.206e-7),
    (((1260,),), 100, 1.201e-7, 1.199e-7),
    (((5040,),), 20, 1.302e-7, 1.299e-7),
    (((100, 0), (0, 100)), 8, 1.239e-7, 1.239e-7),
    (((16384,),), 64, 1.501e-7, 1.502e-7),
    (((65536,),), 16, 1.639e-7, 1.639e-7),
    (((1024, 256), (0, 1024)), 4, 1.874e-7, 1.874e-7),
    (((8209,),), 3, 2.626e-7, 2.645e-7),
    (((2, 0), (0, 2 * 8209)), 2, 2.297e-7, 2.284e-7),
    (((20, -196), (-367, 121)), 2, 2.701e-7, 2.695e-7),
    # a prime of 37 .. 61 in a longer digit: sums, and tight convolutions
    (((444,),), 100, 1.364e-7, 1.367e-7),
    (((188,),), 200, 1.399e-7, 1.399e-7),
    (((740,),), 60, 1.467e-7, 1.467e-7),
    (((2368,),), 50, 1.534e-7, 1.539e-7),
    (((1845,),), 50, 1.539e-7, 1.542e-7),
    (((3904,),), 30, 1.729e-7, 1.729e-7),
    (((37, 0), (0, 2368)), 1, 1.878e-7, 1.876e-7),
    (((6, 0), (0, 222)), 8, 1.521e-7, 1.521e-7),
]


@pytest.mark.parametrize("M,batch,forward,inverse", FIGURES, ids=[str(c[0]) for c in FIGURES])
def test_no_further_from_64_bits(M, batch, forward, inverse):
    """Larger radices, convolutions and twiddles from products are no less
    accurate than the plainest kernels, to the 2% by which two orders of
    evaluation differ on one sample."""
    from paper_1107_5415_amd import lfft
    print("case", M, batch, flush=True)
    plan = lfft.LatticePlan(M, batch=batch)
    x = workloads.complex_normal(203, (batch, plan.m))
    xd = torch.from_numpy(x).cuda()
    z = x.astype(np.complex128)
    assert _rel(plan.forward(xd).cpu().numpy(), dft.lattice_dft_hnf(M, z)) < 1.02 * forward
    back = dft.lattice_dft_hnf(M, z, inverse=True)
    assert _rel(plan.inverse(xd).cpu().numpy(), back) < 1.02 * inverse
