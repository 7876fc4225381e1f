"""The performance cases of this framework.

A case is one call (or one pair of calls) that a user's program makes through
the public entry points: the lattice FFT in both directions, the wavelet
pyramid and its inverse, a differentiated pyramid step and the batched launch.
Sizes are those of the repository's workloads, parity tests and benchmark;
`draw` spreads more cases over the same ranges.

`exact` states what `run` computes in plain 64-bit torch operations: the
lattice DFT through the Hermite form of M (row and column FFTs with a twiddle
in between), the fiber split by index tables.  It shares no code with the
library.

The split-BF16 plan flag is left out: it is slower and less accurate than the
FP32 path, and kept for the matrix-core layout it shows.
"""
import math

import numpy as np
import torch

from paper_1107_5415_amd import autograd, lfft

QUINCUNX = "1,1;1,-1"
TWO_I = "2,0;0,2"
JX = "2,0;0,1"
DILATIONS = (QUINCUNX, JX, "1,0;0,2", "1,-1;1,1")


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


# ---------------------------------------------------------------------------
# Cases

def listed():
    return [
        # the smallest call: one signal of 1088 points (elementary divisors 8
        # and 136 = 8 x 17), where the host path and the launch are the time
        dict(name="fft_small", kind="fft", M="32,8;-8,32", batch=1, dir="forward"),
        # one decomposition and reconstruction of a 512 x 512 picture given by
        # its point values (the experiment of the paper's Section 6.2): few,
        # short kernels
        dict(name="pyramid_picture", kind="pyramid", M="512,0;0,512", J=JX, levels=1, batch=1,
             samples=True),
        # a row of the paper's timing table (Section 6.1) in the order whose
        # last pass scatters long pencils onto an unaligned side
        dict(name="fft_table_row", kind="fft", M="2048,8;0,2048", batch=1, dir="forward"),
        # odd cycles without large primes (105 = 3 5 7 and 1287 = 9 11 13),
        # several signals, from frequencies to samples
        dict(name="fft_odd", kind="fft", M="105,0;0,1287", batch=8, dir="inverse"),
        # matrices as they come: random integer entries give one cycle with a
        # large prime, here 2 x 23 x 1229 ...
        dict(name="fft_random_d3", kind="fft", M="45,-60,-17;51,7,11;-50,18,16", batch=2,
             dir="forward"),
        # ... and 8 x 8689, whose prime does not fit one on-chip pencil
        dict(name="fft_random_d2", kind="fft", M="20,-196;-367,121", batch=2, dir="both"),
        # the benchmark's lattice: a large signal transformed and back
        dict(name="fft_large", kind="fft", M="4096,2048;0,4096", batch=1, dir="both"),
        # the three-dimensional lattice of the same size
        dict(name="fft_d3", kind="fft", M="256,64,0;0,256,64;0,0,256", batch=1, dir="forward"),
        # many lattices of different M in one call, as a graph replay (512
        # matrices of 2^10 .. 2^18 points)
        dict(name="batch_512", kind="batch", count=512, mseed=4, dir="forward"),
        # the benchmark's eight-level pyramid and its inverse
        dict(name="pyramid_large", kind="pyramid", M="4096,2048;0,4096", J=QUINCUNX, levels=8,
             batch=1, samples=False),
        # four channels per level down to the same resolution
        dict(name="pyramid_four", kind="pyramid", M="4096,2048;0,4096", J=TWO_I, levels=4, batch=1,
             samples=False),
        # learning the masks: 16 signals through the pyramid and its inverse,
        # and the gradients of samples and masks back
        dict(name="train_masks", kind="train", M="1024,256;0,1024", J=QUINCUNX, levels=4, batch=16),
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], uniform over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _text(M):
    return ";".join(",".join(str(int(v)) for v in row) for row in M)


def _largest_prime(n):
    p, big = 2, 1
    while p * p <= n:
        while n % p == 0:
            big, n = p, n // p
        p += 1
    return max(big, n)


def _draw_fft(rng):
    direction = rng.choice(["forward", "inverse", "both"])
    family = rng.choice(["pow2", "pow2", "pow2_d3", "smooth", "smooth", "random", "random"])
    if family == "pow2":       # the paper's normal form [[2^a, c], [0, 2^b]]
        s = rng.randint(10, 24)
        a = rng.randint(0, s)
        m, M = 1 << s, [[1 << a, rng.randrange(1 << a)], [0, 1 << (s - a)]]
    elif family == "pow2_d3":  # sheared cubes
        e = [rng.randint(3, 8) for _ in range(3)]
        m = 1 << sum(e)
        M = [[1 << e[0], rng.randrange(1 << e[0]), 0], [0, 1 << e[1], rng.randrange(1 << e[1])],
             [0, 0, 1 << e[2]]]
    elif family == "smooth":   # boxes whose sides have the primes up to 17
        sides = []
        while len(sides) < 2:
            n = _log_int(rng, 24, 1500)
            if _largest_prime(n) <= 17:
                sides.append(n)
        m, M = sides[0] * sides[1], [[sides[0], rng.randrange(sides[0])], [0, sides[1]]]
    else:                      # random entries; the listed cases hold the largest prime
        while True:            # of an on-chip cycle, larger ones leave the pencil
            d = rng.choice([2, 3])
            r = 450 if d == 2 else 60
            M = [[rng.randint(-r, r) for _ in range(d)] for _ in range(d)]
            m = abs(_det(M))
            if 512 <= m <= 1 << 17 and not 1229 < _largest_prime(m) <= 8192:
                break
    batch = max(1, min(_log_int(rng, 1, 16), (1 << 24) // m))
    return dict(kind="fft", M=_text(M), batch=batch, dir=direction)


def _draw_pyramid(rng, train):
    four = rng.random() < 0.25
    J = TWO_I if four else rng.choice(DILATIONS)
    q = 4 if four else 2
    batch = rng.choice([1, 2, 4, 8, 16]) if train else rng.choice([1, 1, 1, 2, 4])
    top = (1 << 22) // batch if train else (1 << 23) // batch
    while True:
        levels = rng.randint(1, 4 if four or train else 8)
        sides = [rng.choice([1, 1, 3, 5]) << rng.randint(2, 10) for _ in range(2)]
        m = sides[0] * sides[1] * q ** levels
        if 1 << 12 <= m <= top:
            break
    M = [[sides[0], rng.randrange(sides[0])], [0, sides[1]]]
    for _ in range(levels):
        M = _mul(_matrix(J), M)
    case = dict(kind="train" if train else "pyramid", M=_text(M), J=J, levels=levels, batch=batch)
    if not train:
        case["samples"] = rng.random() < 0.3
    return case


def draw(rng):
    kind = rng.choice(["fft", "fft", "fft", "pyramid", "pyramid", "train", "batch"])
    if kind == "fft":
        return _draw_fft(rng)
    if kind == "batch":
        return dict(kind="batch", count=_log_int(rng, 32, 512), mseed=rng.randrange(5, 1 << 20),
                    dir=rng.choice(["forward", "inverse"]))
    return _draw_pyramid(rng, kind == "train")


# ---------------------------------------------------------------------------
# What the program has before the call, and the call

def _normal(case, seed, n, k=0):
    """n complex samples on the GPU, real and imaginary parts N(0, 1)."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(1000003 * (seed % (1 << 40)) + k)
    return torch.view_as_complex(torch.randn((n, 2), device=dev, generator=g))


def _batch_matrices(case):
    """[[2^a, c], [0, 2^b]] with a + b in 10 .. 18."""
    rng = np.random.default_rng(case["mseed"])
    out = []
    for _ in range(case["count"]):
        s = int(rng.integers(10, 19))
        a = int(rng.integers(0, s + 1))
        out.append([[1 << a, int(rng.integers(0, 1 << a))], [0, 1 << (s - a)]])
    return out


def _learned(masks, seed):
    """Masks some way into their training: the Dirichlet masks perturbed."""
    g = torch.Generator(device=masks[0].device).manual_seed(seed % (1 << 40) + 7)
    return [a + 0.1 * torch.randn(a.shape, device=a.device, generator=g) for a in masks]


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    if case["kind"] == "batch":
        return dict(x=_normal(case, seed, sum(abs(_det(M)) for M in _batch_matrices(case))))
    M, B = _matrix(case["M"]), case["batch"]
    m = abs(_det(M))
    t = dict(x=_normal(case, seed, B * m).reshape(B, m))
    if case["kind"] in ("pyramid", "train"):
        masks = [a.float() for a in _dirichlet_masks(M, _matrix(case["J"]), case["levels"])]
        t["masks"] = masks if case["kind"] == "pyramid" else _learned(masks, seed)
    if case["kind"] == "train":
        t["gc"] = _normal(case, seed, B * m, 1).reshape(B, m)
        t["gr"] = _normal(case, seed, B * m, 2).reshape(B, m)
    return t


def prepare(case, seed):
    st = _inputs(case, seed)
    kind = case["kind"]
    st["kind"] = kind
    if kind == "fft":
        st["plan"] = lfft.LatticePlan(_matrix(case["M"]), batch=case["batch"])
        st["dir"] = case["dir"]
    elif kind == "batch":
        st["plan"] = lfft.BatchPlan(_batch_matrices(case))
        st["out"] = torch.empty_like(st["x"])
        st["inverse"] = case["dir"] == "inverse"
    else:
        st["plan"] = lfft.WaveletPlan(_matrix(case["M"]), _matrix(case["J"]), case["levels"],
                                      batch=case["batch"], samples=case.get("samples", False))
        if kind == "train":
            st["leaves"] = [st["x"].requires_grad_(True)] + [a.requires_grad_(True)
                                                             for a in st["masks"]]
    return st


def run(st):
    plan, kind = st["plan"], st["kind"]
    if kind == "fft":
        if st["dir"] == "forward":
            return plan.forward(st["x"])
        if st["dir"] == "inverse":
            return plan.inverse(st["x"])
        X = plan.forward(st["x"])
        return [X, plan.inverse(X)]
    if kind == "batch":
        return plan.execute(st["x"], inverse=st["inverse"], out=st["out"])
    if kind == "pyramid":
        c = plan.decompose(st["x"], st["masks"])
        return [c, plan.reconstruct(c, st["masks"])]
    c = autograd.wavelet_decompose(st["x"], plan, st["masks"])
    r = autograd.wavelet_reconstruct(c, plan, st["masks"])
    g = torch.autograd.grad((c, r), st["leaves"], (st["gc"], st["gr"]))
    return [c.detach(), r.detach(), *g]


def work(case):
    """Each input read and each output written once; 5 m log2 m per FFT."""
    def fft(m):
        return 5.0 * m * math.log2(max(m, 2))

    if case["kind"] == "batch":
        ms = [abs(_det(M)) for M in _batch_matrices(case)]
        return dict(bytes=16.0 * sum(ms), flops=sum(fft(m) for m in ms))
    M, B = _matrix(case["M"]), case["batch"]
    m = abs(_det(M))
    if case["kind"] == "fft":
        n = 2 if case["dir"] == "both" else 1
        # both: the samples in, the frequencies out, the samples back out
        return dict(bytes=8.0 * (n + 1) * B * m, flops=n * B * fft(m))
    q = abs(_det(_matrix(case["J"])))
    sizes = [m // q ** l for l in range(case["levels"] + 1)]
    one = fft(m) + sum((q - 1) * fft(n) + 2.0 * q * q * n for n in sizes[1:]) + fft(sizes[-1])
    masks = 4.0 * sum(sizes[:-1])
    if case["kind"] == "pyramid":
        return dict(bytes=24.0 * B * m + masks, flops=2 * B * one)
    return dict(bytes=48.0 * B * m + 2 * masks, flops=4 * B * one)


# ---------------------------------------------------------------------------
# The same in 64 bits, without the library

def _matrix(text):
    return [[int(v) for v in row.split(",")] for row in text.split(";")]


def _mul(A, B):
    return [[sum(A[i][k] * B[k][j] for k in range(len(B))) for j in range(len(B[0]))]
            for i in range(len(A))]


def _transpose(M):
    return [list(r) for r in zip(*M)]


def _det(M):
    if len(M) == 1:
        return M[0][0]
    return sum((-1) ** j * M[0][j] * _det([r[:j] + r[j + 1:] for r in M[1:]])
               for j in range(len(M)) if M[0][j])


def _adjugate(M):
    d = len(M)
    if d == 1:
        return [[1]]
    return [[(-1) ** (i + j) * _det([r[:i] + r[i + 1:] for k, r in enumerate(M) if k != j])
             for j in range(d)] for i in range(d)]


def _divide(J, M):
    """J^{-1} M."""
    D = _det(J)
    return [[v // D for v in row] for row in _mul(_adjugate(J), M)]


def _hermite(M):
    """(H, U): H = M U upper triangular, positive diagonal, 0 <= H_ij < H_ii."""
    d = len(M)
    H = [list(r) for r in M]
    U = [[int(i == j) for j in range(d)] for i in range(d)]

    def add(dst, src, k):
        for A in (H, U):
            for row in A:
                row[dst] += k * row[src]

    for i in range(d - 1, -1, -1):
        for j in range(i):
            while H[i][j]:
                add(i, j, -(H[i][i] // H[i][j]))
                for A in (H, U):
                    for row in A:
                        row[i], row[j] = row[j], row[i]
        if H[i][i] < 0:
            for A in (H, U):
                for row in A:
                    row[i] = -row[i]
        for j in range(i + 1, d):
            add(j, i, -(H[i][j] // H[i][i]))
    return H, U


def _box(H):
    """The points of the box prod [0, H_ii) in C order, one column each."""
    sides = [H[i][i] for i in range(len(H))]
    n = torch.arange(math.prod(sides), device=_device())
    out = []
    for s in reversed(sides):
        out.insert(0, n % s)
        n = n // s
    return out


def _floor(a, b):
    return torch.div(a, b, rounding_mode="floor")


def _index(H, v):
    """Natural index of integer points v, reduced into the box of H."""
    d, v = len(H), list(v)
    for i in range(d - 1, -1, -1):
        t = _floor(v[i], H[i][i])
        v = [v[r] - t * H[r][i] if r <= i else v[r] for r in range(d)]
    n = v[0]
    for i in range(1, d):
        n = n * H[i][i] + v[i]
    return n


def _dft(M, x, sign):
    """m^{-1/2} sum_g x_g exp(sign 2 pi i h^T M^{-1} g) for x (batch, m) in the
    natural order of Z^d / M Z^d, h in that of Z^d / M^T Z^d.

    With H = M U and f = U^T h the phase is w . g, w = H^{-T} f: one FFT per
    coordinate of g, the coordinates before it entering as a twiddle."""
    H, U = _hermite(M)
    d = len(M)
    sides = [H[i][i] for i in range(d)]
    m = math.prod(sides)
    y = x.to(torch.complex128).reshape(-1, *sides)
    num, den = [], []      # w_i = num_i / den_i over the frequencies before axis i
    D = 1
    for i in range(d):
        shape = [1] * i + [sides[i]] + [1] * (d - i - 1)
        f = torch.arange(sides[i], device=y.device).reshape(shape)
        back = sum((H[j][i] * num[j] * (D // den[j]) for j in range(i)), torch.zeros_like(f[:1]))
        if i and any(H[j][i] for j in range(i)):
            r = (-back * f) % (D * sides[i])
            y = y * torch.polar(torch.ones((), dtype=torch.float64, device=y.device),
                                sign * 2 * math.pi / (D * sides[i]) * r.double())
        y = torch.fft.fft(y, dim=1 + i) if sign < 0 else torch.fft.ifft(y, dim=1 + i,
                                                                        norm="forward")
        num.append(f * D - back)
        D *= sides[i]
        den.append(D)
    h = _box(_hermite(_transpose(M))[0])
    f = [sum(U[j][i] * h[j] for j in range(d)) for i in range(d)]
    for i in range(d):     # reduce by the columns of H^T
        t = _floor(f[i], sides[i])
        f = [f[k] - t * H[i][k] if k >= i else f[k] for k in range(d)]
    n = f[0]
    for i in range(1, d):
        n = n * sides[i] + f[i]
    return y.reshape(-1, m).index_select(1, n) / math.sqrt(m)


def _inverse_dft(M, X):
    return _dft(_transpose(M), X, 1)


def _levels(M, J, levels):
    out = []
    for _ in range(levels):
        N = _divide(J, M)
        out.append((M, N))
        M = N
    return out


def _symmetric(M):
    """(t, h, m): M^{-T} h = t / m with t in [-m/2, m/2), and h reduced so."""
    d, D = len(M), _det(M)
    m, s, A = abs(D), (1 if D > 0 else -1), _adjugate(M)
    h = _box(_hermite(_transpose(M))[0])
    t = [(s * sum(A[k][j] * h[k] for k in range(d)) + m // 2) % m - m // 2 for j in range(d)]
    return t, [_floor(sum(M[j][i] * t[j] for j in range(d)), m) for i in range(d)], m


def _dirichlet_masks(M, J, levels):
    """sqrt(q) 2^{(r_M - r_N) / 2} in the closed box of N, 0 outside."""
    out = []
    for Ml, N in _levels(M, J, levels):
        t, h, m = _symmetric(Ml)
        n, A, s = abs(_det(N)), _adjugate(N), (1 if _det(N) > 0 else -1)
        e = sum((2 * a == -m).long() for a in t)
        inside = torch.ones_like(e, dtype=torch.bool)
        for j in range(len(M)):
            w = 2 * s * sum(A[k][j] * h[k] for k in range(len(M)))
            inside &= w.abs() <= n
            e = e - (w.abs() == n).long()
        out.append(torch.where(inside, math.sqrt(m // n) * torch.exp2(0.5 * e.double()), 0.0))
    return out


class _Fibers:
    """The fibers of one level: natural indices of their members, and for two
    channels the phase of the wavelet."""

    def __init__(self, M, N, J):
        d = len(M)
        HM = _hermite(_transpose(M))[0]
        HJ = _hermite(_transpose(J))[0]
        k = _box(_hermite(_transpose(N))[0])
        classes = [[int(c[l]) for c in _box(HJ)] for l in range(abs(_det(J)))]
        self.i = []
        for g in classes:
            s = [sum(N[j][i] * g[j] for j in range(d)) for i in range(d)]
            self.i.append(_index(HM, [k[i] + s[i] for i in range(d)]))
        self.q = len(classes)
        self.m = abs(_det(M))
        order = torch.cat(self.i)
        self.where = torch.empty_like(order)
        self.where[order] = torch.arange(self.m, device=order.device)
        if self.q == 2:
            A, D = _adjugate(J), _det(J)
            y = next([-(A[r][i] % D != 0) for r in range(d)] for i in range(d)
                     if any(A[r][i] % D for r in range(d)))     # twice the point of P(J)
            v = [sum(J[r][c] * y[c] for c in range(d)) // 2 for r in range(d)]
            B, sg = _adjugate(M), (1 if _det(M) > 0 else -1)
            c = [sg * sum(B[i][j] * v[j] for j in range(d)) for i in range(d)]
            sides = [HM[i][i] for i in range(d)]
            n, h = self.i[0], []
            for s in reversed(sides):
                h.insert(0, n % s)
                n = n // s
            rho = sum((c[i] % self.m) * h[i] for i in range(d)) % self.m
            self.phi = torch.polar(torch.ones((), dtype=torch.float64, device=rho.device),
                                   -2 * math.pi / self.m * rho.double())

    def matrix(self, mask):
        """Rows of the channel matrix over the fiber members (q > 2)."""
        u = [mask[i] / math.sqrt(self.q) for i in self.i]
        sg = torch.where(u[0] >= 0, 1.0, -1.0)
        v = [u[0] + sg] + u[1:]
        c = 2 / sum(a * a for a in v)
        return [u] + [[(1.0 if j == l else 0.0) - c * v[j] * v[l] for l in range(self.q)]
                      for j in range(1, self.q)]

    def split(self, X, mask):
        x = [X.index_select(1, i) for i in self.i]
        if self.q == 2:
            a, b = mask[self.i[0]], mask[self.i[1]]
            r = math.sqrt(0.5)
            return [(a * x[0] + b * x[1]) * r, self.phi.conj() * (b * x[0] - a * x[1]) * r]
        return [sum(row[l] * x[l] for l in range(self.q)) for row in self.matrix(mask)]

    def join(self, d, mask):
        if self.q == 2:
            a, b = mask[self.i[0]], mask[self.i[1]]
            r = math.sqrt(0.5)
            w = self.phi * d[1]
            x = [(a * d[0] + b * w) * r, (b * d[0] - a * w) * r]
        else:
            S = self.matrix(mask)
            x = [sum(S[j][l] * d[j] for j in range(self.q)) for l in range(self.q)]
        return torch.cat(x, 1).index_select(1, self.where)


def _pyramid(case, x, masks, samples=False):
    """(coefficients, reconstruction) in 64 bits."""
    M, J = _matrix(case["M"]), _matrix(case["J"])
    levels = [(Ml, N, _Fibers(Ml, N, J)) for Ml, N in _levels(M, J, case["levels"])]
    if samples:            # sqrt(m) 2^{r/2} between point values and coefficients
        t, _, m = _symmetric(M)
        w = math.sqrt(m) * torch.exp2(0.5 * sum((2 * a == -m).double() for a in t))
    X = _dft(M, x, -1)
    X = X / w if samples else X
    blocks = []
    for (Ml, N, F), mask in zip(levels, masks):
        d = F.split(X, mask)
        blocks += [_inverse_dft(N, b) for b in d[1:]]
        X = d[0]
    c = torch.cat(blocks + [_inverse_dft(levels[-1][1], X)], 1)
    at = c.shape[1] - X.shape[1]
    X = _dft(levels[-1][1], c[:, at:], -1)
    for (Ml, N, F), mask in zip(reversed(levels), reversed(masks)):
        n, d = F.m // F.q, [X]
        at -= (F.q - 1) * n
        d += [_dft(N, c[:, at + j * n:at + (j + 1) * n], -1) for j in range(F.q - 1)]
        X = F.join(d, mask)
    return c, _inverse_dft(M, X * w if samples else X)


def exact(case, seed):
    t = _inputs(case, seed)
    x = t["x"].to(torch.complex128)
    if case["kind"] == "fft":
        M = _matrix(case["M"])
        if case["dir"] == "inverse":
            return _inverse_dft(M, x)
        X = _dft(M, x, -1)
        return X if case["dir"] == "forward" else [X, x]
    if case["kind"] == "batch":
        out, at = [], 0
        for M in _batch_matrices(case):
            y = x[at:at + abs(_det(M))].reshape(1, -1)
            at += y.numel()
            out.append((_dft(M, y, -1) if case["dir"] == "forward" else _inverse_dft(M, y))[0])
        return torch.cat(out)
    masks = [a.double() for a in t["masks"]]
    if case["kind"] == "pyramid":
        return list(_pyramid(case, x, masks, case.get("samples", False)))
    leaves = [x.requires_grad_(True)] + [a.requires_grad_(True) for a in masks]
    c, r = _pyramid(case, x, masks)
    g = torch.autograd.grad((c, r), leaves, (t["gc"].to(torch.complex128),
                                             t["gr"].to(torch.complex128)))
    return [c.detach(), r.detach(), *g]
