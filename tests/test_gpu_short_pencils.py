"""Strided passes of short lengths without an FFT plan, on both sides of the lines between one thread
per output and the sine products (6, 12 and 18 intervals; 200 kB a row of columns).

Transforms: every output within N eps of the sum of its terms' absolute values (at most N
roundings each of at most half an eps, and the table's).  Dirichlet solves: the Poisson bars."""
import numpy as np
import pytest

from oracle import fast
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [4, 5, 6, 7, 11, 13, 17, 18, 19]


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


@pytest.mark.parametrize("N", LENGTHS)
@pytest.mark.parametrize("columns", [37, 24999, 25000, 50021])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_transform(ah, N, columns, prec):
    dt = torch.float64 if prec == "fp64" else torch.float32
    x = torch.randn(N - 1, columns, dtype=dt, device="cuda")
    k = np.arange(1, N)
    r = np.outer(k, k) % (2 * N)  # sin(pi r / N) from its first quarter, to the last bit
    sign, r = np.where(r > N, -1.0, 1.0), np.where(r > N, 2 * N - r, r)
    S = torch.from_numpy(sign * np.sin(np.pi * np.minimum(r, N - r) / N)).cuda()
    ref, bound = S @ x.double(), S.abs() @ x.double().abs()
    outs = [ah.dst1(x, 1, ah.FP64 if prec == "fp64" else ah.MIXED) for _ in range(2)]
    assert torch.equal(*outs)
    eps = torch.finfo(dt).eps
    assert bool(((outs[0].double() - ref).abs() <= N * eps * bound).all())


@pytest.mark.parametrize("N", LENGTHS)
@pytest.mark.parametrize("n", [(150, 20), (300, 130)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_dirichlet(ah, N, n, prec):
    for shape in (n + (N,), (n[0], N, n[1])):
        hi = tuple(m / max(shape) for m in shape)
        nodes = tuple(m + 1 for m in reversed(shape))
        pb = W.Problem(shape, (0.0,) * 3, hi, np.ones(nodes), np.zeros(nodes))
        g = np.random.default_rng(N).standard_normal([m - 1 for m in reversed(shape)])
        ref = fast.FastTier(pb).poisson(g)
        gt = torch.from_numpy(g).cuda()
        p = ah.FP64 if prec == "fp64" else ah.MIXED
        with ah.Solver(pb, precision=p) as s:
            outs = [s.poisson(gt), ah.poisson_noalloc(shape, (0.0,) * 3, hi, gt, precision=p)]
        for w in outs:
            assert float(np.abs(w.cpu().numpy() - ref).max()) <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(ref).max()
