"""3-D Dirichlet solves with both axes of a plane in one launch, at the edges of its tiles (16
columns of x, 32 outputs of either parity of y, eight planes per turn of the XCDs) and on both
sides of its rule (128 in, 129 out in either axis; the slowest axis as products to 96 and where
no FFT kernel is specialised on its length): against the oracle, and against the same
solve as separate passes (variant 5).  Bars of the other Poisson parity tests."""
import numpy as np
import pytest

from oracle import fast
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


@pytest.mark.parametrize("n", [(4, 4, 4), (5, 33, 9), (17, 16, 10), (33, 5, 34), (32, 65, 17), (64, 64, 8), (65, 31, 5),
                               (66, 34, 12), (96, 97, 20), (99, 100, 7), (127, 128, 6), (128, 127, 24), (128, 4, 130),
                               (129, 20, 9), (20, 129, 9), (33, 20, 32), (20, 9, 64), (12, 30, 96), (9, 8, 97),
                               (8, 8, 128)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_plane_poisson(ah, n, prec):
    lo, hi = (0.0,) * 3, (1.0, 0.7, 1.2)
    shape = tuple(m + 1 for m in reversed(n))
    pb = W.Problem(n, lo, hi, np.ones(shape), np.zeros(shape))
    ft = fast.FastTier(pb)
    g = np.random.default_rng(n[0]).standard_normal(ft.g.interior_shape)
    ref = ft.poisson(g)
    p = ah.FP64 if prec == "fp64" else ah.MIXED
    gt = torch.from_numpy(g).cuda()
    bad = torch.full((40, 40, 40), float("nan"), dtype=torch.float64, device="cuda")
    ah.poisson_noalloc((41, 41, 41), lo, (1.0,) * 3, bad, precision=p)
    with ah.Solver(pb, precision=p) as s:
        outs = [s.poisson(gt), s.poisson(gt), ah.poisson_noalloc(n, lo, hi, gt, precision=p)]
        ah.set_dst_variant(5)
        outs.append(s.poisson(gt))
        ah.set_dst_variant(0)
    inplace = gt.clone()
    ah.poisson_noalloc(n, lo, hi, inplace, precision=p, out=inplace)
    assert torch.equal(inplace, outs[2]) and torch.equal(outs[0], outs[1])
    err = [float(np.abs(w.cpu().numpy() - ref).max() / np.abs(ref).max()) for w in outs]
    print(n, prec, err)
    assert max(err) <= (1e-12 if prec == "fp64" else 1e-5)
