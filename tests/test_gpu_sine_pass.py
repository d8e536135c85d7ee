"""DST-I passes of lengths without an FFT plan (the half-size sine products on the matrix
cores) against the naive sum, at the edges of their tiles: 16 outputs of either parity, 16 or
32 pencils, the chunks of the summation index, whole pencils or outputs split over work-groups,
and the in-place pass of a length beyond what one work-group holds.

Tolerance: an output is a sum of N/2 products of e_m = x_m +- x_{N-m}; with unit roundoff u
each term carries at most the roundings of e_m, of the sine, of the product and of at most N/2
additions, so |error| <= (N/2 + 4) u sum |x_m| for each pencil."""
import numpy as np
import pytest

from oracle import dst as odst, fast
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


def _inplace(ah, x, axis, prec):
    dim = x.dim()
    nint = (ah.c_int * 3)(*([x.shape[dim - 1 - a] for a in range(dim)] + [1] * (3 - dim)))
    y = x.clone()
    rc = ah._lib.ahoc_dst1(prec, dim, nint, axis, ah._ptr(y), ah._ptr(y), ah._stream())
    assert rc == ah.OK
    return y


@pytest.mark.parametrize("N", [4, 5, 33, 34, 35, 65, 127, 130, 255, 257, 500, 511, 514, 1025, 2047, 2050])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sine_pass_matches_naive_sum(ah, N, prec):
    rng = np.random.default_rng(N)
    p, dt, u = (ah.FP64, torch.float64, 2.0 ** -53) if prec == "fp64" else (ah.MIXED, torch.float32, 2.0 ** -24)
    for axis, shp in ((0, (1, 17, N - 1)), (1, (1, N - 1, 2)), (1, (2, N - 1, 33)), (2, (N - 1, 1, 16))):
        x = torch.from_numpy(rng.standard_normal(shp)).to(dt)
        xin = x.double().numpy()
        ref = odst.dst1(xin, axis=2 - axis)
        tol = (N / 2 + 4) * u * np.abs(xin).sum(axis=2 - axis, keepdims=True)
        for out in (ah.dst1(x.cuda(), axis, p), _inplace(ah, x.cuda(), axis, p)):
            assert (np.abs(out.double().cpu().numpy() - ref) <= tol).all(), (N, axis, shp)


@pytest.mark.parametrize("N", [20, 100, 260, 600])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sine_pass_many_pencils(ah, N, prec):
    """Enough pencils for the 32-pencil tiles: sampled pencils against the naive sum."""
    p, dt, u = (ah.FP64, torch.float64, 2.0 ** -53) if prec == "fp64" else (ah.MIXED, torch.float32, 2.0 ** -24)
    for axis, shp in ((0, (65, 257, N - 1)), (1, (65, N - 1, 257))):
        x = torch.randn(shp, dtype=dt, device="cuda", generator=torch.Generator("cuda").manual_seed(N))
        out = ah.dst1(x, axis, p)
        same = _inplace(ah, x, axis, p)
        assert torch.equal(out, same)
        pick = [0, 1, 31, 64]
        xs = x[pick].double().cpu().numpy()
        tol = (N / 2 + 4) * u * np.abs(xs).sum(axis=2 - axis, keepdims=True)
        assert (np.abs(out[pick].double().cpu().numpy() - odst.dst1(xs, axis=2 - axis)) <= tol).all(), (N, axis)


@pytest.mark.parametrize("n", [(34, 50), (64, 35), (35, 64), (50, 16, 21), (16, 50, 64), (21, 24, 10)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_poisson_mixed_length_axes(ah, n, prec):
    """Axes with and without an FFT plan in one solve (every order of the two work arrays),
    through the handle and without one, on a scratch array that an earlier call left NaN in."""
    hi = (1.0, 1.3, 0.8)[:len(n)]
    shape = tuple(m + 1 for m in reversed(n))
    pb = W.Problem(n, (0.0,) * len(n), hi, np.ones(shape), np.zeros(shape))
    ft = fast.FastTier(pb)
    g = np.random.default_rng(3).standard_normal(ft.g.interior_shape)
    ref = ft.poisson(g)
    p = ah.FP64 if prec == "fp64" else ah.MIXED
    bad = torch.full((40, 40, 40), float("nan"), dtype=torch.float64, device="cuda")
    ah.poisson_noalloc((41, 41, 41), (0.0,) * 3, (1.0,) * 3, bad, precision=p)
    with ah.Solver(pb, precision=p) as s:
        outs = [s.poisson(g), s.poisson(g), ah.poisson_noalloc(n, (0.0,) * len(n), hi, torch.from_numpy(g).cuda(), precision=p)]
    for w in outs:  # the bars of the other Poisson parity tests
        assert np.abs(w.cpu().numpy() - ref).max() <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("n", [(32, 32), (32, 1024), (1024, 64), (192, 256), (2048, 64), (32, 64, 96), (256, 32, 64),
                               (64, 512, 128)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_face_transforms_match_fft_passes(ah, n, prec):
    """The Schur operator and the preconditioner with all face transforms in one launch per pass
    (split sums and not; 2048: beyond its lengths) against the one-tile FFT family, which transforms
    each face pair by its own passes.  Bars of the Schur parity tests."""
    hi = tuple(m / max(n) for m in n)
    p = (W.manufactured("1 + 0.5*sin(2*pi*x)*cos(2*pi*y)", "sin(pi*x)**2*sin(pi*y)**2*exp(x)", n, (0.0,) * 2, hi)
         if len(n) == 2 else W.manufactured(W.C3_ALPHA, "sin(pi*x)*sin(pi*y)*cos(pi*z)*exp(x)", n, (0.0,) * 3, hi))
    tol = 1e-11 if prec == "fp64" else 1e-4
    with ah.Solver(p, precision=ah.FP64 if prec == "fp64" else ah.MIXED) as s:
        q = np.random.default_rng(4).standard_normal(s.nq)
        got = [s.schur_apply(q), s.precond_apply(q)]
        try:
            ah.set_dst_variant(3)
            ref = [s.schur_apply(q), s.precond_apply(q)]
        finally:
            ah.set_dst_variant(0)
    for k, (a, b) in enumerate(zip(got, ref)):
        assert float((a - b).abs().max()) <= (tol if k == 0 else 1e-11) * float(b.abs().max()), (n, k)


# the one-work-group solve at the edges of its tiles (16 pencils, 16 outputs of either parity)
# and on both sides of its rule (64 x 64 in, 97 x 96 out; 20 x 130 the longest axis)
@pytest.mark.parametrize("n", [(4, 4), (4, 33), (33, 5), (17, 16), (34, 31), (64, 64), (65, 64), (96, 96), (97, 96),
                               (100, 96), (20, 130), (130, 20), (101, 101)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_small_plane_poisson(ah, n, prec):
    hi = (1.0, 0.7)
    shape = tuple(m + 1 for m in reversed(n))
    pb = W.Problem(n, (0.0, 0.0), hi, np.ones(shape), np.zeros(shape))
    ft = fast.FastTier(pb)
    g = np.random.default_rng(n[0]).standard_normal(ft.g.interior_shape)
    ref = ft.poisson(g)
    p = ah.FP64 if prec == "fp64" else ah.MIXED
    gt = torch.from_numpy(g).cuda()
    with ah.Solver(pb, precision=p) as s:
        outs = [s.poisson(gt), ah.poisson_noalloc(n, (0.0, 0.0), hi, gt, precision=p)]
        ah.set_dst_variant(5)  # as separate passes
        outs.append(s.poisson(gt))
        ah.set_dst_variant(0)
    inplace = gt.clone()
    ah.poisson_noalloc(n, (0.0, 0.0), hi, inplace, precision=p, out=inplace)
    assert torch.equal(inplace, outs[1])
    for w in outs:
        assert np.abs(w.cpu().numpy() - ref).max() <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(ref).max()
