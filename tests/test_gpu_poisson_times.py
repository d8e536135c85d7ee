"""Per-kernel-class timing of ahoc_poisson: every route of the Dirichlet solve is recorded (small
planes in one launch, planes of a 3-D grid, separate passes)."""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,want", [((32, 32), {"dst_fused": 1}), ((64, 50), {"dst_fused": 1}),
                                    ((100, 90, 75), {"dst_rows": 2, "dst_fused": 1}),
                                    ((128, 96, 64), {"dst_rows": 2, "dst_fused": 1}),
                                    ((256, 128), {"dst_rows": 2, "dst_fused": 1}),
                                    ((150, 64, 40), {"dst_rows": 2, "dst_strided": 2, "dst_fused": 1})])
def test_poisson_is_timed(n, want, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as ah
    src = ("1 + 0*x", "sin(pi*x)**2*sin(pi*y)**2") if len(n) == 2 else (W.C3_ALPHA, "sin(pi*x)**2*sin(pi*y)**2*exp(z)")
    p = W.manufactured(*src, n, (0.0,) * len(n), (1.0,) * len(n))
    g = torch.ones([m - 1 for m in reversed(n)], dtype=torch.float64, device="cuda")
    with ah.Solver(p, precision=ah.FP64 if prec == "fp64" else ah.MIXED) as s:
        s.poisson(g)
        s.profile(True)
        s.poisson(g)
        s.poisson(g)
        kt = s.kernel_times()
        s.profile(False)
    assert {k: v[1] for k, v in kt.items() if v[1]} == {k: 2 * c for k, c in want.items()}
    for k in want:
        ms, _, nbytes = kt[k]
        assert ms > 0 and nbytes >= 8 * g.numel()


# thin planes: few of them in one pass each, many as separate passes, on both sides of the rule
# (n_y >= 8 per 32 columns of x, or fewer than 128 n_y groups of columns)
@pytest.mark.parametrize("n,planes", [((128, 8, 200), True), ((128, 8, 600), False), ((128, 16, 512), True),
                                      ((128, 16, 2048), False), ((100, 31, 2100), False), ((100, 32, 2100), True),
                                      ((64, 15, 1100), False), ((64, 16, 1100), True), ((30, 8, 1030), True),
                                      ((30, 7, 1030), False)])
def test_thin_planes(n, planes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    import paper_2609_16478_amd as ah
    from oracle import fast
    hi = tuple(m / max(n) for m in n)
    shape = tuple(m + 1 for m in reversed(n))
    pb = W.Problem(n, (0.0,) * 3, hi, np.ones(shape), np.zeros(shape))
    g = np.random.default_rng(n[1]).standard_normal([m - 1 for m in reversed(n)])
    ref = fast.FastTier(pb).poisson(g)
    gt = torch.from_numpy(g).cuda()
    for prec in (ah.FP64, ah.MIXED):
        with ah.Solver(pb, precision=prec) as s:
            s.profile(True)
            w = s.poisson(gt)
            kt = s.kernel_times()
        assert kt["dst_strided"][1] == (0 if planes else 2) and kt["dst_rows"][1] == 2, kt
        if prec == ah.FP64:
            assert float(np.abs(w.cpu().numpy() - ref).max()) <= 1e-12 * np.abs(ref).max()
