"""The 2-D operator on square grids, whose boundary lines one work-group per instance takes through
the preconditioner, the lifts and the transforms, against the one-tile FFT family, which runs
them as separate passes: every length it is built for, both precisions, with Navier faces and
as a batch.  Bars of the Schur parity tests; solutions 1e-10 (mixed 1e-9) of max|U| between two
solves to 1e-12."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

A2, U2 = "1 + 0.5*sin(2*pi*x)*cos(2*pi*y)", "sin(pi*x)**2*sin(pi*y)**2*exp(x + y)"


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    yield mod
    mod.set_dst_variant(0)


@pytest.mark.parametrize("N", [32, 64, 96, 128, 192, 256, 384, 512, 768, 1024])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_lines_match_separate_passes(ah, N, prec):
    # spacings differ (h_x = 2 h_y), one Navier face
    p = W.manufactured(A2, U2, (N, N), (0.0, 0.0), (1.0, 0.5), navier=(False, False, True, False))
    mode = ah.FP64 if prec == "fp64" else ah.MIXED
    with ah.Solver(p, precision=mode, tol=1e-12) as s:
        q = np.random.default_rng(N).standard_normal(s.nq)
        ah.set_dst_variant(0)
        y = s.schur_apply(q)
        u, _, _, st = s.solve()
        u = u.clone()
        ah.set_dst_variant(3)
        y3 = s.schur_apply(q)
        u3, _, _, st3 = s.solve()
        ah.set_dst_variant(0)
    assert float((y - y3).abs().max()) <= (1e-11 if prec == "fp64" else 1e-4) * float(y3.abs().max())
    assert st.converged == st3.converged
    assert float((u - u3).abs().max()) <= (1e-10 if prec == "fp64" else 1e-9) * float(u3.abs().max())


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("precond", [0, 1])
def test_lines_in_a_batch(ah, prec, precond):
    """Instances of two sizes, each instance's lines in its own work-group, against single solves."""
    ps = []
    for k, n in enumerate((64, 96, 64, 96, 64)):
        p = W.manufactured("1 + c*sin(2*pi*x)*cos(2*pi*y)", U2, (n, n), params=("c",), pvals=(0.1 * (k + 1),))
        ps.append(p)
    mode = ah.FP64 if prec == "fp64" else ah.MIXED
    outs, stats, rc = ah.solve_batched(ps, precision=mode, tol=1e-11, precond=precond)
    assert rc == ah.OK and all(s.converged for s in stats)
    for p, u in zip(ps, outs):
        with ah.Solver(p, tol=1e-12) as s:
            ref = s.solve()[0]
        assert float((u - ref).abs().max()) <= 1e-9 * float(ref.abs().max())


@pytest.mark.parametrize("N", [32, 128, 512, 1024])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_both_forms_reach_the_tolerance(ah, N, prec):
    """The premise of the comparison above: both solves are done to the tolerance, or to the
    operator's rounding (a few 1e-13 times a condition number below N: 1e-10 at the most)."""
    p = W.manufactured(A2, U2, (N, N), (0.0, 0.0), (1.0, 0.5), navier=(False, False, True, False))
    with ah.Solver(p, precision=ah.FP64 if prec == "fp64" else ah.MIXED, tol=1e-12) as s:
        for variant in (0, 3):
            ah.set_dst_variant(variant)
            _, _, q, st = s.solve(want_q=True)
            ah.set_dst_variant(0)
            print(N, prec, variant, st.converged, st.schur_relres)
            assert st.converged or st.schur_relres <= 1e-10, st
