"""The Arnoldi step at the lengths where its kernels change: one work-group with 1, 2, 4 or 8
entries per thread (up to 512, 1024, 2048, 4096 augmented unknowns), slices summed by every
work-group, and a restart inside the solve.

The residual estimate of GMRES is the residual norm of its iterate up to rounding: with the
tolerance 1e-8 and FP64 operators (a few 1e-13 relative at these grids), the estimate and
||b - S q|| / ||b|| agree to 1e-11."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


A2, U2 = "1 + 0.5*sin(2*pi*x)*cos(2*pi*y)", "sin(pi*x)**2*sin(pi*y)**2*exp(x + y)"
# N_q: 18, 512, 514, 1024, 1026, 2048, 2050, 4096, 4098 (2-D) and 7686, 135300 (3-D)
GRIDS = [(6, 5), (130, 128), (130, 129), (258, 256), (259, 256), (514, 512), (515, 512), (1026, 1024), (1027, 1024),
         (36, 38, 36), (151, 152, 150)]


@pytest.mark.parametrize("restart", [30, 4])
@pytest.mark.parametrize("n", GRIDS)
def test_residual_estimate_is_the_residual(ah, n, restart):
    hi = tuple(m / max(n) for m in n)
    src = (A2, U2) if len(n) == 2 else (W.C3_ALPHA, "sin(pi*x)**2*sin(pi*y)**2*exp(z)")
    p = W.manufactured(*src, n, (0.0,) * len(n), hi)
    with ah.Solver(p, tol=1e-8, restart=restart) as s:
        b = s.schur_rhs()
        _, _, q, st = s.solve(want_q=True)
        r = float((b - s.schur_apply(q)).norm() / b.norm())
        again = s.solve(want_q=True)[2]
    assert st.converged and st.schur_relres <= 1e-8
    assert abs(r - st.schur_relres) <= 1e-11, (r, st)
    assert torch.equal(q, again)


def test_long_segments_in_a_batch(ah):
    """Two instances of more than 4096 unknowns in one bucket, one of them finished early (f = 0),
    against single solves."""
    ps = [W.manufactured(A2, U2, (1030, 1026), (0.0, 0.0), (1.0, 1.0)) for _ in range(3)]
    ps[1].f = np.zeros_like(ps[1].f)
    ps[1].gD = ps[1].gN = ps[1].lapgD = None
    ps[2].f = ps[2].f * (1.0 + 0.5 * np.linspace(0.0, 1.0, ps[2].f.shape[1])[None, :])
    outs, stats, rc = ah.solve_batched(ps, tol=1e-11)
    assert rc == ah.OK and all(s.converged for s in stats)
    for p, u in zip(ps, outs):
        with ah.Solver(p, tol=1e-11) as s:
            ref = s.solve()[0]
        assert float((u - ref).abs().max()) <= 1e-9 * max(float(ref.abs().max()), 1e-30)


ROUGH = "1 + 0.95*sin(12*pi*x)*cos(10*pi*y)"


@pytest.mark.parametrize("restart", [60, 200])
@pytest.mark.parametrize("n,steps", [((130, 128), 32), ((258, 256), 64), ((514, 512), 64)])
def test_more_vectors_than_the_registers_hold(ah, n, steps, restart):
    """Long cycles (rough data, no preconditioner) whose basis outgrows the 32 or 16 vectors that
    one work-group keeps in registers, and the 64 rows of one turn of the back substitution.  The
    second Gram-Schmidt sweep and the sum of the two columns must not meet: with a column
    subtracted twice the estimate leaves the residual by orders of magnitude.  Both carry the
    operator's error of 1e-13 ||S|| ||q|| / ||b||, at most the condition number, which is below N."""
    p = W.manufactured(ROUGH, U2, n, (0.0, 0.0), tuple(m / max(n) for m in n))
    rng = np.random.default_rng(1)
    p.f = rng.standard_normal(p.f.shape)
    p.gN = rng.standard_normal(p.f.shape)
    with ah.Solver(p, tol=1e-10, restart=restart, precond=0) as s:
        b = s.schur_rhs()
        _, _, q, st = s.solve(want_q=True)
        r = float((b - s.schur_apply(q)).norm() / b.norm())
    assert st.converged and st.schur_relres <= 1e-10
    assert st.gmres_iters > min(steps, restart), st.gmres_iters
    assert abs(r - st.schur_relres) <= 1e-13 * max(n), (r, st)
