"""The tiled 3-D stencil kernels at the seams of their tiles (64 x 8 columns, chunks of 4 to 32
planes), on grids without length-specialised transforms, whose Schur operator forms M(V/alpha)
with them.

Tolerances: the physical gather divides differences of U by h^2, so the FP64 operator carries
about 10 N^2 unit roundoffs (N <= 70: 1e-11); solutions of the two V-solve algorithms as in the
variable-beta tests (1e-11)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import fast

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def _box(n):
    hi = tuple(m / max(n) for m in n)
    return W.manufactured(W.C3_ALPHA, "sin(pi*x)*sin(pi*y)*cos(pi*z)*exp(x)", n, (0, 0, 0), hi)


@pytest.mark.parametrize("n", [(65, 9, 5), (66, 10, 6), (33, 17, 39), (70, 8, 37)])
def test_rhs_u_tile_seams(ah, n):
    p = _box(n)
    z = np.zeros(tuple(m + 1 for m in reversed(n)))
    ft = fast.FastTier(dataclasses.replace(p, f=z, gD=None, gN=None, lapgD=None))
    q = np.random.default_rng(5).standard_normal(ft.g.n_q)
    with ah.Solver(p) as s:
        assert _rel(s.schur_apply(q).cpu().numpy(), ft.R_of(q)) < 1e-11
        assert _rel(s.schur_rhs().cpu().numpy(), fast.FastTier(p).schur_rhs()) < 1e-11


@pytest.mark.parametrize("n", [(65, 9, 5), (66, 10, 6), (34, 17, 40)])
def test_vapply_tile_seams(ah, n):
    hi = tuple(m / max(n) for m in n)
    p = W.manufactured("2", "sin(pi*x)*sin(pi*y)**2*sin(pi*z)*exp(x)", n, (0.0,) * 3, hi, beta=-1.5)
    with ah.Solver(p, tol=1e-13) as s:
        u0, _, _, st0 = s.solve()
    p.beta = np.full(tuple(m + 1 for m in reversed(n)), p.beta)
    with ah.Solver(p, tol=1e-13) as s:
        u1, _, _, st1 = s.solve()
    assert st0.converged and st1.converged and st1.vsolve_iters > 0
    assert _rel(u1.cpu().numpy(), u0.cpu().numpy()) < 1e-11
