"""Variable-beta solves at the edges of the V-solve operator's tiles (64 x 8 columns, chunks of
four planes and more): its output, the parts of its dot products and the faces' part alone,
against the direct solve of the coupled system.  Bars of the other variable-beta tests."""
import numpy as np
import pytest

import workloads as W
from oracle import direct

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


@pytest.mark.parametrize("n", [(65, 9, 5), (66, 10, 6), (4, 17, 7), (130, 8, 4), (20, 18, 34)])
def test_varbeta_tile_edges(ah, n):
    hi = tuple(1.0 + 0.01 * m for m in n)
    p = W.manufactured(W.EX2_ALPHA, "sin(pi*x)*sin(pi*y)**2*sin(pi*z)", n, (0.0,) * 3, hi, beta=W.EX2_BETA)
    U, V, Q, asm = direct.solve(p)
    with ah.Solver(p, tol=1e-13) as s:
        u, _, q, st = s.solve(want_q=True)
    assert st.converged and st.vsolve_iters > 0, st
    for got, ref, bar in ((u, U, 1e-11), (q, Q, 1e-10)):
        assert np.abs(got.cpu().numpy() - np.asarray(ref)).max() <= bar * np.abs(np.asarray(ref)).max(), n
