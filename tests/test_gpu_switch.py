"""The process-wide kernel-family switch may move while other threads' calls run: a call then takes
either family for a pass, and its results are right all the same.  Bars of the parity tests
between two families."""
import threading

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
    return mod


class Flipping:
    def __init__(self, ah, to):
        self.ah, self.to, self.stop = ah, to, threading.Event()
        self.t = threading.Thread(target=self.run)

    def run(self):
        while not self.stop.is_set():
            self.ah.set_dst_variant(self.to)
            self.ah.set_dst_variant(0)

    def __enter__(self):
        self.t.start()

    def __exit__(self, *exc):
        self.stop.set()
        self.t.join()
        self.ah.set_dst_variant(0)


# rectangular (faces as sine products, two arrays in turn) and square (lines in one launch)
@pytest.mark.parametrize("n", [(256, 128), (128, 128)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_operator(ah, n, prec):
    p = W.manufactured(A2, U2, n, (0.0, 0.0), tuple(m / max(n) for m in n))
    with ah.Solver(p, precision=ah.FP64 if prec == "fp64" else ah.MIXED, tol=1e-10) as s:
        q = torch.from_numpy(np.random.default_rng(3).standard_normal(s.nq)).cuda()
        y, u = s.schur_apply(q), s.solve()[0].clone()
        bad = []
        with Flipping(ah, 3):
            for _ in range(400):
                bad.append(float((s.schur_apply(q) - y).abs().max() / y.abs().max()))
            solves = [s.solve() for _ in range(20)]
            errs = [float((k[0] - u).abs().max() / u.abs().max()) for k in solves]
    assert max(bad) <= (1e-11 if prec == "fp64" else 1e-4), (max(bad), sum(b > 1e-4 for b in bad))
    assert all(k[3].converged for k in solves) and max(errs) <= 1e-8, max(errs)


def test_small_dirichlet_solves(ah):
    g = torch.randn(31, 31, dtype=torch.float64, device="cuda")
    args = ((32, 32), (0.0, 0.0), (1.0, 1.0), g)
    w = ah.poisson_noalloc(*args)
    with Flipping(ah, 3):
        bad = [float((ah.poisson_noalloc(*args) - w).abs().max() / w.abs().max()) for _ in range(3000)]
    assert max(bad) <= 1e-12
