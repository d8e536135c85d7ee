"""Calls on one handle do not see what earlier calls left in its work arrays (the strided FFT passes
pair the last column of a row with the padding next to it): the same input gives the same bits
again.  Equality is exact; there is no tolerance to derive."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

A2, U2 = "1 + 0.5*sin(2*pi*x)*cos(2*pi*y)", "sin(pi*x)**2*sin(pi*y)**2*exp(x + y)"
ROUGH = "1 + 0.95*sin(12*pi*x)*cos(10*pi*y)"


@pytest.fixture(scope="module")
def ah():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_16478_amd as mod
    return mod


def problem(n, alpha=A2, seed=1):
    src = (alpha, U2) if len(n) == 2 else (W.C3_ALPHA, "sin(pi*x)**2*sin(pi*y)**2*exp(z)")
    p = W.manufactured(*src, n, (0.0,) * len(n), tuple(m / max(n) for m in n))
    rng = np.random.default_rng(seed)
    p.f = rng.standard_normal(p.f.shape)
    p.gN = rng.standard_normal(p.f.shape)
    return p


# rows by each kind of kernel (FFT, short matrix products, split and whole sine products, more than
# 2048 points), before strided FFT passes; 2-D and 3-D, with and without the plane passes
GRIDS = [(130, 128), (258, 256), (514, 512), (70, 256), (35, 32), (48, 36), (70, 4096), (64, 4096), (2050, 48), (256, 256),
         (1024, 1024), (150, 128, 36), (36, 150, 36), (192, 192, 32), (70, 150, 36), (130, 32, 32), (64, 64, 64)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", GRIDS)
def test_calls_do_not_see_earlier_ones(ah, n, prec):
    """Every call of a handle gives the bits it gave at first, after calls with data 1e6 times as
    large and with NaN."""
    with ah.Solver(problem(n), precision=ah.FP64 if prec == "fp64" else ah.MIXED, tol=1e-9) as s:
        g = torch.randn([m - 1 for m in reversed(n)], dtype=torch.float64, device="cuda")
        q = torch.randn(s.nq, dtype=torch.float64, device="cuda")
        calls = {"poisson": lambda x: s.poisson(g * x), "schur": lambda x: s.schur_apply(q * x),
                 "precond": lambda x: s.precond_apply(q * x)}
        wanted = {"rhs": lambda: s.schur_rhs(), "solve": lambda: s.solve()[0]}
        wanted.update({k: lambda f=f: f(1.0) for k, f in calls.items()})
        first = {k: f().clone() for k, f in wanted.items()}
        seen = []
        for x in (1.0, 1e6, float("nan")):
            for k, f in wanted.items():
                for call in calls.values():
                    call(x)
                if not torch.equal(first[k], f()):
                    seen.append((x, k))
    assert not seen, seen


@pytest.mark.parametrize("n", [(130, 36, 32), (40, 36, 32)])
def test_variable_beta_repeats(ah, n):
    p = problem(n)
    x = [np.linspace(0.0, m / max(n), m + 1) for m in n]
    p.beta = np.broadcast_to(10.0 + x[0][None, None, :] + x[1][None, :, None] + x[2][:, None, None], p.f.shape).copy()
    p.navier = (False,) + (True,) * 5
    with ah.Solver(p, tol=1e-9) as s:
        first = s.solve()[0].clone()
        s.poisson(torch.full([m - 1 for m in reversed(n)], float("nan"), dtype=torch.float64, device="cuda"))
        assert torch.equal(first, s.solve()[0])


@pytest.mark.parametrize("alpha", [A2, ROUGH])
@pytest.mark.parametrize("n", [(130, 128), (258, 256), (514, 512)])
def test_solve_repeats(ah, n, alpha):
    with ah.Solver(problem(n, alpha), tol=1e-10, restart=60, precond=0) as s:
        runs = [s.solve(want_q=True) for _ in range(6)]
    assert all(torch.equal(runs[0][0], k[0]) and torch.equal(runs[0][2], k[2]) for k in runs)
