"""Device memory of a handle: arrays that only make passes faster are taken where they do, last of
all, and are done without where the allocator has no room for them.  Bars of the parity and batch
tests (solutions of two solves to 1e-11 within 1e-9)."""
import ctypes

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


class Budget:
    """An allocator over PyTorch's that records the sizes asked for and refuses beyond `limit`."""

    def __init__(self, ah, limit=None):
        self.held, self.sizes, self.refused = {}, [], 0

        def alloc(nbytes, ctx):
            if limit is not None and sum(self.held.values()) + nbytes > limit:
                self.refused += 1
                return None
            p = ah._TORCH_ALLOC(nbytes, 1)
            self.held[p] = nbytes
            self.sizes.append(nbytes)
            return p

        def free(p, ctx):
            if p:
                self.held.pop(p)
                ah._TORCH_FREE(p, 1)

        self.arg = ah._Allocator(ah._ALLOC_FN(alloc), ah._FREE_FN(free), ctypes.c_void_p(1))


def problem(n):
    u = "sin(pi*x)**2*sin(pi*y)**2*exp(x + y)" if len(n) == 2 else "sin(pi*x)**2*sin(pi*y)**2*sin(pi*z)**2*exp(x)"
    a = "1 + 0.5*sin(2*pi*x)*cos(2*pi*y)" if len(n) == 2 else W.C3_ALPHA
    return W.manufactured(a, u, n, (0.0,) * len(n), tuple(m / max(n) for m in n))



@pytest.mark.parametrize("n", [(150, 140, 130), (130, 66, 132)])
def test_no_array_beyond_source_v_and_u(ah, n):
    """Grids whose passes fill the chip from one array to the same: no second work array."""
    rows = (n[0] - 1 + 31) // 32 * 32
    size = 8 * rows * (n[1] - 1) * (n[2] - 1)
    b = Budget(ah)
    p = problem(n)
    p.gD = None  # without its source: M f, V and U
    with ah.Solver(p, allocator=b.arg):
        assert b.sizes.count(size) == 3, b.sizes
    assert not b.held


# a second work array for rows of few pencils and for the planes of a 3-D grid; faces as sine products
@pytest.mark.parametrize("n", [(500, 300), (130, 128), (2500, 40), (100, 90, 75), (64, 64, 64)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_setup_fits_without_the_optional_arrays(ah, n, prec):
    p = problem(n)
    mode = ah.FP64 if prec == "fp64" else ah.MIXED
    g = np.random.default_rng(1).standard_normal([m - 1 for m in reversed(n)])
    ref = fast.FastTier(p).poisson(g)
    free = Budget(ah)
    with ah.Solver(p, precision=mode, allocator=free.arg, tol=1e-11) as s:
        u, q = s.solve()[0].clone(), torch.randn(s.nq, dtype=torch.float64, device="cuda")
        y, z = s.schur_apply(q).clone(), s.precond_apply(q).clone()
    total = sum(free.sizes)
    rows = (n[0] - 1 + 31) // 32 * 32
    size = (8 if prec == "fp64" else 4) * rows * int(np.prod([m - 1 for m in n[1:]]))
    tight = Budget(ah, total - size)  # no room for one interior array of the operator's precision
    with ah.Solver(p, precision=mode, allocator=tight.arg, tol=1e-11) as s:
        assert tight.refused >= 1
        w = s.poisson(torch.from_numpy(g).cuda()).cpu().numpy()
        u2, _, _, st = s.solve()
        y2, z2 = s.schur_apply(q), s.precond_apply(q)
    assert np.abs(w - ref).max() <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(ref).max()
    assert st.converged
    assert float((u - u2).abs().max()) <= 1e-9 * float(u.abs().max())
    assert float((y - y2).abs().max()) <= (1e-11 if prec == "fp64" else 1e-4) * float(y.abs().max())
    assert float((z - z2).abs().max()) <= 1e-11 * float(z.abs().max())
    assert not tight.held and not free.held
