"""An explicit tile of the transform passes (options.tile_fp64, tile_fp32) is taken by the passes per
axis, also where an automatic handle would run a whole plane or a whole small grid in one launch, and
one that no pass can take is refused there too."""
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


def problem(n):
    shape = tuple(m + 1 for m in reversed(n))
    return W.Problem(n, (0.0,) * len(n), tuple(m / max(n) for m in n), np.ones(shape), np.zeros(shape))


GRIDS = [(32, 32), (64, 64), (48, 40), (32, 32, 32), (64, 64, 64), (48, 36, 40), (128, 96, 64)]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("tile,code", [(3, "INVALID"), (1024, "UNSUPPORTED")])
def test_impossible_tiles_are_refused(ah, n, prec, tile, code):
    g = torch.zeros([m - 1 for m in reversed(n)], dtype=torch.float64, device="cuda")
    with ah.Solver(problem(n), precision=ah.FP64 if prec == "fp64" else ah.MIXED, tile_fp64=tile, tile_fp32=tile) as s:
        with pytest.raises(ah.AhocError) as e:
            s.poisson(g)
    assert e.value.code == {"INVALID": -1, "UNSUPPORTED": -5}[code]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_tiles_are_taken(ah, n, prec):
    pb = problem(n)
    g = np.random.default_rng(2).standard_normal([m - 1 for m in reversed(n)])
    ref = fast.FastTier(pb).poisson(g)
    with ah.Solver(pb, precision=ah.FP64 if prec == "fp64" else ah.MIXED, tile_fp64=8, tile_fp32=8) as s:
        s.profile(True)
        w = s.poisson(torch.from_numpy(g).cuda()).cpu().numpy()
        kt = s.kernel_times()
    assert kt["dst_rows"][1] == 2 and kt["dst_fused"][1] == 1 and kt["dst_strided"][1] == (2 if len(n) == 3 else 0)
    assert np.abs(w - ref).max() <= (1e-12 if prec == "fp64" else 1e-5) * np.abs(ref).max()
