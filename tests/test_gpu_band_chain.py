"""GPU parity of the band factorisation's group of four 64-column panels.

Unsplit matrices (order below 384 or below three bandwidths) around the edges of the 16-column
blocks, the 64-row blocks and the 256-column groups, with bandwidths that leave blocks of a
group empty, against SciPy's banded Cholesky (1e-10 of the largest entry in FP64, kappa < 1e3:
diagonally dominant; 1e-4 with FP32 factors); a non-positive pivot in every position that one
of the stages could miss is reported.
"""
import numpy as np
import pytest
import scipy.linalg as sla

pytestmark = pytest.mark.gpu

SHAPES = [(1, 0), (15, 3), (16, 15), (17, 5), (63, 62), (64, 63), (65, 64), (80, 79), (128, 16),
          (191, 64), (192, 127), (255, 80), (256, 255), (257, 128), (257, 15), (320, 144),
          (383, 200), (512, 208), (513, 300), (700, 260)]


@pytest.fixture(scope="module")
def solver():
    import paper_1707_04228_amd as gx
    s = gx.Solver()
    yield gx, s
    s.close()


def _band(n, B, rng):
    """Diagonally dominant: row-major band storage and LAPACK's lower form."""
    lo = np.zeros((B + 1, n))
    total = np.zeros(n)
    for d in range(1, B + 1):
        lo[d, : n - d] = rng.uniform(-1.0, 1.0, n - d)
        total[: n - d] += np.abs(lo[d, : n - d])
        total[d:] += np.abs(lo[d, : n - d])
    lo[0] = total + rng.uniform(1.0, 2.0, n)
    band = np.zeros((n, B + 1))
    for d in range(B + 1):
        band[d:, B - d] = lo[d, : n - d]
    return band, lo


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_group_edges(solver, precision):
    import torch
    gx, s = solver
    rng = np.random.default_rng(5)
    mats = [_band(n, B, rng) for n, B in SHAPES]
    xs = [rng.standard_normal((n, 8)) for n, _ in SHAPES]
    x_t = torch.tensor(np.concatenate([x.ravel() for x in xs]), device="cuda")
    s.band_factor_solve([n for n, _ in SHAPES], [B for _, B in SHAPES],
                        torch.tensor(np.concatenate([m[0].ravel() for m in mats]), device="cuda"),
                        x_t, precision=gx.GX_FP64 if precision == "fp64" else gx.GX_MIXED)
    got, o = x_t.cpu().numpy(), 0
    tol = 1e-10 if precision == "fp64" else 1e-4
    for (n, B), (_, lo), x in zip(SHAPES, mats, xs):
        ref = sla.cho_solve_banded((sla.cholesky_banded(lo, lower=True), True), x)
        g = got[o: o + 8 * n].reshape(n, 8)
        o += 8 * n
        assert np.abs(g - ref).max() <= tol * np.abs(ref).max(), (n, B)


@pytest.mark.parametrize("pivot", [0, 15, 16, 47, 63, 64, 130, 255, 256, 299])
def test_non_positive_pivot(solver, pivot):
    import torch
    gx, s = solver
    rng = np.random.default_rng(pivot)
    n, B = 300, 140
    band, _ = _band(n, B, rng)
    band[pivot, B] = -band[pivot, B]
    with pytest.raises(gx.GxError, match="non-positive pivot"):
        s.band_factor_solve([n], [B], torch.tensor(band.ravel(), device="cuda"),
                            torch.ones(8 * n, dtype=torch.float64, device="cuda"))
