"""GPU parity of the band solver where matrices are eliminated from both ends in two parts.

A matrix of order n >= 3 bw (and six 64-row blocks) is split around a separator of at least
one bandwidth; the orders here lie on both sides of that rule, leave separators that are and
are not whole blocks, and mix split and unsplit matrices in one launch, with every
right-hand-side path (one, several, column panels), forced group counts up to the largest,
and more work-groups than the device holds at a time (the two parts of a matrix wait for
each other).  Reference and tolerances as for the unsplit solver: SciPy's banded Cholesky,
1e-10 of the largest entry in FP64 (kappa < 1e3: diagonally dominant), 1e-4 with FP32
factors.
"""
import numpy as np
import pytest
import scipy.linalg as sla

pytestmark = pytest.mark.gpu

EDGES = [(383, 20), (384, 127), (384, 128), (384, 129), (385, 1), (448, 0), (639, 192),
         (705, 235), (704, 235), (1000, 333), (1000, 17), (2049, 640), (1600, 63), (130, 5)]


@pytest.fixture(scope="module")
def solver():
    import paper_1707_04228_amd as gx
    s = gx.Solver()
    yield gx, s
    s.close()


def _matrix(n, B, rng):
    """Diagonally dominant band matrix: row-major band storage and LAPACK's lower form."""
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
    return band.ravel(), lo


def _check(solver, shapes, nrhs, precision, groups):
    import torch
    gx, s = solver
    rng = np.random.default_rng(nrhs + 17 * groups + len(shapes))
    mats = [_matrix(n, B, rng) for n, B in shapes]
    xs = [rng.standard_normal((n, nrhs)) for n, _ in shapes]
    x_t = torch.tensor(np.concatenate([x.ravel() for x in xs]), device="cuda")
    s.band_factor_solve([n for n, _ in shapes], [B for _, B in shapes],
                        torch.tensor(np.concatenate([m[0] for m in mats]), device="cuda"), x_t,
                        precision=gx.GX_FP64 if precision == "fp64" else gx.GX_MIXED,
                        groups=groups)
    got, o = x_t.cpu().numpy(), 0
    tol = 1e-10 if precision == "fp64" else 1e-4
    for (n, B), (_, lo), x in zip(shapes, mats, xs):
        ref = sla.cho_solve_banded((sla.cholesky_banded(lo, lower=True), True), x)
        g = got[o: o + n * nrhs].reshape(n, nrhs)
        o += n * nrhs
        assert np.abs(g - ref).max() <= tol * np.abs(ref).max(), (n, B)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nrhs", [1, 8, 32, 40])
@pytest.mark.parametrize("groups", [0, 1, 2, 8])
def test_split_edges(solver, precision, nrhs, groups):
    _check(solver, EDGES, nrhs, precision, groups)


@pytest.mark.parametrize("nrhs", [1, 16])
def test_more_parts_than_fit_at_once(solver, nrhs):
    _check(solver, [(400 + k % 7, 20 + k % 11) for k in range(300)], nrhs, "fp64", 0)
