"""Solves with links between neighbouring blocks against solves without.

With one work-group to a part (groups=1) a one-right-hand-side solve takes a block's inverse and
its off-diagonal block one after the other, sums in FP64; with several it takes their product,
formed beforehand.  On the same factors, in either precision, the two differ by FP64 rounding
alone: the five-point Laplacian on a strip, shifted to a condition number of 8e4, so
8e4 x 1.1e-16 per rounding, and some hundred of them meet in an entry: 1e-9.  (Products kept in
FP32 are off by 1e-6 here.)
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w", [(4000, 40), (12000, 100)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_links_round_as_the_blocks_do(n, w, precision):
    import torch
    import paper_1707_04228_amd as gx
    band = np.zeros((n, w + 1))
    band[:, w] = 4.0 + 1e-4
    band[1:, w - 1] = -1.0
    band[w:, 0] = -1.0
    b = np.random.default_rng(n).standard_normal(n)
    s = gx.Solver()
    x = []
    for groups in (0, 1):
        g = torch.tensor(b, device="cuda")
        s.band_factor_solve([n], [w], torch.tensor(band.ravel(), device="cuda"), g,
                            precision=gx.GX_FP64 if precision == "fp64" else gx.GX_MIXED,
                            groups=groups)
        x.append(g.cpu().numpy())
    s.close()
    assert np.linalg.norm(x[0] - x[1]) <= 1e-9 * np.linalg.norm(x[1])
