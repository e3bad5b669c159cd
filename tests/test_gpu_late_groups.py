"""Solves whose groups do not all come in time: the result is the same bit for bit.

The groups that share a matrix wait for each other only so long; then those present solve it.
Contexts that are told that no more than k groups of each part come (gx_tune, param 2) have to
return the bytes that contexts with all of them return: for the band solver's edge shapes with
one and several right-hand sides in both precisions, and for the solutions of a batch, whose
subdomain solves go in one launch.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

SHAPES = [(384, 127), (385, 1), (448, 0), (705, 235), (1000, 333), (2049, 640), (1600, 63),
          (383, 20), (3000, 90), (5000, 300)]


def results(present):
    import torch
    import paper_1707_04228_amd as gx
    out = {}
    rng = np.random.default_rng(11)
    bands = []
    for n, B in SHAPES:
        band = rng.uniform(-1.0, 1.0, (n, B + 1))
        for r in range(min(B, n)):
            band[r, :B - r] = 0.0
        band[:, B] = 2.0 * B + rng.uniform(1.0, 2.0, n)
        bands.append(band.ravel())
    band = torch.tensor(np.concatenate(bands), device="cuda")
    s = gx.Solver()
    s.tune(2, present)
    for name, prec in (("fp64", gx.GX_FP64), ("mixed", gx.GX_MIXED)):
        for nrhs in (1, 16):
            x = torch.tensor(rng.standard_normal(nrhs * sum(n for n, _ in SHAPES)), device="cuda")
            s.band_factor_solve([n for n, _ in SHAPES], [B for _, B in SHAPES], band, x,
                                precision=prec)
            out[f"{name}{nrhs}"] = x.cpu().numpy()
    s.close()
    cfgs = []
    for k in range(3):
        cfg = workloads.small_lsection(nx=36, ny=2, amp=0.05 * k, wlen=6.0)
        cfg["solver"].update(px=2, py=1)
        cfgs.append(cfg)
    for name, prec in (("fp64", gx.GX_FP64), ("mixed", gx.GX_MIXED)):
        b = gx.Batch(cfgs, precision=prec)
        for ctx in b.solvers:
            ctx.tune(2, present)
        b.setup(concurrent=1)
        xs, it, _, st = b.solve(rtol=1e-10, maxit=500)
        assert np.all(st == gx.GX_OK)
        out[f"batch_{name}"] = np.concatenate([x.cpu().numpy() for x in xs])
        out[f"iters_{name}"] = np.asarray(it)
        b.close()
    return out


@pytest.mark.parametrize("present", [1, 3])
def test_late_groups_change_no_bit(present):
    ref, late = results(0), results(present)
    for key, v in ref.items():
        assert late[key].tobytes() == v.tobytes(), key
