"""GPU parity of the element kernels over element counts that do not fill their work-groups.

The element matrices take four elements per work-group, the stress kernels eight (two per
wavefront), with elements outside the region or the selected layers between the others.
Parts of 1 to 75 elements: K through its product with a random vector (1e-13 of its largest
entry, as for the assembled matrix), the delamination criterion at every Gauss point and J
for a random displacement (1e-11: sums of at most 81 products of strains of one size, formed in
another order).  A NaN in one element's displacement stays with the elements that use it.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_K_with_identity

pytestmark = pytest.mark.gpu

LAYERS = [{"mat": "ply", "t": 0.25, "nel": 1, "angle": 30.0},
          {"mat": "resin", "t": 0.05, "nel": 1, "angle": 0.0},
          {"mat": "ply", "t": 0.25, "nel": 3, "angle": -60.0}]


def _parts():
    one = [dict(LAYERS[1])]
    out = [workloads.small_flat(nx=1, ny=1, layers=one, length=1.0, width=1.0),
           workloads.small_flat(nx=3, ny=1, layers=one, length=3.0, width=1.0),
           workloads.small_flat(nx=3, ny=3, layers=one, length=3.0, width=3.0),
           workloads.small_flat(nx=5, ny=3, layers=LAYERS, length=5.0, width=3.0),
           workloads.small_lsection(nx=7, ny=1, layers=LAYERS)]
    return out


@pytest.mark.parametrize("cfg", _parts(), ids=lambda c: f"{c['geometry']}{c['nx']}x{c['ny']}")
def test_element_kernels(cfg):
    import torch
    import paper_1707_04228_amd as gx
    from oracle import adjoint, failure, fem
    s = gx.Solver()
    s.laminate(cfg)
    s.assemble()
    prob = fem.Problem(cfg)
    rng = np.random.default_rng(cfg["nx"])
    x = rng.standard_normal(prob.mesh.n_dofs)
    y = s.spmv(torch.tensor(x, device="cuda")).cpu().numpy()
    ref = oracle_K_with_identity(prob) @ x
    assert np.abs(y - ref).max() <= 1e-13 * np.abs(ref).max()
    u = 1e-3 * rng.standard_normal(prob.mesh.n_dofs)
    ut = torch.tensor(u, device="cuda")
    resin = [k for k, L in enumerate(cfg["layers"]) if L["mat"] == "resin"]
    sel = np.nonzero(np.isin(prob.mesh.elayer, resin))[0]
    F = np.zeros((prob.mesh.n_elems, 27))
    F[sel] = failure.camanho(failure.local_stresses(prob.mesh, u, sel))
    r = s.failure(ut, per_gauss=True)
    got = r["F_gauss"].cpu().numpy().reshape(-1, 27)
    assert np.abs(got - F).max() <= 1e-11 * F.max()
    assert r["F_max"] == got.max() and (r["elem"], r["gauss"]) == divmod(int(got.argmax()), 27)
    assert np.array_equal(r["F_elem"].cpu().numpy(), got.max(axis=1))
    J, Jo = s.objective(ut), adjoint.objective(prob.mesh, u)
    assert abs(J - Jo) <= 1e-11 * abs(Jo)
    if len(sel) > 1:                               # a NaN at one selected element's own node
        own = np.setdiff1d(prob.mesh.conn[sel[-1]], np.delete(prob.mesh.conn, sel[-1], axis=0))
        if own.size:
            u[3 * own[0]] = np.nan
            bad = s.failure(torch.tensor(u, device="cuda"), per_gauss=True)
            g = bad["F_gauss"].cpu().numpy().reshape(-1, 27)
            keep = np.arange(len(g)) != sel[-1]
            assert np.array_equal(g[keep], got[keep]) and np.isnan(g[sel[-1]]).any()
            assert bad["F_max"] == got[keep].max()
    s.close()
