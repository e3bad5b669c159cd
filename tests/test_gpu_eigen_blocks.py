"""GPU parity of the eigensolver's block kernels over every block width.

A fixed number of modes gives a block of that many columns plus eight guard vectors, rounded
up to eight: 16 to 48 columns, one to three 16-column tiles of the matrix instruction, full
and half-filled last tiles, with row counts that are not multiples of a chunk.  Eigenvalues
and the two-level P r against the oracle with the tolerances of the other GenEO parity tests
(1e-8 relative plus 1e-10 absolute at a backward error of 1e-12; 1e-8 for P r).  Six modes at
least: a floating subdomain has six zero eigenvalues, and fewer would not be a unique span.
"""
import numpy as np
import pytest

import workloads
from gpu_helpers import rel_err
from test_gpu_schwarz import _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nev", [6, 8, 9, 16, 24, 25, 33, 40])
def test_block_widths(nev):
    import torch
    import paper_1707_04228_amd as gx
    from oracle import pcg
    cfg = workloads.small_flat(nx=13, ny=3, length=13.0, width=3.0)
    cfg["name"] = f"blocks_{nev}"
    cfg["solver"].update(px=3, py=1, overlap=1, nev=nev)
    R = pcg.solve(cfg, rtol=1e-8, maxit=1)
    prob, co = R["prob"], R["coarse"]
    s, _, _ = _setup(gx, cfg, coarse=True, eig_tol=1e-12)
    assert list(s.nev) == co.nev
    for j in range(len(co.nev)):
        lg, lo = s.eigenvalues(j), co.lams[j]
        assert np.all(np.abs(lg - lo) <= 1e-8 * np.abs(lo) + 1e-10), (j, lg, lo)
    r = np.random.default_rng(nev).standard_normal(prob.n)
    z = s.precond(torch.tensor(prob.to_full(r), device="cuda")).cpu().numpy()
    assert rel_err(z[prob.free], R["P"].apply(r)) <= 1e-8
