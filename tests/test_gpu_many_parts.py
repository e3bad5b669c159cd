"""A batch of more than 65,535 parts: 33 strips of 1,024 narrow subdomains, each matrix in two
parts, within the 65,535 matrices that a joint solve takes.

Two iterations of the lockstep PCG give what each context's own two give (the same sums in
another distribution over work-groups: FP64 rounding, 1e-10 of the largest entry).
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_more_parts_than_a_grid_has_rows():
    import torch
    import paper_1707_04228_amd as gx
    cfg = workloads.small_flat(nx=1024, ny=1, length=1024.0, width=1.0,
                               layers=[{"mat": "ply", "t": 12.0, "nel": 12, "angle": 20.0}])
    cfg["solver"].update(px=1024, py=1, nev=1)
    b = gx.Batch([cfg] * 33)
    b.setup()
    ni, _, hb = b.solvers[0].subdomain_info()
    split = sum(n >= max(3 * w, 6 * 64) for n, w in zip(ni, hb))
    print("matrices", len(ni), "of two parts", split, "orders", min(ni), max(ni), "widths", max(hb))
    assert 33 * (len(ni) + split) > 65535 and 33 * len(ni) <= 65535
    assert 8 * max(hb) <= 1400                             # (wider ones are kept whole)
    xs, its, _, st = b.solve(rtol=1e-8, maxit=2)
    assert all(s == gx.GX_ENOCONV for s in st) and all(i == 2 for i in its)
    torch.cuda.synchronize()
    s = b.solvers[0]
    own = s.pcg(b.f[0], rtol=1e-8, maxit=2, allow_noconv=True)["x"]
    torch.cuda.synchronize()
    for x in (xs[0], xs[32]):
        assert (x - own).abs().max() <= 1e-10 * own.abs().max()
    b.close()
