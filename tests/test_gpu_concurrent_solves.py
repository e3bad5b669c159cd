"""Band solves of several contexts at once, each on a thread and a stream of its own.

Every launch has as many work-groups as stay resident when it runs alone, and its groups wait
for each other; launches of other contexts hold slots meanwhile.  All solves have to end, with
the solution of a lone solve up to the grouping of its sums (1e-10 of the largest entry, FP64,
diagonally dominant matrices).
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("contexts,nrhs", [(2, 1), (4, 1), (4, 32)])
def test_contexts_on_threads(contexts, nrhs):
    import torch
    import paper_1707_04228_amd as gx
    n, B, n_mat = 2304, 300, 3
    g = torch.Generator().manual_seed(3)
    band = torch.rand((n_mat * n, B + 1), generator=g, dtype=torch.float64) - 0.5
    band[:, B] = 2.0 * B
    rows = torch.arange(B)[:, None] - B + torch.arange(B + 1)[None, :] < 0
    for j in range(n_mat):
        band[j * n: j * n + B][rows] = 0
    band = band.reshape(-1).cuda()
    b = torch.rand(n_mat * n * nrhs, generator=g, dtype=torch.float64).cuda()
    one = gx.Solver(stream=torch.cuda.Stream())
    ref = one.band_factor_solve([n] * n_mat, [B] * n_mat, band, b.clone()).cpu().numpy()
    one.close()
    torch.cuda.synchronize()
    worst, errors = [0.0] * contexts, []

    def work(k):
        try:
            s = gx.Solver(stream=torch.cuda.Stream())
            for _ in range(12):
                x = b.clone()
                torch.cuda.synchronize()
                got = s.band_factor_solve([n] * n_mat, [B] * n_mat, band, x).cpu().numpy()
                worst[k] = max(worst[k], float(np.abs(got - ref).max()))
            s.close()
        except Exception as e:                      # reported by the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(contexts)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert max(worst) <= 1e-10 * np.abs(ref).max()
