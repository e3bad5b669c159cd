"""Joint solves of several batches at once, each batch on a thread of its own.

A batch's subdomain solves go in one launch that is sized for the whole device, and the groups
of a matrix wait for each other; the launches of another batch hold slots meanwhile.  Few
matrices per batch, so that one wants most of an XCD's slots.  Every system has to converge, in
the iterations of the batch alone (within one) and to its solution (1e-9 relative: the tolerance
of the other batch tests, for solutions of two runs to a residual of 1e-10).
"""
import threading

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batches_on_threads(precision):
    import torch
    import paper_1707_04228_amd as gx
    prec = gx.GX_FP64 if precision == "fp64" else gx.GX_MIXED
    cfgs = []
    for k in range(4):
        cfg = workloads.small_lsection(nx=24, ny=2, amp=0.05 * k, wlen=6.0)
        cfg["solver"].update(px=2, py=1)
        cfgs.append(cfg)
    batches, ref = [], []
    for _ in range(2):
        b = gx.Batch(cfgs, precision=prec)
        b.setup()
        xs, it, _, st = b.solve(rtol=1e-10, maxit=500)
        assert np.all(st == gx.GX_OK)
        ref.append(([x.cpu().numpy() for x in xs], it))
        batches.append(b)
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            for _ in range(5):
                xs, it, _, st = batches[k].solve(rtol=1e-10, maxit=500)
                assert np.all(st == gx.GX_OK), st
                assert np.all(np.abs(it - ref[k][1]) <= 1), (it, ref[k][1])
                for x, r in zip(xs, ref[k][0]):
                    assert np.abs(x.cpu().numpy() - r).max() <= 1e-9 * np.abs(r).max()
        except BaseException as e:                  # reported by the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for b in batches:
        b.close()
    assert not errors, errors
