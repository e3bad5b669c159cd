"""The autotuner weighs the library's own choice of work-groups too.

The automatic choice goes up to 16 work-groups, more than gx_tune takes, so a tuner that only
tried fixed counts left the solves slower than they were untuned.
"""
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_autotuned_solves_are_no_slower_than_untuned():
    import paper_1707_04228_amd as gx
    cfg = workloads.small_lsection(nx=60, ny=4)
    cfg["solver"].update(px=2, py=1)
    batch = gx.Batch([cfg])
    batch.setup()
    s = batch.solvers[0]
    untuned = min(s.kernel_time(1, reps=20)[0] for _ in range(3))
    times = s.autotune(reps=20)
    assert 0 in times                                      # the automatic choice
    tuned = min(s.kernel_time(1, reps=20)[0] for _ in range(3))
    assert tuned <= 1.3 * untuned, (untuned, times)
    batch.close()
