"""The gathering of a matrix's work-groups before a solve, restated on the host.

The groups of a matrix wait for each other's blocks.  A launch hands its places out in a list,
a matrix's places next to each other, so a launch that has the device to itself always
completes the first matrix of its list.  Two launches that start together (contexts on threads
of their own, joint solves of two batches) can each hold some of an XCD's slots with a matrix
that is not complete: without the gathering they then wait for each other until the poll limit.
Checked here for one XCD, over interleavings of the launches' starts: with the gathering every
launch ends and no matrix is left out or taken up by fewer groups than it has parts; without it
two launches whose matrices want most of the slots stop.
"""
import os
import random

import pytest

SLOTS = 32                                     # work-groups resident on an XCD
HIP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1707_04228_amd", "csrc", "band.hip")


def run(launches, gathers, rng):
    """launches: per launch the list of (parts, groups per part) of its matrices.  Returns
    (True if all ended, per matrix the number of groups per part that solved it)."""
    queue = [[(k, m) for m, (np_, G) in enumerate(ms) for _ in range(np_ * G)]
             for k, ms in enumerate(launches)]
    arrived = {}                               # (launch, matrix): work-groups gathered
    settled = {}                               # the same: groups per part that take part
    running = []
    while any(queue) or running:
        while len(running) < SLOTS and any(queue):
            k = rng.choice([i for i, q in enumerate(queue) if q])
            w = queue[k].pop(0)
            if w in settled:                   # late: leaves
                continue
            running.append(w)
            arrived[w] = arrived.get(w, 0) + 1
            np_, G = launches[w[0]][w[1]]
            if np_ == 1 and G == 1 or arrived[w] == np_ * G:
                settled[w] = G
        if not running:                        # (only latecomers were left)
            continue
        done = [w for w in running if w in settled]
        if not done and gathers:               # the wait of the longest waiting has passed
            w = next((w for w in running if arrived[w] >= launches[w[0]][w[1]][0] and
                      launches[w[0]][w[1]][1] > 1), None)
            if w:
                settled[w] = arrived[w] // launches[w[0]][w[1]][0]
                done = [v for v in running if v == w]
        if not done:
            return False, settled
        running = [w for w in running if w not in done]
    return True, settled


@pytest.mark.parametrize("n_launch", [1, 2, 3, 4])
def test_every_launch_ends(n_launch):
    rng = random.Random(n_launch)
    for _ in range(300):
        launches = [[(rng.choice([1, 2]), rng.choice([1, 2, 3, 8, 15, 16]))
                     for _ in range(rng.randint(1, 6))] for _ in range(n_launch)]
        ended, settled = run(launches, True, rng)
        assert ended
        for k, ms in enumerate(launches):
            for m, (_, G) in enumerate(ms):
                assert 1 <= settled[k, m] <= G
        if n_launch == 1:                      # alone: every matrix has all its groups
            assert all(settled[0, m] == G for m, (_, G) in enumerate(launches[0]))


def test_without_it_two_launches_stop():
    rng = random.Random(1)
    launches = [[(2, 16)], [(2, 16)]]
    ends = [run(launches, False, rng)[0] for _ in range(50)]
    assert not all(ends)
    assert all(run([[(2, 16)] * 3], False, rng)[0] for _ in range(50))


def test_every_solve_kernel_gathers():
    """All kernels whose work-groups wait for one another and take their places in a list."""
    src = open(HIP).read()
    place = src[src.index("inline Place set_place("):]
    assert "gather(" in place[:place.index("\n}")]
    for name in ("k_band_solve_1", "k_band_solve_1_multi", "k_band_solve_m"):
        at = src.index(f" {name}(\n") if f" {name}(\n" in src else src.index(f" {name}(")
        body = src[at:src.index("\n}", at)]
        assert "set_place(" in body or "gather(" in body, name
