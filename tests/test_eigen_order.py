"""The order in which the eigensolver takes its Ritz values is a permutation whatever they are.

Values of a basis that lost rank may be NaN; every place of the order has to be given out all
the same, because the places index the vectors.  The ranking function is compiled for the host
from paper_1707_04228_amd/csrc/geneo.hip.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HIP = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1707_04228_amd", "csrc", "geneo.hip")


@pytest.fixture(scope="module")
def rank(tmp_path_factory):
    src = open(HIP).read()
    i = src.index("__device__ inline int rank_down(")
    fn = src[i:src.index("\n}", i) + 2].replace("__device__ inline", 'extern "C"')
    d = tmp_path_factory.mktemp("rank")
    (d / "r.cpp").write_text(fn)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(d / "r.so"), str(d / "r.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(d / "r.so"))
    return lambda v: [lib.rank_down(v.ctypes.data_as(ctypes.c_void_p), len(v), t)
                      for t in range(len(v))]


def test_ranks_are_a_permutation(rank):
    rng = np.random.default_rng(3)
    for _ in range(300):
        v = rng.choice([1.0, 2.0, 2.0, 0.0, -0.0, -3.0, np.nan, np.inf, -np.inf], rng.integers(1, 40))
        r = rank(v)
        assert sorted(r) == list(range(len(v)))
        w = np.empty(len(v))
        w[r] = v
        real = w[: int((v == v).sum())]
        assert (real == real).all() and (real[:-1] >= real[1:]).all()
        for x in set(real):                               # ties: the lower index first
            same = [r[i] for i in range(len(v)) if v[i] == x]
            assert same == sorted(same)
