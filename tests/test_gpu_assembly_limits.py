"""Meshes whose 32-bit offsets would wrap are refused on the host, before a kernel uses them.

More than 2^31 / 20 elements, or load faces, are refused from their counts alone (the arrays are
not read).  A mesh of 45 million nodes, each in five elements of nodes drawn at random, has rows
of 96 blocks and 4.3e9 blocks in all, more than 2^32: the 32-bit total has wrapped to a positive
number, and the exact one is what has to be tested.  A mesh just as dense and small is taken.
"""
import ctypes as C

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _assemble(gx, s, n_nodes, n_elems, conn, n_faces=0, faces=None):
    """gx_assemble of an unclamped mesh of one layer; returns the status."""
    import torch
    eng = np.array([[3500.0, 0, 0, 0, 0, 0, 0.3, 0, 0]])
    ang = np.zeros(1)
    xyz = torch.rand(3 * n_nodes, dtype=torch.float64, device="cuda")
    layer = torch.zeros(min(n_elems, len(conn) // 20), dtype=torch.int32, device="cuda")
    f = torch.zeros(3 * n_nodes, dtype=torch.float64, device="cuda")
    ps = gx.PlyStack(1, eng.ctypes.data_as(gx.f64p), ang.ctypes.data_as(gx.f64p))
    ms = gx.Mesh(n_nodes, n_elems, C.c_void_p(xyz.data_ptr()), C.c_void_p(conn.data_ptr()),
                 C.c_void_p(layer.data_ptr()), None, (C.c_double * 3)(0, 0, 0))
    fp = C.c_void_p(faces.data_ptr()) if faces is not None else None
    ld = gx.Loads(0, None, n_faces, fp, fp, gx.Traction())
    return gx.lib.gx_assemble(s.h, C.byref(ms), C.byref(ps), C.byref(ld),
                              C.c_void_p(f.data_ptr()))


def _error(gx, s):
    return gx.lib.gx_last_error(s.h).decode()


@pytest.mark.parametrize("extra", [1, 2 ** 27])
def test_counts_beyond_the_offsets_are_refused(extra):
    import torch
    import paper_1707_04228_amd as gx
    s = gx.Solver()
    conn = torch.arange(20, dtype=torch.int32, device="cuda")
    limit = (2 ** 31 - 1) // 20
    assert _assemble(gx, s, 20, limit + extra, conn) == gx.GX_EINVAL
    assert _error(gx, s) == "too many elements"
    assert _assemble(gx, s, 20, 1, conn, limit + extra, conn) == gx.GX_EINVAL
    assert _error(gx, s) == "too many load faces"
    s.laminate(workloads.small_flat(nx=3, ny=3))     # the context goes on
    s.assemble()
    s.close()


def test_block_total_beyond_32_bits_is_refused():
    import torch
    import paper_1707_04228_amd as gx
    s = gx.Solver()
    g = torch.Generator(device="cuda").manual_seed(7)
    for N, code in ((45_000_000, gx.GX_EINVAL), (2_000, None)):
        conn = torch.empty(5 * N, dtype=torch.int32, device="cuda")
        for k in range(5):                         # every node once per pass of N / 20 elements
            conn[k * N:(k + 1) * N] = torch.randperm(N, generator=g, device="cuda",
                                                     dtype=torch.int64).to(torch.int32)
        torch.cuda.synchronize()
        got = _assemble(gx, s, N, N // 4, conn)
        if code is not None:
            assert got == code and _error(gx, s) == "matrix too large"
        else:                                      # (random nodes: its elements are inside out)
            assert _error(gx, s) == "non-positive Jacobian determinant in an element"
        del conn
    s.close()
