"""Band matrices where there is no room for the rows that two parts store twice.

A matrix of order n = 3 B is stored in two parts of 2 B rows each, a third more than whole.  With
so much of the device's memory held that only the whole matrix fits, the factorisation and the
solve still have to be done: against b = A x for a chosen x (diagonally dominant, kappa < 3:
1e-12 of the largest entry).  The held memory leaves 100 MB beyond the whole matrix.
"""
import pytest

pytestmark = pytest.mark.gpu


def _system(n, B):
    """A = 4 I - 1 on the sub- and superdiagonals 1 and B, x and b = A x."""
    import torch
    band = torch.zeros((n, B + 1), dtype=torch.float64, device="cuda")
    band[:, B] = 5.0
    band[1:, B - 1] = -1.0
    band[B:, 0] = -1.0
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.rand(n, dtype=torch.float64, device="cuda", generator=g)
    b = 5.0 * x
    for d in (1, B):
        b[d:] -= x[:-d]
        b[:-d] -= x[d:]
    return band.reshape(-1), x, b


def test_whole_matrix_where_two_parts_do_not_fit():
    import torch
    import paper_1707_04228_amd as gx
    n, B = 36000, 12000
    whole = 8 * n * (B + 16)                       # bytes of the matrix, band rounded up
    band, x, b = _system(n, B)
    s = gx.Solver()
    # (before any memory is held: what the device allocates for the kernels themselves)
    small = _system(400, 20)
    torch.cuda.synchronize()                       # (the solver has a stream of its own)
    s.band_factor_solve([400], [20], small[0], small[2])
    torch.cuda.empty_cache()
    held = torch.empty(torch.cuda.mem_get_info()[0] - whole - 100_000_000, dtype=torch.uint8,
                       device="cuda")
    got = s.band_factor_solve([n], [B], band, b)
    del held
    torch.cuda.empty_cache()
    assert (got - x).abs().max() <= 1e-12 * x.abs().max()
    s.close()


def test_set_up_where_two_parts_do_not_fit():
    """Three elements through the thickness: subdomain matrices of about three bandwidths.  The
    memory left holds both sets of factors whole and a quarter of what two parts add."""
    import numpy as np
    import torch
    import paper_1707_04228_amd as gx
    import workloads
    cfg = workloads.small_flat(nx=30, ny=26, length=30.0, width=26.0,
                               layers=workloads.ply_layers([0, 90], 0.25, 1, 0.05, 1))
    runs, whole, extra = [], 0, 0
    for hold in (False, True):
        s = gx.Solver()
        s.laminate(cfg)
        f = s.assemble()
        part = s.partition(cfg, 2, 1)
        held = None
        if hold:
            # a request that cannot be met empties the library's cache of released blocks
            band = torch.zeros(8_000_000 * 101, dtype=torch.float64, device="cuda")
            x = torch.zeros(8_000_000, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            torch.cuda.empty_cache()
            full = torch.empty(torch.cuda.mem_get_info()[0] - 300_000_000, dtype=torch.uint8,
                               device="cuda")
            with pytest.raises(gx.GxError, match="GX_ENOMEM"):
                s.band_factor_solve([8_000_000], [100], band, x)
            del full, band, x
            torch.cuda.empty_cache()
            held = torch.empty(torch.cuda.mem_get_info()[0] - whole - extra // 4,
                               dtype=torch.uint8, device="cuda")
        nev, n0 = s.geneo_setup(part, 2, overlap=1, nev=6)
        out = s.pcg(f, rtol=1e-10, maxit=200)
        runs.append((list(nev), n0, out["iters"], out["x"].cpu().numpy()))
        if not hold:
            stats = np.zeros(5, dtype=np.int64)
            gx.lib.gx_stats(s.h, stats.ctypes.data_as(gx.i64p))
            ni, nn, hb = s.subdomain_info()
            assert all(n >= 3 * b for n, b in zip(ni, hb))
            whole = 8 * int(stats[2] + stats[3])
            extra = 2 * 8 * int(sum(b * b for b in hb))
            print("whole", whole, "extra", extra, ni, nn, hb, flush=True)
        del held, f, part, out
        s.close()
        torch.cuda.empty_cache()
    (nev, n0, it, x), (nev2, n02, it2, x2) = runs
    assert nev == nev2 and n0 == n02 and abs(it - it2) <= 1
    assert np.abs(x - x2).max() <= 1e-8 * np.abs(x).max()


def test_whole_matrix_where_the_scratch_of_two_parts_does_not_fit():
    """The factors of both parts fit (the storage with its padding, the inverse blocks), the
    scratch of a solve with 16 right-hand sides does not: 25 MB, 8 MB are left."""
    import torch
    import paper_1707_04228_amd as gx
    n, B, m = 36000, 12000, 16
    band, x, b = _system(n, B)
    rhs = b[:, None] * torch.arange(1.0, m + 1, dtype=torch.float64, device="cuda")
    s = gx.Solver()
    small = _system(400, 20)
    torch.cuda.synchronize()                       # (the solver has a stream of its own)
    s.band_factor_solve([400], [20], small[0], small[2])
    # a request that cannot be met empties the library's cache of released blocks
    full = torch.empty(20_000_000_000, dtype=torch.float64, device="cuda")
    y = torch.zeros(40_000_000, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with pytest.raises(gx.GxError, match="GX_ENOMEM"):
        s.band_factor_solve([40_000_000], [499], full, y)
    del full, y
    torch.cuda.empty_cache()
    sep = n - (n - B) // 64 * 64
    two = 8 * ((n + sep + 128) * (B + 1) + 1024) + 8 * 64 * n + 8_000_000
    held = []                                      # (the device counts late what was given back)
    while len(held) < 8 and torch.cuda.mem_get_info()[0] > two + 4_000_000:
        held.append(torch.empty(torch.cuda.mem_get_info()[0] - two, dtype=torch.uint8,
                                device="cuda"))
    assert torch.cuda.mem_get_info()[0] <= two + 4_000_000
    got = s.band_factor_solve([n], [B], band, rhs.reshape(-1)).reshape(n, m)
    del held
    torch.cuda.empty_cache()
    ref = x[:, None] * torch.arange(1.0, m + 1, dtype=torch.float64, device="cuda")
    assert (got - ref).abs().max() <= 1e-12 * ref.abs().max()
    s.close()
