"""GPU parity of the band solver on sets that fill the device, on both sides of the rule that
keeps their matrices whole.

With a work-group per compute unit a set of 256 matrices has one group each, and its matrices
are stored in two parts up to a bandwidth of 1,500 bytes (187 entries in FP64, 375 in FP32) and
whole from there on; one wide matrix keeps the others whole too.  Against a chosen x, with the
tolerances of the other band tests (1e-10 of the largest entry in FP64, kappa < 1e3: diagonally
dominant; 1e-4 with FP32 factors).
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,B,wide", [("fp64", 187, 0), ("fp64", 188, 0), ("fp64", 40, 188),
                                              ("mixed", 375, 0), ("mixed", 376, 0)])
@pytest.mark.parametrize("nrhs", [1, 16])
def test_sets_that_fill_the_device(precision, B, wide, nrhs):
    import torch
    import paper_1707_04228_amd as gx
    g = torch.Generator(device="cuda").manual_seed(B + nrhs)
    shapes = [(256, 3 * B + 70, B)] if not wide else [(255, 3 * B + 300, B), (1, 3 * wide + 9, wide)]
    bands, xs, rhs, n_all, B_all = [], [], [], [], []
    for m, n, b in shapes:
        band = 2.0 * torch.rand((m, n, b + 1), dtype=torch.float64, device="cuda", generator=g) - 1.0
        band[:, :, b] += 2.0 * b + 2.0
        x = torch.rand((m, n, nrhs), dtype=torch.float64, device="cuda", generator=g)
        y = band[:, :, b, None] * x
        for d in range(1, b + 1):
            v = band[:, d:, b - d, None]
            y[:, d:] += v * x[:, :-d]
            y[:, :-d] += v * x[:, d:]
        bands.append(band.reshape(-1))
        xs.append(x.reshape(-1))
        rhs.append(y.reshape(-1))
        n_all += [n] * m
        B_all += [b] * m
    band, x, b = torch.cat(bands), torch.cat(xs), torch.cat(rhs)
    s = gx.Solver()
    torch.cuda.synchronize()                       # (the solver has a stream of its own)
    got = s.band_factor_solve(n_all, B_all, band, b,
                              precision=gx.GX_FP64 if precision == "fp64" else gx.GX_MIXED)
    assert (got - x).abs().max() <= (1e-10 if precision == "fp64" else 1e-4) * x.abs().max()
    s.close()
