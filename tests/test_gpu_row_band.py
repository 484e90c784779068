"""Moments and bins of the angular-spectrum path from the fused temporal and row
transform, at every frame width and window length, for bands that fill its LDS to
every degree and bands that do not fit it (the field path), with overlapping
windows.  Reference: the field of hv_propagate (held to the oracle elsewhere),
transformed in time in float64.  1e-5 is the FP32 form's tolerance, 2e-3 the
mixed form's."""

import numpy as np
import pytest

from oracle import temporal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [64, 128, 256, 320, 384, 512, 800, 1024, 1280])
@pytest.mark.parametrize("w", [8, 16, 32, 64])
def test_moments_and_bins(hv, nx, w):
    import torch
    ny = 128 if nx == 64 else 64
    ctx = hv.Context(0)
    stride = w // 2 - 1 if nx % 128 else w
    n = w + 2 * stride + 1
    x = np.random.default_rng(nx + w).integers(0, 256, (n, ny, nx)).astype(np.uint8)
    xd = torch.from_numpy(x).cuda()
    op = hv.Optics(852e-9, 20e-6, 18e-6, -0.19, hv.HV_AS)
    u = ctx.hv_propagate(xd, op).to(torch.complex128)
    for lo, hi, sym in ((1, 1, False), (1, w // 2 - 1, False), (0, w // 2, True)):
        tp = hv.Temporal(w, stride, float(w), float(lo), float(hi), sym)
        bins, freqs = temporal.band_bins(w, float(w), lo, hi, sym)
        f = torch.from_numpy(freqs).cuda()[:, None, None]
        s = torch.stack([torch.fft.fft(u[j * stride:j * stride + w], dim=0)[torch.from_numpy(bins).cuda()]
                         for j in range(3)])
        for prec, tol in ((hv.HV_PREC_FP32, 1e-5), (hv.HV_PREC_MIXED, 2e-3)):
            got = ctx.hv_stft_moments(xd, op, tp, prec)
            for k in range(3):
                want = (s.abs() ** 2 * f ** k).sum(dim=1)
                for j in range(3):
                    assert (got[k][j] - want[j]).norm() <= tol * want[j].norm(), (lo, hi, prec, k, j)
            spec = ctx.hv_stft_bins(xd, op, tp, prec)
            assert (spec - s).norm() <= tol * s.norm(), (lo, hi, prec)
            only = ctx.hv_stft_moments(xd, op, tp, prec, want=(False, True, False))
            assert torch.equal(only[1], got[1])
    ctx.close()
