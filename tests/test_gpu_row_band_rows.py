"""The fused temporal and row transform with several rows to a workgroup (narrow
frames of enough windows) and with overlapping windows, whose workgroups are numbered
by rows of a die first, at every window length.  Reference: the field of
hv_propagate (held to the oracle elsewhere), transformed in time in float64.  1e-5 is the FP32
form's tolerance, 2e-3 the mixed form's."""

import numpy as np
import pytest

from oracle import temporal

pytestmark = pytest.mark.gpu


# 512 workgroups of 4 or 2 rows, or more: 128 x 4 windows, 256 x 2 (64 wide), 256 x 2 (128 wide)
@pytest.mark.parametrize("ny,nx,windows", [(512, 64, 5), (1024, 64, 2), (512, 128, 3), (320, 128, 4), (64, 256, 3),
                                           (64, 512, 3), (64, 1024, 3), (128, 384, 3)])
@pytest.mark.parametrize("w", [8, 16, 32, 64])
@pytest.mark.parametrize("overlap", [False, True])
def test_moments_and_bins(hv, ny, nx, windows, w, overlap):
    import torch
    ctx = hv.Context(0)
    stride = w // 2 + 1 if overlap else w
    n = (windows - 1) * stride + w
    x = np.random.default_rng(nx + ny + w).integers(0, 256, (n, ny, nx)).astype(np.uint8)
    xd = torch.from_numpy(x).cuda()
    op = hv.Optics(852e-9, 20e-6, 18e-6, -0.19, hv.HV_AS)
    ctx.set_chunk_frames(n)  # one launch of all windows
    u = ctx.hv_propagate(xd, op)
    lo, hi = 1, max(2, w // 4)  # few enough bins for the fused kernel under overlap
    tp = hv.Temporal(w, stride, float(w), float(lo), float(hi), False)
    bins, freqs = temporal.band_bins(w, float(w), lo, hi, False)
    f = torch.from_numpy(freqs).cuda()[:, None, None]
    k = torch.from_numpy(bins).cuda()
    for prec, tol in ((hv.HV_PREC_FP32, 1e-5), (hv.HV_PREC_MIXED, 2e-3)):
        ctx.set_timing(True)
        got = ctx.hv_stft_moments(xd, op, tp, prec)
        fused = ctx.kernel_time("rowinv_coef")[1]
        ctx.set_timing(False)
        assert fused == 1 or prec == hv.HV_PREC_MIXED or nx == 384 and w == 8
        spec = ctx.hv_stft_bins(xd, op, tp, prec)
        for j in range(windows):
            s = torch.fft.fft(u[j * stride:j * stride + w].to(torch.complex128), dim=0)[k]
            for m in range(3):
                want = (s.abs() ** 2 * f ** m).sum(dim=0)
                assert (got[m][j] - want).norm() <= tol * want.norm(), (prec, m, j)
            assert (spec[j] - s).norm() <= tol * s.norm(), (prec, j)
    ctx.close()
