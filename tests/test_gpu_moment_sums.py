"""The rounding of the sum over a band's bins: moments against the float64 sums of the
powers of the bins that hv_stft_bins returns, from the kernel of a field in memory and
from the fused temporal and row kernel, for every number of bins up to the whole window.

Tolerance, rms over an image, u = 2^-24: an addition rounds its result by at most u,
u / sqrt(3) rms at the worst mantissa.  Over four partial sums of nb / 4 equal terms
the results are k / nb of the total, k = 2 .. nb / 4 in each, then 1/2, 1/2 and 1:
sum of squares 4 (nb / 4)^3 / 3 / nb^2 + 1.5 = nb / 48 + 1.5.  Random terms and a last
partial sum that is short add to the roundings of a power (two, over the square root of
nb bins) and of the scale (one): (nb / 48 + 1.5 + 2 / nb + 1) u^2 / 3 with half as much again for the
spread of the terms.  A single chain of nb additions has nb / 3 in place of nb / 48
+ 1.5."""

import math

import pytest

pytestmark = pytest.mark.gpu


def _check(ctx, x, op, w, lo, hi, sym, hv):
    import torch
    tp = hv.Temporal(w, w, float(w), float(lo), float(hi), sym)
    nb = len(hv.band_bins(tp)[0])
    p = ctx.hv_stft_bins(x, op, tp).to(torch.complex128)
    want = (p.real ** 2 + p.imag ** 2).sum(dim=1)
    got = ctx.hv_stft_moments(x, op, tp)[0].double()
    rms = (((got - want) / want) ** 2).mean().sqrt().item()
    tol = 2.0 ** -24 * math.sqrt(1.5 * (nb / 48 + 2 / nb + 2.5) / 3)
    print(f"w={w} nb={nb} rms {rms:.2e} tol {tol:.2e}", flush=True)
    assert rms <= tol


@pytest.mark.parametrize("w,lo,hi,sym", [(8, 1, 4, False), (32, 2, 15, False), (32, 0, 16, True), (64, 2, 31, False),
                                         (64, 0, 32, True), (64, 5, 5, False)])
def test_sums_over_bins(hv, w, lo, hi, sym):
    import torch
    ctx = hv.Context(0)
    g = torch.Generator(device="cuda").manual_seed(w + hi)
    x = torch.complex(*(torch.randn(2 * w, 64, 128, device="cuda", generator=g) for _ in range(2)))
    _check(ctx, x, None, w, lo, hi, sym, hv)  # a field in memory
    x = torch.randint(0, 256, (2 * w, 64, 128), device="cuda", generator=g, dtype=torch.uint8)
    _check(ctx, x, hv.Optics(852e-9, 20e-6, 18e-6, -0.2, hv.HV_AS), w, lo, hi, sym, hv)  # the fused kernel
    ctx.close()
