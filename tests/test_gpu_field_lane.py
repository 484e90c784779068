"""The lane-per-pixel temporal kernel on fields in memory, against float64:
moments, band bins, the energy of component ranges and the SSA filter, on both
sides of the rules that choose between taking components out, summing them and
the coefficient GEMM.

The references of PCA and SSA use the eigenvectors of the covariance that the
GPU itself returns, so only the single-precision image arithmetic is compared;
1e-5 is the FP32 form's tolerance."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-5
NY = NX = 64


def _field(w, seed):
    """[2w][64][64] with well separated components over a dominant one."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(2):
        a = rng.standard_normal((w, NY * NX)) + 1j * rng.standard_normal((w, NY * NX))
        q, _ = np.linalg.qr(rng.standard_normal((w, w)) + 1j * rng.standard_normal((w, w)))
        s = np.linspace(2.0, 1.0, w)
        s[0] = 30.0
        out.append(q @ (s[:, None] * a))
    return np.concatenate(out).reshape(2 * w, NY, NX).astype(np.complex64)


def _rel(got, want):
    got, want = np.asarray(got.cpu(), np.complex128), np.asarray(want)
    return np.linalg.norm(got - want) / np.linalg.norm(want)


@pytest.mark.parametrize("w", [8, 16, 32, 64])
@pytest.mark.parametrize("band", ["one", "dc", "half", "symmetric"])
@pytest.mark.parametrize("prec", [0, 1])
def test_moments_and_bins(w, band, prec):
    import torch

    from oracle import temporal
    from paper_2508_03911_amd import hv
    lo, hi, sym = {"one": (2, 2, False), "dc": (0, 1, True), "half": (1, w // 2, False),
                   "symmetric": (1, w // 2, True)}[band]
    ctx = hv.Context(0)
    x = _field(w, 3)
    xd = torch.from_numpy(x).cuda()
    tp = hv.Temporal(w, w // 2, float(w), float(lo), float(hi), sym)
    bins, freqs = temporal.band_bins(w, float(w), lo, hi, sym)
    s = temporal.stft(x, w, w // 2)
    want = temporal.moments(s, bins, freqs)
    got = ctx.hv_stft_moments(xd, None, tp, prec)
    for g, r in zip(got, want):
        if np.linalg.norm(r) > 0:
            assert _rel(g, r) <= TOL
    assert _rel(ctx.hv_stft_bins(xd, None, tp, prec), s[:, bins]) <= TOL
    only = ctx.hv_stft_moments(xd, None, tp, prec, want=(False, False, True))
    assert torch.equal(only[2], got[2])
    ctx.close()


def _ranges(w):
    """Component ranges on both sides of the rules (12 kept, 6 and 8 left out)."""
    return [(0, 0), (1, w - 1), (0, w - 1), (2, w - 3), (3, w - 4), (3, w - 5), (4, w - 5), (4, w - 6),
            (w - 1, w - 1), (0, 7), (0, 11), (0, 12), (w - 8, w - 1)]


@pytest.mark.parametrize("w", [16, 32, 64])
def test_component_ranges(w):
    import torch

    from paper_2508_03911_amd import hv
    ctx = hv.Context(0)
    x = _field(w, 5)
    xd = torch.from_numpy(x).cuda()
    tp = hv.Temporal(w, w, float(w), 1.0, float(w // 2 - 1))
    bins, freqs = hv.band_bins(tp)
    for lo, hi in _ranges(w):
        r = ctx.hv_pca(xd, None, w, w, lo, hi, want_cov=True)
        m = ctx.hv_ssa_moments(xd, None, tp, lo, hi)
        for j in range(2):
            _, v = np.linalg.eigh(r["cov"][j].cpu().numpy())
            vs = v[:, ::-1][:, lo:hi + 1]
            y = x[j * w:(j + 1) * w].astype(np.complex128).reshape(w, -1).T @ vs  # [P, kept]
            assert _rel(r["m0"][j].reshape(-1), (np.abs(y) ** 2).sum(axis=1)) <= TOL, (lo, hi)
            s = np.fft.fft((y @ vs.conj().T).T, axis=0)[bins]
            for n in range(3):
                want = (np.abs(s) ** 2 * (np.array(freqs) ** n)[:, None]).sum(axis=0)
                assert _rel(m[f"m{n}"][j].reshape(-1), want) <= TOL, (lo, hi, n)
    ctx.close()
