"""The FP64 Jacobi solver behind hv_pca, on fields in memory, against LAPACK on
the covariance the same call returns, for every window length: full-rank
windows, windows with repeated and zero eigenvalues, and an exact tie.

Tolerance: a rotation step rounds each entry by a few eps of the matrix norm;
(W - 1) steps times at most 16 sweeps times 4 eps is 9e-13 of the largest
eigenvalue at W = 64."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 9e-13


def _field(kind, w, seed):
    rng = np.random.default_rng(seed)
    p = 64 * 64
    x = rng.standard_normal((w, p)) + 1j * rng.standard_normal((w, p))
    if kind == "static":  # one dominant component over noise
        x = x + 40.0 * (rng.standard_normal(p) + 1j * rng.standard_normal(p))[None, :]
    elif kind == "rank2":  # two components, the others zero: W - 2 repeated eigenvalues
        x = x[:1] * np.exp(0.3j * np.arange(w))[:, None] + 0.5 * x[1:2] * np.exp(-1.1j * np.arange(w))[:, None]
    elif kind == "diagonal":  # disjoint supports: the covariance is diagonal, in ascending order
        m = np.zeros((w, p), bool)
        for t in range(w):
            m[t, t * (p // w):t * (p // w) + p // w] = True
        x = np.where(m, 1.0 + np.arange(w)[:, None], 0.0).astype(complex)
    elif kind == "ties":  # equal frame energies on disjoint supports: every eigenvalue equal
        m = np.zeros((w, p), bool)
        for t in range(w):
            m[t, t * (p // w):t * (p // w) + p // w] = True
        x = m.astype(complex)
    elif kind == "zero":
        x = np.zeros((w, p), complex)
    return x.reshape(w, 64, 64).astype(np.complex64)


@pytest.mark.parametrize("w", [16, 32, 64])
@pytest.mark.parametrize("kind", ["noise", "static", "rank2", "diagonal", "ties", "zero"])
def test_eigenpairs(w, kind):
    import torch

    from paper_2508_03911_amd import hv
    ctx = hv.Context(0)
    x = np.concatenate([_field(kind, w, s) for s in (1, 2, 3)])
    xd = torch.from_numpy(x).cuda()
    r = ctx.hv_pca(xd, None, w, w, 0, w - 1, want_cov=True)
    ev, cov = (r[k].cpu().numpy() for k in ("eigvals", "cov"))
    assert (r["offdiag"].cpu().numpy() < 1e-14).all()
    for j in range(3):
        c = cov[j]
        assert np.array_equal(c, c.conj().T)
        lam = np.linalg.eigvalsh(c)[::-1]
        assert np.abs(ev[j] - lam).max() <= TOL * max(lam[0], 0.0)
        assert (np.diff(ev[j]) <= 0).all()
    ctx.close()
