"""The eigenvectors of the FP64 Jacobi solver, through the images that use them, on
full-rank windows and on repeated, tied and zero eigenvalues: V is unitary, so the
energies of the single components add up to the pixel's whole energy, as do those
of two complementary ranges, and component c carries the energy lambda_c.

Tolerance, u = 2^-24: a component is a sum of W products in four partial sums of W / 4
(or, over a wide range, one chain of 2 W products in the matrix cores), off by at
most (W / 4 + 3) u |x| with the rounding of V; its energy by twice that times |y|, and
the sum over components by 2 (W / 4 + 3) sqrt(W) u |x|^2, four times that for the
chain.  lambda is that of a covariance summed in single precision, whose entries'
tolerance elsewhere is 1e-6 of the largest."""

import numpy as np
import pytest

from tests.test_gpu_eigensolver import _field

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("w", [16, 32, 64])
@pytest.mark.parametrize("kind", ["noise", "static", "rank2", "diagonal", "ties", "zero"])
def test_components_add_up(hv, w, kind):
    import torch
    ctx = hv.Context(0)
    x = np.concatenate([_field(kind, w, s) for s in (1, 2)])
    xd = torch.from_numpy(x).cuda()
    e = (xd.to(torch.complex128).abs() ** 2).reshape(2, w, 64, 64).sum(dim=1)
    each = 2 * (w / 4 + 3) * U
    total = torch.zeros_like(e)
    for c in range(w):
        r = ctx.hv_pca(xd, None, w, w, c, c)
        m = r["m0"].double()
        total += m
        lam, trace = r["eigvals"].clamp(min=0), e.sum(dim=(1, 2))
        tol = each * (lam[:, c] * trace).sqrt() + each ** 2 * trace + 1e-6 * lam[:, 0]
        assert ((m.sum(dim=(1, 2)) - lam[:, c]).abs() <= tol).all(), c
    assert ((total - e).abs() <= each * w ** 0.5 * e).all()
    for k in {0, 1, w // 4, w // 2, w - 2}:  # few kept, few left out and neither
        two = ctx.hv_pca(xd, None, w, w, 0, k)["m0"].double() + ctx.hv_pca(xd, None, w, w, k + 1, w - 1)["m0"].double()
        assert ((two - e).abs() <= 4 * each * w ** 0.5 * e).all(), k
    ctx.close()
