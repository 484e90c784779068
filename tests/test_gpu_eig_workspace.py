"""Device memory of the PCA path over small frames with a short stride: a call of
few windows holds scratch for those windows alone, and the eigensolver's rotation
log is bounded, its windows taken a part at a time.  A window's outputs are the
same bits in a call of its own.

Bounds: a call of one window of 64 frames of 64 x 64 needs three complex64 fields
(6.3 MB), a rotation log of 40 sweeps of 63 * 32 rotations of 24 bytes (1.9 MB) and
some 0.5 MB of covariances, vectors and tables.  2048 frames need 201 MB of fields,
at most 1 GiB of log, and per window 4 W^2 floats of partial sums, W^2 complex128
of covariance and of vectors and W^2 complex64 of vectors (56 W^2 bytes)."""

import pytest

pytestmark = pytest.mark.gpu


def _frames(n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    return torch.randint(0, 256, (n, 64, 64), device="cuda", generator=g, dtype=torch.uint8)


def test_one_window(hv):
    ctx = hv.Context(0)
    op = hv.Optics(852e-9, 20e-6, 20e-6, -0.2, hv.HV_AS)
    ctx.hv_pca(_frames(64), op, 64, 1, 1)
    assert ctx.workspace_bytes() < 12 << 20
    ctx.close()


@pytest.mark.parametrize("w", [32, 64])
def test_many_windows(hv, w):
    import torch
    n = 2048
    x = _frames(n)
    op = hv.Optics(852e-9, 20e-6, 20e-6, -0.2, hv.HV_AS)
    ctx = hv.Context(0)
    r = ctx.hv_pca(x, op, w, 1, 1)
    nwin = n - w + 1
    assert ctx.workspace_bytes() < 3 * n * 4096 * 8 + (1 << 30) + nwin * 56 * w * w + (8 << 20)
    part = (1 << 30) // (40 * (w - 1) * (w // 2) * 24)  # windows of a full log, about
    for j in {0, part // 2, part - 1, part, part + 1, 2 * part, nwin - 1} & set(range(nwin)):
        one = ctx.hv_pca(x[j:j + w].contiguous(), op, w, 1, 1)
        for k in ("m0", "eigvals"):
            assert torch.equal(one[k][0], r[k][j]), (j, k)
    ctx.close()


def test_no_double_precision_vectors_where_none_are_read(hv):
    """A range that leaves few components out reads the single-precision vectors
    only: 40 W^2 bytes a window."""
    n, w = 2048, 64
    ctx = hv.Context(0)
    ctx.hv_pca(_frames(n), hv.Optics(852e-9, 20e-6, 20e-6, -0.2, hv.HV_AS), w, 1, 1)
    assert ctx.workspace_bytes() < 3 * n * 4096 * 8 + (1 << 30) + (n - w + 1) * 40 * w * w + (8 << 20)
    ctx.close()
