"""The row and column passes at every frame side, on few frames, so that the
last group of workgroups is partial and waves hold from a fraction of a
sequence to eight of them: every side once as the width and once as the height,
against the oracle.  1e-5 is the FP32 form's tolerance, 2e-3 the mixed form's."""

import numpy as np
import pytest

from oracle import optics
from tests.conftest import rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1280), (1280, 64), (128, 800), (800, 128), (256, 320), (320, 256), (384, 512), (512, 384),
          (1024, 64), (64, 1024), (320, 320), (64, 64)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("method", ["as", "fresnel", "fresnel+"])
def test_few_frames(hv, shape, method):
    import torch
    ny, nx = shape
    ctx = hv.Context(0)
    lam, dx, dy = 852e-9, 20e-6, 17e-6
    z = 0.21 if method == "fresnel+" else -0.21
    op = hv.Optics(lam, dx, dy, z, hv.HV_AS if method == "as" else hv.HV_FRESNEL)
    rng = np.random.default_rng(nx + 3 * ny)
    for n, dtype in ((1, np.uint8), (3, np.uint16)):
        x = rng.integers(0, 256 if dtype == np.uint8 else 4096, (n, ny, nx)).astype(dtype)
        want = (optics.angular_spectrum if method == "as" else optics.fresnel)(x.astype(float), lam, dx, dy, z)
        xd = torch.from_numpy(x if dtype == np.uint8 else x.view(np.int16)).cuda()
        for prec, tol in ((hv.HV_PREC_FP32, 1e-5), (hv.HV_PREC_MIXED, 2e-3)):
            got = ctx.hv_propagate(xd, op, prec)
            for j in range(n):
                assert rel_l2(got[j].cpu().numpy(), want[j]) < tol
        c = torch.from_numpy(x.astype(np.complex64)).cuda()
        assert rel_l2(ctx.hv_propagate(c, op).cpu().numpy(), want) < 1e-5
    ctx.close()
