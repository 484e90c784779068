"""Frames 800 high and 64 or 128 wide: 800 rows are no whole number of 64-row
tiles, which the narrow row passes use."""

import numpy as np
import pytest

from oracle import optics
from tests.conftest import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [64, 128])
@pytest.mark.parametrize("method", ["as", "fresnel"])
def test_every_row_is_transformed(hv, nx, method):
    import torch
    ctx = hv.Context(0)
    x = np.random.default_rng(nx).integers(0, 256, (2, 800, nx)).astype(np.uint8)
    want = (optics.angular_spectrum if method == "as" else optics.fresnel)(x.astype(float), 852e-9, 20e-6, 20e-6, -0.2)
    op = hv.Optics(852e-9, 20e-6, 20e-6, -0.2, hv.HV_AS if method == "as" else hv.HV_FRESNEL)
    got = ctx.hv_propagate(torch.from_numpy(x).cuda(), op).cpu().numpy()
    assert rel_l2(got, want) < 1e-5  # the FP32 form's tolerance
    ctx.close()
