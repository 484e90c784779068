"""Post-processing where an image is reduced by several workgroups: sizes that
fill no whole run, one run, and the most runs; the peak in the last run; ties."""

import numpy as np
import pytest
import torch

from oracle import post
from tests.conftest import rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(hv):
    c = hv.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("shape", [(16, 16), (17, 33), (64, 64), (91, 91), (100, 130), (384, 384), (371, 353)])
def test_mean(ctx, shape):
    # one rounding of the reciprocal mean, one of the product: 1.2e-7 a value
    x = np.random.default_rng(1).uniform(0.5, 2.0, (3, *shape)).astype(np.float32)
    got, _ = ctx.hv_postprocess(torch.from_numpy(x).cuda(), renormalise=True)
    assert rel_l2(got.cpu().numpy(), post.renormalise(x)) < 1.3e-7


@pytest.mark.parametrize("shape", [(64, 64), (64, 128), (320, 384), (800, 1280)])
def test_peak_in_every_part(ctx, shape):
    ny, nx = shape
    moves = [(0, 0), (0, nx - 1), (ny - 1, nx - 1), (ny // 2, 3), (ny - 2, 1), (1, 0)]
    rng = np.random.default_rng(4)
    base = rng.uniform(1, 2, shape)
    base[ny // 3: ny // 2, nx // 4: nx // 3] += 3.0
    x = np.stack([np.roll(base, m, axis=(0, 1)) for m in moves]).astype(np.float32)
    got, sh = ctx.hv_postprocess(torch.from_numpy(x).cuda(), ref_count=1, mask_radius=0.9)
    assert np.array_equal(sh.cpu().numpy(), np.array(moves, np.int32))
    for j in range(len(moves)):
        assert np.array_equal(got[j].cpu().numpy(), x[0])


def test_ties_take_the_lowest_index(ctx):
    x = torch.zeros((2, 128, 256), device="cuda")
    got, sh = ctx.hv_postprocess(x, ref_count=1)
    assert (sh == 0).all() and (got == 0).all()
