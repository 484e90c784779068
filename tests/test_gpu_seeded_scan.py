"""Scores of a scan over a hologram's own range, for candidate counts that fill
part of a workgroup's block of eight, whole blocks and one past, against the
oracle's FP64 scores at the same distances (1e-4, the bound of the other scan
tests: FP32 transforms of 64 x 64 and a variance that cancels to a tenth)."""

import numpy as np
import pytest

from oracle import autofocus as oaf
from synth.autofocus import af_hologram
from tests.conftest import rel_l2

pytestmark = pytest.mark.gpu
LAM, PITCH = 852e-9, 20e-6


@pytest.mark.parametrize("nc", [2, 7, 8, 17])
def test_scores_of_own_ranges(hv, nc):
    import torch
    ctx = hv.Context(0)
    zs = np.array([0.11, 0.27, 0.44])
    h = np.stack([af_hologram(z, 30 + i) for i, z in enumerate(zs)])
    lo = np.array([0.09, 0.2, 0.44], np.float32)
    hi = np.array([0.15, 0.3, 0.46], np.float32)
    _, sc = ctx.hv_af_scan_ranges(torch.from_numpy(h).cuda(), LAM, PITCH, torch.from_numpy(lo).cuda(),
                                  torch.from_numpy(hi).cuda(), nc, want_scores=True)
    sc = sc.cpu().numpy()
    for i in range(len(h)):
        zc = lo[i].astype(np.float64) + (hi[i].astype(np.float64) - lo[i]) * np.arange(nc) / (nc - 1)
        assert rel_l2(sc[i], oaf.scan_scores(h[i], LAM, PITCH, zc)) < 1e-4, i
    ctx.close()
