"""Workspaces of a call whose second and last chunk is a smaller one: the second stream
holds that chunk's frames, not a full chunk's.  Chunks of 256 x 256 FP32 frames hold 128
frames of 1.5 complex64 values per pixel (786,432 bytes a frame); the tables take 2 MiB
at most."""

import pytest

pytestmark = pytest.mark.gpu


def test_second_stream_holds_its_own_chunk(hv):
    import torch
    x = torch.randint(0, 256, (160, 256, 256), device="cuda", dtype=torch.uint8)
    op = hv.Optics(852e-9, 20e-6, 20e-6, -0.2, hv.HV_AS)
    ctx = hv.Context(0)
    ctx.hv_stft_moments(x, op, hv.Temporal(32, 32, 32.0, 2.0, 15.0))
    assert ctx.workspace_bytes() <= 160 * 786432 + (2 << 20)
    ctx.close()
