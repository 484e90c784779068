"""Calls of few frames, some of which take smaller tiles in the FP32 form, on both
sides of the frame counts where the tiles change, against the same call with more
frames: a frame's values are the same bits whatever its company, as the images of
a stream have to be."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,edge", [((64, 64), 512), ((128, 128), 256), ((256, 256), 32), ((128, 256), 64),
                                        ((256, 128), 64), ((64, 1024), 32), ((256, 64), 256)])
def test_frames_do_not_depend_on_their_number(hv, shape, edge):
    import torch
    ctx = hv.Context(0)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(0, 256, (2 * edge + 1, *shape), device="cuda", generator=g, dtype=torch.uint8)
    op = hv.Optics(852e-9, 20e-6, 19e-6, -0.2, hv.HV_AS)
    ctx.set_chunk_frames(4 * edge)
    whole = ctx.hv_propagate(x, op)
    tp = hv.Temporal(8, 8, 8.0, 1.0, 3.0)
    images = ctx.hv_stft_moments(x, op, tp)
    for n in (1, 8, edge - 1, edge, edge + 1):
        got = ctx.hv_propagate(x[:n].contiguous(), op)
        assert torch.equal(got, whole[:n]), n
        if n >= 8:
            m = ctx.hv_stft_moments(x[:n].contiguous(), op, tp)
            for a, b in zip(m, images):
                assert torch.equal(a, b[:a.shape[0]]), n
    ctx.close()
