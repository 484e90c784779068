"""The row pass of real frames on calls that take its smaller tiles, against the same
frames in a call that takes the full ones, for every width that has both, tall and
low frames and both storage forms: the same bits."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [128, 256, 512, 1024])
@pytest.mark.parametrize("ny", [64, 320, 1024])
def test_small_tiles_give_the_same_bits(hv, nx, ny):
    import torch
    ctx = hv.Context(0)
    rows = min(64, 16384 // nx)
    edge = -(-256 * rows // ny)  # frames that fill 256 tiles
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    for dtype, top in ((torch.uint8, 256), (torch.int16, 4096)):
        x = torch.randint(0, top, (edge, ny, nx), device="cuda", generator=g, dtype=dtype)
        op = hv.Optics(852e-9, 20e-6, 19e-6, -0.2, hv.HV_AS)
        ctx.set_chunk_frames(edge)
        for prec in (hv.HV_PREC_FP32, hv.HV_PREC_MIXED):
            whole = ctx.hv_propagate(x, op, prec)
            for n in {1, edge // 2, edge - 1} - {0}:
                assert torch.equal(ctx.hv_propagate(x[:n].contiguous(), op, prec), whole[:n]), (dtype, prec, n)
    ctx.close()
