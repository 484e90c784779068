"""Heights 320 and 384 under power-of-two widths: real frames, which go
through the packed row and column passes, against the same values as a complex
field, which take the complex ones.  Either is within a few 1e-7 of the exact
transform in FP32, so 2e-6 between them; the mixed form keeps one path, so its
frames are held to the field type's 2e-3."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [320, 384])
@pytest.mark.parametrize("nx", [64, 128, 256, 512, 1024])
def test_real_frames_match_complex_ones(hv, ny, nx):
    import torch
    ctx = hv.Context(0)
    g = torch.Generator(device="cuda").manual_seed(ny + nx)
    op = hv.Optics(852e-9, 20e-6, 17e-6, -0.21, hv.HV_AS)
    for n, hi, dtype in ((1, 256, torch.uint8), (9, 4096, torch.int16)):
        x = torch.randint(0, hi, (n, ny, nx), device="cuda", generator=g, dtype=torch.int32).to(dtype)
        want = ctx.hv_propagate(x.to(torch.float32).to(torch.complex64), op)
        got = ctx.hv_propagate(x, op)
        assert (got - want).norm() <= 2e-6 * want.norm(), (n, dtype)
        mixed = ctx.hv_propagate(x, op, hv.HV_PREC_MIXED)
        assert (mixed - want).norm() <= 2e-3 * want.norm(), (n, dtype)
    ctx.close()
