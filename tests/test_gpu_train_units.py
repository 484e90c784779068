"""Training batches whose tiles outnumber the workgroups, so that a workgroup
walks several of them, against the same samples one at a time (which the oracle
tests cover): the forward bits of a sample do not depend on its company, and the
gradient is the mean of the samples' to FP32 summation, sqrt(4096) 2^-24 of the
terms' norms on either side (1e-5 together)."""

import numpy as np
import pytest

from oracle import autofocus as oaf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [31, 32, 33, 65, 100])
def test_batch_gradient_is_the_mean_of_its_samples(hv, b):
    import torch
    ctx = hv.Context(0)
    rng = np.random.default_rng(b)
    x = torch.from_numpy(rng.standard_normal((b, 64, 64)).astype(np.float16)).cuda()
    z = torch.from_numpy(rng.uniform(0.05, 0.5, b).astype(np.float32)).cuda()
    m = ctx.af_model(oaf.init_params(11).astype(np.float32), b, 0.275, 0.13)
    out = m.forward(x).clone()
    loss, grad = m.loss_grad(x, z)
    loss, grad = loss.item(), grad.double().cpu()
    losses, mean, norm = [], torch.zeros_like(grad), 0.0
    for i in range(b):
        assert torch.equal(m.forward(x[i:i + 1].contiguous())[0], out[i]), i
        li, gi = m.loss_grad(x[i:i + 1].contiguous(), z[i:i + 1].contiguous())
        losses.append(li.item())
        gi = gi.double().cpu()
        mean += gi / b
        norm += gi.norm().item() / b
    assert abs(loss - np.mean(losses)) <= 1e-5 * np.mean(np.abs(losses))
    assert (grad - mean).norm().item() <= 1e-5 * norm
    m.close()
    ctx.close()
