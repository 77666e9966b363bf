"""The temporal layers in one pass against normalisation, im2col, product, bias
and ReLU one after the other. An image of a pixel count that is no multiple of
64 takes the latter alone and the former in a batch whose pixel count is one;
the sums are the same, so the logits are too, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2403_16438_amd.surrogate import Surrogate, he_init

pytestmark = pytest.mark.gpu


# one wave's 64 pixels over several images; several workgroups; more tiles than the launch has waves
@pytest.mark.parametrize("B,H,W", [(4, 4, 4), (4, 12, 12), (8, 20, 36), (8, 132, 132)])
def test_batched_equals_single(B, H, W):
    assert (H * W) % 64 and (B * H * W) % 64 == 0
    rng = np.random.default_rng(B * H + W)
    frames = rng.poisson(600.0, size=(B, 50, H, W)).astype(np.uint16)
    frames[0, 20:30, : H // 2] += 300
    frames[-1, :, 0, 0] = 65535
    frames[-1, :, 1, 1] = 0
    fd = torch.from_numpy(frames.view(np.int16)).cuda()
    labels = torch.zeros((B, H, W), dtype=torch.float32, device="cuda")
    labels[:, H // 4:H // 2] = 1
    theta = he_init(5)
    theta += (0.01 * rng.standard_normal(theta.size)).astype(np.float32)
    net = Surrogate(B, H, W, theta)
    net.backward(fd, labels)
    got = net.logits().clone().reshape(B, H, W)
    net.close()
    one = Surrogate(1, H, W, theta)
    for b in range(B):
        one.backward(fd[b:b + 1].contiguous(), labels[b:b + 1].contiguous())
        ref = one.logits().reshape(H, W)
        torch.cuda.synchronize()
        assert torch.equal(got[b], ref), (b, (got[b] - ref).abs().max().item())
    one.close()
