"""The temporal layers in one pass against normalisation, im2col, product, bias
and ReLU one after the other. An image of a pixel count that is no multiple of
64 takes the latter alone and the former in a batch whose pixel count is one;
the sums are the same, so the logits are too, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2403_16438_amd.surrogate import Surrogate, he_init, param_layout

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


@pytest.mark.parametrize("H,W", [(4, 4), (12, 12), (20, 36)])
def test_gradients_of_copies(H, W):
    """One segment, whose pixel count is no multiple of 32, takes the products,
    the gather and the mask passes of the temporal input gradients; 16 copies
    take the one kernel. The loss is a mean, so the gradients agree up to the
    FP32 order of the sums over pixels (at most 2,048 terms in groups of 16,
    each rounding by 2^-24 of a partial sum): below 1e-4 norm-wise."""
    assert (H * W) % 32
    rng = np.random.default_rng(H * 40 + W)
    frames = rng.poisson(1000, size=(1, 50, H, W)).astype(np.uint16)
    frames[:, 20:23, 1:3, 1:3] += 250
    labels = np.zeros((1, H, W), np.float32)
    labels[:, 1:3, 1:3] = 1
    theta = he_init(9)
    got = []
    for B in (1, 16):
        net = Surrogate(B, H, W, theta)
        _, g = net.backward(torch.from_numpy(np.repeat(frames, B, 0).view(np.int16)).cuda(),
                            torch.from_numpy(np.repeat(labels, B, 0)).cuda(), want_grad=True)
        got.append(g.cpu().numpy().astype(np.float64))
        net.close()
    for name, r, c, wo, bo in param_layout():
        sl = slice(wo, bo + (r // 4 if name in ("u2", "u1") else r))
        assert np.linalg.norm(got[1][sl] - got[0][sl]) <= 1e-4 * np.linalg.norm(got[0][sl]), name
