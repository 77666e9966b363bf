"""Gradients of both networks at the shapes where the direct backward kernels
change: column blocks of 8 to 64 and a ragged 72, images lower than a tile,
pixel ranges shorter than a step and of one step's length, samples of the
temporal gather shorter than a step, and batches large enough for two pixel
blocks per wave.

The reference rounds where the kernels round, so what separates them are BF16
roundings on either side of a boundary: one in 2^-9 of an operand, with random
signs over the ten layers that a gradient passes, is below 2e-2 norm-wise; a
bound of 5e-2 leaves room for the few-pixel layers, where an indexing or
padding mistake gives 0.3 and more."""
import numpy as np
import pytest
import torch

from oracle import nn_ref, unet_st
from paper_2403_16438_amd import surrogate, unet

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
BF16 = nn_ref.Numerics(bf16=True)


def _rounded(theta, layout):
    t = theta.astype(np.float64).copy()
    for name, r, c, wo, bo in layout:
        t[wo:wo + r * c] = nn_ref.bf16_round(theta[wo:wo + r * c])
    return t


def _check(g, rg, layout):
    errs = {}
    for name, r, c, wo, bo in layout:
        sl = slice(wo, bo + (r // 4 if name in ("u2", "u1") else r))
        errs[name] = np.linalg.norm(g[sl] - rg[sl]) / max(np.linalg.norm(rg[sl]), 1e-30)
    print({k: f"{v:.1e}" for k, v in errs.items()})
    assert max(errs.values()) <= 5e-2, errs


def _summaries(B, H, W, seed):
    rng = np.random.default_rng(seed)
    st = np.stack([rng.uniform(800, 1200, (B, H, W)), rng.uniform(0, 60, (B, H, W))], axis=1).astype(np.float32)
    st[:, 1, 2:6, 3:8] += 180
    labels = np.zeros((B, H, W), np.float32)
    labels[:, 2:6, 3:8] = 1
    return st, labels


@pytest.mark.parametrize("B,H,W", [(1, 8, 8), (3, 8, 32), (2, 12, 64), (1, 8, 72), (2, 16, 128), (4, 36, 32)])
def test_summary_network(B, H, W):
    st, labels = _summaries(B, H, W, B * 1000 + H * W)
    theta = unet.he_init(6)
    net = unet.SummaryUNet(B, H, W, theta)
    _, g = net.backward(torch.from_numpy(st).to(DEV), torch.from_numpy(labels).to(DEV), want_grad=True)
    layout = unet.param_layout()
    _, rg = unet_st.loss_and_grad(_rounded(theta, layout), st.astype(np.float64), labels, BF16)
    _check(g.cpu().numpy().astype(np.float64), rg, layout)
    net.close()


def test_copies_of_a_patch():
    """The loss is a mean over the batch, so 16 copies of a patch have the
    gradient of one: every value inside is 1/16 (a power of two) of the single
    patch's with the same roundings, and only the FP32 order of the sums over
    pixels differs. Those have at most 2,048 terms per range in groups of 16,
    each rounding by 2^-24 of a partial sum, below 1e-4 norm-wise also where
    most of a sum cancels. The large batch takes two pixel blocks per wave."""
    st, labels = _summaries(1, 64, 64, 9)
    theta = unet.he_init(8)
    got = []
    for B in (1, 16):
        net = unet.SummaryUNet(B, 64, 64, theta)
        _, g = net.backward(torch.from_numpy(np.repeat(st, B, 0)).to(DEV),
                            torch.from_numpy(np.repeat(labels, B, 0)).to(DEV), want_grad=True)
        got.append(g.cpu().numpy().astype(np.float64))
        net.close()
    for name, r, c, wo, bo in unet.param_layout():
        sl = slice(wo, bo + (r // 4 if name in ("u2", "u1") else r))
        assert np.linalg.norm(got[1][sl] - got[0][sl]) <= 1e-4 * np.linalg.norm(got[0][sl]), name


@pytest.mark.parametrize("H,W", [(8, 8), (8, 24), (16, 32)])
def test_copies_of_a_segment(H, W):
    """The same for the frame network, whose forward pass rounds differently
    from its reference at a few pixels' normalisation: one segment against 16
    copies, where the temporal gather's samples are shorter than a step of the
    weight gradient and where they are longer."""
    rng = np.random.default_rng(100 + H * W)
    frames = rng.poisson(1000, size=(1, 50, H, W)).astype(np.uint16)
    frames[:, 20:23, 2:6, 3:8] += 250
    labels = np.zeros((1, H, W), np.float32)
    labels[:, 2:6, 3:8] = 1
    theta = surrogate.he_init(7)
    got = []
    for B in (1, 16):
        net = surrogate.Surrogate(B, H, W, theta)
        _, g = net.backward(torch.from_numpy(np.repeat(frames, B, 0).view(np.int16)).to(DEV),
                            torch.from_numpy(np.repeat(labels, B, 0)).to(DEV), want_grad=True)
        got.append(g.cpu().numpy().astype(np.float64))
        net.close()
    for name, r, c, wo, bo in surrogate.param_layout():
        sl = slice(wo, bo + (r // 4 if name in ("u2", "u1") else r))
        assert np.linalg.norm(got[1][sl] - got[0][sl]) <= 1e-4 * np.linalg.norm(got[0][sl]), name
