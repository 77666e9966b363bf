"""The input normalisation of the summary network deals a patch to four, two or
one workgroups by the number of patches: a patch's probabilities have the same
bits in every batch."""
import numpy as np
import pytest
import torch

from paper_2403_16438_amd import unet

pytestmark = pytest.mark.gpu


def test_patch_in_any_batch():
    rng = np.random.default_rng(2)
    st = np.stack([rng.uniform(700, 1300, (129, 32, 64)), rng.uniform(0, 80, (129, 32, 64))], axis=1).astype(np.float32)
    st = torch.from_numpy(st).cuda()
    net = unet.SummaryUNet(129, 32, 64, unet.he_init(4))
    got = {b: net.forward(st[:b].contiguous()).clone() for b in (1, 64, 65, 128, 129)}
    net.close()
    for b, p in got.items():
        assert torch.equal(p, got[129][:b]), b
