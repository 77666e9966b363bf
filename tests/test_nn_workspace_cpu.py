"""Workspace sizes of the networks: a size that was enough for a network before
its backward pass had kernels of its own is enough with them."""
import ctypes as C

import pytest

from paper_2403_16438_amd import abi


def _bytes(f, shape):
    n = C.c_size_t()
    abi.check(f(*shape, C.byref(n)), "workspace_bytes")
    return n.value


@pytest.mark.parametrize("shape,frames,summaries", [
    ((1, 4, 4), 43657216, 43387904),
    ((1, 64, 64), 91180032, 73415680),
    ((1, 8, 72), 50179072, 47508480),          # some layers without direct kernels
    ((3, 20, 36), 68630016, 59167232),
    ((32, 64, 64), 1570198528, 1007961088),
    ((49, 64, 64), 2381273088, 1520453632),
    ((8, 256, 256), 6150384640, 3902036992),
])
def test_former_sizes_are_enough(shape, frames, summaries):
    assert _bytes(abi.lib.seg_nn_workspace_bytes, shape) <= frames
    assert _bytes(abi.lib.seg_nn_st_workspace_bytes, shape) <= summaries
