"""The segment summaries over the ranges of values at which the smoothing
changes from fixed point to FP64 sums, against the FP64 oracle.

Bars. Fixed point (|V - R| at most m = 2000 / 2^e in a tile): the intermediate
is rounded to 2^-(20 + e), the weights to 2^-30 (25 taps, two passes), three
byte products of at most 25 x 128^2 x (1 + 2 x 2^8) x 2^-(50 + e) in sum are
left out, and the result is rounded to FP32. General path: two FP32 roundings.
Both are below m 2^-23 + 7e-7 per smoothed value, with m the largest |V - R|
within the halo. T is the difference of two values and D at most the mean of
such differences: twice that, plus the rounding of the result itself."""
import numpy as np
import pytest
import torch
from scipy.ndimage import maximum_filter

import oracle
from paper_2403_16438_amd import Session, abi, to_device_frames

from parity import assert_image_close, params_from_config

pytestmark = pytest.mark.gpu


def _video(kind, K, H, W, rng):
    n = 50 * K
    v = rng.poisson(1000, size=(n, H, W)).astype(np.int64)
    if kind == "full":                    # no tile fits any scale
        v = rng.integers(0, 65536, size=(n, H, W))
    elif kind == "flash":                 # one corner of one segment leaves its scale late
        v[50 + 47, :3, :3] += 60000
    elif kind == "step":                  # a segment whose values pass the scale by one, or just do not
        v[:] = 5000                       # quiet: e = 7, up to 15
        v[10:20] += 15
        v[60:70] += 16
        v[110:120] -= 15
    elif kind == "ends":                  # the type's lowest and highest values
        v = np.where(rng.random((n, H, W)) < 0.5, 0, 65535)
        v[50:100] = rng.integers(0, 2, size=(50, H, W))
        v[100:] = 65535 - rng.integers(0, 2, size=(n - 100, H, W))
    elif kind == "wide":                  # noise of several hundred: the smallest power of two
        v = 3000 + rng.integers(-240, 241, size=(n, H, W))
    return np.clip(v, 0, 65535).astype(np.uint16)


@pytest.mark.parametrize("shape", [(3, 3), (2, 1), (7, 4), (40, 5), (17, 64), (33, 131)])
@pytest.mark.parametrize("kind", ["poisson", "full", "flash", "step", "ends", "wide"])
def test_value_ranges(kind, shape):
    H, W = shape
    rng = np.random.default_rng(100 * H + W)
    video = _video(kind, 3, H, W, rng)
    s = Session(H, W, len(video))
    s.push(to_device_frames(video))
    s.finalize()
    torch.cuda.synchronize()
    prm = params_from_config(s.cfg)
    S, T, D = (s.segment_maps(k).cpu().numpy() for k in (abi.SEG_MAP_S, abi.SEG_MAP_T, abi.SEG_MAP_D))
    C = np.zeros((5, H, W))
    for i in range(3):
        seg = video[50 * i:50 * i + 50]
        r = oracle.summarize_segment(seg, prm)
        C += oracle.segment_moments(seg)
        m = np.abs(seg.astype(np.int64) - np.median(seg[:3], axis=0).astype(np.int64)).max(axis=0).astype(np.float64)
        # the largest value of the tile (64 x 16) and its halo that a pixel may share
        m = maximum_filter(m, size=(2 * (16 + 12) + 1, 2 * (64 + 12) + 1))
        bar = 2.0 * (m * 2.0 ** -23 + 7e-7)
        assert np.array_equal(S[i], r["S"].astype(np.float32)), i
        assert (np.abs(T[i] - r["T"]) <= bar + np.abs(r["T"]) * 2.0 ** -24).all(), i
        assert (np.abs(D[i] - r["D"]) <= bar + np.abs(r["D"]) * 2.0 ** -24).all(), i
    if H > 1 and kind != "ends":
        assert_image_close(s.image(abi.SEG_IMG_CORR), oracle.correlation_image(C), what="corr")
    s.close()


@pytest.mark.parametrize("sigma,radius", [(0.5, 1), (1.0, 4), (6.0, 12)])
def test_other_smoothing_widths(sigma, radius):
    rng = np.random.default_rng(radius)
    video = rng.poisson(900, size=(50, 30, 83)).astype(np.uint16)
    s = Session(30, 83, 50, gauss_sigma=sigma, gauss_radius=radius)
    s.push(to_device_frames(video))
    s.finalize()
    torch.cuda.synchronize()
    r = oracle.summarize_segment(video, params_from_config(s.cfg))
    bar = 2.0 * (512 * 2.0 ** -23 + 7e-7)
    T, D = (s.segment_maps(k).cpu().numpy()[0] for k in (abi.SEG_MAP_T, abi.SEG_MAP_D))
    assert np.abs(T - r["T"]).max() <= bar + np.abs(r["T"]).max() * 2.0 ** -24
    assert np.abs(D - r["D"]).max() <= bar + np.abs(r["D"]).max() * 2.0 ** -24
    s.close()
