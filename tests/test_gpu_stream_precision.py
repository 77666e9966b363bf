"""T and D of quiet pixels beside loud ones, in frames that leave their tile's
fixed-point scale, and where pixels hardly vary: against FP64, the error is to
be no larger than that of FP64 sums whose intermediate and result are rounded
to FP32 (the same order of passes, formed here).

Bars. The mean over 5,000 and more pixels of a relative error of two roundings
differs between two such computations by a percent or two: 5 %. Single pixels
stay below half of the window around the event threshold in which decisions
are not compared (1e-6), or below the largest error of the FP64 form where that
is more (D where the median lies far from R)."""
import numpy as np
import pytest
import torch

from oracle import smoothing_matrix
from paper_2403_16438_amd import Session, abi, to_device_frames
from paper_2403_16438_amd.serve import Batch

pytestmark = pytest.mark.gpu
H, W = 40, 131


def _video(kind, rng, h=H, w=W):
    loud, quiet = kind if isinstance(kind, tuple) else (0, 20)
    v = 10000 + quiet * rng.standard_normal((50, h, w))
    if loud:
        v[:, h // 2:h // 2 + 4, w // 3:w // 3 + 4] += loud * rng.standard_normal((50, 4, min(4, w - w // 3)))
    if kind == "flash":                    # bright frames, the first of the segment among them
        v[[0, 7, 48]] += 2500
    if kind == "jump":                     # a step that does not fit the fixed point
        v[30:33, :2, :2] += 40000
    if kind == "full":
        v = rng.integers(0, 65536, (50, h, w))
    if kind == "sparse":                   # single counts
        v = 100 + rng.poisson(0.01, (50, h, w))
    if kind == "border":                   # a constant border wider than the smoothing reaches
        v[:, :16] = v[:, :, -16:] = 300
    return np.clip(np.rint(v), 0, 65535).astype(np.uint16)


def _summaries(s):
    order = np.sort(s, axis=0)
    med = 0.5 * (order[24] + order[25])
    return order[-1] - med, np.maximum(0.0, med - s).mean(axis=0)


def _forms(video, sigma, radius):
    """T and D in FP64, and with both passes rounded to FP32."""
    d = video.astype(np.float64) - np.median(video[:3], axis=0)
    gy, gx = smoothing_matrix(video.shape[1], sigma, radius), smoothing_matrix(video.shape[2], sigma, radius)
    up = gy @ d
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    return _summaries(up @ gx.T), [f32(a) for a in _summaries(f32(f32(up) @ gx.T))]


@pytest.mark.parametrize("sigma,radius", [(3.0, 12), (0.6, 2), (6.0, 12)])
@pytest.mark.parametrize("kind", [(0, 33), (0, 0.3), (400, 10), (400, 3), (450, 1), (3000, 10), (3000, 3), (3000, 1),
                                  (9000, 2), "flash", "jump", "full", "sparse", "border"], ids=str)
def test_error_is_that_of_float64_sums(kind, sigma, radius):
    rng = np.random.default_rng(17)
    video = _video(kind, rng)
    s = Session(H, W, 50, gauss_sigma=sigma, gauss_radius=radius)
    s.push(to_device_frames(video))
    got = [s.segment_maps(m).cpu().numpy()[0].astype(np.float64) for m in (abi.SEG_MAP_T, abi.SEG_MAP_D)]
    s.close()
    exact, form = _forms(video, float(np.float32(sigma)), radius)
    own = (video != video[0]).any(axis=0)   # pixels with a signal of their own
    assert own.sum() >= (1000 if kind == "sparse" else 2000)
    for name, g, x, f in zip("TD", got, exact, form):
        at = own & (x >= 1e-3)              # D of a rare count may be next to nothing
        if not at.any():
            assert kind == "sparse" and name == "D"
            continue
        e, ef = np.abs(g - x)[at] / x[at], np.abs(f - x)[at] / x[at]
        print(kind, name, f"mean {e.mean():.2e} (form {ef.mean():.2e}) max {e.max():.2e} ({ef.max():.2e})")
        assert e.mean() <= 1.05 * ef.mean(), name
        assert e.max() <= max(5e-7, ef.max()), name


def test_batch_takes_the_same_paths():
    """Segments of every kind pushed in one batch have the bits that they have
    when each is pushed by itself, frames of three columns among them."""
    rng = np.random.default_rng(4)
    kinds = [(0, 33), (450, 1), "flash", "jump", "full", "sparse", "border"]
    sizes = [(40, 131), (33, 64), (40, 131), (50, 70), (64, 128), (40, 131), (48, 90)]
    videos = [_video(k, rng, h, w) for k, (h, w) in zip(kinds, sizes)] + [_video("full", rng, 20, 3)]
    frames = [to_device_frames(v) for v in videos]
    alone, together = [], []
    for f in frames:
        s = Session(f.shape[1], f.shape[2], 50)
        s.push(f)
        alone.append([s.segment_maps(m).cpu() for m in (abi.SEG_MAP_S, abi.SEG_MAP_T, abi.SEG_MAP_D)])
        s.close()
    sessions = [Session(f.shape[1], f.shape[2], 50) for f in frames]
    batch = Batch(len(sessions), "cuda")
    batch.push(sessions, frames)
    torch.cuda.synchronize()
    for s in sessions:
        together.append([s.segment_maps(m).cpu() for m in (abi.SEG_MAP_S, abi.SEG_MAP_T, abi.SEG_MAP_D)])
        s.close()
    for k, (a, b) in enumerate(zip(alone, together)):
        assert all(torch.equal(x, y) for x, y in zip(a, b)), k
