"""The split NMF (each component over several co-resident workgroups) against
the oracle and against the one-workgroup-per-component kernel.

Both paths compute the same factorisation (Eq. 3) and differ only in the
order of the sums over a component's pixels, so the bar is the oracle's:
same components with the same number of footprints, mask IoU >= 0.99; on top,
the two GPU paths agree closely in weights and the split path is
bit-reproducible from run to run.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_16438_amd import Session, abi, segment_video
from synth import preset, simulate

from parity import compare_footprints, params_from_config
from scenes import ring_video

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wide():
    """256 x 256, 30 neurons, 2,000 frames: components of 200-1,000 pixels,
    i.e. up to ~30 workgroups per component."""
    video, _ = simulate(preset(2, frames=2000), 2000)
    sess = segment_video(video, nmf_path=abi.SEG_NMF_SPLIT)
    ref = oracle.segment(video, params_from_config(sess.cfg))
    return video, sess, ref


def test_split_matches_oracle(wide):
    video, sess, ref = wide
    assert len(ref.footprints) >= 20
    compare_footprints(sess.footprints(), ref.footprints)


def test_split_matches_single_workgroup(wide):
    video, sess, ref = wide
    one = segment_video(video, nmf_path=abi.SEG_NMF_SINGLE).footprints()
    two = sess.footprints()
    assert np.array_equal(one["component"], two["component"])
    assert np.array_equal(one["masks"], two["masks"])
    assert np.abs(one["weights"] - two["weights"]).max() <= 1e-5
    rel = np.abs(one["activity"] - two["activity"]).max() / np.abs(one["activity"]).max()
    assert rel <= 1e-5


def test_split_is_reproducible(wide):
    video, sess, ref = wide
    again = segment_video(video, nmf_path=abi.SEG_NMF_SPLIT).footprints()
    first = sess.footprints()
    assert np.array_equal(again["weights"], first["weights"])
    assert np.array_equal(again["activity"], first["activity"])


def test_auto_path_small_case():
    """64 x 64 x 1,000 (20 segments): the automatic choice (split: the
    exchange slots of its few workgroups fit the workspace) against the
    oracle."""
    video, _ = simulate(preset(1), 0)
    sess = segment_video(video)
    assert sess.profile()["nmf_path"] == abi.SEG_NMF_SPLIT
    ref = oracle.segment(video, params_from_config(sess.cfg))
    compare_footprints(sess.footprints(), ref.footprints)


def test_split_refuses_too_many_segments():
    """4,096 segments do not fit a 32-pixel slice in LDS: the forced split
    path reports SEG_E_CAPACITY, the automatic path falls back."""
    rng = np.random.default_rng(5)
    T, H, W = 4096 * 50, 16, 16
    video = rng.poisson(400.0, size=(T, H, W)).astype(np.uint16)
    for k in (3, 700, 2500):                     # a 6 x 6 blob fires in three segments
        video[k * 50 + 20:k * 50 + 23, 5:11, 5:11] += 600
    with pytest.raises(abi.SegError) as e:
        segment_video(video, block=20000, nmf_path=abi.SEG_NMF_SPLIT)
    assert e.value.code == abi.SEG_E_CAPACITY
    sess = segment_video(video, block=20000)
    fp = sess.footprints()
    assert fp["masks"].shape[0] == 1
    assert fp["masks"][0, 5:11, 5:11].all()


def test_profile_reports_the_finalize(wide):
    """seg_get_profile: event-timed device work of the last finalize and the
    NMF's algorithmic operation count (formula recomputed here from the
    components and ranks)."""
    video, sess, ref = wide
    prof = sess.profile()
    labels = sess.image(abi.SEG_IMG_LABELS)
    assert prof["components"] == labels.max() == ref.n_comp
    assert prof["nmf_path"] == abi.SEG_NMF_SPLIT
    assert prof["nmf_ms"] > 0.0 and prof["maps_ms"] > 0.0
    assert 1 <= prof["max_rank"] <= sess.cfg.nmf_max_rank
    K, S = sess.num_segments, sess.cfg.nmf_sweeps
    sizes = np.bincount(labels.ravel())[1:]
    # lower bound with rank 1 for every component, upper with the largest rank
    lo = sum(8 * m * K + (S + 1) * (2 * m * K + 2 * m + 2 * K) + S * (2 * m * K + 2 * K + 2 * m) for m in sizes)
    N = prof["max_rank"]
    hi = sum((6 * N + 2) * m * K + (S + 1) * (2 * m * K * N + m * N * (N + 1) + 2 * K * N * N)
             + S * (2 * m * K * N + K * N * (N + 1) + 2 * m * N * N) for m in sizes)
    assert lo <= prof["nmf_flops"] <= hi


def test_profile_needs_a_finalize():
    s = Session(32, 32, 100)
    with pytest.raises(abi.SegError) as e:
        s.profile()
    assert e.value.code == abi.SEG_E_STATE


def test_split_over_several_launches():
    """512 x 512 frames with about 90 components need more workgroups than
    compute units: the split plan packs them into several cooperative
    launches, and the result matches the one-workgroup-per-component path."""
    from synth.gpu import GpuScene
    cfg = preset(2, height=512, width=512, frames=5000, n_neurons=120, n_overlap=24)
    video = GpuScene(cfg, 4242).render(0, cfg.frames)
    out = {}
    for path in (abi.SEG_NMF_SPLIT, abi.SEG_NMF_SINGLE):
        s = Session(512, 512, cfg.frames, nmf_path=path)
        s.push(video)
        s.finalize()
        out[path] = (s.footprints(), s.profile())
    fs, ps = out[abi.SEG_NMF_SPLIT]
    f1, p1 = out[abi.SEG_NMF_SINGLE]
    assert ps["nmf_path"] == abi.SEG_NMF_SPLIT and p1["nmf_path"] == abi.SEG_NMF_SINGLE
    assert ps["nmf_workgroups"] > 256          # more than one launch
    assert np.array_equal(fs["component"], f1["component"])
    assert np.array_equal(fs["masks"], f1["masks"])
    assert np.abs(fs["weights"] - f1["weights"]).max() <= 1e-5


@pytest.mark.parametrize("K", [3, 96, 97])
def test_component_sizes_of_every_exchange(K):
    """Components of one slice (which exchange nothing), of a few and of more
    than eight (polled in two rounds), on both sides of the segment count where
    the slice width changes: both paths, which differ in the order of FP64 sums
    only, to the bars of the comparison above."""
    rng = np.random.default_rng(K)
    H, W = 96, 192
    yy, xx = np.mgrid[0:H, 0:W]
    T = rng.uniform(0.5, 1.5, (K, H, W)).astype(np.float32)
    discs = [(12, 12, 5), (14, 40, 9), (40, 24, 14), (46, 100, 20), (46, 112, 20), (30, 160, 16), (66, 160, 16)]
    for j, (cy, cx, r) in enumerate(discs):
        d2 = (yy - cy) ** 2 + (xx - cx) ** 2
        on = rng.random(K) < 0.4
        on[j % K] = True
        for i in np.flatnonzero(on):
            T[i] += np.where(d2 <= r * r, rng.uniform(8, 14) * (1.3 - d2 / (r * r + 1.0)), 0.0).astype(np.float32)
    D = np.full((K, H, W), 1.0 / np.sqrt(2 * np.pi), np.float32)
    got = []
    for path in (abi.SEG_NMF_SINGLE, abi.SEG_NMF_SPLIT):
        s = Session(H, W, 50 * K, nmf_path=path, min_event_segs=1, area_max=4000)
        s.load_summaries(T, np.ones_like(T), D)
        s.finalize()
        torch.cuda.synchronize()
        assert s.profile()["nmf_path"] == path
        got.append(s.footprints())
        s.close()
    one, two = got
    assert len(one["component"]) >= 5
    assert np.array_equal(one["component"], two["component"])
    assert np.array_equal(one["masks"], two["masks"])
    assert np.abs(one["weights"] - two["weights"]).max() <= 1e-5
    assert np.abs(one["activity"] - two["activity"]).max() <= 1e-5 * np.abs(one["activity"]).max()


@pytest.mark.parametrize("K", [3, 13, 15, 29, 31, 44, 45])
def test_sweeps_in_registers(K):
    """Components of at most 512 pixels over at most 44 segments: one or two
    rows per thread, ranks one to three and above, on both sides of every block
    of 16 columns (and one segment more, which takes the other path): against
    the one-workgroup-per-component kernel, to the bars of the comparison
    above."""
    rng = np.random.default_rng(10 * K)
    H, W = 96, 160
    yy, xx = np.mgrid[0:H, 0:W]
    T = rng.uniform(0.5, 1.5, (K, H, W)).astype(np.float32)
    discs = [(10, 10, 4), (14, 36, 9), (16, 70, 12), (50, 12, 6), (50, 19, 6), (50, 50, 6), (50, 57, 6), (56, 53, 6),
             (50, 100, 5), (50, 107, 5), (57, 100, 5), (57, 107, 5), (50, 114, 5), (84, 30, 5), (84, 132, 9)]
    for j, (cy, cx, r) in enumerate(discs):
        d2 = (yy - cy) ** 2 + (xx - cx) ** 2
        on = rng.random(K) < 0.3
        on[j % K] = True
        for i in np.flatnonzero(on):
            T[i] += np.where(d2 <= r * r, rng.uniform(8, 14) * (1.3 - d2 / (r * r + 1.0)), 0.0).astype(np.float32)
    D = np.full((K, H, W), 1.0 / np.sqrt(2 * np.pi), np.float32)
    got = []
    for path in (abi.SEG_NMF_SINGLE, abi.SEG_NMF_SPLIT):
        s = Session(H, W, 50 * K, nmf_path=path, min_event_segs=1, area_max=4000)
        s.load_summaries(T, np.ones_like(T), D)
        s.finalize()
        torch.cuda.synchronize()
        assert s.profile()["nmf_path"] == path
        sizes = np.bincount(s.image(abi.SEG_IMG_LABELS).ravel())[1:]
        assert sizes.max() <= 512 and sizes.max() > 256 and sizes.min() <= 256
        got.append(s.footprints())
        s.close()
    one, two = got
    assert len(one["component"]) >= 6
    assert np.array_equal(one["component"], two["component"])
    assert np.array_equal(one["masks"], two["masks"])
    assert np.abs(one["weights"] - two["weights"]).max() <= 1e-5
    assert np.abs(one["activity"] - two["activity"]).max() <= 1e-5 * np.abs(one["activity"]).max()


def _cluster(T, cy, cx, n, q, r, rng):
    """n cells of radius r on a ring of radius q, one at a time active: one
    component of rank n."""
    yy, xx = np.mgrid[0:T.shape[1], 0:T.shape[2]]
    for i in range(len(T)):
        a = 2 * np.pi * (i % n) / n
        d2 = (yy - cy - q * np.sin(a)) ** 2 + (xx - cx - q * np.cos(a)) ** 2
        T[i] += np.where(d2 <= r * r, rng.uniform(8, 14) * (1.3 - d2 / (r * r + 1.0)), 0.0).astype(np.float32)


@pytest.mark.parametrize("K", [8, 20, 44])
@pytest.mark.parametrize("n,q,r", [(4, 7.5, 6.5), (5, 7.5, 6), (6, 7.5, 6), (7, 8, 5.5), (8, 8.5, 5)])
def test_higher_ranks_in_short_recordings(n, q, r, K):
    """Components of at most 512 pixels over at most 44 segments whose rank is
    more than the sweeps in registers take, beside some of rank 1 to 3 (of more
    and of less than 256 pixels) that they do take: both paths, which differ in
    the order of FP64 sums only, to the bars of the comparison above."""
    rng = np.random.default_rng(100 * n + K)
    T = rng.uniform(0.5, 1.5, (K, 64, 192)).astype(np.float32)
    _cluster(T, 32, 32, n, q, r, rng)
    _cluster(T, 32, 96, 3, 6, 6.5, rng)
    _cluster(T, 16, 150, 2, 3, 4, rng)
    _cluster(T, 48, 150, 1, 0, 4, rng)
    D = np.full(T.shape, 1.0 / np.sqrt(2 * np.pi), np.float32)
    got = []
    for path in (abi.SEG_NMF_SINGLE, abi.SEG_NMF_SPLIT):
        s = Session(64, 192, 50 * K, nmf_path=path, min_event_segs=1, nmf_max_rank=8)
        s.load_summaries(T, np.ones_like(T), D)
        s.finalize()
        torch.cuda.synchronize()
        prof = s.profile()
        assert prof["nmf_path"] == path and prof["max_rank"] == n
        sizes = np.sort(np.bincount(s.image(abi.SEG_IMG_LABELS).ravel())[1:])
        assert len(sizes) == 4 and 450 <= sizes[-1] <= 512 and 256 < sizes[-2] <= 512
        got.append(s.footprints())
        s.close()
    one, two = got
    assert len(one["component"]) == n + 6
    assert np.array_equal(one["component"], two["component"])
    assert np.array_equal(one["masks"], two["masks"])
    assert np.abs(one["weights"] - two["weights"]).max() <= 1e-5
    assert np.abs(one["activity"] - two["activity"]).max() <= 1e-5 * np.abs(one["activity"]).max()


@pytest.mark.parametrize("n,radius,sigma,frames", [(6, 5.0, 2.0, 1000), (5, 5.0, 2.0, 500), (4, 5.0, 2.5, 500)])
def test_short_recordings_of_a_ring(n, radius, sigma, frames):
    """The same from frames, with the default limits: against the oracle."""
    video = ring_video(n_cells=n, radius=radius, sigma=sigma, frames=frames)
    sess = segment_video(video)
    ref = oracle.segment(video, params_from_config(sess.cfg))
    prof = sess.profile()
    assert prof["nmf_path"] == abi.SEG_NMF_SPLIT and prof["max_rank"] >= 4
    compare_footprints(sess.footprints(), ref.footprints)
