"""The workloads whose speed this framework answers for.

Each case is one call (or the few calls that belong together) of the public
entry points on inputs as they are met in use: voltage-imaging recordings of
a structured background, spiking cells and shot noise, generated from a seed.

Kinds:
  push      frames appended to an open session (the streaming summaries)
  segment   a whole recording: push, finalize, footprints on the host
  serve     one 500-frame block of several recordings pushed in one batch
  motion    motion of every frame against a template, corrected frames
  traces    voltage traces of a finalized session's footprints
  unet      probability map of one segment by the summary-image U-Net
  unet_train, surrogate, surrogate_train
            one training step of that U-Net; the frame-input network's maps
            and its training step
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2403_16438_amd import MotionCorrector, Session, abi
from paper_2403_16438_amd.surrogate import Surrogate
from paper_2403_16438_amd.unet import SummaryUNet

SEG = 50
DEV = "cuda"
SERVE_MIX = [(128, 128), (256, 256), (512, 128), (512, 512)]


def listed():
    return [
        # one segment of the smallest recording, as a live session pushes it
        dict(name="push_64x64x50", kind="push", h=64, w=64, frames=50),
        # a block of the paper's 450 x 138 recording: a width that is no
        # multiple of four, and a frame that ends inside a tile both ways
        dict(name="push_450x138x500", kind="push", h=138, w=450, frames=500),
        # one block of each frame size of the serving mix, in one batch
        dict(name="serve_mix_500", kind="serve", sizes=4, frames=500),
        # a short recording from the first frame to the footprints
        dict(name="segment_64x64x1000", kind="segment", h=64, w=64, frames=1000),
        # the benchmark recording from the first frame to the footprints
        dict(name="segment_256x256x10000", kind="segment", h=256, w=256, frames=10000),
        # motion correction of one live segment, the template being kept
        dict(name="motion_128x128x50", kind="motion", h=128, w=128, frames=50, radius=8, template=False),
        # motion correction of a recording, its template included
        dict(name="motion_256x256x2000", kind="motion", h=256, w=256, frames=2000, radius=8, template=True),
        # the traces of one block of a live session
        dict(name="traces_256x256x500", kind="traces", h=256, w=256, frames=500),
        # the paper's detector on one segment (49 patches of 64 x 64)
        dict(name="unet_256x256", kind="unet", h=256, w=256),
        # its training step at the trainer's batch and patch size
        dict(name="unet_train_32", kind="unet_train", batch=32, h=64, w=64),
        # the frame-input network on eight segments
        dict(name="surrogate_8x256x256", kind="surrogate", batch=8, h=256, w=256),
        # its training step at the trainer's batch and video size
        dict(name="surrogate_train_16", kind="surrogate_train", batch=16, h=64, w=64),
    ]


def _log(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    """A case of one kind: frame sizes, lengths and batches over the range
    that the listed ones span, odd sizes among them."""
    kind = rng.choice(["push", "push", "segment", "segment", "serve", "motion", "motion", "traces", "unet",
                       "unet_train", "surrogate", "surrogate_train"])
    if kind == "push":
        return dict(kind=kind, h=_log(rng, 32, 512), w=_log(rng, 32, 512), frames=_log(rng, 50, 1000))
    if kind == "segment":
        return dict(kind=kind, h=_log(rng, 64, 256), w=_log(rng, 64, 256), frames=_log(rng, 300, 8000))
    if kind == "serve":
        return dict(kind=kind, sizes=rng.randint(2, 4), frames=_log(rng, 50, 500))
    if kind == "motion":
        return dict(kind=kind, h=_log(rng, 64, 256), w=_log(rng, 64, 300), frames=_log(rng, 10, 1500),
                    radius=rng.randint(2, 10), template=rng.random() < 0.5)
    if kind == "traces":
        return dict(kind=kind, h=_log(rng, 64, 300), w=_log(rng, 64, 300), frames=_log(rng, 50, 2000))
    if kind == "unet":
        return dict(kind=kind, h=_log(rng, 64, 400), w=_log(rng, 64, 400))
    if kind == "unet_train":
        return dict(kind=kind, batch=_log(rng, 2, 32), h=64, w=rng.choice([32, 64]))
    if kind == "surrogate":
        return dict(kind=kind, batch=rng.randint(1, 8), h=_log(rng, 64, 256, 4), w=_log(rng, 64, 256, 4))
    return dict(kind=kind, batch=_log(rng, 2, 16), h=64, w=rng.choice([32, 64]))


# ---- inputs ------------------------------------------------------------------

def _scene(h, w, seed):
    """Background [h, w] and cells (footprints [n, h * w], rest, spike size)."""
    r = np.random.default_rng([seed, h, w])
    yy, xx = torch.meshgrid(torch.arange(h, device=DEV, dtype=torch.float32),
                            torch.arange(w, device=DEV, dtype=torch.float32), indexing="ij")
    b = torch.ones((h, w), device=DEV)
    for _ in range(1 + h * w // 16384):
        cy, cx, s, a = r.uniform(0, h), r.uniform(0, w), r.uniform(15, 80), r.uniform(0.2, 0.6)
        b += a * torch.exp(-((xx - cx) ** 2 + (yy - cy) ** 2) / (2 * s * s))
    b *= 1000.0 / float(b.mean())
    n, m, at = max(3, h * w // 2184), 8.0, []
    for _ in range(50 * n):
        c = (r.uniform(m, h - 1 - m), r.uniform(m, w - 1 - m))
        # a few cells may lie close to another one
        if len(at) < n and all(math.hypot(c[0] - p[0], c[1] - p[1]) > (16 if len(at) % 5 else 8) for p in at):
            at.append(c)
    g = []
    for cy, cx in at:
        s1, s2, th = r.uniform(3, 5), r.uniform(3, 5), r.uniform(0, math.pi)
        u = (xx - cx) * math.cos(th) + (yy - cy) * math.sin(th)
        v = (yy - cy) * math.cos(th) - (xx - cx) * math.sin(th)
        g.append(torch.exp(-u * u / (2 * s1 * s1) - v * v / (2 * s2 * s2)).reshape(-1))
    bc = np.array([float(b[int(cy), int(cx)]) for cy, cx in at])
    rest = r.uniform(0.03, 0.10, len(at)) * bc
    dff = r.uniform(0.05, 0.15, len(at)) * (bc + rest)
    rate = r.uniform(5.0, 20.0, len(at)) / 741.0
    return b, torch.stack(g), rest, dff, rate


def _frames(n, h, w, seed, spiking=None):
    """uint16 video (as int16) [n, h, w] and, on request, where cells spike
    in each segment."""
    b, g, rest, dff, rate = _scene(h, w, seed)
    r = np.random.default_rng([seed, n])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    s = (r.random((n, len(rate))) < rate).astype(np.float32)
    act = s + 0.5 * np.concatenate([np.zeros((1, len(rate)), np.float32), s[:-1]])
    act = torch.from_numpy((rest + dff * act).astype(np.float32)).to(DEV)
    out = torch.empty((n, h, w), dtype=torch.int16, device=DEV)
    step = max(1, (1 << 25) // (h * w))
    for t in range(0, n, step):
        lam = act[t:t + step] @ g + b.reshape(1, -1)
        lam += torch.sqrt(lam + 25.0) * torch.randn(lam.shape, device=DEV, generator=gen)
        out[t:t + step] = lam.round_().clamp_(0, 32767).to(torch.int16).reshape(-1, h, w)
    if spiking is not None:
        on = torch.from_numpy(s[:n // SEG * SEG].reshape(-1, SEG, len(rate)).max(axis=1)).to(DEV)
        spiking.append(((on @ (g >= 0.25).float()) > 0).float().reshape(-1, h, w))
    return out


def _segments(batch, h, w, seed):
    """[batch, 50, h, w] segments of recordings, and where cells spike."""
    lab = []
    v = _frames(batch * SEG, h, w, seed, lab)
    return v.reshape(batch, SEG, h, w), lab[0]


def _moving(n, h, w, radius, seed):
    """A recording whose frames after the first 50 drift by whole pixels."""
    v = _frames(n, h, w, seed)
    r = np.random.default_rng([seed, radius])
    lim = min(radius, 6)
    step = (r.random((n, 2)) < 0.05) * r.choice([-1, 1], (n, 2))
    d = np.zeros((n, 2), np.int64)
    for t in range(1, n):
        d[t] = np.clip(d[t - 1] + step[t], -lim, lim) if t >= SEG or n <= SEG else 0
    out = torch.empty_like(v)
    dd = torch.from_numpy(d).to(DEV)
    ys, xs = torch.arange(h, device=DEV), torch.arange(w, device=DEV)
    for t in range(0, n, 100):
        k = torch.arange(t, min(n, t + 100), device=DEV)
        yi = (ys[None] - dd[k, :1]).clamp(0, h - 1)
        xi = (xs[None] - dd[k, 1:]).clamp(0, w - 1)
        out[k] = v[k[:, None, None], yi[:, :, None], xi[:, None, :]]
    return out


def _summaries(h, w, seed):
    """One segment's mean image and its max-minus-median image."""
    b, g, rest, dff, rate = _scene(h, w, seed)
    r = np.random.default_rng([seed, 7])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    on = torch.from_numpy((dff * (r.random(len(rate)) < rate * SEG)).astype(np.float32)).to(DEV)
    noise = torch.sqrt(b + 25.0)
    S = b + (torch.from_numpy(rest.astype(np.float32)).to(DEV) @ g).reshape(h, w)
    S = S + noise / 7.07 * torch.randn((h, w), device=DEV, generator=gen)
    T = noise * (0.2 + 0.03 * torch.randn((h, w), device=DEV, generator=gen)) + 0.5 * (on @ g).reshape(h, w)
    return S.contiguous(), T.contiguous()


# ---- the two networks ---------------------------------------------------------

TEMPORAL = [("t1", 32, 5), ("t2", 32, 160), ("t3", 32, 160)]
UNET = [("e1b", 32, 288), ("e2a", 64, 288), ("e2b", 64, 576), ("e3a", 128, 576), ("e3b", 128, 1152),
        ("u2", 256, 128), ("d2a", 64, 1152), ("d2b", 64, 576), ("u1", 128, 64), ("d1a", 32, 576),
        ("d1b", 32, 288), ("out", 1, 32)]
ST_TABLE = [("e1a", 32, 18)] + UNET
SUR_TABLE = TEMPORAL + [("e1a", 32, 288)] + UNET
RES = dict(e2a=4, e2b=4, d2a=4, d2b=4, u1=4, e3a=16, e3b=16, u2=16)   # pixels per output of a layer


def _bias(name, rows):
    return rows // 4 if name in ("u1", "u2") else rows


def _weights(table, seed):
    """He-normal weights and small biases, laid out as the library's table."""
    r = np.random.default_rng([seed, len(table)])
    out = []
    for name, rows, cols in table:
        out.append(r.standard_normal(rows * cols) * np.sqrt(2.0 / cols) * (0.2 if name == "out" else 1.0))
        out.append(0.02 * r.standard_normal(_bias(name, rows)))
    return np.concatenate(out).astype(np.float32)


def _macs(table, h, w):
    """Multiply-adds of one item of h x w."""
    mac = 0.0
    for name, rows, cols in table:
        per = dict(t1=10, t2=5).get(name, 1.0 / RES.get(name, 1))
        mac += rows * cols * h * w * per
    return mac


# ---- prepare, run ---------------------------------------------------------------

class _Live:
    """An open session that is pushed to block by block, and started anew
    over the same workspace when its recording is full."""

    def __init__(self, h, w, block):
        self.h, self.w, self.cap = h, w, max(SEG, block) * max(2, min(64, (1 << 25) // (h * w * max(SEG, block))))
        self.workspace = None
        self.session = None

    def room(self, n):
        if self.session is None or self.done + n > self.cap:
            if self.session is not None:
                self.session.close()
            self.session = Session(self.h, self.w, self.cap, workspace=self.workspace)
            self.workspace = self.session.workspace
            self.done = 0
        self.done += n
        return self.session

    def maps(self, n):
        s, k = self.session, n // SEG
        first = s.num_segments - k
        return [s.segment_maps(m, first, k) for m in (abi.SEG_MAP_S, abi.SEG_MAP_T, abi.SEG_MAP_D)]


class _Batch:
    """A batch object and its device table."""

    def __init__(self, slots):
        nb = abi.seg_batch_bytes(slots)
        self.table = torch.empty(nb + 256, dtype=torch.uint8, device=DEV)
        self.handle = abi.seg_batch_create(slots, (self.table.data_ptr() + 255) & ~255, nb)

    def __del__(self):
        abi.seg_batch_destroy(self.handle)


def prepare(case, seed):
    k = case["kind"]
    if k == "push":
        n = case["frames"] // SEG * SEG
        live = _Live(case["h"], case["w"], n)
        live.room(0)
        return dict(kind=k, n=n, live=live, video=_frames(n, case["h"], case["w"], seed))
    if k == "segment":
        v = _frames(case["frames"], case["h"], case["w"], seed)
        s = Session(case["h"], case["w"], case["frames"])
        ws = s.workspace
        s.close()
        # result arrays for up to twice the cells that the scene may hold
        h, w, K = case["h"], case["w"], case["frames"] // SEG
        cap = 2 * max(3, h * w // 2184) + 8
        out = dict(weights=np.zeros((cap, h, w), np.float32), masks=np.zeros((cap, h, w), np.uint8),
                   activity=np.zeros((cap, K), np.float32), component=np.zeros(cap, np.int32))
        return dict(kind=k, video=v, workspace=ws, cap=cap, out=out)
    if k == "serve":
        n = case["frames"] // SEG * SEG
        sizes = SERVE_MIX[:case["sizes"]]
        lives = [_Live(h, w, n) for h, w in sizes]
        for x in lives:
            x.room(0)
        return dict(kind=k, n=n, lives=lives, batch=_Batch(len(sizes)),
                    videos=[_frames(n, h, w, seed + i) for i, (h, w) in enumerate(sizes)])
    if k == "motion":
        h, w, n = case["h"], case["w"], case["frames"]
        v = _moving(max(n, 2 * SEG), h, w, case["radius"], seed)
        mc = MotionCorrector(h, w, radius=case["radius"])
        first, v = v[:SEG].clone(), (v if n >= 2 * SEG else v[-n:]).clone()
        mc.set_template(first)
        return dict(kind=k, mc=mc, video=v, first=first if case["template"] else None)
    if k == "traces":
        h, w, n = case["h"], case["w"], case["frames"]
        v = _frames(1000, h, w, seed)
        s = Session(h, w, 1000)
        s.push(v)
        s.finalize()
        video = v[:n].clone() if n <= 1000 else _frames(n, h, w, seed)
        # a result array for up to twice the cells that the scene may hold
        full = torch.zeros((2 * max(3, h * w // 2184) + 8, n), dtype=torch.float32, device=DEV)
        out = full[:s.traces(video[:1]).shape[0]]
        return dict(kind=k, session=s, video=video, full=full, out=out)
    if k == "unet":
        S, T = _summaries(case["h"], case["w"], seed)
        theta = _weights(ST_TABLE, seed)
        return dict(kind=k, S=S, T=T, net=SummaryUNet(_patches(case["h"], case["w"]), theta=theta))
    if k == "unet_train":
        st, y = _train_patches(case, seed)
        return dict(kind=k, net=SummaryUNet(case["batch"], case["h"], case["w"], _weights(ST_TABLE, seed)), x=st, y=y)
    x, y = _segments(case["batch"], case["h"], case["w"], seed)
    return dict(kind=k, net=Surrogate(case["batch"], case["h"], case["w"], _weights(SUR_TABLE, seed)), x=x, y=y)


def _train_patches(case, seed):
    S, T, y = [], [], []
    for b in range(case["batch"]):
        s, t = _summaries(case["h"], case["w"], seed * 1000 + b)
        S.append(s)
        T.append(t)
        y.append((t > 12.0).float())
    return torch.stack([torch.stack(S), torch.stack(T)], dim=1).contiguous(), torch.stack(y).contiguous()


def run(state):
    k = state["kind"]
    if k == "push":
        state["live"].room(state["n"]).push(state["video"])
        return state["live"].maps(state["n"])
    if k == "segment":
        v = state["video"]
        s = Session(v.shape[1], v.shape[2], v.shape[0], workspace=state["workspace"])
        s.push(v)
        s.finalize()
        out = state["out"]
        out["n"] = abi.seg_get_footprints(s.handle, state["cap"], out["weights"], out["masks"], out["activity"],
                                          out["component"])
        out.update(mean=s.image(abi.SEG_IMG_MEAN), corr=s.image(abi.SEG_IMG_CORR), noise=s.image(abi.SEG_IMG_NOISE),
                   labels=s.image(abi.SEG_IMG_LABELS))
        s.close()
        return out
    if k == "serve":
        n = state["n"]
        sessions = [x.room(n).handle for x in state["lives"]]
        abi.seg_push_batch(state["batch"].handle, sessions, [v.data_ptr() for v in state["videos"]], [n] * len(sessions),
                           torch.cuda.current_stream().cuda_stream)
        return [x.maps(n) for x in state["lives"]]
    if k == "motion":
        mc = state["mc"]
        if state["first"] is not None:
            mc.set_template(state["first"])
        motion, scores = mc.estimate(state["video"], scores=True)
        return motion, scores, mc.apply(state["video"], motion)
    if k == "traces":
        state["session"].traces(state["video"], out=state["out"])
        return state["full"]
    net = state["net"]
    if k == "unet":
        return net.segment_map(state["S"], state["T"])
    if k == "surrogate":
        return net.forward(state["x"]), net.logits()
    loss, grad = net.backward(state["x"], state["y"], want_grad=True)
    net.step()
    return loss, grad, net.params


# ---- work -------------------------------------------------------------------------

def _origins(n):
    """Origins of the 64-pixel patches along an axis."""
    o = list(range(0, n - 63, 32))
    return o if o[-1] == n - 64 else o + [n - 64]


def _patches(h, w):
    return len(_origins(h)) * len(_origins(w))


def _push_work(h, w, n):
    # the frames in, nine FP32 planes per segment out; two 25-tap passes
    return 2.0 * n * h * w + 36.0 * (n // SEG) * h * w, 100.0 * n * h * w


def work(case):
    k = case["kind"]
    h, w = case.get("h", 0), case.get("w", 0)
    n = case.get("frames", 0)
    if k in ("push", "segment"):
        b, f = _push_work(h, w, n // SEG * SEG)
        return dict(bytes=b, flops=f)
    if k == "serve":
        got = [_push_work(y, x, n // SEG * SEG) for y, x in SERVE_MIX[:case["sizes"]]]
        return dict(bytes=sum(g[0] for g in got), flops=sum(g[1] for g in got))
    if k == "motion":
        r = case["radius"]
        tiles, vec = ((h - 2 * r) // 21) * ((w - 2 * r) // 21), (2 * r + 1) ** 2
        return dict(bytes=4.0 * n * h * w, flops=2.0 * 441 * tiles * vec * n)
    if k == "traces":
        # about 7 % of the pixels lie in a mask, at about 165 pixels a cell
        return dict(bytes=2.0 * 0.07 * h * w * n + 4.0 * n * 0.07 * h * w / 165, flops=0.07 * h * w * n)
    if k == "unet":
        return dict(bytes=12.0 * h * w, flops=2 * _macs(ST_TABLE, 64, 64) * _patches(h, w))
    b = case["batch"]
    if k == "unet_train":
        return dict(bytes=12.0 * b * h * w, flops=6 * _macs(ST_TABLE, h, w) * b)
    flops = 2 * _macs(SUR_TABLE, h, w) * b
    return dict(bytes=(2.0 * SEG + 8.0) * b * h * w, flops=flops if k == "surrogate" else 3 * flops)


# ---- 64-bit values ------------------------------------------------------------------

def _taps():
    w = np.exp(-np.arange(-12, 13) ** 2 / (2.0 * 9.0))
    return w / w.sum()


def _fold(n):
    j = np.arange(-12, n + 12) % (2 * n)
    return torch.from_numpy(np.where(j >= n, 2 * n - 1 - j, j)).to(DEV)


def _seg64(v):
    """S, T, D of one segment [50, h, w] (int16) in 64 bits."""
    x = v.double()
    h, w = x.shape[1:]
    taps, fy, fx = _taps(), _fold(h), _fold(w)
    a = sum(float(t) * x[:, fy[k:k + h]] for k, t in enumerate(taps))
    s = sum(float(t) * a[:, :, fx[k:k + w]] for k, t in enumerate(taps))
    o = torch.sort(s, dim=0).values
    med = 0.5 * (o[24] + o[25])
    return x.mean(0), o[-1] - med, (med[None] - s).clamp_(min=0).mean(0)


def _maps64(v):
    got = [_seg64(v[i:i + SEG]) for i in range(0, v.shape[0] // SEG * SEG, SEG)]
    return [torch.stack([g[j] for g in got]) for j in range(3)]


NEAR = [(0, 1), (1, 0), (1, 1), (1, -1)]


def _images64(v):
    """Mean, correlation and noise images of a recording."""
    h, w = v.shape[1:]
    K = v.shape[0] // SEG
    S, D = torch.zeros((h, w), device=DEV, dtype=torch.float64), torch.zeros((h, w), device=DEV, dtype=torch.float64)
    var, C = torch.zeros_like(S), [torch.zeros_like(S) for _ in NEAR]

    def pair(dy, dx):   # the pixels x and x + (dy, dx) that both lie in the frame
        x0, x1 = max(0, -dx), w - max(0, dx)
        return (slice(0, h - dy), slice(x0, x1)), (slice(dy, h), slice(x0 + dx, x1 + dx))

    for i in range(K):
        x = v[i * SEG:(i + 1) * SEG]
        s, _, d = _seg64(x)
        S += s / K
        D += d / K
        c = x.double() - s
        var += (c * c).sum(0)
        for q, o in enumerate(NEAR):
            a, b = pair(*o)
            C[q][a] += (c[:, a[0], a[1]] * c[:, b[0], b[1]]).sum(0)
    rho, cnt = torch.zeros_like(S), torch.zeros_like(S)
    for q, o in enumerate(NEAR):
        a, b = pair(*o)
        r = C[q][a] / torch.sqrt(var[a] * var[b])
        for at in (a, b):
            rho[at] += r
            cnt[at] += 1
    return S, rho / cnt, math.sqrt(2 * math.pi) * D


def _scores64(first, v, R):
    h, w = v.shape[1:]
    t = ((first.to(torch.int64).sum(0) + first.shape[0] // 2) // first.shape[0]).double()
    ny, nx = (h - 2 * R) // 21, (w - 2 * R) // 21
    oy, ox = R + (h - 2 * R - 21 * ny) // 2, R + (w - 2 * R - 21 * nx) // 2
    side = 2 * R + 1
    out = torch.zeros((v.shape[0], side * side), device=DEV, dtype=torch.float64)

    def unit(a):
        a = a - a.mean(1, keepdim=True)
        n = a.norm(dim=1, keepdim=True)
        return torch.where(n > 0, a / n.clamp(min=1e-300), torch.zeros_like(a))

    for p in range(ny * nx):
        y, x = oy + 21 * (p // nx), ox + 21 * (p % nx)
        win = t[y - R:y + 21 + R, x - R:x + 21 + R].unfold(0, 21, 1).unfold(1, 21, 1).reshape(side * side, 441)
        tile = v[:, y:y + 21, x:x + 21].reshape(-1, 441).double()
        out += unit(tile) @ unit(win).T.contiguous()
    return out


def _unpack(theta, table):
    p, at = {}, 0
    for name, rows, cols in table:
        p[name] = (theta[at:at + rows * cols].reshape(rows, cols),
                   theta[at + rows * cols:at + rows * cols + _bias(name, rows)])
        at += rows * cols + _bias(name, rows)
    return p


def _conv64(x, p):
    w, b = p
    c, B, h, wd = x.shape
    xp = F.pad(x, (1, 1, 1, 1))
    w = w.reshape(w.shape[0], c, 9)
    y = b.reshape(-1, 1)
    for k in range(9):
        y = y + w[:, :, k].contiguous() @ xp[:, :, k // 3:k // 3 + h, k % 3:k % 3 + wd].reshape(c, -1)
    return torch.relu(y).reshape(-1, B, h, wd)


def _up64(x, p):
    w, b = p
    c, B, h, wd = x.shape
    z = (w @ x.reshape(c, -1)).reshape(-1, 2, 2, B, h, wd)
    return z.permute(0, 3, 4, 1, 5, 2).reshape(-1, B, 2 * h, 2 * wd) + b.reshape(-1, 1, 1, 1)


def _unet64(x, p):
    """Logits [B, h, w] of the input [channels, B, h, w]."""
    pool = lambda a: a.reshape(a.shape[0], a.shape[1], a.shape[2] // 2, 2, a.shape[3] // 2, 2).amax(dim=(3, 5))
    s1 = _conv64(_conv64(x, p["e1a"]), p["e1b"])
    s2 = _conv64(_conv64(pool(s1), p["e2a"]), p["e2b"])
    b3 = _conv64(_conv64(pool(s2), p["e3a"]), p["e3b"])
    d2 = _conv64(_conv64(torch.cat([_up64(b3, p["u2"]), s2]), p["d2a"]), p["d2b"])
    d1 = _conv64(_conv64(torch.cat([_up64(d2, p["u1"]), s1]), p["d1a"]), p["d1b"])
    w, b = p["out"]
    return (w @ d1.reshape(32, -1)).reshape(d1.shape[1:]) + b


def _st64(st):
    S, T = st[:, 0].double(), st[:, 1].double()
    m = S.mean(dim=(1, 2), keepdim=True)
    sd = ((S - m) ** 2).mean(dim=(1, 2), keepdim=True).sqrt().clamp(min=1e-3)
    return torch.stack([(S - m) / sd, T / torch.sqrt(S + 25.0)])


def _temporal64(frames, p):
    B, _, h, w = frames.shape
    x = frames.double()
    m = x.mean(1, keepdim=True)
    x = ((x - m) / torch.sqrt(m + 25.0)).permute(1, 0, 2, 3).reshape(SEG, -1)
    lin = lambda q, a: torch.relu(q[0] @ a + q[1].reshape(-1, 1))
    a1 = torch.stack([lin(p["t1"], x[5 * j:5 * j + 5]) for j in range(10)], dim=1)
    a1 = F.pad(a1, (0, 0, 2, 2))
    a2 = torch.stack([lin(p["t2"], a1[:, 2 * j:2 * j + 5].reshape(160, -1)) for j in range(5)], dim=1)
    return lin(p["t3"], a2.reshape(160, -1)).reshape(32, B, h, w)


def exact(case, seed):
    k = case["kind"]
    h, w = case.get("h", 0), case.get("w", 0)
    if k == "push":
        return _maps64(_frames(case["frames"] // SEG * SEG, h, w, seed))
    if k == "serve":
        n = case["frames"] // SEG * SEG
        return [_maps64(_frames(n, y, x, seed + i)) for i, (y, x) in enumerate(SERVE_MIX[:case["sizes"]])]
    if k == "segment":
        mean, corr, noise = _images64(_frames(case["frames"], h, w, seed))
        return dict(weights=None, masks=None, activity=None, component=None, n=None, mean=mean, corr=corr,
                    noise=noise, labels=None)
    if k == "motion":
        n = case["frames"]
        v = _moving(max(n, 2 * SEG), h, w, case["radius"], seed)
        return None, _scores64(v[:SEG], v if n >= 2 * SEG else v[-n:], case["radius"]), None
    if k == "traces":
        return None   # the footprints come from the session
    if k == "unet":
        S, T = _summaries(h, w, seed)
        p = _unpack(torch.from_numpy(_weights(ST_TABLE, seed)).to(DEV).double(), ST_TABLE)
        oy, ox = _origins(h), _origins(w)
        st = torch.stack([torch.stack([S[y:y + 64, x:x + 64], T[y:y + 64, x:x + 64]]) for y in oy for x in ox])
        prob = torch.sigmoid(_unet64(_st64(st), p))
        tent = 1.0 - (torch.arange(64, device=DEV, dtype=torch.float64) - 31.5).abs() / 32.0
        num, den = torch.zeros((h, w), device=DEV, dtype=torch.float64), torch.zeros((h, w), device=DEV, dtype=torch.float64)
        for i, (y, x) in enumerate((y, x) for y in oy for x in ox):
            num[y:y + 64, x:x + 64] += prob[i] * tent[:, None] * tent[None]
            den[y:y + 64, x:x + 64] += tent[:, None] * tent[None]
        return num / den
    table = ST_TABLE if k == "unet_train" else SUR_TABLE
    theta = torch.from_numpy(_weights(table, seed)).to(DEV).double()
    if k == "surrogate":
        x, _ = _segments(case["batch"], h, w, seed)
        p = _unpack(theta, table)
        z = _unet64(_temporal64(x, p), p)
        return torch.sigmoid(z), z
    theta.requires_grad_(True)
    p = _unpack(theta, table)
    if k == "unet_train":
        x, y = _train_patches(case, seed)
        z = _unet64(_st64(x), p)
    else:
        x, y = _segments(case["batch"], h, w, seed)
        z = _unet64(_temporal64(x, p), p)
    loss = F.binary_cross_entropy_with_logits(z, y.double())
    loss.backward()
    g = theta.grad
    # one RMSProp step: v = 0.1 g^2
    return float(loss.detach()), g, theta.detach() - 1e-3 * g / (torch.sqrt(0.1 * g * g) + 1e-7)
