"""The calls that this library is used for, as measured cases.

A case is one call (for the cached step: two) through the Python binding on
frames that are already on the GPU, as a training or serving step makes it:
the data loader has sampled the frame indices and chosen the target sizes, the
call plans the batch, resamples, normalises and writes the rows.  Sizes are
those of the benchmark configurations (240x320 and 480x854 clips, 1080p, the
ragged batch of 12 videos and 20 images, the 64-video 720p batch at a quarter
of its length), of the full-resolution video and image budgets that the tests
use, and generic ones.

`path` of a case:
  "resize"  vp.preprocess: resample + normalise + patchify;
  "cached"  vp.patchify on frames already at the target size, then
            vp.vp_position_ids of the same batch: what each later stage does
            with cached frames;
  "writer"  vp.resize_u8: the frames of an offline cache, resized to bytes.
A batch holds `videos` videos and `images` images.  With `H`, `W` every video
has that size; with `mix` the sizes and lengths are drawn from that number,
over the ranges that the case names.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2604_16893_amd as vp

DEV = "cuda:0"
MEAN, STD = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)
RESOLUTIONS = ((360, 640), (480, 854), (720, 1280), (1080, 1920))


def _case(path, **kw):
    c = dict(path=path, videos=0, images=0, frames=0, sources=0, H=0, W=0, mix=0, patch=16, dtype="bf16",
             video_max=262144, video_min=0, image_max=1048576, image_min=65536, side_min=256, side_max=1024,
             frames_min=32, frames_max=256, tallest=720, portrait=False)
    c.update(kw)
    return c


def listed():
    return [
        # one photo of a chat request: the smallest call a server makes
        _case("resize", name="image_one", images=1, side_min=0, H=1200, W=1600),
        # a short clip in float32 (the tiny configuration): latency and launches
        _case("resize", name="clip_small_f32", videos=1, frames=8, sources=16, H=240, W=320,
              video_max=24576, dtype="f32"),
        # images as they come, from thumbnails raised to the minimum to 12-megapixel photos
        _case("resize", name="images_ragged", images=24, mix=11, side_min=72, side_max=4032),
        # one 480p video at 2 of 8 fps in float32
        _case("resize", name="video_480p_f32", videos=1, frames=64, sources=256, H=480, W=854,
              video_max=230400, dtype="f32"),
        # one long 1080p video
        _case("resize", name="video_1080p", videos=1, frames=128, sources=192, H=1080, W=1920, video_max=360448),
        # one 4K video at the training budget: long filter windows
        _case("resize", name="video_4k", videos=1, frames=64, sources=64, H=2160, W=3840),
        # the ragged batch of joint image and video training
        _case("resize", name="mixed_ragged", videos=12, images=20, mix=3, video_max=200704, image_max=1003520),
        # the rollout batch: many 720p videos at a small budget (the largest call)
        _case("resize", name="videos_720p", videos=16, frames=256, sources=256, H=720, W=1280, video_max=122880),
        # the ragged batch for models with patches of 14
        _case("resize", name="mixed_ragged_p14", videos=8, images=12, mix=5, patch=14, video_max=200704,
              image_max=1003520, frames_max=128),
        # a later stage on cached frames: rows and position tables
        _case("cached", name="cached_step", videos=64, frames=64, sources=64, H=256, W=448),
        # the same for patches of 14, ragged, in float32
        _case("cached", name="cached_step_p14_f32", videos=12, images=8, mix=7, patch=14, dtype="f32",
              video_max=200704, image_max=1003520, frames_max=96),
        # the offline cache writer over videos of several resolutions
        _case("writer", name="cache_writer", videos=12, mix=9, frames_max=192, tallest=1080),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(("resize", "resize", "resize", "cached", "writer"))
    kind = rng.choice(("video", "images", "mix"))
    c = _case(path, patch=rng.choice((16, 16, 14)), dtype=rng.choice(("bf16", "bf16", "f32")),
              video_max=_log_int(rng, 65536, 401408), image_max=_log_int(rng, 262144, 1048576))
    if kind == "video":
        h = _log_int(rng, 120, 2160)
        w = max(96, int(h * rng.uniform(0.5, 2.2)))
        n = _log_int(rng, 2, 256)
        c.update(H=h, W=w, videos=_log_int(rng, 1, 16), video_min=rng.choice((0, 131072)))
        c["video_max"] = max(c["video_max"], c["video_min"])
        most = int(3e9 / (h * w * 3 * c["videos"]))   # about 3 GB of sampled frames
        c["frames"] = max(1, min(n, most))
        c["sources"] = c["frames"] + rng.randint(0, c["frames"])
    elif kind == "images":
        c.update(images=_log_int(rng, 1, 48), mix=rng.randint(1, 1 << 20), side_min=_log_int(rng, 64, 384),
                 side_max=_log_int(rng, 640, 4096))
    else:
        c.update(videos=rng.randint(1, 8), images=rng.randint(1, 16), mix=rng.randint(1, 1 << 20),
                 frames_min=8, frames_max=_log_int(rng, 16, 128), tallest=rng.choice((480, 720, 1080)),
                 portrait=True)
    return c


# ---------------------------------------------------------------- the batch

def _rhe(num, den):
    q, r = divmod(num, den)
    return q + (2 * r > den or (2 * r == den and q % 2 == 1))


def _target(H, W, factor, lo, hi):
    """smart_resize: multiples of `factor` with lo <= h * w <= hi."""
    h = max(factor, round(H / factor) * factor)
    w = max(factor, round(W / factor) * factor)
    if h * w > hi:
        beta = math.sqrt(H * W / hi)
        h = max(factor, math.floor(H / beta / factor) * factor)
        w = max(factor, math.floor(W / beta / factor) * factor)
    elif h * w < lo:
        beta = math.sqrt(lo / (H * W))
        h = math.ceil(H * beta / factor) * factor
        w = math.ceil(W * beta / factor) * factor
    return h, w


def _sources(case):
    """The batch's items as (source frames, sampled frames, H, W, min, max)."""
    rng = random.Random(case["mix"])
    vid, img = (case["video_min"], case["video_max"]), (case["image_min"], case["image_max"])
    got = []
    for _ in range(case["videos"]):
        if case["mix"]:
            H, W = rng.choice([r for r in RESOLUTIONS if r[0] <= case["tallest"]])
            if case["portrait"] and rng.random() < 0.3:
                H, W = W, H
            n = 2 * rng.randint(case["frames_min"] // 2, case["frames_max"] // 2)
            got.append((rng.randint(n, 2 * n), n, H, W) + vid)
        else:
            got.append((case["sources"], case["frames"], case["H"], case["W"]) + vid)
    for _ in range(case["images"]):
        if case["mix"]:
            a, b = (_log_int(rng, case["side_min"], case["side_max"]) for _ in range(2))
            b = min(max(b, a // 3), 3 * a)
            got.append((1, 1, a, b) + img)
        else:
            got.append((1, 1, case["H"], case["W"]) + img)
    if case["mix"]:
        rng.shuffle(got)
    return got


def _plan(case):
    """Per item (source frames, indices, H, W, h, w)."""
    F = 2 * case["patch"]
    out = []
    for n_src, n, H, W, lo, hi in _sources(case):
        h, w = _target(H, W, F, lo, hi)
        if case["path"] == "cached":   # the cache holds the sampled frames at the target size
            n_src, H, W = n, h, w
        idx = [_rhe(i * (n_src - 1), n - 1) if n > 1 else 0 for i in range(n)]
        out.append((n_src, idx, H, W, h, w))
    return out


def _frames(gen, n, H, W):
    """Decoded-looking frames: a smooth gradient that drifts from frame to frame, sensor noise, some flat areas."""
    out = torch.empty((n, H, W, 3), dtype=torch.uint8, device=DEV)
    ramp = (torch.arange(H, device=DEV).view(H, 1, 1) * (96.0 / max(H - 1, 1))
            + torch.arange(W, device=DEV).view(1, W, 1) * (80.0 / max(W - 1, 1))
            + torch.arange(3, device=DEV).view(1, 1, 3) * 6.0)
    level = int(torch.randint(8, 24, (1,), generator=gen, device=DEV))
    ramp = (ramp + level).to(torch.uint8)
    step = max(1, (1 << 28) // (H * W * 3))
    for a in range(0, n, step):
        part = out[a:a + step]
        part.random_(0, 30, generator=gen)
        part += ramp
        part += (torch.arange(a, a + part.shape[0], device=DEV) % 16).to(torch.uint8).view(-1, 1, 1, 1)
    out[:, H // 8:H // 3, W // 2:W // 2 + W // 5] = torch.tensor([250, 8, 120], dtype=torch.uint8, device=DEV)
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    F = 2 * case["patch"]
    items = []
    for n_src, n, H, W, lo, hi in _sources(case):
        h, w = vp.vp_smart_resize_dims(H, W, F, lo, hi)
        if case["path"] == "cached":
            n_src, H, W = n, h, w
        idx = vp.vp_sample_indices(n_src, vp.VP_SAMPLE_UNIFORM, n)
        items.append(vp.Item(_frames(gen, n_src, H, W), idx, h, w, case["patch"]))
    state = {"path": case["path"], "dtype": case["dtype"], "items": items}
    if case["path"] == "cached":
        _, _, rows, ws = vp.vp_batch_layout(items)
        state["vit"] = torch.empty((rows, 3), dtype=torch.int32, device=DEV)
        state["llm"] = torch.empty((rows // 4, 3), dtype=torch.int32, device=DEV)
        state["work"] = torch.empty(ws, dtype=torch.uint8, device=DEV)
    return state


def run(state):
    items = state["items"]
    if state["path"] == "resize":
        rows, grid, cu = vp.preprocess(items, MEAN, STD, state["dtype"])
        return {"rows": rows, "grid": grid, "cu": cu}
    if state["path"] == "cached":
        rows, grid, cu = vp.patchify(items, MEAN, STD, state["dtype"])
        seg = vp.vp_position_ids(items, state["vit"], state["llm"], state["work"])
        return {"rows": rows, "grid": grid, "cu": cu, "vit": state["vit"], "llm": state["llm"], "seg": seg}
    # one buffer, as the writer fills it: the frames are views of it
    frames = vp.resize_u8(items)
    return {"frames": frames[0]._base if frames[0]._base is not None else frames[0]}


# ---------------------------------------------------------------- what it takes

def _taps(n_in, n_out):
    return min(n_in, 4 * max(n_in / n_out, 1.0))


def work(case):
    size = {"f32": 4, "bf16": 2}[case["dtype"]]
    read = write = flops = 0
    for n_src, idx, H, W, h, w in _plan(case):
        n, P = len(idx), case["patch"]
        pairs = (n + 1) // 2
        distinct = len(set(idx))
        read += distinct * H * W * 3
        if case["path"] == "writer":
            write += n * h * w * 3
        else:
            write += 2 * pairs * h * w * 3 * size
        if case["path"] == "cached":
            rows = pairs * (h // P) * (w // P)
            write += rows * 12 + rows // 4 * 12
            flops += 2 * n * h * w * 3
        else:   # the cheaper order of the two passes
            y, x = _taps(H, h), _taps(W, w)
            flops += 2 * distinct * 3 * min(h * W * y + h * w * x, H * w * x + h * w * y)
    return {"bytes": read + write, "flops": flops}


def tolerance(case):
    if case["path"] == "writer":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    return {"rel": 6e-3, "max": 1.6e-2}


# ---------------------------------------------------------------- in 64 bits

def _matrix(n_in, n_out):
    """The antialiased Keys cubic (a = -1/2) as an [n_out, n_in] matrix."""
    scale = n_in / n_out
    s = max(scale, 1.0)
    m = np.zeros((n_out, n_in))
    for i in range(n_out):
        c = (i + 0.5) * scale
        lo, hi = max(0, math.floor(c - 2 * s + 0.5)), min(n_in, math.floor(c + 2 * s + 0.5))
        t = np.abs((np.arange(lo, hi) + 0.5 - c) / s)
        k = np.where(t < 1, 1.5 * t ** 3 - 2.5 * t ** 2 + 1, np.where(t < 2, -0.5 * t ** 3 + 2.5 * t ** 2 - 4 * t + 2, 0.0))
        m[i, lo:hi] = k / k.sum()
    return torch.from_numpy(m).to(DEV)


def exact(case, seed):
    if case["path"] == "writer":
        return None   # bytes: compared as they are
    P = case["patch"]
    state = prepare(case, seed)
    mean = torch.tensor(MEAN, dtype=torch.float32, device=DEV).double().view(1, 3, 1, 1)
    std = torch.tensor(STD, dtype=torch.float32, device=DEV).double().view(1, 3, 1, 1)
    parts = []
    for item, (_, idx, H, W, h, w) in zip(state["items"], _plan(case)):
        idx = idx + idx[-1:] if len(idx) % 2 else idx
        my = mx = None
        if case["path"] == "resize":
            my, mx = _matrix(H, h), _matrix(W, w).t().contiguous()
        rows = torch.empty(len(idx) // 2 * (h // P) * (w // P), 6 * P * P, dtype=torch.float64, device=DEV)
        step = max(1, (1 << 26) // (H * W * 3)) * 2
        at = 0
        for a in range(0, len(idx), step):
            f = item.frames[torch.tensor(idx[a:a + step], device=DEV)].permute(0, 3, 1, 2).double().contiguous()
            if my is not None:
                f = torch.matmul(torch.matmul(my, f), mx)
            v = (f / 255.0 - mean) / std
            t = v.shape[0] // 2
            # [t, dt, c, bh, mh, y, bw, mw, x] -> [t, bh, bw, mh, mw, c, dt, y, x]
            v = v.view(t, 2, 3, h // (2 * P), 2, P, w // (2 * P), 2, P).permute(0, 3, 6, 4, 7, 2, 1, 5, 8)
            v = v.reshape(-1, 6 * P * P)
            rows[at:at + v.shape[0]] = v
            at += v.shape[0]
        parts.append(rows)
    out = {"rows": torch.cat(parts), "grid": None, "cu": None}
    if case["path"] == "cached":
        out.update(vit=None, llm=None, seg=None)
    return out
