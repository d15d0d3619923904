"""vp_preprocess_batch_noalloc (the entry point that allocates nothing: its
plan goes to the library's fixed device memory) against vp_preprocess_batch
through the C ABI: the same rows, bit for bit, with the same grid_thw and
cu_seqlens, on two calls in a row -- the second with a smaller batch, whose
plan is shorter than the one the fixed memory still holds -- in both output
types; the plan copied whole and in pieces, its tables computed on the device
or filled on the host; calls in flight one behind another.  Rows past the
batch must stay untouched.
"""
import sys

import numpy as np
import pytest

import paper_2604_16893_amd as vp
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def log(msg):
    print(f"[no-alloc] {msg}", flush=True)
    sys.stdout.flush()


def _items(specs, seed):
    out = []
    for k, (n_src, H, W, idx, h, w) in enumerate(specs):
        it = workloads.Item("video", n_src, H, W, "uniform", seed + k, {"mode": "uniform", "n": 1})
        out.append(vp.Item(workloads.frames_torch(it, DEV), np.asarray(idx, np.int32), h, w))
    return out


# a ragged batch of five kernel shapes (several launches), then a smaller one
FIRST = [(9, 120, 200, [0, 3, 8, 5], 96, 160), (1, 333, 257, [0], 320, 256),
         (7, 45, 80, [6], 64, 64), (3, 480, 854, [0, 1, 2], 128, 224),
         (2, 300, 3000, [1, 0], 32, 96), (4, 720, 1280, [3, 1, 0, 2], 256, 448)]
SECOND = [(3, 75, 101, [2, 0, 1], 64, 96), (1, 250, 333, [0], 256, 320)]


def _run_both(items, dtype):
    mean, std = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)
    code = vp.VP_OUT_BF16 if dtype == "bf16" else vp.VP_OUT_F32
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    grid, cu, rows, ws = vp.vp_batch_layout(items)
    assert ws <= vp.VP_NOALLOC_PLAN_BYTES
    ref = torch.full((rows + 4, 1536), float("nan"), dtype=tdt, device=DEV)
    work = torch.empty(ws, dtype=torch.uint8, device=DEV)
    g1, c1 = vp.vp_preprocess_batch(items, mean, std, code, ref, work)
    got = torch.full((rows + 4, 1536), float("nan"), dtype=tdt, device=DEV)
    g2, c2 = vp.vp_preprocess_batch_noalloc(items, mean, std, code, got)
    torch.cuda.synchronize()
    assert g1.tolist() == g2.tolist() == grid.tolist()
    assert c1.tolist() == c2.tolist() == cu.tolist()
    assert torch.isnan(got[rows:].float()).all(), "rows past the batch were written"
    a = got[:rows].view(torch.int16 if dtype == "bf16" else torch.int32)
    b = ref[:rows].view(torch.int16 if dtype == "bf16" else torch.int32)
    same = torch.equal(a, b)
    log(f"{len(items)} items, {rows} rows, plan {ws} bytes, {dtype}: bit-identical {same}")
    assert same


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_noalloc_matches_workspace_entry_twice(dtype):
    first = _items(FIRST, 300)
    second = _items(SECOND, 400)
    assert vp.vp_batch_layout(second)[3] < vp.vp_batch_layout(first)[3]
    _run_both(first, dtype)
    _run_both(second, dtype)


def test_noalloc_on_a_side_stream_in_order():
    """Two calls on one non-default stream are ordered: the second (smaller)
    call's plan copy waits for the first call's kernels."""
    first = _items(FIRST, 500)
    second = _items(SECOND, 600)
    mean, std = (0.5, 0.5, 0.5), (0.5, 0.5, 0.5)
    outs = []
    s = torch.cuda.Stream()
    for items in (first, second):
        _, _, rows, _ = vp.vp_batch_layout(items)
        outs.append(torch.full((rows, 1536), float("nan"), dtype=torch.bfloat16, device=DEV))
    with torch.cuda.stream(s):
        vp.vp_preprocess_batch_noalloc(first, mean, std, vp.VP_OUT_BF16, outs[0], s)
        vp.vp_preprocess_batch_noalloc(second, mean, std, vp.VP_OUT_BF16, outs[1], s)
    torch.cuda.synchronize()
    for items, got in zip((first, second), outs):
        ref, _, _ = vp.preprocess(items, mean, std, "bf16")
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16))


# The ways this entry's plan reaches the device: in one to four pieces of
# 16 KiB with the tables computed there, and (many small frames: few tables
# beside many units, `host`) in one copy with the tables filled on the host --
# both patches and kernels, twelve slots, windows of 138 rows, long column
# windows.  The workspace entry computes all tables on the device.
PLANS = [
    # n, H, W, h, w, patch, host
    (2, 130, 170, 96, 128, 16, False),
    (8, 480, 854, 352, 640, 16, False),
    (48, 480, 854, 320, 576, 16, False),
    (1, 18, 19, 32, 32, 16, False),     # the tables in the pieces that the plan takes anyway: x-first,
    (1, 57, 17, 168, 56, 14, False),    # many slots,
    (3, 400, 300, 32, 64, 16, False),   # the general kernel, without any,
    (124, 52, 78, 64, 96, 16, False),   # two pieces
    (2600, 60, 90, 32, 64, 16, True),
    (4096, 47, 45, 96, 96, 16, True),
    (2600, 1100, 40, 32, 32, 16, True),
    (2600, 40, 200, 32, 32, 16, True),
    (6000, 56, 70, 56, 56, 14, True),
    (9000, 90, 70, 28, 56, 14, True),
]


@pytest.mark.parametrize("n,H,W,h,w,patch,host", PLANS)
def test_noalloc_plan_copies(n, H, W, h, w, patch, host):
    it = workloads.Item("video", min(n, 64), H, W, "uniform", 700, {"mode": "uniform", "n": 1})
    items = [vp.Item(workloads.frames_torch(it, DEV), np.arange(n, dtype=np.int32) % min(n, 64), h, w, patch)]
    ws = vp.vp_batch_layout(items)[3]
    log(f"plan of {ws} bytes: {n} x {H}x{W} -> {h}x{w} patch {patch}")
    assert (ws > 4 * 16384 + 4 * 8192) if host else ws < 4 * 16384 + 4 * 8192
    mean, std = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)
    ref, _, _ = vp.preprocess(items, mean, std, "f32")
    got = torch.full_like(ref, float("nan"))
    vp.vp_preprocess_batch_noalloc(items, mean, std, vp.VP_OUT_F32, got)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), ref.view(torch.int32))


def test_noalloc_calls_in_flight_keep_their_plans():
    """Calls one after another on one stream, none waited for, with other
    frames and sizes in turn: the host memory that a plan is copied from is
    written again by the next call while earlier ones are still in flight."""
    it = workloads.Item("video", 16, 480, 854, "uniform", 710, {"mode": "uniform", "n": 1})
    f = workloads.frames_torch(it, DEV)
    mean, std = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)
    batches = [[vp.Item(f, (np.arange(n, dtype=np.int32) * step + k) % 16, h, w)]
               for k, (n, step, h, w) in enumerate([(16, 1, 352, 640), (15, 3, 320, 576), (64, 5, 64, 96), (2, 7, 256, 448)])]
    refs = [vp.preprocess(b, mean, std, "f32")[0] for b in batches]
    outs = [[torch.full_like(r, float("nan")) for r in refs] for _ in range(5)]
    torch.cuda.synchronize()
    for turn in outs:
        for b, out in zip(batches, turn):
            vp.vp_preprocess_batch_noalloc(b, mean, std, vp.VP_OUT_F32, out)
    torch.cuda.synchronize()
    for turn in outs:
        for ref, out in zip(refs, turn):
            assert torch.equal(out.view(torch.int32), ref.view(torch.int32))


@pytest.mark.parametrize("specs", [
    [(2, 130, 170, 96, 128)],                                                # one copy, tables on the device
    [(8, 480, 854, 352, 640), (1, 1000, 700, 320, 224), (3, 90, 60, 96, 64)],   # several pieces, several kernels
    [(64, 270, 480, 128, 224)] * 20,                                         # one copy with its tables
], ids=["one_piece", "pieces", "whole"])
def test_noalloc_captured_and_replayed(specs):
    """A captured call replayed over frames that change, with the library's
    other entry and torch's work between the replays: each replay's rows are
    the eager call's."""
    items = [vp.Item(torch.randint(0, 256, (n, H, W, 3), dtype=torch.uint8, device=DEV),
                     np.arange(n, dtype=np.int32), h, w) for n, H, W, h, w in specs]
    mean, std = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)
    out = torch.empty_like(vp.preprocess(items, mean, std, "f32")[0])
    vp.vp_preprocess_batch_noalloc(items, mean, std, vp.VP_OUT_F32, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        vp.vp_preprocess_batch_noalloc(items, mean, std, vp.VP_OUT_F32, out)
    for _ in range(4):
        items[0].frames.random_(0, 256)
        out.fill_(float("nan"))
        ref = vp.preprocess(items, mean, std, "f32")[0]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), ref.view(torch.int32))
