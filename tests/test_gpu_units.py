"""GPU parity of the unit split: a small batch is cut into short units of
output rows, a large one into units of ten or more filter windows; the rows
are the same bits either way, and match the oracle."""
import numpy as np
import pytest

import oracle
from oracle import compare
import paper_2604_16893_amd as vp
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MEAN, STD = (0.481, 0.458, 0.408), (0.269, 0.261, 0.276)

# (n_src, H, W, indices, h, w, patch): y-first, x-first, an upscale whose
# rows close several at a time, long windows, patch 14 with an odd count
CASES = [
    (2, 421, 611, [1, 0], 160, 256, 16),
    (2, 240, 321, [0, 1], 192, 256, 16),
    (3, 90, 131, [2, 0, 1], 160, 224, 16),
    (1, 900, 1501, [0], 192, 288, 16),
    (3, 411, 600, [2, 0, 1], 224, 280, 14),
]


def _workgroups(items):
    return int(sum(r[5] for r in vp.vp_batch_kernels(items)))


@pytest.mark.parametrize("n_src,H,W,idx,h,w,patch", CASES)
def test_short_units_match_long_ones(n_src, H, W, idx, h, w, patch):
    it = workloads.Item("video", n_src, H, W, "uniform", 41, {"mode": "uniform", "n": n_src})
    frames = workloads.frames_torch(it, DEV)
    one = vp.Item(frames, np.asarray(idx, np.int32), h, w, patch)
    copies = 64
    while _workgroups([one] * copies) * 2 > _workgroups([one]) * copies:   # units of the single item: twice as many
        copies *= 2
        assert copies <= 16384, "the batch never took longer units"
    print(f"[units] {H}x{W} -> {h}x{w} patch {patch}: {copies} copies", flush=True)
    rows, _, cu = vp.preprocess([one], MEAN, STD, "f32")
    many, _, cu_many = vp.preprocess([one] * copies, MEAN, STD, "f32")
    torch.cuda.synchronize()
    assert torch.equal(many[:rows.shape[0]], rows) and torch.equal(many[-rows.shape[0]:], rows)
    ref = oracle.preprocess_item(workloads.frames_np(it), idx, h, w, MEAN, STD, patch=patch)
    res = compare.check_f32(rows.cpu().numpy(), ref)
    assert res["ok"], res


@pytest.mark.parametrize("n_src,H,W,idx,h,w,form", [
    (2, 421, 611, [1, 0], 160, 256, vp.VP_WRITER_MATRIX),
    (2, 700, 1291, [0, 1], 256, 448, vp.VP_WRITER_MATRIX),
    (2, 900, 320, [1, 0], 128, 160, vp.VP_WRITER_DOT),
    (2, 640, 1984, [0, 1], 96, 320, vp.VP_WRITER_DOT),
])
def test_writer_short_units_match_long_ones(n_src, H, W, idx, h, w, form):
    """The uint8 writer's forms in units: bytes equal the oracle's for one item
    alone, in short units, and for the first and last of many, in long ones."""
    it = workloads.Item("video", n_src, H, W, "uniform", 43, {"mode": "uniform", "n": n_src})
    one = vp.Item(workloads.frames_torch(it, DEV), np.asarray(idx, np.int32), h, w)
    copies = 512
    few, lots = vp.vp_resize_kernels([one]), vp.vp_resize_kernels([one] * copies)
    assert [int(r[0]) for r in few] == [int(r[0]) for r in lots] == [form]
    assert 2 * int(lots[0][5]) <= copies * int(few[0][5]), "the batch never took longer units"
    print(f"[units] writer {H}x{W} -> {h}x{w}: {few.tolist()} {lots.tolist()}", flush=True)
    alone = vp.resize_u8([one])[0]
    many = vp.resize_u8([one] * copies)
    torch.cuda.synchronize()
    src = workloads.frames_np(it)
    ref = np.stack([oracle.resize_u8(src[i], h, w) for i in idx])
    assert np.array_equal(alone.cpu().numpy(), ref)
    assert torch.equal(many[0], alone) and torch.equal(many[-1], alone)


# Patch 14: pairs of bands of up to 63 columns.  Widths of one window, of a
# second band with no, some or all of its columns, of several workgroups; x
# scales that give 4 to 8 taps on the x-first kernel (M up to 8 slots), and
# y-first bands that are no whole number of patches (49 and 63 columns)
BANDS14 = [
    # H, W, h, w, kind, taps
    (60, 31, 56, 28, vp.VP_KERNEL_XFIRST, 5),
    (56, 112, 56, 112, vp.VP_KERNEL_XFIRST, 4),
    (121, 181, 84, 140, vp.VP_KERNEL_XFIRST, 6),
    (75, 409, 112, 252, vp.VP_KERNEL_XFIRST, 7),
    (40, 511, 56, 280, vp.VP_KERNEL_XFIRST, 8),
    (61, 131, 112, 252, vp.VP_KERNEL_XFIRST, 4),
    (243, 641, 112, 280, vp.VP_KERNEL_YFIRST, 10),
    (240, 427, 112, 196, vp.VP_KERNEL_YFIRST, 9),
    (300, 421, 168, 364, vp.VP_KERNEL_YFIRST, 5),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,W,h,w,kind,taps", BANDS14)
def test_patch14_bands(H, W, h, w, kind, taps, dtype):
    it = workloads.Item("video", 3, H, W, "uniform", 47, {"mode": "uniform", "n": 3})
    idx = [2, 0, 1]   # a pair, and an odd frame that stands for both of its pair
    item = vp.Item(workloads.frames_torch(it, DEV), np.asarray(idx, np.int32), h, w, 14)
    launches = vp.vp_batch_kernels([item])
    assert [(int(r[0]), int(r[2])) for r in launches] == [(kind, taps)], launches.tolist()
    print(f"[patch14 bands] {H}x{W} -> {h}x{w} {dtype} {launches.tolist()}", flush=True)
    rows, _, _ = vp.preprocess([item], MEAN, STD, dtype)
    torch.cuda.synchronize()
    ref = oracle.preprocess_item(workloads.frames_np(it), idx, h, w, MEAN, STD, patch=14)
    if dtype == "bf16":
        res = compare.check_bf16(rows.view(torch.int16).cpu().numpy().view(np.uint16), ref)
    else:
        res = compare.check_f32(rows.cpu().numpy(), ref)
    assert res["ok"], res


@pytest.mark.parametrize("H,W,h,w", [(37, 53, 64, 96), (97, 131, 96, 128), (241, 330, 160, 224), (700, 1291, 256, 448),
                                     (64, 64, 64, 64), (540, 3840, 96, 672), (33, 5, 32, 32), (1201, 40, 32, 32),
                                     (9001, 70, 32, 64)])
def test_device_tables_are_the_hosts_bits(H, W, h, w):
    """The column weights that the device computes for a plan are the bits of
    vp_filter_table, for upscales, identity and long windows: the whole table
    (zero-padded to the kernel's taps) stands in the workspace."""
    item = vp.Item(torch.zeros((1, H, W, 3), dtype=torch.uint8, device=DEV), [0], h, w)
    kind, m, kx = (int(v) for v in vp.vp_batch_kernels([item])[0][:3])
    assert kind in (vp.VP_KERNEL_XFIRST, vp.VP_KERNEL_YFIRST)
    _, _, rows, ws = vp.vp_batch_layout([item])
    work = torch.zeros(ws, dtype=torch.uint8, device=DEV)
    out = torch.empty((rows, vp.VP_ROW), dtype=torch.float32, device=DEV)
    vp.vp_preprocess_batch([item], MEAN, STD, vp.VP_OUT_F32, out, work)
    torch.cuda.synchronize()
    plan = work.cpu().numpy()
    start, count, weight = vp.vp_filter_table(W, w)
    words = plan.view(np.int32)
    table = np.zeros((w, kx), np.float32)
    table[:, :weight.shape[1]] = weight[:, :kx]
    at = [k for k in np.flatnonzero(words == table.view(np.int32)[0, 0]) if k + w * kx <= len(words)]
    assert at, "the first column's first weight is not in the plan"
    best = max(at, key=lambda k: int((words[k:k + w * kx] == table.view(np.int32).reshape(-1)).sum()))
    got = words[best:best + w * kx].view(np.float32).reshape(w, kx)
    for j in range(w):   # a column at its band's right edge has its weights shifted
        assert any(np.array_equal(got[j], np.roll(table[j], s)) for s in range(kx)), j
    slots = (weight_slots(H, h, m) * np.float32(2.0 ** 24)).astype(np.float32).tobytes()
    assert slots in plan.tobytes(), "the slot table is not in the plan"


def weight_slots(H, h, m):
    start, count, weight = vp.vp_filter_table(H, h)
    table = np.zeros((H + 6, m), np.float32)
    for i in range(h):
        table[start[i]:start[i] + count[i], i % m] = weight[i, :count[i]]
    return table


# Upscales over 2x on the x-first kernel: 12 and 16 slots (3x and 4x exactly,
# and just past 2x), 4 and 5 column taps, a one-column source, both patches
UPSCALES = [
    # H, W, h, w, patch, slots, taps
    (47, 45, 96, 96, 16, 12, 4),
    (32, 33, 96, 64, 16, 12, 4),
    (24, 70, 96, 64, 16, 16, 5),
    (16, 1, 64, 32, 16, 16, 4),
    (64, 64, 256, 256, 16, 16, 4),
    (20, 66, 56, 56, 14, 12, 5),
    (21, 40, 84, 140, 14, 16, 4),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,W,h,w,patch,slots,taps", UPSCALES)
def test_upscales_of_many_slots(H, W, h, w, patch, slots, taps, dtype):
    it = workloads.Item("video", 3, H, W, "uniform", 53, {"mode": "uniform", "n": 3})
    idx = [1, 2, 0]
    item = vp.Item(workloads.frames_torch(it, DEV), np.asarray(idx, np.int32), h, w, patch)
    launches = vp.vp_batch_kernels([item])
    assert [tuple(int(v) for v in r[:3]) for r in launches] == [(vp.VP_KERNEL_XFIRST, slots, taps)], launches.tolist()
    print(f"[upscales] {H}x{W} -> {h}x{w} patch {patch} {dtype}", flush=True)
    rows, _, _ = vp.preprocess([item], MEAN, STD, dtype)
    torch.cuda.synchronize()
    ref = oracle.preprocess_item(workloads.frames_np(it), idx, h, w, MEAN, STD, patch=patch)
    if dtype == "bf16":
        res = compare.check_bf16(rows.view(torch.int16).cpu().numpy().view(np.uint16), ref)
    else:
        res = compare.check_f32(rows.cpu().numpy(), ref)
    assert res["ok"], res
