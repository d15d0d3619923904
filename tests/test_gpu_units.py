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


@pytest.mark.parametrize("n_src,H,W,idx,h,w", [(2, 421, 611, [1, 0], 160, 256), (2, 700, 1291, [0, 1], 256, 448)])
def test_writer_short_units_match_long_ones(n_src, H, W, idx, h, w):
    """The uint8 writer, on both of its forms: bytes equal the oracle's for
    one item alone and for the first and last of many."""
    it = workloads.Item("video", n_src, H, W, "uniform", 43, {"mode": "uniform", "n": n_src})
    one = vp.Item(workloads.frames_torch(it, DEV), np.asarray(idx, np.int32), h, w)
    alone = vp.resize_u8([one])[0]
    many = vp.resize_u8([one] * 512)
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
