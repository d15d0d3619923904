"""GPU parity of the uint8 cache writer (vp_resize_batch).

The fixed-point resampler is integer arithmetic from the 22-bit weights on,
so the device bytes must equal the oracle's exactly (the oracle itself is
pinned byte for byte to Pillow's bicubic resize): small cases in full, and
sampled frames of the full-size 64 x 256-frame workload and of the ragged
image/video batch.  Bytes beyond the batch must stay untouched.
"""
import sys

import numpy as np
import pytest

import oracle
import paper_2604_16893_amd as vp
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def log(msg):
    print(f"[gpu-resize-u8] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(autouse=True)
def _free_memory():
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def run(items, sentinel=8, patch=16):
    """items: list of (device frames, indices, h, w).  Returns the output
    buffer (without the sentinel bytes) and frame_off."""
    vitems = [vp.Item(f, idx, h, w, patch) for f, idx, h, w in items]
    off, ws = vp.vp_resize_layout(vitems)
    total = int(off[-1])
    out = torch.full((total + sentinel,), 0xA5, dtype=torch.uint8, device=DEV)
    work = torch.empty(max(ws, 1), dtype=torch.uint8, device=DEV)
    off2 = vp.vp_resize_batch(vitems, out, work)
    torch.cuda.synchronize()
    assert off2.tolist() == off.tolist()
    assert (out[total:] == 0xA5).all(), "bytes beyond the batch were written"
    return out[:total], off


def frames_of(out, off, k, n, h, w):
    return out[int(off[k]):int(off[k + 1])].view(n, h, w, 3)


def _video(seed, n, H, W, gen="uniform"):
    it = workloads.Item("video", n, H, W, gen, seed, {"mode": "uniform", "n": n})
    return it, workloads.frames_torch(it, DEV)


CASES = [
    # name, [(n_src, H, W, indices, h, w)]
    ("downscale_2x", [(3, 64, 96, [2, 0], 32, 48 + 16)]),
    ("upscale_1_6x", [(2, 40, 50, [1, 0, 1], 64, 96)]),
    ("upscale_2x_eight_slots", [(2, 48, 80, [1, 0], 96, 160)]),
    ("upscale_2_5x", [(1, 64, 64, [0], 160, 160)]),
    ("identity", [(2, 64, 96, [1], 64, 96)]),
    ("mixed_axes", [(2, 100, 60, [0, 1], 64, 96)]),
    ("odd_width_854", [(2, 60, 854, [1, 0], 32, 640)]),
    ("tall_strong_downscale", [(2, 2400, 100, [1, 0], 64, 32)]),
    ("wide_strong_downscale", [(1, 300, 3000, [0], 32, 96)]),
    ("long_window_4k_width", [(2, 540, 3840, [1, 0], 96, 672)]),
    # x downscale of 3.9x: 16-column blocks read more than 64 pixels, so the
    # matrix-core form takes windows of 128 and bands of 16 columns
    ("wide_blocks_3_9x", [(2, 100, 1000, [0, 1], 64, 256)]),
    # matrix-core form, windows of 10 and more taps, with a vertical upscale
    # that keeps seven rows open
    ("mfma_seven_slots", [(2, 40, 240, [1, 0], 64, 96)]),
    # matrix-core form on rows and frames that start off 4-byte boundaries
    # (3 W = 783 bytes per row, 58,725 bytes per frame)
    ("mfma_unaligned_rows", [(3, 75, 261, [2, 0, 1], 32, 96)]),
    ("single_pixel", [(1, 1, 1, [0], 32, 32)]),
    ("ragged_batch", [(4, 75, 101, [3, 1, 2], 64, 96), (1, 333, 257, [0], 320, 256),
                      (5, 120, 200, [4, 0], 96, 160)]),
]

# One form of the writer each, with its shape (slots and column taps of the
# dot-product form, pixels of a loaded row and columns a workgroup of the
# matrix-core form).  Dot products: uniform downscales over 5.9x (column taps
# 28 and 32, bands of 32 columns, a last one of 28), vertical ones over 5.6x
# beside milder horizontal ones (bands of 64, a last one of 32 columns; four and
# five slots), a target wider than the matrix-core form's 4,094 blocks (eight
# slots); tiles: longer windows than either holds
FORMS = [
    # H, W, h, w, patch, kind and shape
    (400, 1588, 64, 256, 16, [vp.VP_WRITER_DOT, 4, 28, 0, 0]),
    (680, 2176, 96, 320, 16, [vp.VP_WRITER_DOT, 4, 32, 0, 0]),
    (420, 1745, 56, 252, 14, [vp.VP_WRITER_DOT, 4, 32, 0, 0]),
    (700, 700, 96, 224, 16, [vp.VP_WRITER_DOT, 4, 16, 0, 0]),
    (900, 320, 128, 160, 16, [vp.VP_WRITER_DOT, 4, 12, 0, 0]),
    (608, 200, 96, 96, 16, [vp.VP_WRITER_DOT, 5, 12, 0, 0]),
    (4000, 100, 32, 96, 16, [vp.VP_WRITER_DOT, 4, 8, 0, 0]),
    (16, 33000, 32, 66016, 16, [vp.VP_WRITER_DOT, 8, 8, 0, 0]),
    (333, 4001, 64, 160, 16, [vp.VP_WRITER_TILES, 0, 0, 0, 0]),
    (60, 1600, 96, 192, 16, [vp.VP_WRITER_TILES, 0, 0, 0, 0]),
    (300, 3000, 28, 84, 14, [vp.VP_WRITER_TILES, 0, 0, 0, 0]),
    (100, 1000, 64, 256, 16, [vp.VP_WRITER_MATRIX, 0, 0, 128, 16]),
    (200, 301, 64, 128, 16, [vp.VP_WRITER_MATRIX, 0, 0, 128, 32]),
]


@pytest.mark.parametrize("H,W,h,w,patch,form", FORMS)
def test_each_form_exact(H, W, h, w, patch, form):
    it, fd = _video(431, 3, H, W)
    idx = [2, 0, 1]
    launches = vp.vp_resize_kernels([vp.Item(fd, np.array(idx, np.int32), h, w, patch)]).tolist()
    log(f"form {H}x{W} -> {h}x{w} patch {patch}: {launches}")
    assert [r[:5] for r in launches] == [form]
    out, off = run([(fd, np.array(idx, np.int32), h, w)], patch=patch)
    got = frames_of(out, off, 0, 3, h, w).cpu().numpy()
    ref = oracle.resize_u8_item(workloads.frames_np(it), idx, h, w, patch=patch)
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} bytes differ, first at {bad[0]}"


@pytest.mark.parametrize("name,specs", CASES, ids=[c[0] for c in CASES])
def test_resize_u8_small_cases_exact(name, specs):
    items, hosts = [], []
    for k, (n, H, W, idx, h, w) in enumerate(specs):
        it, fd = _video(400 + k, n, H, W)
        items.append((fd, np.asarray(idx, np.int32), h, w))
        hosts.append(workloads.frames_np(it))
    log(f"case {name}: {[(s[0], s[1], s[2], s[4], s[5]) for s in specs]}")
    out, off = run(items)
    for k, (fd, idx, h, w) in enumerate(items):
        got = frames_of(out, off, k, len(idx), h, w).cpu().numpy()
        ref = oracle.resize_u8_item(hosts[k], idx, h, w)
        diff = int((got != ref).sum())
        log(f"{name} item {k}: {diff} differing bytes of {ref.size}")
        assert diff == 0


def _sampled_workload_check(wl, n_check, seed):
    items = []
    for it in wl.items:
        if it.dims is not None:
            h, w = it.dims
        else:
            h, w = vp.vp_smart_resize_dims(it.H, it.W, 32, it.min_pixels, it.max_pixels)
        idx = vp.vp_sample_indices(it.n_src, vp.VP_SAMPLE_UNIFORM, it.sample["n"])
        items.append((workloads.frames_torch(it, DEV, chunk=32), idx, h, w))
    out, off = run(items, sentinel=4)
    rng = np.random.default_rng(seed)
    for _ in range(n_check):
        k = int(rng.integers(0, len(items)))
        fd, idx, h, w = items[k]
        m = int(rng.integers(0, len(idx)))
        got = frames_of(out, off, k, len(idx), h, w)[m].cpu().numpy()
        ref = oracle.resize_u8(workloads.frames_np(wl.items[k], [idx[m]])[0], h, w)
        diff = int((got != ref).sum())
        log(f"{wl.name[:3]} item {k} frame {m}: {diff} differing bytes")
        assert diff == 0
    del items, out


def test_resize_u8_rollout_workload_full_size():
    _sampled_workload_check(workloads.config(4), 6, 51)


def test_resize_u8_ragged_workload_full_size():
    _sampled_workload_check(workloads.config(3), 10, 52)


def test_resize_u8_patch14_widths():
    """Sizes on the patch-14 grid (multiples of 28): column bands of 64 that
    end in a 60-column band (252) or a 48-column one (112), so the stage
    leaves 45 and 36 dwords per band row."""
    specs = [(1, 333, 257, [0], 308, 252), (3, 70, 90, [2, 0, 1], 56, 112), (2, 720, 1280, [1, 0], 252, 448)]
    items, hosts = [], []
    for k, (n, H, W, idx, h, w) in enumerate(specs):
        it, fd = _video(470 + k, n, H, W)
        items.append((fd, np.asarray(idx, np.int32), h, w))
        hosts.append(workloads.frames_np(it))
    log(f"case patch14_widths: {[(s[0], s[1], s[2], s[4], s[5]) for s in specs]}")
    out, off = run(items, patch=14)
    for k, (fd, idx, h, w) in enumerate(items):
        got = frames_of(out, off, k, len(idx), h, w).cpu().numpy()
        ref = oracle.resize_u8_item(hosts[k], idx, h, w, patch=14)
        diff = int((got != ref).sum())
        log(f"patch14_widths item {k}: {diff} differing bytes of {ref.size}")
        assert diff == 0



# The matrix-core form at the edges of its shapes: 2, 4 and 8 loads per chunk
# (spans of up to 32, 64 and 128 pixels), windows on multiples of 16, 8 and 1,
# one product and two in the vertical pass, upscales, a frame of fewer rows
# than one chunk, last bands of 24, 20 and 12 columns, rows that are not 16-byte
# aligned, odd row lengths (every byte alignment), single frames
MM_CASES = [
    # H, W, h, w, patch
    (9, 7, 32, 32, 16),
    (40, 33, 96, 128, 16),
    (33, 61, 32, 64, 16),
    (101, 157, 96, 96, 16),
    (77, 190, 64, 96, 16),
    (181, 271, 64, 96, 16),
    (200, 301, 64, 128, 16),
    (120, 183, 64, 64, 16),
    (290, 365, 96, 128, 16),
    (290, 202, 96, 64, 16),
    (400, 441, 96, 96, 16),     # wide: windows of 128 pixels, 16-column bands
    (372, 373, 64, 64, 16),
    (120, 395, 64, 64, 16),     # wide at any pixel
    (301, 655, 84, 140, 14),
    (203, 199, 64, 64, 16),
    (330, 211, 64, 64, 16),
    (61, 117, 56, 56, 14),
    (150, 245, 56, 140, 14),
    (165, 260, 84, 84, 14),
]


@pytest.mark.parametrize("H,W,h,w,patch", MM_CASES)
def test_matrix_core_form_edges(H, W, h, w, patch):
    it, fd = _video(71, 2, H, W)
    src = workloads.frames_np(it)
    log(f"matrix-core {H}x{W} -> {h}x{w} patch {patch}")
    out, off = run([(fd, np.array([1, 0], np.int32), h, w)], patch=patch)
    got = frames_of(out, off, 0, 2, h, w).cpu().numpy()
    for k, f in enumerate([1, 0]):
        ref = oracle.resize_u8(src[f], h, w)
        bad = np.argwhere(got[k] != ref)
        assert bad.size == 0, f"frame {f}: {len(bad)} bytes differ, first at {bad[0]}"


# Batches whose launches are joined: the kernel of more loads, unaligned windows
# or two products runs items that alone take less
JOINED = [
    # patch, [(H, W, h, w)], {(source pixels per row, columns per workgroup)}
    ("every_form", 16, [c[:4] for c in MM_CASES if c[4] == 16], {(128, 32), (128, 16)}),
    ("every_form_patch14", 14, [c[:4] for c in MM_CASES if c[4] == 14], {(128, 32), (128, 16)}),
    ("loads", 16, [(40, 33, 96, 128), (101, 150, 64, 128)], {(64, 32)}),
    ("second_product", 16, [(96, 150, 96, 128), (400, 150, 96, 128)], {(64, 32)}),
    ("windows_on_8", 16, [(64, 100, 64, 96), (61, 360, 64, 128)], {(128, 32)}),
    ("windows_on_1", 16, [(61, 360, 64, 128), (64, 300, 64, 128), (90, 420, 64, 128)], {(128, 32)}),
    ("wide_windows_on_1", 16, [(120, 395, 64, 64), (100, 500, 64, 128)], {(128, 16)}),
]


@pytest.mark.parametrize("name,patch,specs,shapes", JOINED, ids=[c[0] for c in JOINED])
def test_joined_launches_give_the_same_bytes(name, patch, specs, shapes):
    items, hosts = [], []
    for k, (H, W, h, w) in enumerate(specs):
        it, fd = _video(520 + k, 2, H, W)
        items.append((fd, np.array([1, 0], np.int32), h, w))
        hosts.append(workloads.frames_np(it))
    launches = vp.vp_resize_kernels([vp.Item(f, i, h, w, patch) for f, i, h, w in items]).tolist()
    log(f"joined {name}: {launches}")
    assert len(launches) == len(shapes) and {(r[3], r[4]) for r in launches} == shapes
    assert all(r[0] == vp.VP_WRITER_MATRIX for r in launches)
    out, off = run(items, patch=patch)
    for k, (H, W, h, w) in enumerate(specs):
        got = frames_of(out, off, k, 2, h, w).cpu().numpy()
        for m, f in enumerate([1, 0]):
            bad = np.argwhere(got[m] != oracle.resize_u8(hosts[k][f], h, w))
            assert bad.size == 0, f"{H}x{W} -> {h}x{w}, frame {f}: {len(bad)} bytes differ, first at {bad[0]}"
