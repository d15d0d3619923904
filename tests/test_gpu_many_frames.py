"""The plans of batches of very many frames, which take other forms than the
same frames in a small batch: upscales on the general kernel beyond 2^20 work
units or the no-alloc entry's plan memory, and the uint8 writer's whole-frame
units and its second plan.  Two distinct source frames in turn, so the first
ones are compared with the oracle and every other with the first ones.
"""
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


@pytest.fixture(autouse=True)
def _free_memory():
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _video(H, W, seed):
    it = workloads.Item("video", 2, H, W, "uniform", seed, {"mode": "uniform", "n": 2})
    return workloads.frames_np(it), workloads.frames_torch(it, DEV)


def _all_equal_first(out, n):
    """Whether `out`, n equal parts, repeats its first part throughout."""
    v = out.view(n, -1)
    step = max(1, (1 << 30) // v.shape[1])
    return all(bool((v[a:a + step] == v[:1]).all()) for a in range(0, n, step))


@pytest.mark.parametrize("n,noalloc", [(1100000, False), (700000, True)])
def test_upscaled_frames_beyond_the_plan(n, noalloc):
    src, dev = _video(12, 12, 91)
    item = vp.Item(dev, np.arange(n, dtype=np.int32) % 2, 32, 32)
    small = vp.Item(dev, np.arange(2, dtype=np.int32), 32, 32)
    assert [int(r[0]) for r in vp.vp_batch_kernels([small])] == [vp.VP_KERNEL_XFIRST]
    print(f"[many frames] {n} upscaled, noalloc {noalloc}", flush=True)
    if noalloc:
        rows, ws = vp.vp_batch_layout([item])[2:]
        assert ws > vp.VP_NOALLOC_PLAN_BYTES
        out = torch.empty((rows, vp.VP_ROW), dtype=torch.bfloat16, device=DEV)
        vp.vp_preprocess_batch_noalloc([item], MEAN, STD, vp.VP_OUT_BF16, out)
    else:
        assert [int(r[0]) for r in vp.vp_batch_kernels([item])] == [vp.VP_KERNEL_GENERIC]
        out, _, _ = vp.preprocess([item], MEAN, STD, "bf16")
    torch.cuda.synchronize()
    out = out.view(torch.int16)
    assert _all_equal_first(out, out.shape[0] // 4)
    ref = oracle.preprocess_item(src, [0, 1], 32, 32, MEAN, STD)
    res = compare.check_bf16(out[:4].cpu().numpy().view(np.uint16), ref)
    assert res["ok"], res


# (H, W, h, w, frames) of each item, and the forms its plan takes: whole frames
# on the matrix cores (2^19 units of 128 rows are too many); the second plan,
# where dot-product items and whole frames of the others fill the list, and
# windows over 64 pixels go back to dot products; frames of many open rows on
# the tile kernel, which needs no units
WRITER = [
    ([(300, 60, 160, 32, 300000)], {vp.VP_WRITER_MATRIX}),
    ([(600, 60, 64, 32, 600000), (300, 60, 160, 32, 200000), (40, 160, 32, 32, 100000)], {vp.VP_WRITER_MATRIX, vp.VP_WRITER_DOT}),
    ([(12, 12, 32, 32, 1100000)], {vp.VP_WRITER_TILES}),
]


@pytest.mark.parametrize("specs,forms", WRITER, ids=["whole_frames", "second_plan", "tiles"])
def test_writer_plans_of_many_frames(specs, forms):
    items, hosts = [], []
    for k, (H, W, h, w, n) in enumerate(specs):
        src, dev = _video(H, W, 95 + k)
        items.append(vp.Item(dev, np.arange(n, dtype=np.int32) % 2, h, w))
        hosts.append(src)
    launches = vp.vp_resize_kernels(items).tolist()
    print(f"[many frames] writer {specs}: {launches}", flush=True)
    assert {r[0] for r in launches} == forms
    # no more matrix-core workgroups than whole frames need (in eights, a band of 32 columns each)
    matrix = sum(r[5] for r in launches if r[0] == vp.VP_WRITER_MATRIX)
    assert matrix <= sum(n + 8 for H, W, h, w, n in specs if W <= 64)
    assert not any(r[0] == vp.VP_WRITER_MATRIX and r[4] == 16 for r in launches)
    outs = vp.resize_u8(items)
    torch.cuda.synchronize()
    for out, src, (H, W, h, w, n) in zip(outs, hosts, specs):
        assert _all_equal_first(out, n // 2)
        ref = np.stack([oracle.resize_u8(f, h, w) for f in src])
        assert np.array_equal(out[:2].cpu().numpy(), ref), f"{H}x{W} -> {h}x{w}"
