"""Routes of the sequential variant: calls of fewer than 8 wavefront steps are
one launch per step and nothing else; longer ones of at most 512 blocks a step
run as rows in one launch, unless the device's memory pool refuses the rows'
counters; larger steps are one launch each.  Results on every route are bitwise
those of one launch per step, which stream capture always records.
"""
import ctypes

import numpy as np
import pytest

import synth
from tests.kernel_trace import kernels_of

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ROWS = ["fsr_reuse_rows_reset", "fsr_reuse_rows_s32"]


class Clip:
    """n frames of h x w blocks at B = 4 and what a call on them writes."""

    def __init__(self, n, h, w, iters, seed):
        h, w = 4 * h, 4 * w
        self.ctx = fsr.Context(0)
        self.params = fsr.make_params(iterations=iters)
        imgs = [synth.make_image(h, w, seed + 2 * (f % 5)).astype(np.float32) for f in range(n)]
        self.images = torch.from_numpy(np.stack(imgs)).to(DEV)
        self.masks = torch.from_numpy(np.stack([synth.quarter_mask(h, w, seed + 1 + 2 * f) for f in range(n)])).to(DEV)
        self.outs = torch.full((n, h, w), -7.0, device=DEV)
        self.log = torch.full((n * fsr.fsr_num_blocks(h, w, 4) * max(iters, 1),), -1, dtype=torch.int16, device=DEV)
        fsr.reconstruct(self.images[0], self.masks[0], self.params, ctx=self.ctx)   # the context's tables

    def call(self):
        fsr.fsr_reconstruct_reuse_frames(self.ctx, self.images, self.masks, self.outs, self.params, 0.5, self.log)

    def take(self):
        torch.cuda.synchronize()
        got = self.outs.clone(), self.log.clone()
        self.outs.fill_(-7.0)
        self.log.fill_(-1)
        torch.cuda.synchronize()
        return got

    def captured(self):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            self.call()
        g.replay()
        return self.take()


# (frames, block rows, block columns) and the kernels of the call: 1, 7 and 8
# steps in a row of blocks, 7 and 8 in a column (whose steps lie 5 apart, with
# empty ones between), a frame of 11 steps, and 512 and 516 blocks a step
@pytest.mark.parametrize("n,h,w,want", [
    (1, 1, 1, 1 * ["fsr_reuse_split4_s32"]), (1, 1, 7, 7 * ["fsr_reuse_split4_s32"]), (1, 1, 8, ROWS),
    (3, 7, 1, 7 * ["fsr_reuse_split4_s32"]), (1, 8, 1, ROWS), (2, 2, 6, ROWS), (128, 16, 16, ROWS), (129, 16, 16, None)])
def test_route_and_result(n, h, w, want):
    print(f"\n[gpu case] reuse routes: {n} frames of {h} x {w} blocks", flush=True)
    clip = Clip(n, h, w, 5, 940)
    clip.call()
    a = clip.take()
    names = kernels_of(clip.call)
    b, ref = clip.take(), clip.captured()
    print(f"[route] {names[:3]} ({len(names)})", flush=True)
    if want is None:      # per step: four wavefronts per block up to 512 blocks, one above
        assert set(names) == {"fsr_reuse_split4_s32", "fsr_reuse_s32"}
    else:
        assert names == want
    assert torch.isfinite(ref[0]).all()
    for got in (a, b):
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    if n > 1:             # a frame alone, which may take another route
        alone = fsr.reconstruct_reuse(clip.images[-1], clip.masks[-1], clip.params, 0.5, ctx=clip.ctx)
        assert torch.equal(a[0][-1], alone)


class MemPoolProps(ctypes.Structure):
    """hipMemPoolProps: pinned allocations on device 0, at most max_size bytes."""
    _fields_ = [("alloc_type", ctypes.c_int), ("handle_types", ctypes.c_int), ("location_type", ctypes.c_int),
                ("location_id", ctypes.c_int), ("security", ctypes.c_void_p), ("max_size", ctypes.c_size_t),
                ("reserved", ctypes.c_ubyte * 56)]


def test_pool_without_room():
    """The counters cannot be allocated: one launch per step, no error left."""
    print("\n[gpu case] reuse routes: a memory pool without room for the counters", flush=True)
    clip = Clip(2, 5, 9, 7, 960)
    ref = clip.captured()
    clip.call()
    clip.take()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    old, pool, ptr = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipDeviceGetMemPool(ctypes.byref(old), 0) == 0
    props = MemPoolProps(1, 0, 1, 0, None, 128)
    assert hip.hipMemPoolCreate(ctypes.byref(pool), ctypes.byref(props)) == 0
    assert hip.hipDeviceSetMemPool(0, pool) == 0
    try:
        assert hip.hipMallocAsync(ctypes.byref(ptr), ctypes.c_size_t(256), None) != 0   # it does refuse
        hip.hipGetLastError()
        names = kernels_of(clip.call)
        left = hip.hipGetLastError()
        got = clip.take()
    finally:
        assert hip.hipDeviceSetMemPool(0, old) == 0
        torch.cuda.synchronize()
        assert hip.hipMemPoolDestroy(pool) == 0
    assert names == 29 * ["fsr_reuse_split4_s32"] and left == 0
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    assert kernels_of(clip.call) == ROWS
    again = clip.take()
    assert torch.equal(again[0], ref[0]) and torch.equal(again[1], ref[1])
