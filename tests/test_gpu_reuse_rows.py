"""The sequential variant in one launch against one launch per step.

Outside stream capture a call whose steps hold at most 512 blocks runs as
workgroups that each take a block row and wait for the row above; under
capture the same call is recorded as one launch per wavefront step.  Outputs
and argmax logs of the two have to be bitwise equal.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    return fsr.Context(0)


class Clip:
    def __init__(self, n, h, w, B, iters, seed, pad=0):
        self.params = fsr.make_params(block=B, border=(32 - B) // 2, iterations=iters)
        wide = (n, h, w + pad)
        self.images, self.masks = torch.zeros(wide, device=DEV), torch.zeros(wide, dtype=torch.uint8, device=DEV)
        self.outs = torch.full(wide, -7.0, device=DEV)
        for t in ("images", "masks", "outs"):
            setattr(self, t, getattr(self, t)[:, :, :w])
        for f in range(n):
            self.images[f] = torch.from_numpy(synth.make_image(h, w, seed + 2 * (f % 5)).astype(np.float32)).to(DEV)
            self.masks[f] = torch.from_numpy(synth.quarter_mask(h, w, seed + 1 + 2 * f)).to(DEV)
        self.log = torch.full((n * fsr.fsr_num_blocks(h, w, B) * max(iters, 1),), -1, dtype=torch.int16, device=DEV)

    def call(self, ctx):
        fsr.fsr_reconstruct_reuse_frames(ctx, self.images, self.masks, self.outs, self.params, 0.5, self.log)

    def result(self):
        torch.cuda.synchronize()
        got = self.outs.cpu().numpy().copy(), self.log.cpu().numpy().copy()
        self.outs.fill_(-7.0)
        self.log.fill_(-1)
        torch.cuda.synchronize()
        return got


def captured(ctx, clip):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        clip.call(ctx)
    g.replay()
    return clip.result()


def same(a, b):
    assert np.isfinite(a[0]).all() and (a[0] != -7.0).any()
    assert np.array_equal(a[0], b[0])
    assert np.array_equal(a[1], b[1])


# one block row, one column (every row waits for one block), a slope of 9, a
# clip with ragged edges in a wider buffer, and 512 and 516 blocks a step
CASES = [(1, 4, 130, 4, 12, 0), (1, 130, 4, 4, 12, 0), (1, 37, 50, 2, 15, 0), (3, 90, 75, 8, 20, 5),
         (1, 64, 64, 4, 33, 0), (128, 64, 64, 4, 3, 0), (129, 64, 64, 4, 3, 0), (2, 9, 9, 4, 0, 0)]


@pytest.mark.parametrize("n,h,w,B,iters,pad", CASES)
def test_rows_equal_steps(ctx, n, h, w, B, iters, pad):
    print(f"\n[gpu case] reuse rows: {n} x {h}x{w} B={B} I={iters} pad={pad}", flush=True)
    clip = Clip(n, h, w, B, iters, 930, pad)
    clip.call(ctx)
    a = clip.result()
    same(a, captured(ctx, clip))


def test_two_streams_at_once(ctx):
    print("\n[gpu case] reuse rows: two calls on two streams", flush=True)
    clips = [Clip(2, 72, 88, 4, 20, 950), Clip(3, 60, 100, 4, 20, 970)]
    refs = [captured(ctx, c) for c in clips]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(2):
        for c, s in zip(clips, streams):
            with torch.cuda.stream(s):
                c.call(ctx)
        for c, ref in zip(clips, refs):
            same(c.result(), ref)
