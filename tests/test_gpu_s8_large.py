"""S = 8 with B <= 4 above 4608 blocks, where a wavefront takes eight blocks.

The eight-block kernels against the FP64 oracle (empty supports and ragged
edges, both target layouts), with and without the argmax log, in graph replays
and under the tuned schedule of a batch, and over block counts around whole
stripes of the workgroup order.  The shared-memory argmax kernel, which runs one
block per wavefront at every size, is the bitwise reference.  The frames of the
other tests of this support lie below the line.
"""
import numpy as np
import pytest

import synth
from tests.kernel_trace import kernels_of
from tests.test_gpu_small_supports import exhaustive

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SPLITS = [(4, 2), (2, 3)]
# 70 x 76 = 5320 blocks, the last row and column of blocks short by a pixel
BLOCKS = (70, 76)


@pytest.fixture(scope="module")
def ctx():
    return fsr.Context(0)


def frame(B, kind, seed):
    h, w = BLOCKS[0] * B - 1, BLOCKS[1] * B - 1
    return synth.make_image(h, w, seed).astype(np.float32), synth.make_mask(kind, h, w, seed + 1)


def with_hole(mask, B):
    mask = mask.copy()
    mask[10 * B:30 * B, 20 * B:45 * B] = 0
    return mask


def dev(img, mask):
    return torch.from_numpy(img).to(DEV), torch.from_numpy(mask).to(DEV)


def one(ctx, ti, tm, B, L, iters, log=True, flags=0):
    p = fsr.make_params(block=B, border=L, iterations=iters, flags=flags)
    out = torch.full_like(ti, float("nan"))
    lg = torch.full((fsr.fsr_num_blocks(*ti.shape, B), max(iters, 1)), -1, dtype=torch.int16, device=DEV) if log else None
    fsr.fsr_reconstruct(ctx, ti, tm, out, p, lg)
    return out, lg


@pytest.mark.parametrize("B,L", SPLITS)
@pytest.mark.parametrize("hole,iters", [(False, 100), (True, 25)])
def test_against_the_oracle(ctx, B, L, hole, iters):
    print(f"\n[gpu case] S = 8 (B = {B}), {BLOCKS} blocks, hole {hole}, I = {iters}, every pixel", flush=True)
    img, mask = frame(B, "quarter", 610 + B)
    if hole:
        mask = with_hole(mask, B)
    ti, tm = dev(img, mask)
    ran = kernels_of(lambda: one(ctx, ti, tm, B, L, 1))
    assert ran == [f"fsr_plain_multi<8, {1 if B == 2 else 2}>"]
    _, gl, ol, n_empty = exhaustive(ctx, img, mask, B, L, iters, f"S8 B{B} large hole {hole}")
    if hole:
        empty = np.all(ol == 0xFFFF, axis=1)
        assert n_empty > 0 and np.all(gl[empty] == 0xFFFF)


@pytest.mark.parametrize("B,L", SPLITS)
def test_with_and_without_log(ctx, B, L):
    print(f"\n[gpu case] S = 8 (B = {B}), {BLOCKS} blocks, log and no log, one image and batched", flush=True)
    img, mask = frame(B, "uniform:0.4", 620 + B)
    ti, tm = dev(img, with_hole(mask, B))
    want, want_log = one(ctx, ti, tm, B, L, 60, flags=fsr.FSR_FLAG_LDS_ARGMAX)
    out, log = one(ctx, ti, tm, B, L, 60)
    assert torch.equal(out, want) and torch.equal(log, want_log)
    assert torch.equal(one(ctx, ti, tm, B, L, 60, log=False)[0], want)
    params = fsr.make_params(block=B, border=L, iterations=1)
    for sched in (fsr.make_schedule(1, 0, 10), fsr.make_schedule(2, 8, 5)):
        for with_log in (True, False):
            lg = torch.full_like(want_log, -1) if with_log else None
            item = fsr.BatchItem(ti, tm, torch.full_like(ti, float("nan")), 60, lg)
            fsr.fsr_reconstruct_batched(ctx, [item], params, fsr.Workspace(1, DEV), sched)
            assert torch.equal(item.out, want)
            assert lg is None or torch.equal(lg, want_log)


def test_graph_and_autotune(ctx):
    print("\n[gpu case] S = 8, a batch of more than 4608 blocks: graph replays and the tuned schedule", flush=True)
    sizes = [(150, 203, 40), (37, 50, 25), (1, 1, 10), (211, 251, 17), (8, 9, 0)]
    items, wants = [], []
    for i, (h, w, iters) in enumerate(sizes):
        ti, tm = dev(synth.make_image(h, w, 630 + i).astype(np.float32), synth.make_mask("quarter", h, w, 640 + i))
        wants.append(one(ctx, ti, tm, 4, 2, iters, flags=fsr.FSR_FLAG_LDS_ARGMAX))
        items.append(fsr.BatchItem(ti, tm, torch.empty_like(ti), iters, torch.empty_like(wants[-1][1])))
    p, ws = fsr.make_params(block=4, border=2), fsr.Workspace(len(items), DEV)

    def check(call):
        for item in items:
            item.out.fill_(-5.0)
            item.argmax_log.fill_(-1)
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        for item, (out, log) in zip(items, wants):
            assert torch.equal(item.out, out) and torch.equal(item.argmax_log, log)

    for sched in (fsr.make_schedule(1, 0, 10), fsr.make_schedule(2, 4, 5)):
        g = fsr.BatchGraph(ctx, items, p, ws, sched)
        for _ in range(3):
            check(g.launch)
        g.close()
    check(lambda: fsr.fsr_batch_autotune(ctx, items, p, ws))
    check(lambda: fsr.fsr_reconstruct_batched(ctx, items, p, ws))
    ran = kernels_of(lambda: fsr.fsr_reconstruct_batched(ctx, items, p, ws, fsr.make_schedule(1, 0, 10)))
    assert ran[-1] == "fsr_batched_grid_multi<1, 2>"


# around two, three and four stripes of 256 wavefronts of eight blocks, and the
# smallest count
@pytest.mark.parametrize("n", [4609, 6143, 6144, 6145, 6153, 6207, 8192, 8200])
def test_every_block_once(ctx, n):
    print(f"\n[gpu case] block order S 8, eight blocks per wavefront, n {n}", flush=True)
    img = torch.from_numpy(synth.make_image(4, 4 * n, 71).astype(np.float32) + 1.0).to(DEV)
    mask = torch.from_numpy(synth.make_mask("quarter", 4, 4 * n, 91)).to(DEV)
    want = torch.where(mask != 0, img, torch.zeros_like(img))
    assert torch.equal(one(ctx, img, mask, 4, 2, 0, log=False)[0], want)
    params = fsr.make_params(block=4, border=2, iterations=0)
    for waves in (1, 2, 4):
        item = fsr.BatchItem(img, mask, torch.full_like(img, -1.0), 0)
        fsr.fsr_reconstruct_batched(ctx, [item], params, fsr.Workspace(1, DEV), fsr.make_schedule(waves, 0, 1))
        assert torch.equal(item.out, want)
