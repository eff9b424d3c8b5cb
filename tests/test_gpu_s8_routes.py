"""S = 8 with B <= 4: calls of up to 4608 blocks run one block per wavefront,
larger ones eight.  Both sides of the line, plain and batched, against the
shared-memory argmax kernel, which runs one block per wavefront at every size
and chooses the same bins: output and argmax log must agree bitwise.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# (height, width) in blocks and how many pixels the last row and column lack
SIZES = [((48, 96), (0, 0)),      # 4608
         ((11, 419), (0, 0)),     # 4609
         ((57, 83), (1, 1)),      # 4731, ragged
         ((1, 4615), (1, 0)),
         ((4617, 1), (0, 1))]


@pytest.fixture(scope="module")
def ctx():
    return fsr.Context(0)


def frame(h, w, mask, seed):
    img = torch.from_numpy(synth.make_image(h, w, seed).astype(np.float32)).to(DEV)
    m = torch.from_numpy(synth.make_mask(mask, h, w, seed + 1)).to(DEV)
    return img, m


def run_alone(ctx, img, mask, params, iters, block):
    n = fsr.fsr_num_blocks(*img.shape, block)
    out = torch.full_like(img, -1.0)
    log = torch.full((n, iters), -1, dtype=torch.int16, device=DEV)
    fsr.fsr_reconstruct(ctx, img, mask, out, params, log)
    return out, log


@pytest.mark.parametrize("block,border", [(4, 2), (2, 3)])
@pytest.mark.parametrize("blocks,short", SIZES)
def test_one_image(ctx, block, border, blocks, short):
    iters = 23
    h, w = (n * block - s for n, s in zip(blocks, short))
    print(f"[gpu case] S 8 routes B {block} {h} x {w}", flush=True)
    img, mask = frame(h, w, "quarter", 31)
    mask[h // 3: h // 3 + 24, : w // 2] = 0   # blocks without a known pixel too
    kw = dict(block=block, border=border, iterations=iters)
    out, log = run_alone(ctx, img, mask, fsr.make_params(**kw), iters, block)
    want, want_log = run_alone(ctx, img, mask, fsr.make_params(flags=fsr.FSR_FLAG_LDS_ARGMAX, **kw), iters, block)
    assert torch.equal(out, want) and torch.equal(log, want_log)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("waves,chunk", [(1, 0), (4, 0), (2, 3)])
def test_batch(ctx, large, waves, chunk):
    print(f"[gpu case] S 8 routes batch large {large} waves {waves} chunk {chunk}", flush=True)
    sizes = [(61, 83, 19), (5, 3, 40), (1, 1, 7), (64, 250, 11)] + ([(230, 251, 19)] if large else [])
    items, wants = [], []
    for i, (h, w, iters) in enumerate(sizes):
        img, mask = frame(h, w, "uniform:0.4", 50 + 3 * i)
        flag = fsr.make_params(block=4, border=2, iterations=iters, flags=fsr.FSR_FLAG_LDS_ARGMAX)
        wants.append(run_alone(ctx, img, mask, flag, iters, 4))
        log = torch.full_like(wants[-1][1], -1)
        items.append(fsr.BatchItem(img, mask, torch.full_like(img, -1.0), iters, log))
    params = fsr.make_params(block=4, border=2, iterations=1)
    fsr.fsr_reconstruct_batched(ctx, items, params, fsr.Workspace(len(items), DEV),
                                fsr.make_schedule(waves, chunk, 4))
    for item, (out, log) in zip(items, wants):
        assert torch.equal(item.out, out) and torch.equal(item.argmax_log, log)
