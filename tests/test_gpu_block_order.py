"""Workgroup order of the one-block-per-wavefront launches: every block of a
call is reconstructed exactly once, whatever their number.

With 0 iterations the output is the known pixels and 0 elsewhere, so a block
left out (its output keeps the fill value) shows at once; the exact result is
known without any reconstruction.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# around the eighths of a small call, one stripe (256) and two, and, at S = 8,
# where a wavefront takes eight blocks, 2048
COUNTS = [1, 7, 8, 9, 255, 256, 257, 511, 513, 775, 2047, 2049, 2065]


@pytest.fixture(scope="module")
def ctx():
    return fsr.Context(0)


@pytest.mark.parametrize("support", [8, 16, 24, 32])
def test_every_block_once(ctx, support):
    params = fsr.make_params(block=4, border=(support - 4) // 2, iterations=0)
    frames = []
    for i, n in enumerate(COUNTS):
        img = torch.from_numpy(synth.make_image(4, 4 * n, 70 + i).astype(np.float32) + 1.0).to(DEV)
        mask = torch.from_numpy(synth.make_mask("quarter", 4, 4 * n, 90 + i)).to(DEV)
        frames.append((img, mask, torch.where(mask != 0, img, torch.zeros_like(img))))
    for n, (img, mask, want) in zip(COUNTS, frames):
        print(f"[gpu case] block order S {support} n {n}", flush=True)
        out = torch.full_like(img, -1.0)
        fsr.fsr_reconstruct(ctx, img, mask, out, params)
        assert torch.equal(out, want), f"one image, {n} blocks"
        for waves in (1, 2, 4):
            out.fill_(-1.0)
            items = [fsr.BatchItem(img, mask, out, 0)]
            fsr.fsr_reconstruct_batched(ctx, items, params, fsr.Workspace(1, DEV), fsr.make_schedule(waves, 0, 1))
            assert torch.equal(out, want), f"batch, {n} blocks, {waves} wavefronts per group"
    items = [fsr.BatchItem(img, mask, torch.full_like(img, -1.0), 0) for img, mask, _ in frames]
    fsr.fsr_reconstruct_batched(ctx, items, params, fsr.Workspace(len(items), DEV))
    for item, (_, _, want) in zip(items, frames):
        assert torch.equal(item.out, want)
