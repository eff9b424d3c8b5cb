"""Small calls against one another: what a call that leaves the device mostly
idle takes, measured as the best of several rounds.
"""
import time

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


def frame(rows, cols):
    img = torch.from_numpy(synth.make_image(4 * rows, 4 * cols, 1).astype(np.float32)).to(DEV)
    return img, torch.from_numpy(synth.quarter_mask(4 * rows, 4 * cols, 2)).to(DEV), torch.empty_like(img)


def best_us(*calls):
    """Each call's best round, the rounds taken in turn."""
    best = [float("inf")] * len(calls)
    for _ in range(15):
        for k, call in enumerate(calls):
            call()
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                call()
            torch.cuda.synchronize()
            best[k] = min(best[k], (time.perf_counter() - t) / 20 * 1e6)
    return best


def test_split_bf16_loop_beside_fp32(ctx):
    """The compensated model sum adds six of some 165 instructions to an
    iteration: 1024 blocks, one per SIMD, may take 1.09 times the FP32 call."""
    img, mask, out = frame(32, 32)
    fp32, bf16 = (fsr.make_params(iterations=200, dft=d) for d in (fsr.FSR_DFT_FP32, fsr.FSR_DFT_SPLIT_BF16))
    a, b = best_us(lambda: fsr.fsr_reconstruct(ctx, img, mask, out, fp32),
                   lambda: fsr.fsr_reconstruct(ctx, img, mask, out, bf16))
    print(f"\n[gpu case] 1024 blocks, I = 200: FP32 {a:.1f} us, split-bf16 {b:.1f} us", flush=True)
    assert b <= 1.09 * a


def test_queue_schedule_spreads_small_batches(ctx):
    """Four blocks per wavefront in turn, 64 and 512 wavefronts on 1024 SIMDs:
    both are bound by the latency of four blocks, so the larger batch may take
    1.1 times the smaller."""
    p, ws, sched = fsr.make_params(iterations=100), fsr.Workspace(1, DEV), fsr.make_schedule(4, 4, 2)
    batches = [[fsr.BatchItem(*frame(*blocks), 100)] for blocks in ((16, 16), (32, 64))]
    a, b = best_us(*(lambda items=items: fsr.fsr_reconstruct_batched(ctx, items, p, ws, sched) for items in batches))
    print(f"\n[gpu case] queue schedule, 256 blocks {a:.1f} us, 2048 blocks {b:.1f} us", flush=True)
    assert b <= 1.1 * a
