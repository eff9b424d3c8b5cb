"""A small call on the default stream beside a large one on a stream of
PyTorch's own (which does not wait for the default stream): it has to finish
while the large call is still running, not behind it.

The bound is a quarter of the large call's duration; a workgroup that finds
room only when the large call's last blocks run takes nearly all of it, one of
a single wavefront about a hundredth.  Streams may share a hardware queue, in
which case their work runs in order, so the best of several streams counts.
"""
import time

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def frame(h, w, seed):
    img = torch.from_numpy(synth.make_image(h, w, seed).astype(np.float32)).to(DEV)
    return img, torch.from_numpy(synth.quarter_mask(h, w, seed + 1)).to(DEV), torch.empty_like(img)


@pytest.mark.parametrize("support", [32, 24, 16])
def test_small_call_beside_a_large_one(support):
    print(f"\n[gpu case] 64x64 beside 1080p, S {support}", flush=True)
    ctx = fsr.Context(0)
    large, small = frame(1080, 1920, 801), frame(64, 64, 803)
    p_large = fsr.make_params(block=4, border=(support - 4) // 2, iterations=400)
    p_small = fsr.make_params(block=4, border=(support - 4) // 2, iterations=100)
    durations, waits = [], []
    for _ in range(2):
        fsr.fsr_reconstruct(ctx, *small, p_small)
        torch.cuda.synchronize()
        t = time.perf_counter()
        fsr.fsr_reconstruct(ctx, *large, p_large)
        torch.cuda.synchronize()
        durations.append(time.perf_counter() - t)
    for _ in range(4):
        side = torch.cuda.Stream()
        fsr.fsr_reconstruct(ctx, *large, p_large, None, side)
        time.sleep(durations[1] / 8)           # the large call fills the device
        t = time.perf_counter()
        fsr.fsr_reconstruct(ctx, *small, p_small)
        torch.cuda.current_stream().synchronize()
        waits.append(time.perf_counter() - t)
        torch.cuda.synchronize()
    print(f"[overlap] large {durations[1] * 1e3:.2f} ms, small beside it {[round(w * 1e3, 3) for w in waits]} ms",
          flush=True)
    assert min(waits) < durations[1] / 4
