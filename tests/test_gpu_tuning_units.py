"""Tuned schedules at S = 8 with B <= 4: batches of up to 4608 blocks run one
block per wavefront, larger ones eight, in another kernel, and a schedule tuned
for one is not applied to the other although their work is alike.  The key of
the larger ones is that of schedules saved before there was such a line.
"""
import json

import numpy as np
import pytest

import synth
from tests.kernel_trace import kernels_of

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ITERS = 25
SMALL, LARGE = (67, 68), (69, 68)   # blocks at B = 4: 4556 and 4692, work of one octave


def batch(blocks):
    h, w = 4 * blocks[0], 4 * blocks[1]
    img = torch.from_numpy(synth.make_image(h, w, 17).astype(np.float32)).to(DEV)
    mask = torch.from_numpy(synth.quarter_mask(h, w, 18)).to(DEV)
    return [fsr.BatchItem(img, mask, torch.empty_like(img), ITERS)]


def test_schedules_of_the_two_kernels_are_kept_apart():
    print("\n[gpu case] tuned schedules on both sides of 4608 blocks", flush=True)
    params, ws = fsr.make_params(block=4, border=2, iterations=ITERS), fsr.Workspace(1, DEV)
    small, large = batch(SMALL), batch(LARGE)
    keys = []
    for items in (small, large):
        ctx = fsr.Context(0)
        fsr.fsr_batch_autotune(ctx, items, params, ws)
        entries = json.loads(fsr.fsr_batch_tuning_export(ctx))["entries"]
        assert len(entries) == 1
        keys.append(entries[0][0])
    octave, octave_small = ((b[0] * b[1] * (ITERS + 8)).bit_length() - 1 for b in (LARGE, SMALL))
    assert octave == octave_small
    assert keys[1] == octave << 48 | 8 << 40 | ITERS
    head = json.loads(fsr.fsr_batch_tuning_export(ctx))
    grid_small, grid_large = "fsr_batched_grid_sg<1, 8>", "fsr_batched_grid_multi<1, 2>"
    for key, names in ((keys[0], ("fsr_batched_sg<4, 8>", grid_large)), (keys[1], (grid_small, "fsr_batched_multi<4, 2>"))):
        ctx = fsr.Context(0)
        fsr.fsr_batch_tuning_import(ctx, json.dumps({**head, "entries": [[key, 4, 4, 2]]}))
        for items, want in zip((small, large), names):
            fsr.fsr_reconstruct_batched(ctx, items, params, ws)
            ran = kernels_of(lambda: fsr.fsr_reconstruct_batched(ctx, items, params, ws))
            print(f"[route] key {key:#x}: {ran}", flush=True)
            assert ran[-1] == want
