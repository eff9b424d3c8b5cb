"""Small images at S = 32: a block on four wavefronts.

A one-image call of at most 512 blocks runs each block on four wavefronts,
by the same operations in the same order as the one-wavefront routine, which
the batched path always runs: outputs and argmax logs are held to bitwise
equality on both sides of that line.
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


def frame(h, w, kind):
    img = synth.make_image(h, w, 771).astype(np.float32)
    if kind == "none":
        return img, np.zeros((h, w), np.uint8)
    if kind == "flat":                     # every known pixel equals the mean
        return np.full((h, w), 255.0, np.float32), synth.quarter_mask(h, w, 772)
    if kind == "half":                     # blocks with and without known pixels
        mask = synth.quarter_mask(h, w, 772)
        mask[:, w // 3:] = 0
        return img, mask
    return img, synth.make_mask(kind, h, w, 772)


# 512 blocks (the last size on four wavefronts), 544 (the first on one), a
# single pixel, ragged edges, and the other block sizes of this support
CASES = [(64, 128, 4, 60, "quarter"), (65, 128, 4, 60, "quarter"), (1, 1, 4, 5, "uniform:0.0"),
         (37, 50, 2, 40, "uniform:0.9"), (90, 75, 6, 30, "macroblock"), (61, 67, 8, 30, "quarter"),
         (40, 120, 4, 25, "half"), (33, 30, 4, 10, "none"), (48, 44, 4, 25, "flat"), (30, 34, 4, 0, "quarter")]


@pytest.mark.parametrize("h,w,B,iters,kind", CASES)
def test_same_as_one_wavefront_per_block(ctx, h, w, B, iters, kind):
    print(f"\n[gpu case] {h}x{w} B={B} I={iters} {kind}: one-image against batched", flush=True)
    img, mask = frame(h, w, kind)
    ti, tm = torch.from_numpy(img).to(DEV), torch.from_numpy(mask).to(DEV)
    p = fsr.make_params(block=B, border=(32 - B) // 2, iterations=iters)
    n = fsr.fsr_num_blocks(h, w, B)
    got, ref = [], []
    for res, batched in ((got, False), (ref, True)):
        out = torch.full_like(ti, float("nan"))
        log = torch.full((n, max(iters, 1)), -1, dtype=torch.int16, device=DEV)
        if batched:
            fsr.fsr_reconstruct_batched(ctx, [fsr.BatchItem(ti, tm, out, iters, log)], p, fsr.Workspace(1, DEV),
                                        fsr.make_schedule(1, 0, 1))
        else:
            fsr.fsr_reconstruct(ctx, ti, tm, out, p, log)
        torch.cuda.synchronize()
        res += [out.cpu().numpy(), log.cpu().numpy()]
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0], ref[0])
    assert np.array_equal(got[1], ref[1])


def test_own_stream_equals_null_stream(ctx):
    """On a stream of the caller's own a block runs on one wavefront."""
    print("\n[gpu case] 61x128, null stream against own stream", flush=True)
    img, mask = frame(61, 128, "half")
    ti, tm = torch.from_numpy(img).to(DEV), torch.from_numpy(mask).to(DEV)
    p = fsr.make_params(iterations=45)
    torch.cuda.synchronize()
    res = []
    for stream in (None, torch.cuda.Stream()):
        out = torch.full_like(ti, float("nan"))
        log = torch.full((fsr.fsr_num_blocks(61, 128, 4), 45), -1, dtype=torch.int16, device=DEV)
        torch.cuda.synchronize()
        fsr.fsr_reconstruct(ctx, ti, tm, out, p, log, stream)
        torch.cuda.synchronize()
        res.append((out, log))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
