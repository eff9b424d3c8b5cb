"""The server's copy in two parts: which frames take it, read from the kernels
that run, and what happens to requests queued behind such a frame.
"""
import numpy as np
import pytest

import synth
from tests.kernel_trace import kernels_of

torch = pytest.importorskip("torch")
import paper_2202_13926_amd as fsr  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    return fsr.Context(0)


def host_frame(h, w, seed):
    return (torch.from_numpy(synth.make_image(h, w, seed).astype(np.float32)),
            torch.from_numpy(synth.make_mask("quarter", h, w, seed + 1)))


def strided(t, pad):
    wide = torch.zeros((t.shape[0], t.shape[1] + pad), dtype=t.dtype).pin_memory()
    wide[:, :t.shape[1]] = t
    return wide[:, :t.shape[1]]


# launches of a frame sent alone to an idle server: pinned frames of more than
# 4 MiB are split; not so smaller ones, pageable or device frames, one row of
# blocks, or a first part that with its border is the whole frame
@pytest.mark.parametrize("block,border,h,w,where,launches", [
    (4, 14, 861, 1027, "pinned", 2), (4, 6, 861, 1027, "strided", 2), (4, 2, 861, 1029, "pinned", 2),
    (4, 6, 861, 1027, "pageable", 1), (4, 6, 861, 1027, "device", 1), (4, 6, 800, 1027, "pinned", 1),
    (4, 2, 3, 300001, "pinned", 1), (8, 12, 18, 50001, "pinned", 1)])
def test_which_frames_are_split(ctx, block, border, h, w, where, launches):
    print(f"\n[gpu case] serve parts: S {block + 2 * border}, {h} x {w} {where}", flush=True)
    img, mask = host_frame(h, w, 14)
    params = fsr.make_params(block=block, border=border, iterations=3)
    want = fsr.reconstruct(img.to(DEV), mask.to(DEV), params, ctx=ctx).cpu()
    send = {"pinned": lambda t: t.pin_memory(), "strided": lambda t: strided(t, 5), "pageable": lambda t: t,
            "device": lambda t: t.to(DEV)}[where]
    img, mask = send(img), send(mask)
    torch.cuda.synchronize()
    with fsr.Server(ctx, params, fsr.make_server_config(hbm_budget=64 << 20)) as srv:
        tickets = []

        def serve():
            tickets.append(srv.submit(img, mask, 3))
            srv.wait(tickets[-1], 20000)

        ran = [k for k in kernels_of(serve) if k.startswith("fsr_batched")]
        print(f"[route] {ran}", flush=True)
        got = torch.empty((h, w))
        srv.result(tickets[0], got)
    assert len(ran) == launches and len(set(ran)) == 1
    assert torch.equal(got, want)


@pytest.mark.parametrize("streams", [1, 2])
@pytest.mark.parametrize("border", [2, 6, 14])
def test_burst_behind_a_split_frame(ctx, streams, border):
    print(f"\n[gpu case] serve burst: S {4 + 2 * border}, {streams} streams", flush=True)
    sizes = [(1000, 1203, 30), (61, 83, 50), (900, 1001, 12), (5, 7, 3), (1000, 1203, 9), (120, 160, 0)]
    frames, wants = [], []
    for i, (h, w, iters) in enumerate(sizes):
        img, mask = host_frame(h, w, 30 + 2 * i)
        p = fsr.make_params(block=4, border=border, iterations=iters)
        wants.append(fsr.reconstruct(img.to(DEV), mask.to(DEV), p, ctx=ctx).cpu())
        frames.append((img.pin_memory(), mask.pin_memory(), iters))
    cfg = fsr.make_server_config(hbm_budget=128 << 20, max_inflight=16, max_batch=4, streams=streams)
    with fsr.Server(ctx, fsr.make_params(block=4, border=border), cfg) as srv:
        for _ in range(3):
            tickets = [srv.submit(*f) for f in frames]
            for k, (t, want) in enumerate(zip(tickets, wants)):
                srv.wait(t, 20000)
                got = torch.full(want.shape, -1.0)
                srv.result(t, got)
                assert torch.equal(got, want), f"frame {k}"
        st = srv.stats()
        assert st["completed"] == st["released"] == 3 * len(frames) and st["bytes_in_use"] == 0
