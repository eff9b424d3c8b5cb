"""Large pinned host frames sent to an idle server are copied, and their blocks
reconstructed, in two parts: the result must be that of the one-image call.
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


# frames of more than 4 MiB with their masks; ragged; at S = 8 the first part's
# block count is no multiple of the eight blocks of a wavefront; one row of
# blocks; a first part that with its border is the whole frame
@pytest.mark.parametrize("block,border,h,w", [(4, 14, 861, 1027), (4, 6, 861, 1027), (4, 2, 861, 1029),
                                              (4, 10, 1300, 701), (4, 2, 3, 300001), (8, 12, 18, 50001)])
def test_two_parts_equal_one_image(ctx, block, border, h, w):
    print(f"[gpu case] serve parts S {block + 2 * border} {h} x {w}", flush=True)
    iters = 4
    img = torch.from_numpy(synth.make_image(h, w, 8).astype(np.float32))
    mask = torch.from_numpy(synth.make_mask("quarter", h, w, 9))
    params = fsr.make_params(block=block, border=border, iterations=iters)
    want = fsr.reconstruct(img.to(DEV), mask.to(DEV), params, ctx=ctx).cpu()
    pinned = (img.pin_memory(), mask.pin_memory())
    wide = torch.zeros((h, w + 5)).pin_memory()      # rows further apart than they are long
    wide[:, :w] = img
    wide_mask = torch.zeros((h, w + 5), dtype=torch.uint8).pin_memory()
    wide_mask[:, :w] = mask
    out = torch.empty((h, w)).pin_memory()
    with fsr.Server(ctx, params, fsr.make_server_config(hbm_budget=64 << 20)) as srv:
        for name, (f, m) in {"pinned": pinned, "strided": (wide[:, :w], wide_mask[:, :w]),
                             "pageable": (img, mask), "again": pinned}.items():
            ticket = srv.submit(f, m, iters)
            srv.wait(ticket, 20000)
            out.fill_(-1.0)
            srv.result(ticket, out)
            assert torch.equal(out, want), name
