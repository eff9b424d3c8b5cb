"""Names of the library's kernels that a piece of code runs on the GPU, in the
order in which they ran, for tests of a route that results cannot show."""
from __future__ import annotations

import re

_NAME = re.compile(r"fsr_\w+(?:<[^>]*>)?")


def kernels_of(fn) -> list[str]:
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    found = []
    for e in prof.events():
        m = _NAME.search(e.name)
        if m and e.device_type != torch.autograd.DeviceType.CPU:
            found.append((e.time_range.start, m.group(0)))
    return [name for _, name in sorted(found)]
