"""Creating an RSD plan waits for no work of the caller's stream.  Streams share a few hardware
queues, and on the one that the uploads take a copy runs behind that stream's work: of several
streams, at least one is still busy when the plan is there.
"""
import numpy as np
import pytest
import torch

from paper_2608_28183_amd import runtime

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["fp32", "bf16"])
def test_plan_creation_does_not_wait_for_the_stream(lib, kernel):
    a = torch.randn(8192, 8192, device="cuda")
    out = torch.empty_like(a)
    torch.mm(a, a, out=out)
    bins = np.arange(8, 16, dtype=np.int32)
    args = (16, 16, 128, 0.02, 0.02, 32.0, 2, bins, np.ones(8), 8, 0.1, 0.02)
    busy = 0
    for _ in range(6):
        s = torch.cuda.Stream()
        ctx = runtime.Context(0, s)
        runtime.RsdPlan(ctx, *args, kernel_prec=kernel)  # (first use)
        torch.cuda.synchronize()
        done = torch.cuda.Event()
        with torch.cuda.stream(s):
            for _ in range(60):
                torch.mm(a, a, out=out)
            done.record()
        plan = runtime.RsdPlan(ctx, *args, kernel_prec=kernel)
        pending = not done.query()
        busy += pending
        say(f"{kernel} plan created with its stream {'busy' if pending else 'idle'}")
        torch.cuda.synchronize()
        del plan
    assert busy > 0
