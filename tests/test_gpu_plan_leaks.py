"""Plans whose creation fails on the way, or that are created and destroyed, hold no device
memory afterwards."""
import pytest
import torch

from paper_2608_28183_amd import nlos, runtime

from gpu_util import say

pytestmark = pytest.mark.gpu

TIMES = 2000
SLACK = 8 << 20  # bytes (the tables left by 2000 plans are 40 MB)


@pytest.mark.parametrize("k", [3, 4])
def test_phasor_plans_leave_nothing(lib, k):
    """The k-th allocation of a creation fails: the host copy of the tiles' table, its device
    copy (before them: the plan, 16 KB of twiddles, 4 KB of bins)."""
    ctx = runtime.Context(0)
    desc = nlos.bin_desc(8, 8, 2048, 7)
    bins = list(range(1000))

    def create():
        try:
            nlos.nlos_phasor_plan_destroy(nlos.nlos_phasor_plan_create(ctx.handle, desc, bins))
        except nlos.NlosError as e:
            assert e.status in (nlos.NLOS_ERR_OUT_OF_MEMORY, nlos.NLOS_ERR_DEVICE)

    create()
    free0 = torch.cuda.mem_get_info()[0]
    try:
        for _ in range(TIMES):
            nlos.nlos_debug_fail_allocations_after(k, 1)
            create()
    finally:
        nlos.nlos_debug_fail_allocations(0)
    lost = free0 - torch.cuda.mem_get_info()[0]
    say(f"phasor plans, allocation {k} failing {TIMES} times: {lost} bytes lost")
    assert lost < SLACK
