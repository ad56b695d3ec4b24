"""The z-IFFT's image where a line takes one wave, two, four or more (mixed-radix lengths):
the maximum of every volume line, bit for bit."""
import pytest
import torch

from paper_2608_28183_amd import runtime

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return runtime.Context(0)


@pytest.mark.parametrize("nt", [250, 260, 390, 520, 600, 1000, 1500, 2000])
def test_image_is_the_maximum_of_each_line(ctx, nt):
    say("fk zi image", nt)
    gen = torch.Generator(device="cuda").manual_seed(nt)
    tau = torch.poisson(torch.full((10, 12, nt), 0.5, device="cuda"), generator=gen)
    plan = runtime.FkPlan(ctx, 10, 12, nt, 1.0, 1.0, 32.0, 2)
    vol = torch.full((10, 12, nt), -1.0, device="cuda")
    img = torch.full((10, 12), -1.0, device="cuda")
    plan(tau, vol, img, plan.workspace())
    assert float(vol.amax()) > 0
    assert torch.equal(vol.amax(dim=2), img)
