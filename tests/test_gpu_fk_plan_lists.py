"""Work lists only save time, so creating a plan takes and touches nothing that a plan
without lists does not need: where memory for them runs out the plan does without, and a
plan can be created, used and destroyed while a stream is under capture.

The lists leave out exact zeros; the kernels with and without them are compiled apart and may
round the last bit differently.  Both against the FP64 oracle: FP32 DFTs of 2^21 to 2^23 points
err by about 23 2^-24 = 1.4e-6 relative L2, bound 1e-5.
"""
import gc

import numpy as np
import pytest
import torch

from oracle import fk as ofk
from oracle.metrics import rel_l2
from paper_2608_28183_amd import nlos, runtime

from gpu_util import say

pytestmark = pytest.mark.gpu

POW2 = (64, 64, 256, 0.2, 0.2, 32.0, 2)
GENERAL = (72, 60, 250, 0.25, 0.25, 32.0, 2)


def desc(c):
    ny, nx, nt, w, h, bin_ps, pad = c
    return nlos.fk_desc(nx, ny, nt, w, h, bin_ps, pad=pad)


def inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.poisson(torch.full(c[:3], 0.3, device="cuda"), generator=gen)


def outputs(c):
    return torch.full(c[:3], -1.0, device="cuda"), torch.full(c[:2], -1.0, device="cuda")


def run(plan, c, tau):
    vol, img = outputs(c)
    plan(tau, vol, img, plan.workspace())
    torch.cuda.synchronize()
    return vol, img


# (descriptor, allocations of a creation: the plan, a general plan's tables, the lists on the
# host and on the device; how many of them a plan cannot do without)
@pytest.mark.parametrize("case,points,needed", [(POW2, 3, 1), (GENERAL, 4, 2)])
def test_a_plan_does_without_lists_where_memory_runs_out(lib, case, points, needed):
    ctx = runtime.Context(0)
    assert nlos.nlos_debug_fk_lists(desc(case)) > 0
    tau = inputs(case, 1)
    rv, ri = ofk.fk(tau.cpu().numpy().astype(np.float64), *case[3:])
    try:
        for k in range(points):
            say(f"fk plan lists {case}: allocation {k} fails")
            nlos.nlos_debug_fail_allocations_after(k, 1)
            if k < needed:
                with pytest.raises(nlos.NlosError) as e:
                    runtime.FkPlan(ctx, *case)
                assert e.value.status == nlos.NLOS_ERR_OUT_OF_MEMORY
                continue
            plan = runtime.FkPlan(ctx, *case)
            nlos.nlos_debug_fail_allocations(0)
            vol, img = run(plan, case, tau)
            assert rel_l2(vol.cpu().numpy(), rv) < 1e-5 and rel_l2(img.cpu().numpy(), ri) < 1e-5
    finally:
        nlos.nlos_debug_fail_allocations(0)


def test_a_plan_under_capture(lib):
    """Created, used and (another one) destroyed while its stream is captured in the strictest
    mode; the graph replays with new inputs."""
    say("fk plan under capture")
    s = torch.cuda.Stream()
    ctx = runtime.Context(0, s)
    gone = runtime.FkPlan(ctx, *POW2)
    ws = torch.empty(nlos.nlos_fk_desc_workspace_bytes(desc(POW2)), dtype=torch.uint8, device="cuda")
    tau = inputs(POW2, 1)
    vol, img = outputs(POW2)
    torch.cuda.synchronize()
    gc.collect()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s, capture_error_mode="global"):
        plan = runtime.FkPlan(ctx, *POW2)
        plan(tau, vol, img, ws)
        del gone
    ref_ctx = runtime.Context(0)
    ref_plan = runtime.FkPlan(ref_ctx, *POW2)
    for seed in (1, 2, 3):
        tau.copy_(inputs(POW2, seed))
        ref = run(ref_plan, POW2, tau)  # eager work between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(vol, ref[0]) and torch.equal(img, ref[1])


@pytest.mark.parametrize("how", ["stream", "graph"])
def test_a_graph_outlives_its_plan(lib, how):
    """The plan is destroyed after its call was captured (by the caller on the context's stream,
    or by nlos_fk_graph_create), and memory like its lists' is taken and filled, before the
    graph is replayed."""
    say("fk graph outlives its plan:", how)
    s = torch.cuda.Stream()
    ctx = runtime.Context(0, s)
    plan = runtime.FkPlan(ctx, *POW2)
    ws = plan.workspace()
    tau = inputs(POW2, 1)
    vol, img = outputs(POW2)
    torch.cuda.synchronize()
    if how == "stream":
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            plan(tau, vol, img, ws)
    else:
        g = plan.graph(tau, vol, img, ws)
        g.plan = None  # (the helper would keep it)
    del plan
    gc.collect()
    others = [runtime.FkPlan(ctx, 64, 64, 256, 0.02 + 0.03 * k, 0.4, 32.0, 2) for k in range(8)]
    ref_plan = runtime.FkPlan(ctx, *POW2)
    for seed in (2, 3, 4):
        tau.copy_(inputs(POW2, seed))
        torch.cuda.synchronize()  # (the context's stream does not wait for torch's)
        ref = run(ref_plan, POW2, tau)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(vol, ref[0]) and torch.equal(img, ref[1])
    if how == "graph":
        g.close()
    del others
