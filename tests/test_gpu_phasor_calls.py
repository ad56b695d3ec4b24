"""nlos_phasor_bin as a call: it enqueues and returns (its workspace grows without waiting for
the stream), it needs no memory of its own to succeed, and it can be captured.

Against the DFT of the oracle histogram (FP64), relative L2 within 1e-5 as in
test_gpu_phasor_tiles.py.
"""
import numpy as np
import pytest
import torch

import scenes
from oracle import rsd as orsd
from oracle.metrics import rel_l2
from paper_2608_28183_amd import nlos, runtime

from gpu_util import say

pytestmark = pytest.mark.gpu

NX, NY, NT = 32, 16, 256
BINS = [3 * f + 1 for f in range(20)]
DESC = nlos.bin_desc(NX, NY, NT, 7, 0, False)


def events(n, seed):
    ev = scenes.random_events(n, NX, NY, NT, 7, seed=seed, invalid_frac=0.05)
    return ev, torch.from_numpy(np.frombuffer(ev.tobytes(), dtype=np.uint8).copy()).cuda()


def outputs():
    return torch.full((NY, NX, len(BINS), 2), 3.0, device="cuda"), torch.full((1,), 5, dtype=torch.int64, device="cuda")


def check(ev, P, dropped):
    R, rd = orsd.phasor_from_events(ev["pixel"], ev["t_ps"], NX, NY, NT, 7, 0, BINS)
    got = torch.view_as_complex(P).cpu().numpy().astype(np.complex128)
    assert int(dropped.item()) == rd
    assert rel_l2(got, np.moveaxis(R, 0, 2)) < 1e-5


def test_the_call_does_not_wait_for_its_stream(lib):
    """Work is pending on the stream when the call asks for more workspace than the context
    has; it is still pending when the call returns."""
    s = torch.cuda.Stream()
    ctx = runtime.Context(0, s)
    plan = nlos.nlos_phasor_plan_create(ctx.handle, DESC, BINS)
    a = torch.randn(8192, 8192, device="cuda")
    out = torch.empty_like(a)
    jobs = [(*events(n, n), *outputs()) for n in (2000, 50000, 400000)]
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    for ev, d_ev, P, dropped in jobs:
        done = torch.cuda.Event()
        with torch.cuda.stream(s):
            for _ in range(40):
                torch.mm(a, a, out=out)
            done.record()
        nlos.nlos_phasor_bin(ctx.handle, plan, d_ev, len(ev), P, dropped)
        pending = not done.query()
        say(f"phasor_bin of {len(ev)} events returned with its stream {'busy' if pending else 'idle'}")
        torch.cuda.synchronize()
        assert pending
        check(ev, P, dropped)
    nlos.nlos_phasor_plan_destroy(plan)


def test_the_call_needs_no_memory(lib):
    """Allocations of a plan (handle, table, bins, tiles' table on the host and on the device)
    and of its first call (workspace): the first three are needed, the others save time."""
    ctx = runtime.Context(0)
    ev, d_ev = events(30000, 4)
    try:
        for k in range(6):
            say("phasor: allocation", k, "fails")
            nlos.nlos_debug_fail_allocations_after(k, 1)
            if k < 3:
                with pytest.raises(nlos.NlosError):
                    nlos.nlos_phasor_plan_create(ctx.handle, DESC, BINS)
                continue
            plan = nlos.nlos_phasor_plan_create(ctx.handle, DESC, BINS)
            P, dropped = outputs()
            nlos.nlos_phasor_bin(ctx.handle, plan, d_ev, len(ev), P, dropped)
            nlos.nlos_debug_fail_allocations(0)
            check(ev, P, dropped)
            nlos.nlos_phasor_plan_destroy(plan)
    finally:
        nlos.nlos_debug_fail_allocations(0)


def test_the_call_under_capture(lib):
    """Captured, replayed on new events, with eager calls of the same context that need more
    workspace between the replays."""
    say("phasor under capture")
    s = torch.cuda.Stream()
    ctx = runtime.Context(0, s)
    plan = nlos.nlos_phasor_plan_create(ctx.handle, DESC, BINS)
    n = 20000
    ev, d_ev = events(n, 1)
    P, dropped = outputs()
    torch.cuda.synchronize()
    nlos.nlos_phasor_bin(ctx.handle, plan, d_ev, n, P, dropped)
    torch.cuda.synchronize()
    check(ev, P, dropped)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        nlos.nlos_phasor_bin(ctx.handle, plan, d_ev, n, P, dropped)
    for seed in (2, 3, 4):
        ev, new = events(n, seed)
        d_ev.copy_(new)
        big, d_big = events(n * 4 ** seed, seed + 10)
        Pb, db = outputs()
        torch.cuda.synchronize()
        nlos.nlos_phasor_bin(ctx.handle, plan, d_big, len(big), Pb, db)
        torch.cuda.synchronize()
        check(big, Pb, db)
        g.replay()
        torch.cuda.synchronize()
        check(ev, P, dropped)
    nlos.nlos_phasor_plan_destroy(plan)
