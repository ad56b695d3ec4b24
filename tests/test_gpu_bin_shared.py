"""Accumulating binnings that share a counter or a phasor buffer across streams: every add
must arrive.  Two contexts on two streams, launches interleaved from the host.

Counts are exact.  A phasor is a sum of `rounds` equal contributions in FP32: relative L2
within rounds 2^-24 of them, 2.4e-5 for 400.
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

NX, NY, NT, N, ROUNDS = 16, 8, 64, 4000, 200


def events(seed):
    ev = scenes.random_events(N, NX, NY, NT, 7, seed=seed, invalid_frac=0.3)
    return ev, torch.from_numpy(np.frombuffer(ev.tobytes(), dtype=np.uint8).copy()).cuda()


def test_dropped_counter_shared_by_two_streams(lib):
    say("bin shared counter")
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [runtime.Context(0, s) for s in streams]
    ev, d_ev = events(1)
    ok = (ev["pixel"] >= 0) & (ev["pixel"] < NX * NY) & (ev["t_ps"] // 7 < NT)
    hists = [torch.zeros((NY, NX, NT), dtype=torch.int32, device="cuda") for _ in range(2)]
    dropped = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(ROUNDS):
        for c, h in zip(ctxs, hists):
            nlos.nlos_bin(c.handle, nlos.bin_desc(NX, NY, NT, 7, 0, True), d_ev, N, h, dropped)
    torch.cuda.synchronize()
    assert int(dropped.item()) == 2 * ROUNDS * int((~ok).sum())
    assert torch.equal(hists[0], hists[1]) and int(hists[0].sum()) == ROUNDS * int(ok.sum())


def test_phasors_shared_by_two_streams(lib):
    say("phasor shared buffer")
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [runtime.Context(0, s) for s in streams]
    ev, d_ev = events(2)
    bins = list(range(1, 10))
    plan = nlos.nlos_phasor_plan_create(ctxs[0].handle, nlos.bin_desc(NX, NY, NT, 7, 0, True), bins)
    P = torch.zeros((NY, NX, len(bins), 2), device="cuda")
    dropped = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    for _ in range(ROUNDS):
        for c in ctxs:
            nlos.nlos_phasor_bin(c.handle, plan, d_ev, N, P, dropped)
    torch.cuda.synchronize()
    R, rd = orsd.phasor_from_events(ev["pixel"], ev["t_ps"], NX, NY, NT, 7, 0, bins)
    got = torch.view_as_complex(P).cpu().numpy().astype(np.complex128)
    nlos.nlos_phasor_plan_destroy(plan)
    assert int(dropped.item()) == 2 * ROUNDS * rd
    assert rel_l2(got, 2 * ROUNDS * np.moveaxis(R, 0, 2)) < 2 * ROUNDS * 2.0 ** -24
