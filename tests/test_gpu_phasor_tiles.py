"""Phasor binning by pixel tiles at the edges of its tiles and splits, and the plans that keep
the per-event atomics, against the DFT of the oracle histogram (FP64).

A phasor is a sum over the bins of count times a unit twiddle, the twiddles rounded once
(2^-24) and the FP32 sums of at most nt terms: relative L2 within 1e-5 as in
test_gpu_phasor_bin.py.
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

# nx, ny, nt, frequencies, events
CASES = [
    (1, 1, 4, 1, 10),              # one pixel, one row block split over all the waves
    (16, 1, 512, 4, 5000),         # a full tile of 16 pixels, 8 of 16 rows
    (17, 3, 512, 8, 20000),        # a tile of 3 pixels at the end, one whole row block
    (9, 7, 514, 9, 20000),         # bins not a multiple of 4, rows a little over a block
    (40, 5, 60, 13, 30000),        # several blocks of pixels per tile, 60 bins a row of 64 + 4
    (8, 8, 61, 24, 30000),         # odd bins at the edge of the row stride
    (8, 5, 1024, 129, 30000),      # more units than waves
    (5, 5, 1500, 40, 30000),
    (5, 3, 2048, 100, 50000),      # 8 pixels a tile
    (64, 64, 512, 39, 300000),     # many tiles, long chunks
    (96, 96, 1024, 40, 1000),      # few events on a large plan: atomics
    (300, 300, 2048, 2, 400000),   # more tiles than the tiled path takes: atomics
]


@pytest.fixture(scope="module")
def ctx(lib):
    return runtime.Context(0)


@pytest.mark.parametrize("nx,ny,nt,nf,n", CASES)
@pytest.mark.parametrize("accumulate", [False, True])
def test_phasor_tiles(ctx, nx, ny, nt, nf, n, accumulate):
    say(f"phasor tiles {nx}x{ny}x{nt} nf={nf} n={n} accumulate={accumulate}")
    ev = scenes.random_events(n, nx, ny, nt, 7, seed=nt + nf, invalid_frac=0.05)
    bins = [(5 * f + 1) % nt for f in range(nf)]
    plan = nlos.nlos_phasor_plan_create(ctx.handle, nlos.bin_desc(nx, ny, nt, 7, 0, accumulate), bins)
    d_ev = torch.from_numpy(np.frombuffer(ev.tobytes(), dtype=np.uint8).copy()).cuda()
    P = torch.full((ny, nx, nf, 2), 3.0, device="cuda")
    dropped = torch.full((1,), 5, dtype=torch.int64, device="cuda")
    nlos.nlos_phasor_bin(ctx.handle, plan, d_ev, n, P, dropped)
    R, rd = orsd.phasor_from_events(ev["pixel"], ev["t_ps"], nx, ny, nt, 7, 0, bins)
    got = torch.view_as_complex(P).cpu().numpy().astype(np.complex128)
    nlos.nlos_phasor_plan_destroy(plan)
    want = np.moveaxis(R, 0, 2) + ((3 + 3j) if accumulate else 0)
    assert int(dropped.item()) == rd + (5 if accumulate else 0)
    assert rel_l2(got, want) < 1e-5
