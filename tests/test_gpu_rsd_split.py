"""The FP32 radial propagation as sums of bfloat16 products, at the edges of its steps (8
frequencies), rounds (two steps), depth tiles (32) and half chunks (32 pixels), against the
FP64 oracle.

Each FP32 operand is the exact sum of three bfloat16 values and the products left out are below
2^-24 of the term, so a propagated value carries FP32's own error: at most about N 2^-24 of
the sum of its N <= 2 Nf terms' magnitudes, in L2 well below 1e-5 for the N <= 60 here.
"""
import dataclasses

import numpy as np
import pytest
import torch

import scenes
from oracle import rsd as orsd
from oracle.metrics import rel_l2
from paper_2608_28183_amd import runtime

from gpu_util import rsd_plan_for, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return runtime.Context(0)


@pytest.mark.parametrize("nf,nd", [(1, 1), (7, 33), (8, 32), (9, 31), (16, 64), (17, 65), (24, 8), (30, 96)])
@pytest.mark.parametrize("ny,nx,pad", [(16, 8, 2), (8, 32, 1)])
def test_rsd_split_edges(ctx, ny, nx, pad, nf, nd):
    say(f"rsd split {ny}x{nx} pad {pad} nf {nf} nd {nd}")
    cfg = scenes.small_config(nx, ny, 128, bin_ps=64, pad=pad, n_depth=nd)
    p = scenes.rsd_params(cfg, nd)
    rng = np.random.Generator(np.random.PCG64(nf * 100 + nd))
    p = dataclasses.replace(p, freq_bins=np.arange(3, 3 + nf, dtype=np.int32),
                            weights=rng.uniform(0.2, 1, nf) * np.exp(1j * rng.uniform(0, 6, nf)))
    tau = rng.poisson(0.7, (ny, nx, 128)).astype(np.float32)
    plan, _ = rsd_plan_for(ctx, cfg, pad=pad, params=p)
    ws = plan.workspace()
    ws.fill_(0xFF)  # NaN
    vol = torch.full((ny, nx, nd), -1.0, device="cuda")
    img = torch.full((ny, nx), -1.0, device="cuda")
    plan(to_dev(tau), vol, img, ws)
    depths = p.depth0 + p.depth_step * np.arange(nd)
    rv, ri = orsd.rsd(tau.astype(np.float64), cfg.dx, cfg.dy, 64.0, pad, p.freq_bins, p.weights, depths)
    assert rel_l2(np.moveaxis(vol.cpu().numpy(), 2, 0), rv) < 1e-5
    assert rel_l2(img.cpu().numpy(), ri) < 1e-5
