"""The FP32 radial propagation at FP32's own error, tight enough to tell six bfloat16 products
from fewer (test_rsd_split_model.py): transforms of log2(128) + 2 log2(My Mx) <= 25 stages and
sums of up to 60 terms, each rounding 2^-24, give (25 + sqrt(60)) 2^-24 = 2e-6 relative L2;
three products alone would lose 4e-6.
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


@pytest.mark.parametrize("nf,nd", [(1, 1), (7, 33), (16, 64), (17, 65), (30, 96)])
@pytest.mark.parametrize("ny,nx,pad", [(16, 8, 2), (8, 32, 1)])
def test_rsd_split_bound(lib, ny, nx, pad, nf, nd):
    ctx = runtime.Context(0)
    cfg = scenes.small_config(nx, ny, 128, bin_ps=64, pad=pad, n_depth=nd)
    p = scenes.rsd_params(cfg, nd)
    rng = np.random.Generator(np.random.PCG64(nf * 100 + nd))
    p = dataclasses.replace(p, freq_bins=np.arange(3, 3 + nf, dtype=np.int32),
                            weights=rng.uniform(0.2, 1, nf) * np.exp(1j * rng.uniform(0, 6, nf)))
    tau = rng.poisson(0.7, (ny, nx, 128)).astype(np.float32)
    plan, _ = rsd_plan_for(ctx, cfg, pad=pad, params=p)
    vol = torch.full((ny, nx, nd), -1.0, device="cuda")
    plan(to_dev(tau), vol, None, plan.workspace())
    depths = p.depth0 + p.depth_step * np.arange(nd)
    rv, _ = orsd.rsd(tau.astype(np.float64), cfg.dx, cfg.dy, 64.0, pad, p.freq_bins, p.weights, depths)
    e = rel_l2(np.moveaxis(vol.cpu().numpy(), 2, 0), rv)
    say(f"rsd split bound {ny}x{nx} pad {pad} nf {nf} nd {nd}: {e:.2e}")
    assert e < 2e-6
