"""f-k plans whose Stolt remap leaves much of the spectrum zero: bins long against the scan
pitch (or no padding in time) put columns beyond the frequency grid, and the passes then
run over lists of the tiles and columns that can be non-zero.  Everything against the FP64
oracle, from a workspace filled with NaNs: a sample that is read must have been written.

FP32 within the parity bar of the other f-k tests (relative L2 1e-4); FP16 / BF16 storage
within 10 u as derived in test_gpu_fk_prec.py.  The shapes take each listed kernel: 256- and
512-point lines of the resident and matrix-core passes, shorter lines, mixed radices, with
the bound at its extremes (a wall so small that only the axis kx = 0 survives; a depth
limit that ends inside a tile).
"""
import numpy as np
import pytest
import torch

import scenes
from oracle import fk as ofk
from oracle.metrics import rel_l2
from paper_2608_28183_amd import nlos, runtime

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# ny, nx, nt, wall_w, wall_h, bin_ps, pad, precision
CASES = [
    (64, 64, 256, 0.20, 0.20, 32.0, 2, "fp32"),
    (64, 64, 256, 0.004, 0.004, 32.0, 2, "fp32"),
    (128, 16, 512, 0.12, 0.8, 32.0, 2, "fp32"),
    (16, 128, 512, 0.8, 0.06, 32.0, 2, "fp32"),
    (16, 256, 256, 1.0, 0.05, 32.0, 2, "fp32"),
    (256, 16, 256, 0.06, 0.9, 32.0, 2, "fp32"),
    (128, 64, 512, 1.0, 1.0, 16.0, 1, "fp32"),
    (72, 60, 250, 0.25, 0.25, 32.0, 2, "fp32"),
    (35, 110, 300, 0.5, 0.11, 32.0, 2, "fp32"),
    (128, 64, 512, 0.5, 0.2, 32.0, 2, "fp16"),
    (128, 64, 512, 0.5, 0.2, 32.0, 2, "bf16"),
    (32, 256, 512, 1.0, 0.05, 32.0, 2, "fp16"),
    (64, 64, 512, 0.2, 0.2, 32.0, 2, "bf16"),
]
UNIT = {"fp16": 2.0 ** -11, "bf16": 2.0 ** -8}


@pytest.fixture(scope="module")
def ctx(lib):
    return runtime.Context(0)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_fk_lists(ctx, case):
    ny, nx, nt, w, h, bin_ps, pad, prec = case
    say("fk lists", case)
    rng = np.random.Generator(np.random.PCG64(3))
    tau = rng.poisson(0.05, (ny, nx, nt)).astype(np.float32)
    tau[ny // 3, nx // 2, nt // 2] += 60.0  # some structure over the noise
    plan = runtime.FkPlan(ctx, ny, nx, nt, w, h, bin_ps, pad, prec)
    ws = plan.workspace()
    ws.fill_(0xFF)  # NaN in every storage format
    vol = torch.full((ny, nx, nt), -1.0, device="cuda")
    img = torch.full((ny, nx), -1.0, device="cuda")
    plan(to_dev(tau), vol, img, ws)
    rv, ri = ofk.fk(tau.astype(np.float64), w, h, bin_ps, pad)
    assert rv.max() > 0
    tol = 1e-4 if prec == "fp32" else 10 * UNIT[prec]
    e_v, e_i = rel_l2(vol.cpu().numpy(), rv), rel_l2(img.cpu().numpy(), ri)
    say("  rel_l2 vol %.3e img %.3e" % (e_v, e_i))
    assert e_v < tol and e_i < tol
    if prec == "fp32":
        psi = torch.full((ny, nx, nt, 2), -1.0, device="cuda")
        ws.fill_(0xFF)
        nlos.nlos_fk_complex(ctx.handle, plan.handle, to_dev(tau), psi, ws)
        assert rel_l2(psi.square().sum(-1).cpu().numpy(), rv) < tol
