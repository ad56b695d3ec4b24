"""Listed f-k passes that test_gpu_fk_lists.py does not reach: 256-point lines on the y axis
(the resident forward pass and y-IFFT) and unpadded scans, mixed radices and powers of two,
where half the depth samples are zero.  Every plan here has lists.  Against the FP64 oracle
from a workspace filled with NaNs; FP32 within 1e-5 (DFTs of up to 2^24 points err by about
24 2^-24 = 1.4e-6), BF16 storage within 10 u as in test_gpu_fk_prec.py.
"""
import numpy as np
import pytest
import torch

from oracle import fk as ofk
from oracle.metrics import rel_l2
from paper_2608_28183_amd import nlos, runtime

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# ny, nx, nt, wall_w, wall_h, bin_ps, pad, precision
CASES = [
    (128, 32, 512, 0.12, 0.3, 32.0, 2, "fp32"),
    (128, 64, 256, 0.1, 0.1, 32.0, 2, "fp32"),
    (120, 144, 600, 0.2, 0.3, 32.0, 1, "fp32"),
    (100, 128, 500, 0.2, 0.3, 32.0, 1, "fp32"),
    (128, 96, 300, 0.2, 0.2, 32.0, 1, "fp32"),
    (256, 32, 512, 0.1, 0.1, 32.0, 1, "fp32"),
    (32, 256, 400, 0.1, 0.1, 32.0, 1, "fp32"),
    (256, 32, 512, 0.1, 0.1, 32.0, 1, "bf16"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_fk_lists_routes(lib, case):
    ny, nx, nt, w, h, bin_ps, pad, prec = case
    say("fk lists routes", case)
    assert nlos.nlos_debug_fk_lists(nlos.fk_desc(nx, ny, nt, w, h, bin_ps, pad=pad, prec=prec)) > 0
    ctx = runtime.Context(0)
    rng = np.random.Generator(np.random.PCG64(3))
    tau = rng.poisson(0.05, (ny, nx, nt)).astype(np.float32)
    tau[ny // 3, nx // 2, nt // 2] += 60.0
    plan = runtime.FkPlan(ctx, ny, nx, nt, w, h, bin_ps, pad, prec)
    ws = plan.workspace()
    ws.fill_(0xFF)
    vol = torch.full((ny, nx, nt), -1.0, device="cuda")
    img = torch.full((ny, nx), -1.0, device="cuda")
    plan(to_dev(tau), vol, img, ws)
    rv, ri = ofk.fk(tau.astype(np.float64), w, h, bin_ps, pad)
    tol = 1e-5 if prec == "fp32" else 10 * 2.0 ** -8
    e_v, e_i = rel_l2(vol.cpu().numpy(), rv), rel_l2(img.cpu().numpy(), ri)
    say("  rel_l2 vol %.3e img %.3e" % (e_v, e_i))
    assert e_v < tol and e_i < tol
