"""f-k at the edge of 32-bit byte offsets: an unpadded scan whose x-IFFT output is a plane of
4.36 GB for the y-IFFT (520 rows of 512 x 2048 samples), beyond what the listed passes can
address, and one of 4.29 GB just within it.  Against the same algorithm in 64-bit torch.

FP32 DFTs of N points in all err by about log2(N) 2^-24 relative L2, 1.8e-6 for the 2^29
points here; a row read from the wrong place is an error of order 1.  Bound 1e-5.
"""
import pytest
import torch

from paper_2608_28183_amd import nlos, runtime

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(lib):
    return runtime.Context(0)


def signed(m):
    k = torch.arange(m, device="cuda", dtype=torch.float64)
    return torch.where(k < m // 2, k, k - m)


def fk64(tau, wall_w, wall_h, bin_ps):
    """The volume of an unpadded scan: scale, 3D DFT, Stolt remap row by row, inverse, |.|^2."""
    ny, nx, nt = tau.shape
    half = nt // 2
    g = tau.double() * (torch.arange(nt, device="cuda", dtype=torch.float64) / (nt - 1))
    S = torch.fft.rfft(g, dim=2)[:, :, :half].contiguous()
    del g
    S = torch.fft.fft(torch.fft.fft(S, dim=1), dim=0)
    c = 0.5 * 299792458.0 * bin_ps * 1e-12
    X, Y = c * nx / wall_w * nt / nx * signed(nx), c * ny / wall_h * nt / ny * signed(ny)
    Z = torch.arange(half, device="cuda", dtype=torch.float64)
    zero = torch.zeros((), dtype=S.dtype, device="cuda")
    for i in range(ny):
        q = torch.sqrt(X[:, None] ** 2 + Y[i] ** 2 + Z ** 2)
        i0 = q.floor().long().clamp(max=half - 1)
        fr = q - i0
        v = torch.gather(S[i], 1, i0) * (1.0 - fr) + torch.gather(S[i], 1, (i0 + 1).clamp(max=half - 1)) * fr
        S[i] = torch.where(q <= half - 1, v * (Z / q.clamp(min=1e-6)), zero)
    S = torch.fft.ifft(torch.fft.ifft(S, dim=1), dim=0)
    v = torch.fft.ifft(S, n=nt, dim=2)
    return v.real.square() + v.imag.square()


@pytest.mark.parametrize("ny,nx,nt,listed", [(520, 512, 2048, False), (512, 512, 2000, True)])
def test_fk_at_the_edge_of_32_bit_offsets(ctx, ny, nx, nt, listed):
    say(f"fk {ny}x{nx}x{nt} unpadded")
    d = nlos.fk_desc(nx, ny, nt, 2.0, 2.0, 32.0, pad=1)
    assert (nlos.nlos_debug_fk_lists(d) > 0) == listed
    gen = torch.Generator(device="cuda").manual_seed(11)
    tau = torch.poisson(torch.full((ny, nx, nt), 0.05, device="cuda"), generator=gen)
    tau[ny // 3, nx // 2, nt // 2] += 60.0
    plan = runtime.FkPlan(ctx, ny, nx, nt, 2.0, 2.0, 32.0, 1)
    vol = torch.full((ny, nx, nt), -1.0, device="cuda")
    img = torch.full((ny, nx), -1.0, device="cuda")
    plan(tau, vol, img, plan.workspace())
    ref = fk64(tau, 2.0, 2.0, 32.0)
    e = float((vol.double() - ref).norm() / ref.norm())
    say("  rel_l2 %.3e" % e)
    assert e < 1e-5
    assert torch.equal(vol.amax(dim=2), img)
