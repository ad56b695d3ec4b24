"""f-k at the edge of 32-bit byte offsets: an unpadded scan whose x-IFFT output is a plane of
4.36 GB for the y-IFFT (520 rows of 512 x 2048 samples), beyond what the listed passes can
address, one of 4.19 GB just within it, and a padded scan whose planes of 512 rows (4.29 GB)
the resident passes reach to within 4 MB.  Against the same algorithm in 64-bit torch.

FP32 DFTs of N points in all err by about log2(N) 2^-24 relative L2, 1.8e-6 for the 2^30
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


def fk64(tau, wall_w, wall_h, bin_ps, pad):
    """The volume: scale, zero-padded 3D DFT, Stolt remap row by row, inverse, |.|^2."""
    ny, nx, nt = tau.shape
    My, Mx, Mt = pad * ny, pad * nx, pad * nt
    half = Mt // 2
    g = tau.double() * (torch.arange(nt, device="cuda", dtype=torch.float64) / (nt - 1))
    S = torch.fft.rfft(g, n=Mt, dim=2)[:, :, :half].contiguous()
    del g
    S = torch.fft.fft(torch.fft.fft(S, n=Mx, dim=1), n=My, dim=0)
    c = 0.5 * 299792458.0 * bin_ps * 1e-12
    X, Y = c * nx / wall_w * Mt / Mx * signed(Mx), c * ny / wall_h * Mt / My * signed(My)
    Z = torch.arange(half, device="cuda", dtype=torch.float64)
    zero = torch.zeros((), dtype=S.dtype, device="cuda")
    for i in range(My):
        q = torch.sqrt(X[:, None] ** 2 + Y[i] ** 2 + Z ** 2)
        i0 = q.floor().long().clamp(max=half - 1)
        fr = q - i0
        v = torch.gather(S[i], 1, i0) * (1.0 - fr) + torch.gather(S[i], 1, (i0 + 1).clamp(max=half - 1)) * fr
        S[i] = torch.where(q <= half - 1, v * (Z / q.clamp(min=1e-6)), zero)
    S = torch.fft.ifft(S, dim=1)[:, :nx].contiguous()
    S = torch.fft.ifft(S, dim=0)[:ny].contiguous()
    v = torch.fft.ifft(S, n=Mt, dim=2)[:, :, :nt]
    return v.real.square() + v.imag.square()


@pytest.mark.parametrize("ny,nx,nt,pad,listed", [(520, 512, 2048, 1, False), (512, 512, 2000, 1, True),
                                                 (256, 1024, 1024, 2, True)])
def test_fk_at_the_edge_of_32_bit_offsets(ctx, ny, nx, nt, pad, listed):
    say(f"fk {ny}x{nx}x{nt} pad {pad}")
    d = nlos.fk_desc(nx, ny, nt, 2.0, 2.0, 32.0, pad=pad)
    assert (nlos.nlos_debug_fk_lists(d) > 0) == listed
    gen = torch.Generator(device="cuda").manual_seed(11)
    tau = torch.poisson(torch.full((ny, nx, nt), 0.05, device="cuda"), generator=gen)
    tau[ny // 3, nx // 2, nt // 2] += 60.0
    plan = runtime.FkPlan(ctx, ny, nx, nt, 2.0, 2.0, 32.0, pad)
    vol = torch.full((ny, nx, nt), -1.0, device="cuda")
    img = torch.full((ny, nx), -1.0, device="cuda")
    plan(tau, vol, img, plan.workspace())
    ref = fk64(tau, 2.0, 2.0, 32.0, pad)
    e = float((vol.double() - ref).norm() / ref.norm())
    say("  rel_l2 %.3e" % e)
    assert e < 1e-5
    assert torch.equal(vol.amax(dim=2), img)
