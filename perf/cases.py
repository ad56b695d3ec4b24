"""Performance cases of the reconstruction library: the calls a program makes through
``paper_2608_28183_amd`` with its inputs in device memory and its plan, workspace and
outputs kept, at the sizes the configurations, tests and benchmark of this repository use.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare``
makes a case's inputs and handles, ``run`` is one pass through the public entry points,
``work`` the bytes and operations a pass cannot do without, and ``exact`` the same outputs
in 64 bits from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_28183_amd import nlos, runtime

C_LIGHT = 299_792_458.0

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------


def _fk(ny, nx, nt, bin_ps, wall_w, wall_h, pad=2, prec="fp32"):
    return dict(op="fk", ny=ny, nx=nx, nt=nt, bin_ps=bin_ps, wall_w=wall_w, wall_h=wall_h, pad=pad, prec=prec)


def _rsd(ny, nx, nt, bin_ps, wall_w, wall_h, n_depth, pad=2, data="fp32", kernel="fp32", sigma_s=2, sigma_t=0,
         depth_major=False):
    return dict(op="rsd", ny=ny, nx=nx, nt=nt, bin_ps=bin_ps, wall_w=wall_w, wall_h=wall_h, n_depth=n_depth,
                pad=pad, data=data, kernel=kernel, sigma_s=sigma_s, sigma_t=sigma_t, depth_major=depth_major)


def _bin(ny, nx, nt, bin_ps, events):
    return dict(op="bin", ny=ny, nx=nx, nt=nt, bin_ps=bin_ps, wall_w=1.0, wall_h=1.0, events=events)


def _phasor(ny, nx, nt, bin_ps, events, n_depth):
    return dict(op="phasor", ny=ny, nx=nx, nt=nt, bin_ps=bin_ps, wall_w=1.0, wall_h=1.0, events=events,
                n_depth=n_depth, pad=2)


def listed():
    return [
        # a coarse preview scan: the smallest call, launches and latency count
        dict(_fk(32, 32, 256, 32.0, 1.0, 1.0), name="fk_32x32x256"),
        # the small shape of the serving mix
        dict(_fk(64, 64, 512, 16.0, 1.0, 1.0), name="fk_64x64x512"),
        # a fine time axis: the middle shape of the serving mix, 2048-point columns
        dict(_fk(128, 128, 1024, 16.0, 1.0, 1.0), name="fk_128x128x1024"),
        # the benchmark's own volume, in the default storage and in the reduced one
        dict(_fk(256, 256, 512, 32.0, 1.0, 1.0), name="fk_256x256x512"),
        dict(_fk(256, 256, 512, 32.0, 1.0, 1.0, prec="fp16"), name="fk_256x256x512_fp16"),
        # the office scan: neither axis pads to a power of two
        dict(_fk(260, 360, 512, 32.0, 1.8, 1.3), name="fk_office_260x360x512"),
        # RSD of the same scans, the small one at serving rates
        dict(_rsd(64, 64, 512, 16.0, 1.0, 1.0, 64), name="rsd_64x64x512"),
        dict(_rsd(128, 128, 1024, 16.0, 1.0, 1.0, 64), name="rsd_128x128x1024"),
        # RSD with the reduced storage and kernel
        dict(_rsd(128, 128, 1024, 16.0, 1.0, 1.0, 64, data="bf16", kernel="bf16"), name="rsd_128x128x1024_bf16"),
        dict(_rsd(260, 360, 512, 32.0, 1.8, 1.3, 51), name="rsd_office_260x360x512"),
        # one acquisition of a photon-counting detector into its histogram
        dict(_bin(64, 64, 512, 16, 10_000_000), name="bin_64x64x512_1e7"),
        # a short exposure straight to phasors and on to the RSD volume, no histogram
        dict(_phasor(64, 64, 512, 16, 1_000_000, 64), name="phasor_rsd_64x64x512_1e6"),
    ]


def _smooth(n):
    for p in (2, 3, 5, 7, 11, 13):
        while n % p == 0:
            n //= p
    return n == 1


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _axis(rng, lo, hi, pad, pow2):
    """A length whose padded size the library takes: a power of two, or even after padding
    with prime factors up to 13 (odd itself now and then)."""
    while True:
        n = _log_int(rng, lo, hi)
        if pow2:
            return 2 ** int(round(math.log2(n)))
        if _smooth(n) and (pad * n) % 2 == 0:
            return n


def _scan(rng, side, tlo, thi, pad, tpad):
    """ny, nx, nt and the wall's sides: four grids in ten are powers of two throughout, the
    others have a power of two on some axes; the scan's sides differ by at most a factor 4."""
    p = [True] * 3 if rng.random() < 0.4 else [rng.random() < 0.3 for _ in range(3)]
    ny = _axis(rng, 16, side, pad, p[0])
    nx = _axis(rng, max(16, ny // 4), min(side, 4 * ny), pad, p[1])
    return ny, nx, _axis(rng, tlo, thi, tpad, p[2]), round(rng.uniform(0.6, 2.0), 3), round(rng.uniform(0.6, 2.0), 3)


def _all_pow2(*ns):
    return all(n & (n - 1) == 0 for n in ns)


def draw(rng):
    op = rng.choice(("fk", "fk", "fk", "rsd", "rsd", "rsd", "bin", "phasor"))
    bin_ps = rng.choice((8.0, 16.0, 32.0))
    pad = 1 if rng.random() < 0.2 else 2
    if op == "fk":
        while True:
            ny, nx, nt, w, h = _scan(rng, 256, 64, 1024, pad, pad)
            if pad ** 3 * ny * nx * nt <= (2 ** 28 if _all_pow2(ny, nx, nt) else 1.5e8):
                break
        prec = rng.choice(("fp32", "fp32", "fp32", "fp16", "bf16")) if _all_pow2(ny, nx, nt) else "fp32"
        return _fk(ny, nx, nt, bin_ps, w, h, pad, prec)
    if op == "rsd":
        while True:
            ny, nx, nt, w, h = _scan(rng, 256, 64, 1024, pad, 1)
            c = _rsd(ny, nx, nt, bin_ps, w, h, rng.randint(8, 80), pad)
            if pad * pad * ny * nx * len(_band(c)[0]) * c["n_depth"] <= 6e8:
                break
        if rng.random() < 0.25:
            c.update(sigma_s=1, sigma_t=1)
        c["depth_major"] = rng.random() < 0.25
        if _all_pow2(ny, nx, nt):
            p = rng.choice(("fp32", "fp32", "fp16", "bf16"))
            c.update(kernel=p, data=p if rng.random() < 0.7 else "fp32")
        return c
    if op == "bin":
        ny, nx = _log_int(rng, 16, 256), _log_int(rng, 16, 256)
        return _bin(ny, nx, _log_int(rng, 64, 1024), int(bin_ps), _log_int(rng, 10_000, 10_000_000))
    while True:
        ny, nx, nt, _, _ = _scan(rng, 128, 64, 1024, 2, 1)
        c = _phasor(ny, nx, nt, int(bin_ps), _log_int(rng, 10_000, 1_000_000), rng.randint(8, 64))
        if len(_band(c)[0]) * c["events"] <= 6e7:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

_SHARED = {}


def _context():
    """One library context, as a program keeps it."""
    if "ctx" not in _SHARED:
        _SHARED["ctx"] = runtime.Context(0, torch.cuda.current_stream())
    return _SHARED["ctx"]


def _c_dt(case):
    return C_LIGHT * case["bin_ps"] * 1e-12


def _depth_range(case):
    """Depths that the time axis covers with room at both ends."""
    z = case["nt"] * _c_dt(case) / 2
    return 0.3 * z, 0.75 * z


def _band(case):
    """DFT bins and Gaussian weights around the virtual wavelength max(4 dx, 8 c dt)."""
    nt, dx = case["nt"], case["wall_w"] / case["nx"]
    lam = max(4.0 * dx, 8.0 * _c_dt(case))
    kc = max(1, min(int(round(nt * _c_dt(case) / lam)), nt // 2 - 1))
    ks = np.arange(1, nt // 2)
    sigma = kc / 6.0 if kc >= 12 else 2.0
    keep = 2 * np.abs(ks - kc) <= kc if kc >= 12 else np.abs(ks - kc) <= 6
    kb = ks[keep].astype(np.int32)
    return kb, np.exp(-((kb - kc) ** 2) / (2.0 * sigma ** 2))


def _depths(case):
    z0, z1 = _depth_range(case)
    nd = case["n_depth"]
    return z0, (z1 - z0) / max(nd - 1, 1)


def _scene(case, seed, points):
    """Reflecting points in front of the wall: positions (x, y, z) and strengths."""
    r = np.random.Generator(np.random.PCG64(seed + 1))
    z0, z1 = _depth_range(case)
    w, h = case["wall_w"], case["wall_h"]
    return np.stack([r.uniform(-0.4 * w, 0.4 * w, points), r.uniform(-0.4 * h, 0.4 * h, points),
                     r.uniform(z0, z1, points), r.uniform(0.2, 1.0, points)], axis=1)


def _distances(case, p):
    """Distance of every scan point [ny][nx] from the point p, FP64 on the host."""
    x = (np.arange(case["nx"]) + 0.5) * case["wall_w"] / case["nx"] - case["wall_w"] / 2
    y = (np.arange(case["ny"]) + 0.5) * case["wall_h"] / case["ny"] - case["wall_h"] / 2
    return np.sqrt((x[None, :] - p[0]) ** 2 + (y[:, None] - p[1]) ** 2 + p[2] ** 2)


def _transient(case, seed):
    """Poisson photon counts of a confocal scan of the scene, float32 [ny][nx][nt]: each
    point returns a pulse of one bin's width that falls off with the fourth power of the
    distance, 50 photons at the strongest point's brightest bin, over a little background."""
    pts = _scene(case, seed, 16)
    t = torch.arange(case["nt"], device="cuda", dtype=torch.float32) + 0.5
    lam = torch.full((case["ny"], case["nx"], case["nt"]), 0.01, device="cuda")
    amp = [p[3] / _distances(case, p) ** 4 for p in pts]
    scale = 50.0 / max(a.max() for a in amp)
    for p, a in zip(pts, amp):
        tb = torch.from_numpy((2.0 * _distances(case, p) / _c_dt(case)).astype(np.float32)).cuda()
        g = t - tb[:, :, None]
        lam.add_(torch.from_numpy((a * scale).astype(np.float32)).cuda()[:, :, None] * g.square_().mul_(-0.5).exp_())
    gen = torch.Generator(device="cuda").manual_seed(seed + 17)
    return torch.poisson(lam, generator=gen)


def _events(case, seed):
    """Photon records (int32 pixel, uint32 picoseconds) as an int32 tensor [n][2]: 95 % from
    the scene's points with a bin of jitter, the rest uniform, in order of arrival."""
    n, nx, ny, nt = case["events"], case["nx"], case["ny"], case["nt"]
    pts = _scene(case, seed, 16)
    r = np.stack([_distances(case, p) for p in pts])                       # [points][ny][nx]
    cdf = np.cumsum((pts[:, 3, None, None] / r ** 4).ravel())
    gen = torch.Generator(device="cuda").manual_seed(seed + 29)
    u = torch.rand(n, device="cuda", dtype=torch.float64, generator=gen)
    k = torch.searchsorted(torch.from_numpy(cdf / cdf[-1]).cuda(), u).clamp_(max=cdf.size - 1)
    t = torch.from_numpy(2.0 * r.ravel() / C_LIGHT * 1e12).cuda()[k]
    t += torch.randn(n, device="cuda", dtype=torch.float64, generator=gen) * case["bin_ps"]
    back = torch.rand(n, device="cuda", generator=gen) < 0.05
    t = torch.where(back, torch.rand(n, device="cuda", dtype=torch.float64, generator=gen) * nt * case["bin_ps"], t)
    pix = torch.where(back, torch.randint(0, nx * ny, (n,), device="cuda", generator=gen), k % (nx * ny))
    return torch.stack([pix.int(), t.clamp_(min=0).int()], dim=1).contiguous()


def _rsd_plan(ctx, case, data="fp32", kernel="fp32"):
    bins, w = _band(case)
    d0, step = _depths(case)
    return runtime.RsdPlan(ctx, case["ny"], case["nx"], case["nt"], case["wall_w"] / case["nx"],
                           case["wall_h"] / case["ny"], case["bin_ps"], case["pad"], bins, w, case["n_depth"], d0,
                           step, sigma_s=case.get("sigma_s", 2), sigma_t=case.get("sigma_t", 0), data_prec=data,
                           kernel_prec=kernel, vol_depth_major=case.get("depth_major", False))


def prepare(case, seed):
    ctx = _context()
    ny, nx, nt = case["ny"], case["nx"], case["nt"]
    s = {"op": case["op"], "ctx": ctx}
    if case["op"] == "fk":
        s["plan"] = runtime.FkPlan(ctx, ny, nx, nt, case["wall_w"], case["wall_h"], case["bin_ps"], case["pad"],
                                   case["prec"])
        s["tau"], s["vol"] = _transient(case, seed), torch.empty((ny, nx, nt), device="cuda")
    elif case["op"] == "bin":
        s["events"], s["n"], s["bin_ps"] = _events(case, seed), case["events"], case["bin_ps"]
        s["hist"] = torch.empty((ny, nx, nt), device="cuda", dtype=torch.int32)
        s["dropped"] = torch.empty(1, device="cuda", dtype=torch.int64)
        return s
    else:
        nd = case["n_depth"]
        shape = (nd, ny, nx) if case.get("depth_major") else (ny, nx, nd)
        s["plan"] = _rsd_plan(ctx, case, case.get("data", "fp32"), case.get("kernel", "fp32"))
        s["vol"] = torch.empty(shape, device="cuda")
        if case["op"] == "rsd":
            s["tau"] = _transient(case, seed)
        else:
            bins, _ = _band(case)
            s["events"], s["n"] = _events(case, seed), case["events"]
            s["phasor_plan"] = _Phasor(ctx, nlos.bin_desc(nx, ny, nt, case["bin_ps"]), bins)
            s["phasor"] = torch.empty((ny, nx, len(bins), 2), device="cuda")
            s["dropped"] = torch.empty(1, device="cuda", dtype=torch.int64)
    s["img"] = torch.empty((ny, nx), device="cuda")
    s["ws"] = s["plan"].workspace()
    return s


class _Phasor:
    """A phasor plan's handle, destroyed with its owner."""

    def __init__(self, ctx, desc, bins):
        self.handle = nlos.nlos_phasor_plan_create(ctx.handle, desc, bins)

    def __del__(self):
        nlos.nlos_phasor_plan_destroy(self.handle)


def run(s):
    if s["op"] == "bin":
        runtime.bin_events(s["ctx"], s["events"], s["n"], s["hist"], s["bin_ps"], dropped=s["dropped"])
        return {"hist": s["hist"], "dropped": s["dropped"]}
    if s["op"] == "phasor":
        nlos.nlos_phasor_bin(s["ctx"].handle, s["phasor_plan"].handle, s["events"], s["n"], s["phasor"], s["dropped"])
        nlos.nlos_rsd_from_phasors(s["ctx"].handle, s["plan"].handle, s["phasor"], s["vol"], s["img"], s["ws"])
        return {"phasor": s["phasor"], "dropped": s["dropped"], "vol": s["vol"], "img": s["img"]}
    s["plan"](s["tau"], s["vol"], s["img"], s["ws"])
    return {"vol": s["vol"], "img": s["img"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def _fft_flops(n, lines):
    return 5.0 * n * math.log2(n) * lines


def work(case):
    ny, nx, nt = case["ny"], case["nx"], case["nt"]
    if case["op"] == "bin":  # records in, histogram out; an add per record
        return {"bytes": 8 * case["events"] + 4 * ny * nx * nt, "flops": case["events"]}
    My, Mx = case["pad"] * ny, case["pad"] * nx
    if case["op"] == "fk":  # transient in, volume and image out; the lines that are not known to be zero
        Mt = case["pad"] * nt
        flops = (_fft_flops(Mx, ny * nt / 2) + _fft_flops(My, (Mx // 2 + 1) * nt) + _fft_flops(Mt, (Mx // 2 + 1) * My)
                 + _fft_flops(Mx, My * nt) + _fft_flops(My, nx * nt) + _fft_flops(Mt, ny * nx))
        return {"bytes": 8 * ny * nx * nt + 4 * ny * nx, "flops": flops}
    # the transient or records, the kernel table up to its cutoff, volume and image
    nf, nd = len(_band(case)[0]), case["n_depth"]
    g = _geometry(case)
    table = (8 if case.get("kernel", "fp32") == "fp32" else 4) * (g["cut"] + 1) * nf * nd
    data = 8 * case["events"] + 8 * ny * nx * nf if case["op"] == "phasor" else 4 * ny * nx * nt
    flops = (16.0 * My * Mx * nf * nd + _fft_flops(Mx, ny * nf) + _fft_flops(My, Mx * nf) + _fft_flops(My, Mx * nd)
             + _fft_flops(Mx, ny * nd))
    flops += 8.0 * case["events"] * nf if case["op"] == "phasor" else _fft_flops(nt, ny * nx / 2)
    return {"bytes": data + table + 4 * ny * nx * (nd + 1), "flops": flops}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------


def _signed(m):
    k = torch.arange(m, device="cuda", dtype=torch.float64)
    return torch.where(k < m // 2, k, k - m)


def _exact_fk(case, tau):
    """Algorithms 1 and 2: scale, pad, 3D DFT, Stolt remap, inverse DFT, |.|^2."""
    ny, nx, nt, pad = case["ny"], case["nx"], case["nt"], case["pad"]
    My, Mx, Mt = pad * ny, pad * nx, pad * nt
    half = Mt // 2
    g = tau.double() * (torch.arange(nt, device="cuda", dtype=torch.float64) / (nt - 1))
    S = torch.fft.rfft(g, n=Mt, dim=2)[:, :, :half].contiguous()
    S = torch.fft.fft(torch.fft.fft(S, n=Mx, dim=1), n=My, dim=0)
    sx, sy = (_c_dt(case) / (2.0 * case["wall_%s" % a] / case["n%s" % b]) for a, b in (("w", "x"), ("h", "y")))
    # in units of the frequency bins
    X, Y = sx * half * _signed(Mx) / (Mx / 2), sy * half * _signed(My) / (My / 2)
    Z = torch.arange(half, device="cuda", dtype=torch.float64)
    for i in range(My):
        q = torch.sqrt(X[:, None] ** 2 + Y[i] ** 2 + Z[None, :] ** 2)
        jac = Z / q.clamp(min=1e-6)
        i0 = q.floor().long().clamp(max=half - 1)
        fr = q - i0
        v = torch.gather(S[i], 1, i0) * (1.0 - fr) + torch.gather(S[i], 1, (i0 + 1).clamp(max=half - 1)) * fr
        S[i] = torch.where(q <= half - 1, v * jac, torch.zeros((), dtype=v.dtype, device="cuda"))
    S = torch.fft.ifft(S, dim=1)[:, :nx].contiguous()
    S = torch.fft.ifft(S, dim=0)[:ny].contiguous()
    vol = torch.fft.ifft(S, n=Mt, dim=2)[:, :, :nt]
    vol = vol.real.square() + vol.imag.square()
    return {"vol": vol, "img": vol.amax(dim=2)}


def _geometry(case):
    """Radial sampling rules of the supplementary material."""
    My, Mx = case["pad"] * case["ny"], case["pad"] * case["nx"]
    dx, dy = case["wall_w"] / case["nx"], case["wall_h"] / case["ny"]
    ceil = lambda x: int(math.ceil(x - 1e-9 * abs(x)))  # noqa: E731
    pow2 = lambda n: 1 << max(0, (n - 1).bit_length())  # noqa: E731
    r_max = math.hypot(0.5 * Mx * dx, 0.5 * My * dy)
    rho_max = math.hypot(0.5 / dx, 0.5 / dy)
    lam_min = case["nt"] * _c_dt(case) / int(_band(case)[0].max())
    n_r = max(2, pow2(ceil(2.0 * case.get("sigma_s", 2) * r_max / lam_min) + 1))
    n_rho = pow2(ceil(2.0 * r_max * rho_max) + 1)
    cut_bin = min(rho_max, 0.5 * (n_r - 1) / r_max) * (n_rho - 1) / rho_max
    return dict(r_max=r_max, rho_max=rho_max, n_r=n_r, dr=r_max / (n_r - 1), n_rho=n_rho, cut_bin=cut_bin,
                cut=min(n_rho - 1, int(math.ceil(cut_bin))))


def _exact_rsd(case, P):
    """Algorithm 4 from the phasors P [ny][nx][Nf] with the radial kernel of Eq. 4-6."""
    ny, nx, pad, nd = case["ny"], case["nx"], case["pad"], case["n_depth"]
    My, Mx = pad * ny, pad * nx
    ss, st = case.get("sigma_s", 2), case.get("sigma_t", 0)
    bins, w = _band(case)
    g = _geometry(case)
    f64 = dict(device="cuda", dtype=torch.float64)
    kappa = torch.from_numpy(2.0 * np.pi * bins.astype(np.float64) / (case["nt"] * _c_dt(case))).cuda()
    d0, step = _depths(case)
    d = d0 + step * torch.arange(nd, **f64)
    r = torch.arange(g["n_r"], **f64) * g["dr"]
    q = torch.full_like(r, g["dr"])
    q[0] = q[-1] = 0.5 * g["dr"]
    rho = torch.arange(g["n_rho"], **f64) * g["rho_max"] / (g["n_rho"] - 1)
    B = 2.0 * math.pi * r * torch.special.bessel_j0(2.0 * math.pi * rho[:, None] * r)         # [rho][r]
    ph = ss * kappa[:, None, None] * torch.sqrt(r ** 2 + d[:, None] ** 2)                     # [f][d][r]
    K = torch.complex((q * ph.cos()).reshape(-1, r.numel()) @ B.T, (q * ph.sin()).reshape(-1, r.numel()) @ B.T)
    m = kappa[:, None] * (st * d)
    K = K.reshape(len(bins), nd, -1) * torch.complex(m.cos(), m.sin())[:, :, None]
    K[:, :, torch.arange(g["n_rho"], device="cuda") > g["cut_bin"] + 1e-9] = 0
    K = K.permute(2, 0, 1).contiguous()                                                       # [rho][f][d]
    Ph = torch.fft.fft(torch.fft.fft(P, n=Mx, dim=1), n=My, dim=0).reshape(My * Mx, -1)
    Ph = Ph * torch.from_numpy(w).cuda()
    dx, dy = case["wall_w"] / nx, case["wall_h"] / ny
    rt = torch.sqrt((_signed(My) / (My * dy))[:, None] ** 2 + (_signed(Mx) / (Mx * dx)) ** 2).reshape(-1)
    rt = rt * (g["n_rho"] - 1) / g["rho_max"]
    t = (g["cut_bin"] - rt) / 8.0
    a = torch.where(t >= 1, torch.ones_like(t), torch.where(t > 0, t * t * (3.0 - 2.0 * t), torch.zeros_like(t)))
    i0 = rt.floor().long().clamp(0, max(0, min(g["cut"] - 1, g["n_rho"] - 2)))
    i1 = (i0 + 1).clamp(max=g["cut"])
    al = rt - i0
    C = torch.zeros((My * Mx, nd), device="cuda", dtype=torch.complex128)
    n = max(1, (1 << 24) // (len(bins) * nd))
    for s in range(0, My * Mx, n):
        e = slice(s, min(My * Mx, s + n))
        h = K[i0[e]] * ((1.0 - al[e]) * a[e])[:, None, None] + K[i1[e]] * (al[e] * a[e])[:, None, None]
        C[e] = torch.where(a[e, None] > 0, (h * Ph[e][:, :, None]).sum(dim=1), C[e])
    I = torch.fft.ifft(torch.fft.ifft(C.reshape(My, Mx, nd), dim=0)[:ny], dim=1)[:, :nx]
    vol = I.abs()
    img = vol.amax(dim=2)
    return {"vol": vol.permute(2, 0, 1).contiguous() if case.get("depth_major") else vol.contiguous(), "img": img}


def _exact_hist(case, ev):
    ny, nx, nt = case["ny"], case["nx"], case["nt"]
    b = ev[:, 1].long() // int(case["bin_ps"])
    ok = (ev[:, 0] >= 0) & (ev[:, 0] < ny * nx) & (b < nt)
    hist = torch.bincount((ev[:, 0].long() * nt + b)[ok], minlength=ny * nx * nt).reshape(ny, nx, nt)
    return hist, (~ok).sum().reshape(1)


def exact(case, seed):
    if case["op"] == "fk":
        return _exact_fk(case, _transient(case, seed))
    bins = None if case["op"] == "bin" else torch.from_numpy(_band(case)[0].astype(np.int64)).cuda()
    if case["op"] == "rsd":
        return _exact_rsd(case, torch.fft.fft(_transient(case, seed).double(), dim=2)[:, :, bins])
    hist, dropped = _exact_hist(case, _events(case, seed))
    if case["op"] == "bin":
        return {"hist": hist.int(), "dropped": dropped}
    P = torch.fft.fft(hist.double(), dim=2)[:, :, bins]
    return {"phasor": torch.view_as_real(P).contiguous(), "dropped": dropped, **_exact_rsd(case, P)}
