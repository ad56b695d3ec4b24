"""Which f-k plans run over work lists (no GPU): the listed passes address a plane of an
intermediate with 32-bit byte offsets, so no descriptor whose furthest sample lies beyond
them may have lists, and those within keep them where there are zeros to skip.
"""
import random

import pytest

from paper_2608_28183_amd import nlos

REACH = 0xFFFFFFF0  # bytes


def spans(ny, nx, nt, pad, es):
    """Bytes from a plane's first sample to the end of its last, for the y pass (in, out), the
    x-IFFT (in, out) and the y-IFFT (in, out): rows of the half spectrum and of the x-IFFT's
    output are followed by 256 bytes."""
    My, Mx = pad * ny, pad * nx
    half, xi = (Mx // 2 + 1) * nt + 256 // es, nx * nt + 256 // es
    return [es * ((rows - 1) * line + nt) for rows, line in
            ((ny, half), (My, half), (Mx, nt), (nx, nt), (My, xi), (ny, nx * nt))]


def zero_bytes(ny, nx, nt, wall_w, wall_h, bin_ps, pad, es):
    """Lower bound of the zeros of the remapped spectrum: the columns whose kz = 1 is already
    outside the frequency grid."""
    Mt, My, Mx = pad * nt, pad * ny, pad * nx
    h = 0.5 * 299792458.0 * bin_ps * 1e-12
    sx, sy = h / (wall_w / nx) * Mt / Mx, h / (wall_h / ny) * Mt / My
    lim = (Mt // 2 - 1) ** 2
    n = sum(1 for j in range(My // 2 + 1) for k in range(Mx // 2 + 1) if (sx * k) ** 2 + (sy * j) ** 2 + 1 > lim)
    return n * nt * es * 4


BEYOND = [(600, 600, 2048), (520, 512, 2048), (720, 600, 1500), (1000, 1000, 600), (768, 768, 1024),
          (800, 800, 1000), (900, 900, 1024), (512, 1800, 1024)]


@pytest.mark.parametrize("shape", BEYOND, ids=lambda s: "x".join(map(str, s)))
def test_no_lists_beyond_32_bit_offsets(shape):
    ny, nx, nt = shape
    assert max(spans(ny, nx, nt, 1, 8)) > REACH
    assert nlos.nlos_debug_fk_lists(nlos.fk_desc(nx, ny, nt, 2.0, 2.0, 32.0, pad=1)) == 0


@pytest.mark.parametrize("ny,nx,nt,pad", [(1024, 1024, 512, 1), (256, 256, 512, 2), (260, 360, 512, 2),
                                          (512, 512, 2000, 1)])
def test_lists_within_32_bit_offsets(ny, nx, nt, pad):
    assert max(spans(ny, nx, nt, pad, 8)) <= REACH
    assert zero_bytes(ny, nx, nt, 1.0, 1.0, 32.0, pad, 8) > 1 << 24
    assert nlos.nlos_debug_fk_lists(nlos.fk_desc(nx, ny, nt, 1.0, 1.0, 32.0, pad=pad)) > 0


@pytest.mark.parametrize("w,h", [(1e-310, 1.0), (1.0, 1e-312), (5e-324, 5e-324)])
def test_no_lists_where_the_ellipsoid_has_no_extent(w, h):
    """A wall so small that the ratio of bin to pitch overflows: accepted, but without bounds."""
    d = nlos.fk_desc(64, 64, 256, w, h, 32.0)
    assert nlos.nlos_fk_check(d) == nlos.NLOS_OK
    assert nlos.nlos_debug_fk_lists(d) == 0


def test_random_descriptors_stay_within_reach():
    """Over the accepted sizes: lists only where every listed pass stays within reach."""
    r = random.Random(5)
    smooth = [n for n in range(8, 2049, 2) if all(p in (2, 3, 5, 7, 11, 13) for p in factors(n))]
    listed = beyond = 0
    while listed < 30 or beyond < 30:
        pad = r.choice((1, 2))
        ny, nx, nt = (r.choice(smooth[len(smooth) // 2:]) // pad for _ in range(3))
        prec = r.choice(("fp32", "fp16")) if all(n & (n - 1) == 0 for n in (ny, nx, nt)) else "fp32"
        d = nlos.fk_desc(nx, ny, nt, r.uniform(0.5, 3.0), r.uniform(0.5, 3.0), r.choice((8.0, 16.0, 32.0)), pad=pad,
                         prec=prec)
        if ny * nx * nt > 1.2e9 or nlos.nlos_fk_check(d) != nlos.NLOS_OK:
            continue
        far = max(spans(ny, nx, nt, pad, 8 if prec == "fp32" else 4)) > REACH
        n = nlos.nlos_debug_fk_lists(d)
        assert not (far and n), (ny, nx, nt, pad, prec)
        listed += n > 0
        beyond += far


def factors(n):
    out, p = [], 2
    while n > 1:
        while n % p == 0:
            out.append(p)
            n //= p
        p += 1
    return out
