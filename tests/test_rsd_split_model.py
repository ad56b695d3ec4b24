"""What the FP32 propagation's six bfloat16 products are worth, on a CPU model of its sum: six
keep FP32's error, three would not, and the bound of test_gpu_rsd_split_bound.py tells them
apart.
"""
import numpy as np
import pytest

BOUND = 2e-6


def bf16(x):
    """The bfloat16 nearest to float32 x (to nearest even), as float32."""
    u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def parts(x):
    out = []
    for _ in range(3):
        p = bf16(x)
        out.append(p.astype(np.float64))
        x = (x - p).astype(np.float32)
    assert not x.any()  # three parts are the value
    return out


def product_error(products, n, seed):
    """Relative L2 error of sums of n complex FP32 products made of the given part products (in
    64 bits: what the parts leave out, not how they are added)."""
    r = np.random.Generator(np.random.PCG64(seed))
    z = r.standard_normal((2, 4096, n)).astype(np.float32)
    k = r.standard_normal((2, 4096, n)).astype(np.float32)
    zp, kp = [parts(c) for c in z], [parts(c) for c in k]
    mul = lambda a, b: sum(zp[a][i] * kp[b][j] for i, j in products)  # noqa: E731
    got = np.stack([(mul(0, 0) - mul(1, 1)).sum(-1), (mul(0, 1) + mul(1, 0)).sum(-1)])
    z, k = z.astype(np.float64), k.astype(np.float64)
    ref = np.stack([(z[0] * k[0] - z[1] * k[1]).sum(-1), (z[0] * k[1] + z[1] * k[0]).sum(-1)])
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


SIX = [(0, 0), (0, 1), (1, 0), (0, 2), (1, 1), (2, 0)]


@pytest.mark.parametrize("n", [1, 7, 16, 30])
def test_six_products_keep_fp32(n):
    assert product_error(SIX, n, n) < 2.0 ** -24


@pytest.mark.parametrize("n", [1, 7, 16, 30])
def test_fewer_products_fail_the_bound(n):
    assert product_error(SIX[:3], n, n) > BOUND
    for left_out in SIX[3:]:
        assert product_error([p for p in SIX if p != left_out], n, n) > BOUND
