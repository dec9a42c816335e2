"""The three-piece split of fp32 operands (the fp32 heads' arithmetic), in numpy:
exact, and what its six products leave out.  CPU only."""
import numpy as np
import pytest


def bf16(v):
    """float32 rounded to bfloat16 (to nearest, ties to even), as float32."""
    b = np.ascontiguousarray(v, np.float32).view(np.uint32).astype(np.uint64)
    b = (b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000
    return b.astype(np.uint32).view(np.float32)


def split(v):
    p0 = bf16(v)
    p1 = bf16(v - p0)
    return p0, p1, bf16(v - p0 - p1)


def left_out(a, b):
    """|a b - the six products|, relative, in float64 (every product is exact there)."""
    p, q = [x.astype(np.float64) for x in split(a)], [x.astype(np.float64) for x in split(b)]
    out = p[1] * q[2] + p[2] * q[1] + p[2] * q[2]
    return np.abs(out) / np.abs(a.astype(np.float64) * b.astype(np.float64))


@pytest.mark.parametrize("lo,hi", [(1.0, 2.0), (1.0, 1.0 + 2.0 ** -7)])
def test_split_is_exact_and_leaves_out_one_rounding_at_most(lo, hi):
    """|x1| <= 2^-8 and |x2| <= 2^-17 of the operand's binade, so what is left out,
    x1 y2 + x2 y1 + x2 y2, is below 2^-24 + 2^-34 of the product: up to the
    rounding of one fp32 product, and close to it for operands just above a power
    of two."""
    rng = np.random.Generator(np.random.PCG64(4))
    a = rng.uniform(lo, hi, 1 << 20).astype(np.float32)
    b = rng.uniform(lo, hi, 1 << 20).astype(np.float32)
    for v in (a, b):
        assert (sum(x.astype(np.float64) for x in split(v)) == v).all()
    worst = left_out(a, b).max()
    assert worst <= 2.0 ** -24 + 2.0 ** -34
    assert worst > 2.0 ** (-25 if hi == 2.0 else -24.2)
