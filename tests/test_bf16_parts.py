"""The arithmetic of the bf16 split (bf16_split.hpp) emulated in numpy: the
three parts of a scaled fp32 number are that number exactly, for normal and
subnormal ones, and the bounds that the kernels' comments and the GPU tests'
tolerances state hold and are nearly reached.  No GPU needed."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2003_12621_amd", "csrc", "bf16_split.hpp")


def bf16(v):
    """float32 rounded to the nearest bf16, ties to even, as float32."""
    b = v.view(np.uint32).astype(np.uint64)
    b = (b + 0x7fff + ((b >> 16) & 1)) & 0xffff0000
    return b.astype(np.uint32).view(np.float32)


def parts(v):
    out = []
    for _ in range(3):
        out.append(bf16(v))
        v = v - out[-1]
    return out


def scale():
    text = open(HEADER).read()
    return float.fromhex(re.search(r"kSplitScale = (0x1p[0-9-]+)f", text).group(1))


def numbers(lo, hi, n=200000):
    """Random signs and significands, dense (all ones, one bit, runs) among
    them, exponents [lo, hi)."""
    rng = np.random.default_rng(lo + 1000)
    m = rng.integers(0, 1 << 23, n, dtype=np.uint32)
    m[: n // 4] |= rng.integers(0, 2, n // 4, dtype=np.uint32) * 0x7fff
    m[n // 4: n // 2] &= ~np.uint32(0x7fff)
    m[:6] = 0, 1, 0x7fffff, 0x7f8000, 0x8000, 0xffff
    v = np.ldexp(1.0 + m / 2.0 ** 23, rng.integers(lo, hi, n)) * rng.choice((-1.0, 1.0), n)
    return v.astype(np.float32)


@pytest.mark.parametrize("lo,hi", [(-149, -126), (-126, -100), (-100, 0), (0, 103)])
def test_scaled_parts_are_exact(lo, hi):
    v = numbers(lo, hi) * np.float32(scale())
    assert np.isfinite(v).all()
    p = [q.astype(np.float64) for q in parts(v)]
    np.testing.assert_array_equal(p[0] + p[1] + p[2], v.astype(np.float64))
    # no subnormal part: the matrix unit's treatment of those does not count
    for q in p:
        assert (np.abs(q[q != 0]) >= 2.0 ** -126).all()


def test_unscaled_parts_are_not():
    v = numbers(-126, -112)
    p = [q.astype(np.float64) for q in parts(v)]
    assert (p[0] + p[1] + p[2] != v.astype(np.float64)).any()


def test_part_bounds():
    v, w = numbers(0, 1), numbers(-1, 0)
    pv, pw = parts(v), parts(w)
    for p, bound in ((pv[1], 2.0 ** -8), (pv[2], 2.0 ** -17)):
        r = np.abs(p.astype(np.float64)) / np.abs(v.astype(np.float64))
        assert 0.95 * bound < r.max() <= bound
    q = [[a.astype(np.float64) * b.astype(np.float64) for b in pw] for a in pv]
    left_out = np.abs(q[1][2]) + np.abs(q[2][1]) + np.abs(q[2][2])
    r = left_out / np.abs(v.astype(np.float64) * w.astype(np.float64))
    assert r.max() <= 1.01 * 2.0 ** -24
    assert r.max() > 2.0 ** -25
