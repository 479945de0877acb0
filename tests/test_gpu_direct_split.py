"""The direct convolution on the bf16 matrix instruction, at the edges of its
blocks: every block shape (8x8 to 1x64 pixels) with remainders, channel counts
around 32 and 16, one, two and four waves of output channels, and inputs that
are not finite.

Tolerance.  The operands' three bf16 parts are exact and the part products
left out are below 1.01 * 2^-24 of a product; each tap and group of 32 channels
is summed by six matrix instructions and added in fp32, and the bias once, each
rounding below 2^-23 of the sum of absolute products so far:
    |y - ref| <= (7 ceil(cin / 32) K^2 + 2) 2^-23 (|w| * |x| + |b|).
"""
import numpy as np
import pytest

import oracle
from workloads import small_layer, make_random_bias

torch = pytest.importorskip("torch")
fs = pytest.importorskip("paper_2003_12621_amd")

pytestmark = pytest.mark.gpu

CASES = [
    # (n, cin, h, w, cout, k)
    (4, 32, 100, 102, 70, 3),      # 8x8 blocks, two waves
    (2, 47, 76, 128, 250, 3),      # 4x16 blocks, four waves, a last group of 16 channels
    (8, 20, 17, 124, 250, 3),      # 1x64 blocks, four waves
    (6, 70, 63, 95, 190, 3),       # a partial last group
    (11, 96, 40, 40, 256, 9),      # a large filter
    (4, 32, 64, 64, 256, 13),      # the largest one: more than 64 KB of LDS
    (40, 30, 14, 60, 120, 3),      # 2x32 blocks, two waves
]


def _run(shape, x, w, b, relu, split=1):
    plan = fs.Plan(*shape, bias=True, relu=relu)
    assert plan.kernels.direct_split == split
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return plan.direct_conv2d(dev(x), plan.direct_transform_weights(dev(w)), dev(b)).cpu().numpy()


@pytest.mark.parametrize("shape", CASES)
def test_against_float64(shape):
    n, cin, h, w_, cout, k = shape
    print(f"[case] {shape}", flush=True)
    x, w = small_layer(*shape, seed=sum(shape))
    b = make_random_bias(cout, cin, k, seed=3)
    got = _run(shape, x, w, b, False).astype(np.float64)
    ref = oracle.direct_xcorr2d(x, w, b)
    mag = oracle.direct_xcorr2d(np.abs(x), np.abs(w), np.abs(b))
    bound = (7 * -(-cin // 32) * k * k + 2) * 2.0 ** -23
    assert (np.abs(got - ref) <= bound * mag).all(), (np.abs(got - ref) / mag).max() / bound
    np.testing.assert_array_equal(_run(shape, x, w, b, True), np.maximum(got, 0).astype(np.float32))


@pytest.mark.parametrize("shape", CASES[:2])
def test_no_less_precise_and_same_nonfinite_values(shape, monkeypatch):
    """Closer to float64 than the fp32 instruction; infinities, NaN and sums
    that overflow come out as there."""
    x, w = small_layer(*shape, seed=7)
    b = make_random_bias(shape[4], shape[1], shape[5], seed=4)
    ref = oracle.direct_xcorr2d(x, w, b)
    y = _run(shape, x, w, b, False)
    x2, w2 = x.copy(), w.copy()
    x2[0, 3, 5, 6], x2[1, 2, 1, 1], x2[1, 7, 30, 40] = np.inf, np.nan, 3e38
    w2[4, 5, 1, 1] = -np.inf
    y2 = _run(shape, x2, w2, b, False)
    monkeypatch.setenv("FFTSPLIT_DIRECT_SPLIT", "0")
    f = _run(shape, x, w, b, False, 0)
    f2 = _run(shape, x2, w2, b, False, 0)
    err = lambda a: np.linalg.norm(a.astype(np.float64) - ref)
    assert err(y) <= err(f)
    np.testing.assert_array_equal(np.isnan(y2), np.isnan(f2))
    np.testing.assert_array_equal(np.isposinf(y2), np.isposinf(f2))
    np.testing.assert_array_equal(np.isneginf(y2), np.isneginf(f2))
    ok = np.isfinite(f2)
    np.testing.assert_allclose(y2[ok], f2[ok], rtol=1e-5, atol=1e-4)
