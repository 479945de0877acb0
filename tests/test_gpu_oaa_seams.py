"""The packed seam entries of overlap-add at the sizes of the core they leave:
none (T = K - 1, every entry packed), one or two rows, most of the patch, and
no seam at all (K = 1), with ragged last tiles.

Tolerance: rel-L2 2e-6 of the float64 cross-correlation.  The transforms and
the channel sum round to fp32 at each of about 4 log2(L) + Cin steps of random
sign, 2^-24 * sqrt(40) = 4e-7 rms; an entry misplaced or missing changes the
result by a part in its own size.
"""
import numpy as np
import pytest

import oracle
from workloads import make_random_bias, small_layer

from spectra_layout import rel_l2

torch = pytest.importorskip("torch")
fs = pytest.importorskip("paper_2003_12621_amd")

pytestmark = pytest.mark.gpu

CASES = [
    # (n, cin, h, w, cout, k), T
    ((2, 3, 23, 19, 5, 5), 4),      # L = 8, no core
    ((1, 3, 25, 41, 5, 9), 8),      # L = 16, no core
    ((2, 20, 20, 21, 5, 3), 6),     # L = 8, core 4
    ((1, 3, 25, 30, 5, 7), 10),     # L = 16, core 4
    ((3, 3, 31, 29, 5, 3), 14),     # L = 16, core 12
    ((1, 3, 61, 50, 5, 9), 24),     # L = 32, core 16
    ((1, 3, 61, 64, 5, 3), 30),     # L = 32, core 28
    ((2, 3, 17, 19, 5, 1), 8),      # K = 1: all core
]


@pytest.mark.parametrize("shape,tile", CASES, ids=[f"{s}-T{t}" for s, t in CASES])
def test_seams_against_float64(shape, tile):
    n, cin, h, w, cout, k = shape
    print(f"[case] oaa seams {shape} T={tile}", flush=True)
    x, wt = small_layer(n, cin, h, w, cout, k, seed=sum(shape) + tile)
    b = make_random_bias(cout, cin, k, seed=5)
    plan = fs.Plan(n, cin, h, w, cout, k, tile=tile, mode="oaa", bias=True)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, wt, b)]
    ws = plan.new_workspace()
    ws.fill_(0xFF)   # NaN wherever nothing is written
    y = plan.conv2d(dev[0], plan.transform_weights(dev[1]), dev[2], workspace=ws)
    torch.cuda.synchronize()
    ref = oracle.direct_xcorr2d(x, wt, b)
    assert rel_l2(y.cpu().numpy(), ref) <= 2e-6
