"""OaAConv's inverse with the overlap-add in LDS, where its strips can go
wrong: planes split into strips with a ragged last one, several images per
workgroup with a ragged last group, patches taken in several passes, widths
that are and are not a multiple of 4, and images too wide for a strip (the
form through memory): the widest image of strips of four patch rows and the
next column, for each filter.

Tolerance: rel-L2 2e-6 of the float64 cross-correlation.  The transforms and
the channel sum round to fp32 at each of about 2 log2(L^2) + Cin steps of
random sign, 2^-24 * sqrt(40) = 4e-7 rms; a pixel misplaced or a missing
contribution changes the result by a part in its own size.
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
    # (n, cin, h, w, cout, k), patch rows and images per workgroup (0: through memory)
    ((1, 3, 61, 60, 4, 3), (4, 1)),       # strips, ragged last rows, w % 4 == 0
    ((2, 3, 58, 83, 3, 5), (4, 1)),       # strips, several passes, w % 4 != 0
    ((1, 2, 75, 40, 2, 7), (4, 1)),
    ((37, 2, 9, 8, 64, 3), (3, 2)),       # several images per workgroup, ragged last group
    ((33, 2, 14, 14, 70, 5), (3, 2)),
    ((1, 1, 8, 360, 2, 7), (2, 1)),       # two patch rows
    ((1, 1, 22, 1167, 2, 3), (4, 1)),     # widest strips
    ((1, 1, 22, 1168, 2, 3), (0, 0)),
    ((1, 1, 38, 675, 2, 5), (4, 1)),
    ((1, 1, 38, 676, 2, 5), (0, 0)),
    ((1, 1, 53, 469, 2, 7), (4, 1)),
    ((1, 1, 53, 470, 2, 7), (0, 0)),
    ((1, 1, 9, 1500, 2, 3), (0, 0)),      # through memory
    ((1, 1, 15, 700, 2, 7), (0, 0)),
]


@pytest.mark.parametrize("shape,strip", CASES, ids=[str(s) for s, _ in CASES])
def test_strips_against_float64(shape, strip):
    n, cin, h, w, cout, k = shape
    print(f"[case] oaa strip {shape}", flush=True)
    x, wt = small_layer(n, cin, h, w, cout, k, seed=sum(shape))
    b = make_random_bias(cout, cin, k, seed=5)
    plan = fs.Plan(n, cin, h, w, cout, k, tile=k, mode="oaa", bias=True)
    assert (plan.kernels.oaaconv_strip_rows, plan.kernels.oaaconv_strip_images) == strip
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, wt, b)]
    spectra = plan.transform_weights(dev[1])
    y = plan.conv2d(dev[0], spectra, dev[2])
    again = plan.conv2d(dev[0], spectra, dev[2])
    torch.cuda.synchronize()
    assert torch.equal(y, again)
    assert rel_l2(y.cpu().numpy(), oracle.direct_xcorr2d(x, wt, b)) <= 2e-6
