"""The direct convolution on the bf16 matrix instruction with operands whose
smallest parts bf16 does not hold as they stand (below 2^-110, subnormal ones
too): the error against float64 is no larger than on the fp32 instruction."""
import numpy as np
import pytest

import oracle
from workloads import small_layer

torch = pytest.importorskip("torch")
fs = pytest.importorskip("paper_2003_12621_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("xs,ws", [(-118, 0), (0, -118), (40, -116), (-112, 30), (-60, -58), (0, -128), (-136, 0)])
@pytest.mark.parametrize("shape", [(4, 32, 100, 102, 70, 3), (2, 47, 76, 128, 250, 3), (8, 20, 17, 124, 250, 3)])
def test_small_operands(shape, xs, ws, monkeypatch):
    print(f"[case] {shape} x 2^{xs} w 2^{ws}", flush=True)
    x, w = small_layer(*shape, seed=sum(shape))
    x, w = np.ldexp(x, xs), np.ldexp(w, ws)
    # (the operands as they were rounded, in a range that float64 squares)
    ref = oracle.direct_xcorr2d(np.ldexp(x.astype(np.float64), -xs), np.ldexp(w.astype(np.float64), -ws))

    def error(split):
        plan = fs.Plan(*shape)
        assert plan.kernels.direct_split == split
        y = plan.direct_conv2d(torch.from_numpy(x).cuda(), plan.direct_transform_weights(torch.from_numpy(w).cuda()))
        return np.linalg.norm(np.ldexp(y.cpu().numpy().astype(np.float64), -xs - ws) - ref) / np.linalg.norm(ref)
    split = error(1)
    monkeypatch.setenv("FFTSPLIT_DIRECT_SPLIT", "0")
    assert split <= error(0)
