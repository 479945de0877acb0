"""The bf16-split contraction at the ends of the fp32 range, for every tile:
operands whose smallest parts bf16 does not hold as they stand (below 2^-110,
subnormal ones too), infinities, NaN and sums that overflow.  Small operands are
split as exactly as others; a wave whose sums are not finite computes its tile
as the fp32 kernel (FFTSPLIT_CONTRACT_SPLIT=0) does.

The reference is the channel sum in float64 of the spectra that the GPU's own
forward and filter transforms wrote.
"""
import numpy as np
import pytest

from workloads import small_layer

from test_gpu_contract_split import CASES as SPLIT_CASES

torch = pytest.importorskip("torch")
fs = pytest.importorskip("paper_2003_12621_amd")

pytestmark = pytest.mark.gpu

# one shape for each tile, and one whose transforms have no slots of two real bins
CASES = list({kernel: (shape, tile) for shape, tile, kernel in SPLIT_CASES if shape[1] > 16 and tile != shape[5]}
             .values()) + [((2, 18, 25, 25, 20, 5), 5)]


def _spectra(shape, tile, x, w, split=1):
    plan = fs.Plan(*shape, tile=tile, mode="oaa" if tile == shape[5] else "os")
    assert plan.kernels.contract_split == split
    ws = plan.new_workspace()
    wspec = plan.transform_weights(torch.from_numpy(w).cuda())
    plan.forward(torch.from_numpy(x).cuda(), ws)
    plan.contract(wspec, ws)
    nt = plan.info.tiles
    return plan.xspec_view(ws)[:, :, :nt], plan.wspec_view(wspec), plan.yspec_view(ws)[:, :, :nt], plan


def _error(X, W, Y, packed):
    """Relative error (2-norm) over the bins that are products of complex
    numbers."""
    n = X.shape[0] - (2 if packed else 0)
    X, W, Y = (a[:n].to(torch.complex128) for a in (X, W, Y))
    ref = W.transpose(1, 2).contiguous() @ X.contiguous()
    scale = float(ref.abs().max())
    return float(((Y - ref) / scale).abs().pow(2).sum().sqrt() / (ref / scale).abs().pow(2).sum().sqrt())


# scales of x and w: small operands against ordinary and against large ones,
# both small, and subnormal ones
@pytest.mark.parametrize("xs,ws", [(-122, 0), (0, -112), (40, -114), (-112, 30), (-60, -60), (0, -126), (-136, 0)])
@pytest.mark.parametrize("shape,tile", CASES)
def test_small_operands(shape, tile, xs, ws, monkeypatch):
    print(f"[case] {shape} T={tile} x 2^{xs} w 2^{ws}", flush=True)
    x, w = small_layer(*shape, seed=sum(shape))
    x, w = np.ldexp(x, xs), np.ldexp(w, ws)
    packed = shape[5] != tile
    X, W, Y, _ = _spectra(shape, tile, x, w)
    monkeypatch.setenv("FFTSPLIT_CONTRACT_SPLIT", "0")
    assert _error(X, W, Y, packed) <= _error(*_spectra(shape, tile, x, w, 0)[:3], packed)


@pytest.mark.parametrize("shape,tile", CASES)
def test_small_operands_among_ordinary_ones(shape, tile, monkeypatch):
    """One image and one filter far below the others: their own spectra are as
    precise as the fp32 kernel's."""
    print(f"[case] {shape} T={tile} one image, one filter", flush=True)
    x, w = small_layer(*shape, seed=sum(shape))
    x[-1] *= np.float32(2.0 ** -120)
    w[shape[4] // 2] *= np.float32(2.0 ** -112)
    co, packed = shape[4] // 2, shape[5] != tile

    def errors(split):
        X, W, Y, plan = _spectra(shape, tile, x, w, split)
        t = plan.info.tiles - plan.info.tiles_h * plan.info.tiles_w
        return [_error(X[:, :, t:], W[:, :, :co], Y[:, :co, t:], packed),
                _error(X, W[:, :, co:co + 1], Y[:, co:co + 1], packed) if t == 0 else
                _error(X[:, :, :t], W[:, :, co:co + 1], Y[:, co:co + 1, :t], packed)]
    split = errors(1)
    monkeypatch.setenv("FFTSPLIT_CONTRACT_SPLIT", "0")
    for s, f in zip(split, errors(0)):
        assert s <= f


@pytest.mark.parametrize("overflow", [False, True])
@pytest.mark.parametrize("shape,tile", CASES)
def test_nonfinite_values_are_the_fp32_kernels(shape, tile, overflow, monkeypatch):
    """A NaN and infinities of both signs, or bins and sums that overflow: the
    same infinities and NaN, in the output spectra and in the layer's result
    after ReLU.  (Near the largest float the fp32 kernel's third product,
    (Wr + Wi)(Xr + Xi), can overflow where the result does not: there the split
    kernel may stay finite.)"""
    print(f"[case] {shape} T={tile} overflow={overflow}", flush=True)
    x, w = small_layer(*shape, seed=sum(shape))
    if not overflow:
        x[0, 2, 3, 4], x[0, 1, 20, 20], x[-1, 0, 9, 2] = np.nan, np.inf, -np.inf
        w[3, 1, 1, 1] = np.inf
    else:
        # the bins of a patch of s x s pixels are about s times those, 4.5 s
        # times the largest: past the largest float in the first patch
        x[::8] *= np.float32(3.2e37 / (tile if tile == shape[5] else tile + shape[5] - 1))
        x[::8, :, : tile, : tile] *= np.float32(5)
    b = np.zeros(shape[4], np.float32)

    def run(split):
        y = _spectra(shape, tile, x, w, split)[2]
        plan = fs.Plan(*shape, tile=tile, mode="oaa" if tile == shape[5] else "os", bias=True, relu=True)
        out = plan.conv2d(torch.from_numpy(x).cuda(), plan.transform_weights(torch.from_numpy(w).cuda()),
                          torch.from_numpy(b).cuda())
        return torch.view_as_real(y).contiguous(), out
    split = run(1)
    monkeypatch.setenv("FFTSPLIT_CONTRACT_SPLIT", "0")
    for s, f in zip(split, run(0)):
        assert not bool(s.isfinite().all())
        same = (s.isnan() == f.isnan()) & (s.isposinf() == f.isposinf()) & (s.isneginf() == f.isneginf())
        assert bool((same | (s.isfinite() & ~f.isfinite()) if overflow else same).all())
