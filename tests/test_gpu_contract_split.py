"""The bf16-split contraction (k_contract_split.hip) at the edges of its tiles.

Every tile the plan can choose, channel counts below, at and just past a
channel block of 16 (and block counts the wave groups do not divide), patches
that leave whole blocks of padding, and the two slots of real bins, against
the float64 channel sum of the GPU's own spectra.

Tolerance.  An operand is its three bf16 parts exactly, and what six of the
nine part products leave out is below 1.01 * 2^-24 of a product, so at most
1.43 * 2^-24 of a complex one.  Each block of 16 channels is summed by six
matrix instructions, and then added in fp32 or, in wave groups, not; at most 3
further additions join the groups' sums.  With each of those roundings below
2^-23 of the sum of absolute products so far, a single group of ceil(cin / 16)
blocks is within 7 of them a block and the products left out, groups within 6 a
block, 3 and the products left out:
    |Y - ref| <= (7 ceil(cin / 16) + 3) 2^-23 (|W| |X|).
"""
import numpy as np
import pytest

from workloads import small_layer

torch = pytest.importorskip("torch")
fs = pytest.importorskip("paper_2003_12621_amd")

pytestmark = pytest.mark.gpu

# (n, cin, h, w, cout, k), tile T, then what the plan's rule gives: channels x
# patches of the workgroup tile, wave groups
CASES = [
    ((2, 97, 24, 24, 70, 3), 6, (64, 32, 2)),      # a partial block
    ((3, 80, 24, 24, 40, 3), 6, (64, 32, 2)),      # five channel blocks
    ((1, 270, 24, 24, 70, 3), 6, (64, 32, 4)),     # a partial block
    ((3, 256, 24, 24, 40, 3), 6, (64, 32, 4)),
    ((1, 3, 20, 40, 5, 3), 14, (64, 64, 1)),       # one channel block, padding patches
    ((20, 50, 56, 56, 40, 3), 14, (64, 64, 1)),    # a partial block
    ((1, 1, 30, 30, 1, 3), 30, (64, 64, 1)),       # one channel
    ((5, 83, 56, 56, 192, 3), 14, (64, 64, 1)),    # many blocks
    ((10, 23, 112, 112, 70, 3), 14, (64, 64, 1)),  # two blocks, one of them partial
    ((30, 50, 56, 56, 40, 3), 14, (64, 64, 1)),    # four blocks
    ((3, 83, 56, 56, 192, 3), 14, (64, 64, 2)),    # a partial block
    ((4, 96, 56, 40, 192, 3), 14, (64, 64, 2)),    # even blocks
    ((4, 37, 100, 100, 128, 3), 30, (128, 64, 1)),
    ((4, 47, 100, 100, 256, 3), 30, (256, 64, 1)),
    ((8, 35, 110, 120, 128, 3), 30, (128, 128, 1)),
    ((16, 34, 112, 100, 48, 3), 30, (64, 256, 1)),
    ((2, 18, 25, 25, 20, 5), 5, (64, 64, 1)),      # odd transform size: no packed bins
    ((2, 70, 25, 25, 20, 5), 5, (64, 32, 2)),      # odd transform size
]


def _tile(plan):
    k = plan.kernels
    assert k.contract_split
    return k.contract_tile_m, k.contract_tile_n, k.contract_wave_groups


def _spectra(shape, tile, scale=1.0, mean=0.0):
    x, w = small_layer(*shape, seed=sum(shape))
    x = (x + np.float32(mean)) * np.float32(scale)
    plan = fs.Plan(*shape, tile=tile, mode="oaa" if tile == shape[5] else "os")
    ws = plan.new_workspace()
    ws.fill_(0xFF)   # NaN wherever nothing is written
    wspec = plan.transform_weights(torch.from_numpy(w).cuda())
    plan.forward(torch.from_numpy(np.ascontiguousarray(x)).cuda(), ws)
    plan.contract(wspec, ws)
    nt = plan.info.tiles
    X, W = plan.xspec_view(ws)[:, :, :nt], plan.wspec_view(wspec)
    return X.to(torch.complex128), W.to(torch.complex128), plan.yspec_view(ws), plan


def _channel_sum(X, W, packed):
    Y = W.transpose(1, 2).contiguous() @ X
    A = W.abs().transpose(1, 2).contiguous() @ X.abs()
    for f in range(Y.shape[0] - 2, Y.shape[0]) if packed else ():
        Y[f] = torch.complex(W[f].real.T.contiguous() @ X[f].real, W[f].imag.T.contiguous() @ X[f].imag)
    return Y, A


@pytest.mark.parametrize("shape,tile,kernel", CASES)
def test_against_float64(shape, tile, kernel):
    print(f"[case] {shape} T={tile} {kernel}", flush=True)
    X, W, got, plan = _spectra(shape, tile)
    assert _tile(plan) == kernel
    ref, mag = _channel_sum(X, W, plan.nfft % 2 == 0)
    nt = plan.info.tiles
    bound = (7 * -(-shape[1] // 16) + 3) * 2.0 ** -23
    err = (got[:, :, :nt].to(torch.complex128) - ref).abs()
    assert bool((err <= bound * mag).all()), float((err / mag.clamp_min(1e-300)).max()) / bound
    # padded output channels and padding patches are zero spectra
    assert not bool(got[:, shape[4]:].abs().any()) and not bool(got[:, :, nt:].abs().any())


@pytest.mark.parametrize("shape,tile", [((4, 256, 56, 56, 256, 3), 14), ((16, 64, 56, 56, 256, 5), 28),
                                        ((2, 512, 14, 14, 128, 3), 6), ((4, 512, 28, 28, 512, 3), 6),
                                        # long sums in wave groups
                                        ((1, 1024, 28, 28, 64, 3), 6), ((1, 4096, 14, 14, 64, 3), 6),
                                        ((4, 2048, 40, 40, 192, 3), 14)])
@pytest.mark.parametrize("scale,mean", [(1.0, 0.0), (2.0 ** -60, 0.0), (2.0 ** 60, 0.0), (1.0, 3.0)])
def test_no_less_precise_than_fp32(shape, tile, scale, mean, monkeypatch):
    """Its error against float64 is no larger than the fp32 matrix
    instruction's on the same spectra, at any scale of the input, and where
    every pixel is positive and the sums lean one way."""
    def error(split):
        X, W, got, plan = _spectra(shape, tile, scale, mean)
        assert plan.kernels.contract_split == split
        ref, _ = _channel_sum(X, W, True)
        d = got[:, :, :plan.info.tiles].to(torch.complex128) - ref
        return float((d / scale).abs().pow(2).sum().sqrt() / (ref / scale).abs().pow(2).sum().sqrt())
    split = error(1)
    monkeypatch.setenv("FFTSPLIT_CONTRACT_SPLIT", "0")
    fp32 = error(0)
    print(f"[case] {shape} scale={scale:g} mean={mean}: split {split:.3e} fp32 {fp32:.3e}", flush=True)
    assert split <= fp32
