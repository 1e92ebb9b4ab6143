"""FP32 matrix-core convolutions (conv_f32m.hip) at the sizes where their
tiles can go wrong: windows shorter than a tile, one column past a tile, odd
multiples of the networks' strides, and rows that do not start 16-byte
aligned.  Tolerance: the FP32 path's stated bound, 1e-5 normwise against the
FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOUND = 1e-5


def rel(a, r):
    return float(np.max(np.abs(np.asarray(a, np.float64) - r)) / np.max(np.abs(r)))


# last-stage lengths 1, 9, 127, 128, 129, 256 (128-column tiles); W = 8 L
@pytest.mark.parametrize("n,L", [(1, 1), (3, 9), (2, 127), (1, 128), (2, 129), (5, 256)])
def test_bbhnet_fp32_tile_edges(n, L):
    params = synth.bbhnet_params(3)
    m = gs.BBHnet(torch.from_numpy(params).to(DEV), synth.bbhnet_stages())
    x = synth.gaussian(70 + L, (n, 2, 8 * L))
    got = m.forward(x=torch.from_numpy(x).to(DEV)).cpu().numpy()
    assert rel(got, ref.bbhnet_forward(params, x)) <= BOUND
    # the same windows at an address 4 bytes past 16-byte alignment, bitwise
    buf = torch.empty(x.size + 1, device=DEV)
    buf[1:] = torch.from_numpy(x.reshape(-1)).to(DEV)
    off = buf[1:].view(n, 2, 8 * L)
    assert np.array_equal(m.forward(x=off).cpu().numpy(), got)


def train(m, x, dn, flags, precision):
    n, W = dn.shape
    noise = torch.empty((n, W), device=DEV)
    ws = m.forward(x=x, noise=noise, flags=flags, precision=precision)
    dp = torch.empty_like(m.params)
    m.backward(x, dn, ws, dp, flags=flags, precision=precision)
    return noise.cpu().numpy(), dp.cpu().numpy()


# W / 16 = 2, 3, 33, 129: every layer's length straddles its tile differently
# (W = 16 is left out: batch statistics over two or three values amplify
# rounding by 1 / (their difference), far past any FP32 bound)
@pytest.mark.parametrize("n,q", [(2, 2), (3, 3), (1, 33), (2, 129)])
def test_training_fp32_tile_edges(n, q):
    layers = synth.deepclean_layers()
    params = synth.deepclean_params(2)
    m = gs.DeepClean(torch.from_numpy(params).to(DEV), layers)
    W = 16 * q
    x = synth.gaussian(80 + q, (n, 21, W))
    dn = synth.gaussian(90 + q, (n, W))
    xt, dnt = torch.from_numpy(x).to(DEV), torch.from_numpy(dn).to(DEV)
    en = ref.deepclean_forward(params, x, layers, train=True)
    eg = ref.deepclean_grad(params, x, dn, layers)
    for flags in (gs.TRAIN, gs.TRAIN | gs.RECOMPUTE):
        noise, dp = train(m, xt, dnt, flags, gs.FP32)
        assert rel(noise, en) <= BOUND
        assert rel(dp, eg) <= BOUND
        # split-BF16 forward: its stated bound
        noise, dp = train(m, xt, dnt, flags, gs.BF16)
        assert rel(noise, en) <= 2e-2
        assert rel(dp, eg) <= 2e-2


def test_training_unaligned_windows_bitwise():
    """Windows at an address 4 bytes past 16-byte alignment train to the same bits."""
    m = gs.DeepClean(torch.from_numpy(synth.deepclean_params(2)).to(DEV), synth.deepclean_layers())
    x = torch.from_numpy(synth.gaussian(11, (2, 21, 528))).to(DEV)
    dn = torch.from_numpy(synth.gaussian(12, (2, 528))).to(DEV)
    shifted = []
    for t in (x, dn):
        buf = torch.empty(t.numel() + 1, device=DEV)
        buf[1:] = t.reshape(-1)
        shifted.append(buf[1:].view(t.shape))
    for precision in (gs.FP32, gs.BF16):
        a = train(m, x, dn, gs.TRAIN | gs.RECOMPUTE, precision)
        b = train(m, *shifted, gs.TRAIN | gs.RECOMPUTE, precision)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
