"""The band-passed loss and gradient at the edges of their tiles: 16 windows,
16 bins and 128 samples a block.

Tolerance: the residual (2^-24 of a sample), the angle 2 m / W and the basis
value (together below 1e-6 of a basis value of order one), the rounding of a
projection and the FP32 sum over the bins each enter the result linearly; 1e-5
of its norm leaves several times their sum.
"""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,W,k_lo,k_hi", [
    (1, 2, 0, 1),          # the smallest row: its bins are DC and Nyquist
    (1, 128, 5, 5),        # one bin, one block of samples
    (16, 129, 0, 15),      # one window tile, one bin tile, one sample past a block
    (17, 130, 1, 17),      # one window and one bin past a tile
    (32, 4095, 3, 34),     # odd rows, two whole bin tiles
    (33, 1024, 0, 512),    # every bin, one window past the largest tile
    (5, 40000, 500, 508),  # more blocks of samples than slices
])
@pytest.mark.parametrize("shift", [0, 1])
def test_bandpass_tile_edges(n, W, k_lo, k_hi, shift):
    strain = synth.gaussian(60, (n, W)).astype(np.float32)
    noise = synth.gaussian(61, (n, W), 0.5).astype(np.float32)

    def dev(a):  # shift: rows that are not 16-byte aligned
        buf = torch.empty(n * W + shift, device=DEV)
        buf[shift:] = torch.from_numpy(a).to(DEV).reshape(-1)
        return buf[shift:].reshape(n, W)

    fs = float(W)  # bin k lies at k Hz
    loss, dn = gs.bandpass_mse(dev(strain), dev(noise), fs, k_lo - 0.25 if k_lo else 0.0, k_hi + 0.25)
    el, edn = ref.bandpass_mse(strain, noise, fs, k_lo - 0.25 if k_lo else 0.0, k_hi + 0.25)
    got = dn.cpu().numpy().astype(np.float64)
    print(n, W, shift, abs(loss.item() / el - 1), np.linalg.norm(got - edn) / np.linalg.norm(edn), flush=True)
    assert abs(loss.item() - el) <= 1e-5 * abs(el)
    assert np.linalg.norm(got - edn) <= 1e-5 * np.linalg.norm(edn)
    only, none = gs.bandpass_mse(dev(strain), dev(noise), fs, k_lo - 0.25 if k_lo else 0.0, k_hi + 0.25,
                                 want_grad=False)
    assert none is None and only.item() == loss.item()
