"""The band-passed loss and gradient on every route: up to four windows and
more, one slice of the samples and several, bins split among a block's waves and
not, sums added in a launch of their own or with the loss.

Tolerance: a basis value's angle 2 m / W is off by up to 2^-23 of itself (its
scale and its product are rounded), up to 7.5e-7 rad, and the value by 2^-23
besides; the residual and a projection are rounded once (2^-24 each) and the
products and sums are FP64.  Both directions take a basis value: 2e-6 of the
gradient's norm, and of the loss, whose terms are squares, twice that of one
direction.
"""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(n, W, k_lo, k_hi, shift):
    strain = synth.gaussian(62, (n, W)).astype(np.float32)
    noise = synth.gaussian(63, (n, W), 0.5).astype(np.float32)

    def dev(a):  # shift: rows that are not 16-byte aligned
        buf = torch.empty(n * W + shift, device=DEV)
        buf[shift:] = torch.from_numpy(a).to(DEV).reshape(-1)
        return buf[shift:].reshape(n, W)

    fs = float(W)  # bin k lies at k Hz
    lo, hi = k_lo - 0.25 if k_lo else 0.0, k_hi + 0.25
    el, edn = ref.bandpass_mse(strain, noise, fs, lo, hi)
    s, x = dev(strain), dev(noise)
    loss, dn = gs.bandpass_mse(s, x, fs, lo, hi)
    got = dn.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - el) <= 2e-6 * abs(el)
    assert np.linalg.norm(got - edn) <= 2e-6 * np.linalg.norm(edn)
    only, none = gs.bandpass_mse(s, x, fs, lo, hi, want_grad=False)
    assert none is None and only.item() == loss.item()


@pytest.mark.parametrize("n,W,k_lo,k_hi", [
    (1, 2, 0, 1), (1, 63, 0, 31), (2, 64, 0, 32), (3, 65, 1, 4),  # around one round of samples
    (4, 1023, 3, 7), (1, 1024, 0, 512), (2, 1025, 5, 5),          # one slice, two
    (4, 8191, 100, 104), (1, 8192, 0, 4096), (3, 8193, 4090, 4096),  # the gradient's two kernels
    (4, 40001, 437, 520), (2, 32768, 440, 520),                   # many slices, rows of any alignment
    (5, 8192, 0, 300),                                            # one window past them
])
def test_few_windows(n, W, k_lo, k_hi):
    check(n, W, k_lo, k_hi, 1)


@pytest.mark.parametrize("n,W,k_lo,k_hi", [
    (5, 511, 0, 62), (5, 512, 1, 64),          # one bin below the split, and at it
    (16, 1031, 3, 70), (17, 1031, 3, 270),     # one window tile of either kind; samples not whole tiles
    (33, 527, 0, 263), (32, 33, 0, 16),        # every bin; a few
    (5, 16384, 1, 64), (5, 16400, 1, 64),      # 256 blocks unsplit, 257
    (5, 16400, 1, 255), (5, 16400, 1, 256),    # the latter's bound
    (6, 65472, 10, 265), (6, 65536, 10, 265),  # 1023 blocks, 1024
])
@pytest.mark.parametrize("shift", [0, 1])
def test_split_bins(n, W, k_lo, k_hi, shift):
    check(n, W, k_lo, k_hi, shift)


@pytest.mark.parametrize("n,W,k_lo,k_hi", [
    (16, 1024, 9, 136), (16, 1024, 9, 137),               # eight slices of 4096 values, and of more
    (5, 250, 0, 20), (7, 800, 30, 30), (128, 600, 3, 9),  # two, seven and five slices
    (2, 4096, 60, 66), (5, 4096, 60, 66),                 # eight, and more
])
def test_loss_alone(n, W, k_lo, k_hi):
    check(n, W, k_lo, k_hi, 0)
