"""The reference network's cached forward (dc_band.hip) at the sizes where its
tiles and zones can go wrong, bitwise against the general cached kernel
(cache.hip).  The same weights with a 22nd witness channel of zero weights are
a network the general kernel takes: its sums gain exact zeros only."""
import numpy as np
import pytest
import torch

from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def models():
    p21 = synth.deepclean_params(4)
    n0 = 8 * 21 * 7
    w0 = np.zeros((8, 22, 7), np.float32)
    w0[:, :21] = p21[:n0].reshape(8, 21, 7)
    p22 = np.concatenate([w0.ravel(), p21[n0:]])
    return (gs.DeepClean(torch.from_numpy(p21).to(DEV), synth.deepclean_layers(21)),
            gs.DeepClean(torch.from_numpy(p22).to(DEV), synth.deepclean_layers(22)))


class Side:
    def __init__(self, m, c, W, n):
        self.m, self.W, self.n = m, W, n
        self.pool = gs.Pool(n * W * c * 8 + (8 << 20), max_slots=n, max_items=n)
        self.slots = [self.pool.open(c, W) for _ in range(n)]
        self.caches = [m.new_cache(W) for _ in self.slots]
        for s, b in zip(self.slots, self.caches):
            self.pool.attach_cache(s, b)

    def step(self, x, strides, strain, delays, noise):
        off = np.cumsum([0] + [b.numel() for b in x[:-1]])
        self.pool.update(self.slots, strides, torch.cat([b.reshape(-1) for b in x]), off)
        out = torch.full((self.n, self.W), float("nan"), device=DEV) if noise else None
        clean = torch.full((int(sum(strides)),), float("nan"), device=DEV)
        self.m.forward_cached(pool=self.pool, slots=self.slots, W=self.W, strides=strides, strain=strain, noise=out,
                              clean=clean, delays=delays)
        return clean.cpu().numpy(), None if out is None else out.cpu().numpy()


# windows shorter than the zones, one step around a tile, and long ones;
# strides of one step, odd ones (full recompute) and the whole window
@pytest.mark.parametrize("W,strides", [(16, (16, 5)), (176, (16, 48)), (256, (16, 240)), (272, (32, 13)),
                                       (528, (16, 528)), (2064, (256, 1040)), (4096, (64, 1024))])
def test_band_kernel_equals_general_kernel_bitwise(W, strides):
    a, b = models()
    sa, sb = Side(a, 21, W, 2), Side(b, 22, W, 2)
    for k in range(6):
        x = [torch.from_numpy(synth.gaussian(1000 * k + i, (21, s))).to(DEV) for i, s in enumerate(strides)]
        x22 = [torch.cat([v, torch.full((1, v.shape[1]), 3.0, device=DEV)]) for v in x]
        strain = torch.from_numpy(synth.gaussian(k, (sum(strides),))).to(DEV)
        delays = [min(k * 40, W - s) for s in strides]
        noise = k % 2 == 0
        ca, na = sa.step(x, strides, strain, delays, noise)
        cb, nb = sb.step(x22, strides, strain, delays, noise)
        assert np.array_equal(ca, cb), k
        if noise:
            assert np.array_equal(na, nb), k
