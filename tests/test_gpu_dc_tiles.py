"""The fused kernel's third tile size (512 outputs), taken where it needs a round
of the chip less: with a small budget of compute units a few windows reach it.
Its outputs and the rings it updates are bitwise those of calls that take the
other sizes, at heads of any alignment, with and without the update."""
import numpy as np
import pytest
import torch

from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

STRIDES = [[16, 8, 24], [1, 333, 64], [250, 13, 7], [272, 4, 512]]


def cdiv(a, b):
    return -(-a // b)


@pytest.mark.parametrize("n,W,budget", [
    (3, 4096, 8),     # 18 tiles of 768 (two rounds), 24 of 512 (one, exactly full)
    (3, 2560, 5),     # 12 and 15: whole tiles of 512, a last one of 256 outputs for 768
    (7, 1008, 6),     # 14 and 14: two tiles a window, the last one short
    (1, 13328, 8),    # one long window: 18 and 27 tiles in 2 and 2 rounds (768 stays)
])
@pytest.mark.parametrize("precision", [pytest.param(gs.BF16, id="bf16"), pytest.param(gs.FP16, id="fp16")])
def test_tiles_of_512(n, W, budget, precision):
    r768, r512 = cdiv(n * cdiv(W, 768), 2 * budget), cdiv(n * cdiv(W, 512), 3 * budget)
    assert (r512 < r768) == (W != 13328) and n * cdiv(W, 256) > budget
    params = torch.from_numpy(synth.deepclean_params(3)).to(DEV)
    small, full = (gs.DeepClean(params, synth.deepclean_layers()) for _ in range(2))
    small.set_cu_budget(budget)
    pools = []
    for _ in range(3):
        pool = gs.Pool(n * (W * 21 * 6 + 512) + (8 << 20), max_slots=n, max_items=n)
        pools.append((pool, [pool.open(21, W) for _ in range(n)]))
    rng = np.random.default_rng(n + W)
    for k, tri in enumerate(STRIDES):
        s = [min(W, tri[i % 3]) for i in range(n)]
        off = np.cumsum([0] + [21 * v for v in s[:-1]]) + k
        x = torch.from_numpy(rng.standard_normal(21 * sum(s) + k).astype(np.float32)).to(DEV)
        strain = torch.from_numpy(rng.standard_normal(sum(s)).astype(np.float32)).to(DEV)
        got = []
        for side, (pool, slots) in enumerate(pools):
            clean = torch.full((sum(s),), 7.0, device=DEV)
            noise = torch.full((n, W), 7.0, device=DEV)
            kw = dict(pool=pool, slots=slots, W=W, strides=s, strain=strain, noise=noise, clean=clean,
                      precision=precision)
            if side == 0:    # the whole chip: 256 outputs a tile
                full.update_forward(samples=x, offsets=off, **kw)
            elif side == 1:  # with the update folded in
                small.update_forward(samples=x, offsets=off, **kw)
            else:            # without
                pool.update(slots, s, x, off)
                small.forward(**kw)
            rings = torch.stack([pool.window(i) for i in slots])
            shadows = torch.stack([pool.window(i, bf16=True) for i in slots])
            got.append((clean, noise, rings, shadows))
        for other in got[1:]:
            for a, b in zip(got[0], other):
                assert torch.equal(a, b), k
