"""GW_CAUSAL in tiles of 768 outputs, which a launch takes that has more tiles of
256 than compute units: with a budget of one unit a few windows reach it.  Its
clean outputs, and the rings it updates, are bitwise those of the tiles of 256
and of the update and the forward apart, for spans of any length and alignment
(tiles count from the band's newest end, so the last starts before the band),
and with delays."""
import numpy as np
import pytest
import torch

from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# strides of the three streams, request by request; the largest sets the band
STRIDES = [[16, 8, 24], [1, 333, 64], [769, 13, 7], [256, 512, 1024], [1537, 1, 767], [2560, 2304, 5]]


@pytest.mark.parametrize("W", [272, 2560, 8192])
@pytest.mark.parametrize("precision", [pytest.param(gs.BF16, id="bf16"), pytest.param(gs.FP16, id="fp16")])
def test_causal_tiles_of_768(W, precision):
    n = 3
    params = torch.from_numpy(synth.deepclean_params(3)).to(DEV)
    small, full = (gs.DeepClean(params, synth.deepclean_layers()) for _ in range(2))
    small.set_cu_budget(1)
    pools = []
    for _ in range(3):
        pool = gs.Pool(n * (W * 21 * 6 + 512) + (8 << 20), max_slots=n, max_items=n)
        pools.append((pool, [pool.open(21, W) for _ in range(n)]))
    rng = np.random.default_rng(W)
    for k, tri in enumerate(STRIDES):
        s = [min(W, v) for v in tri]
        off = np.cumsum([0] + [21 * v for v in s[:-1]]) + k
        x = torch.from_numpy(rng.standard_normal(21 * sum(s) + k).astype(np.float32)).to(DEV)
        strain = torch.from_numpy(rng.standard_normal(sum(s)).astype(np.float32)).to(DEV)
        got = []
        for side, (pool, slots) in enumerate(pools):
            clean, late = (torch.full((sum(s),), 7.0, device=DEV) for _ in range(2))
            kw = dict(pool=pool, slots=slots, W=W, strides=s, strain=strain, precision=precision, flags=gs.CAUSAL)
            if side == 0:    # the whole chip: 256 outputs a tile
                full.update_forward(samples=x, offsets=off, clean=clean, **kw)
            elif side == 1:  # with the update folded in
                small.update_forward(samples=x, offsets=off, clean=clean, **kw)
            else:            # without
                pool.update(slots, s, x, off)
                small.forward(clean=clean, **kw)
            # spans that end before the window: tiles are left out at both ends
            m = full if side == 0 else small
            m.forward(clean=late, delays=[min(W - v, d) for v, d in zip(s, (0, 300, 1500))], **kw)
            rings = torch.stack([pool.window(i) for i in slots])
            shadows = torch.stack([pool.window(i, bf16=True) for i in slots])
            got.append((clean, late, rings, shadows))
        for other in got[1:]:
            for a, b in zip(got[0], other):
                assert torch.equal(a, b), k
