"""deepclean_update_forward as one launch (every precision, with and without
GW_CAUSAL), item tables in the kernel arguments (up to 60 items) and in device
memory, rings read at any head, and the fused kernel's two tile sizes: bitwise
against the two calls, dense windows and larger batches."""
import numpy as np
import pytest
import torch

from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PRECISIONS = [pytest.param(p, id=n) for p, n in ((gs.BF16, "bf16"), (gs.FP16, "fp16"), (gs.FP32, "fp32"))]


@pytest.fixture(scope="module")
def dc():
    return gs.DeepClean(torch.from_numpy(synth.deepclean_params(3)).to(DEV), synth.deepclean_layers())


def rings(n, W):
    pool = gs.Pool(n * (W * 21 * 6 + 512) + (8 << 20), max_slots=n, max_items=n)
    return pool, [pool.open(21, W) for _ in range(n)]


def rand(rng, *shape):
    return torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(DEV)


STRIDES = [[16, 8], [1, 333], [250, 13], [272, 272], [4, 999]]


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("n,W", [(2, 1040), (61, 1008), (2, 272)])
def test_one_launch_equals_two_calls(dc, precision, causal, n, W):
    sides = [rings(n, W) for _ in range(2)]
    rng = np.random.default_rng(n + W)
    flags = gs.CAUSAL if causal else 0
    for k, pair in enumerate(STRIDES):
        s = [min(W, pair[i % 2]) for i in range(n)]
        off = np.cumsum([0] + [21 * v for v in s[:-1]]) + k  # source blocks at any alignment
        x, strain = rand(rng, 21 * sum(s) + k), rand(rng, sum(s))
        # delays force the two calls under GW_CAUSAL, and are one launch otherwise
        delays = [min(100 * k, W - v) for v in s] if k % 2 else None
        got = []
        for side, (pool, slots) in enumerate(sides):
            clean = torch.full((sum(s),), 7.0, device=DEV)
            noise = None if causal else torch.full((n, W), 7.0, device=DEV)
            kw = dict(pool=pool, slots=slots, W=W, strides=s, strain=strain, noise=noise, clean=clean,
                      precision=precision, flags=flags, delays=delays)
            if side == 0:
                pool.update(slots, s, x, off)
                dc.forward(**kw)
            else:
                dc.update_forward(samples=x, offsets=off, **kw)
            got.append((clean, noise))
        assert torch.equal(got[0][0], got[1][0]), k
        assert causal or torch.equal(got[0][1], got[1][1]), k
        for a, b in zip(sides[0][1], sides[1][1]):
            assert sides[0][0].info(a) == sides[1][0].info(b)
            assert torch.equal(sides[0][0].window(a), sides[1][0].window(b)), k
            assert torch.equal(sides[0][0].window(a, bf16=True), sides[1][0].window(b, bf16=True)), k


@pytest.mark.parametrize("precision", PRECISIONS)
def test_any_head_equals_dense_and_causal(dc, precision):
    """Rings advanced by odd strides: the noise window equals the dense
    window's, and GW_CAUSAL gives the full window's clean output, also when
    the span ends a delay before the window's end."""
    W, n = 2064, 3
    pool, slots = rings(n, W)
    rng = np.random.default_rng(5)
    for k in range(9):
        s = [[5, 16, 301], [1, 777, 64], [2, 3, 1033]][k % 3]
        off = np.cumsum([0] + [21 * v for v in s[:-1]])
        pool.update(slots, s, rand(rng, 21 * sum(s)), off)
        strain = rand(rng, sum(s))
        delays = [0, 40, 300] if k % 2 else None
        out = torch.full((n, W), 7.0, device=DEV)
        full, band, dense = torch.zeros(sum(s), device=DEV), torch.zeros(sum(s), device=DEV), torch.empty((n, W), device=DEV)
        dc.forward(pool=pool, slots=slots, W=W, strides=s, strain=strain, noise=out, clean=full, precision=precision,
                   delays=delays)
        dc.forward(pool=pool, slots=slots, W=W, strides=s, strain=strain, clean=band, precision=precision,
                   flags=gs.CAUSAL, delays=delays)
        dc.forward(x=torch.stack([pool.window(i) for i in slots]), noise=dense, precision=precision)
        assert torch.equal(out, dense), k
        assert torch.equal(full, band), k


@pytest.mark.parametrize("precision", PRECISIONS)
def test_tile_sizes_and_alignment_agree(dc, precision):
    """A window alone (the small tiles) and among 24 (the large ones), and at
    an address 4 bytes past 16-byte alignment."""
    rng = np.random.default_rng(6)
    x = rand(rng, 24, 21, 4112)
    def fwd(v):
        noise = torch.empty(v.shape[0], 4112, device=DEV)
        dc.forward(x=v, noise=noise, precision=precision)
        return noise
    full = fwd(x)
    for i in (0, 23):
        assert torch.equal(fwd(x[i:i + 1].contiguous()), full[i:i + 1])
    buf = torch.empty(x.numel() + 1, device=DEV)
    buf[1:] = x.reshape(-1)
    assert torch.equal(fwd(buf[1:].view(x.shape)), full)


@pytest.mark.parametrize("precision,flags", [(gs.FP32, 0), (gs.FP16, 0), (gs.BF16, gs.CAUSAL)])
def test_call_refused_by_the_forward_has_made_its_update(dc, precision, flags):
    """Outside BF16 without flags, the update comes before the forward's checks."""
    W = 272
    pool, (slot,) = rings(1, W)
    x = rand(np.random.default_rng(7), 21 * 16)
    ws = torch.empty(256, dtype=torch.uint8, device=DEV)[:0]
    with pytest.raises(gs.GwError):
        dc.update_forward(pool=pool, slots=[slot], strides=[16], samples=x, offsets=[0], W=W,
                          strain=torch.zeros(16, device=DEV), clean=torch.zeros(16, device=DEV), precision=precision,
                          flags=flags, ws=ws)
    assert pool.info(slot) == (21, W, 16)
    assert torch.equal(pool.window(slot)[:, -16:], x.view(21, 16))
