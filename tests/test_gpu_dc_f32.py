"""The fused FP32 DeepClean forward (dc_f32.hip): window lengths around its
tiles, its three tile sizes against each other, ring and dense input, and
samples that are not finite.  Tolerance: the FP32 path's stated bound, 1e-5
normwise against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOUND = 1e-5


@pytest.fixture(scope="module")
def dc():
    params = synth.deepclean_params(1)
    layers = synth.deepclean_layers()
    return gs.DeepClean(torch.from_numpy(params).to(DEV), layers), params, layers


def forward(m, x):
    noise = torch.full((x.shape[0], x.shape[2]), float("nan"), device=DEV)
    m.forward(x=x, noise=noise)
    return noise.cpu().numpy()


# one step of the bottleneck, and one step short of, at and past each tile size
@pytest.mark.parametrize("W", [16, 112, 128, 144, 240, 256, 272, 512, 528, 4000])
def test_tile_edges(dc, W):
    m, params, layers = dc
    x = synth.gaussian(W, (3, 21, W))
    got = forward(m, torch.from_numpy(x).to(DEV))
    exp = ref.deepclean_forward(params, x, layers)
    assert np.max(np.abs(got - exp)) <= BOUND * np.max(np.abs(exp))


def test_tile_sizes_agree_bitwise(dc):
    """Batches of 40, 8 and 1 windows run in tiles of 512, 256 and 128."""
    m = dc[0]
    x = torch.from_numpy(synth.gaussian(7, (40, 21, 8192))).to(DEV)
    full = forward(m, x)
    assert np.array_equal(forward(m, x[:8].contiguous()), full[:8])
    for i in (0, 39):
        assert np.array_equal(forward(m, x[i:i + 1].contiguous()), full[i:i + 1])


@pytest.mark.parametrize("s", [16, 37, 1000])
def test_rings_at_any_head_bitwise(dc, s):
    """Windows read in place from rings whose head is not aligned give the
    dense windows' bits."""
    m, W = dc[0], 1040
    pool = gs.Pool(8 << 20, max_slots=2, max_items=2)
    slots = [pool.open(21, W) for _ in range(2)]
    for k in range(3):
        new = torch.from_numpy(synth.gaussian(100 * s + k, (2, 21, s))).to(DEV)
        pool.update(slots, [s, s], new.reshape(-1), [0, 21 * s])
    noise = torch.empty((2, W), device=DEV)
    m.forward(pool=pool, slots=slots, W=W, noise=noise)
    dense = torch.stack([pool.window(i) for i in slots])
    assert np.array_equal(noise.cpu().numpy(), forward(m, dense))


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("pos", [0, 255, 511, 700, 1023])
def test_non_finite_samples(dc, bad, pos):
    """An infinite sample saturates the first layer's tanh and stays finite;
    a NaN reaches the outputs of its receptive field and no other."""
    m, params, layers = dc
    x = synth.gaussian(5, (2, 21, 1024))
    x[1, 4, pos] = bad
    got = forward(m, torch.from_numpy(x).to(DEV))
    with np.errstate(invalid="ignore"):
        exp = ref.deepclean_forward(params, x, layers)
    assert np.array_equal(np.isnan(got), np.isnan(exp))
    ok = ~np.isnan(exp)
    assert np.max(np.abs(got[ok] - exp[ok])) <= BOUND * np.max(np.abs(exp[ok]))
