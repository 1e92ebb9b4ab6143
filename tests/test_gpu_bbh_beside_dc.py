"""BBHnet's fused forward beside a DeepClean launch that fills the chip.

Free-running on two streams, a bbh_fused launch may reach the chip before the
next step's dc_fused launch.  The blocks that it leaves must not keep dc_fused
blocks waiting for a whole tile: a step was 1.6 times as long with the BBHnet
group as without it.  Results do not depend on the placement.
"""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2108_12430_amd import gwstream as gs, synth

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"
DC_W, BB_W = 32768, 2048


def models():
    dc = gs.DeepClean(torch.from_numpy(synth.deepclean_params(0)).to(DEV), synth.deepclean_layers())
    bb = gs.BBHnet(torch.from_numpy(synth.bbhnet_params(0)).to(DEV), synth.bbhnet_stages())
    return dc, bb


def open_all(n_dc, n_bb):
    pool = gs.Pool(n_dc * (21 * DC_W * 6 + 1024) + n_bb * (2 * BB_W * 6 + 1024) + (32 << 20), max_slots=n_dc + n_bb,
                   max_items=n_dc + n_bb)
    dc_sl = np.array([pool.open(21, DC_W) for _ in range(n_dc)], np.int32)
    bb_sl = np.array([pool.open(2, BB_W) for _ in range(n_bb)], np.int32)
    return pool, dc_sl, bb_sl


# one block a CU from 65 windows (260 blocks) to 112 (448) once the pool's
# DeepClean forward is dense and on another stream; two outside
@pytest.mark.parametrize("n", [3, 64, 65, 112, 113])
def test_logits_do_not_depend_on_the_placement(n):
    dc, bb = models()
    n_dc = 7  # 301 tiles of 768
    pool, dc_sl, bb_sl = open_all(n_dc, n)
    g = torch.Generator(device=DEV).manual_seed(n)
    x = torch.randn((n, 2, BB_W), generator=g, device=DEV)
    pool.update(bb_sl, [BB_W] * n, x.reshape(-1), np.arange(n, dtype=np.int64) * 2 * BB_W)
    ws = torch.empty(bb.workspace_bytes(n, BB_W, gs.BF16), dtype=torch.uint8, device=DEV)
    want, got = torch.empty(n, device=DEV), torch.empty(n, device=DEV)
    bb.forward(x=x, logits=want, precision=gs.BF16, ws=ws)
    before = torch.empty(n, device=DEV)
    bb.forward(pool=pool, slots=bb_sl, W=BB_W, logits=before, precision=gs.BF16, ws=ws)
    noise = torch.empty((n_dc, DC_W), device=DEV)
    wd = torch.empty(dc.workspace_bytes(n_dc, DC_W, gs.BF16), dtype=torch.uint8, device=DEV)
    dc.forward(pool=pool, slots=dc_sl, W=DC_W, noise=noise, precision=gs.BF16, ws=wd)
    torch.cuda.synchronize()
    same = torch.empty(n, device=DEV)
    bb.forward(pool=pool, slots=bb_sl, W=BB_W, logits=same, precision=gs.BF16, ws=ws)
    torch.cuda.synchronize()
    bb.forward(pool=pool, slots=bb_sl, W=BB_W, logits=got, precision=gs.BF16, ws=ws, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(same, want) and torch.equal(before, want)


# 179 DeepClean streams with overlap averaging: per step the time without the
# BBHnet group is about 205 us.  With it 215 where its launch comes into the
# next dc_fused launch's tail; where it comes first, two rounds of its blocks
# (40 us) and the averaging beside it are added: 260, 1.27 times.  A whole tile
# more (before) made it 316 .. 330, 1.55 times.  The bound lies between the two.
@pytest.mark.parametrize("n_bb", [48, 77])
def test_step_is_not_held_up(n_bb):
    dc, bb = models()
    n = 179
    s = 256
    pool, dc_sl, bb_sl = open_all(n, n_bb)
    strides, bstr = np.full(n, s, np.int32), np.full(n_bb, 64, np.int32)
    off, boff = np.arange(n, dtype=np.int64) * 21 * s, np.arange(n_bb, dtype=np.int64) * 2 * 64
    xs, xb = torch.randn(21 * s * n, device=DEV), torch.randn(2 * 64 * n_bb, device=DEV)
    strain = torch.randn(n * s, device=DEV)
    clean = torch.empty_like(strain)
    noise = torch.empty((n, DC_W), device=DEV)
    logits = torch.empty(n_bb, device=DEV)
    ws = torch.empty(dc.workspace_bytes(n, DC_W, gs.BF16), dtype=torch.uint8, device=DEV)
    wb = torch.empty(bb.workspace_bytes(n_bb, BB_W, gs.BF16), dtype=torch.uint8, device=DEV)
    state = torch.zeros(dc.overlap_state_floats(strides, 4), device=DEV)
    sm, sb = torch.cuda.current_stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    done = 0

    def run(steps, group):
        nonlocal done
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            dc.update_forward(pool=pool, slots=dc_sl, strides=strides, samples=xs, offsets=off, W=DC_W, noise=noise,
                              precision=gs.BF16, ws=ws, stream=sm)
            dc.overlap_average(noise=noise, strides=strides, depth=4, counts=[done] * n, state=state, strain=strain,
                               clean=clean)
            if group:
                pool.update(bb_sl, bstr, xb, boff, stream=sb)
                bb.forward(pool=pool, slots=bb_sl, W=BB_W, logits=logits, precision=gs.BF16, ws=wb, stream=sb)
            done += 1
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps

    for group in (False, True):
        run(100, group)
    alone = min(run(200, False) for _ in range(4))
    both = min(run(200, True) for _ in range(4))
    print(f"{1e6 * alone:.1f} us a step, with {n_bb} BBHnet windows {1e6 * both:.1f}")
    assert both < 1.4 * alone
