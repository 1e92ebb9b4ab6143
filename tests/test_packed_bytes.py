"""The packed buffer of a DeepClean model holds what its kernels read.  The
adjoint convolutions of the reference network run from FP32 fragments made by each
backward, so that it packs none of them; a network of another shape does."""
import ctypes as C

import pytest

from paper_2108_12430_amd import gwstream as gs
from paper_2108_12430_amd import synth

TABLE = 32 * 4096 * 56  # the item tables of dense calls


def up(b):
    return -(-b // 256) * 256


def elems(ci, co, transposed):
    """16-bit elements of a k7 layer's fragments: phases x tiles of 16 rows x K steps of 32 x 512."""
    k = (4 if transposed else 7) * (-(-ci // 8) * 8)
    return (2 if transposed else 1) * -(-co // 16) * -(-k // 32) * 512


def packed(layers):
    d, b = gs.deepclean_desc(layers), C.c_size_t()
    gs.check(gs.lib().gw_model_packed_bytes(gs.MODEL_DEEPCLEAN, d.ctypes.data_as(C.c_void_p), len(d), C.byref(b)))
    return b.value - up(TABLE)


@pytest.mark.parametrize("reference", [True, False])
def test_adjoint_fragments(reference):
    layers = synth.deepclean_layers() if reference else synth.deepclean_layers(c_in=20)
    affine = sum(2 * up(4 * co) for _, _, co, *_ in layers)
    own = sum(up(2 * elems(ci, co, t == "convT")) for t, ci, co, *_ in layers)
    adjoint = sum(2 * up(2 * elems(co, ci, t == "conv")) for t, ci, co, _k, s, *_ in layers[1:] if s == 2)
    if not reference:
        assert packed(layers) == affine + 2 * own + adjoint  # high and low terms of each
        return
    # high and low terms, FP16 copies, FP32 fragments (twice the bytes, K steps of
    # 16, rows as above), and the fused kernels' own layouts of five layers
    assert packed(layers) <= affine + 5 * own + 2 * 5 * up(2 * 8 * 512)
