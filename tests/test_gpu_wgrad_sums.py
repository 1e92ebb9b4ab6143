"""Rounding of the weight gradients' FP32 sums, on operands that are exact.

With beta = 20 and gamma = 0 an activation is 1, and with no sums and unit
scale dz is dh, so that a weight's gradient is a plain sum of dh, of values
around one, and FP64 gives it exactly.  A sum is cut into chains that are added
in FP32, and the chains' sums in FP64.

Bound: a chain of K values rounds K times, by ulp(S) / sqrt(12) at a partial sum
S of 1 .. K, together at most 2^-23 K^1.5 / 6.  N / K of them make a relative
error of 2^-23 / 6 K / sqrt(N); the rounding of the gradient itself adds
2^-24 / sqrt(3).  K is N / 256 (N / 512: layers 1, 6, 7 and 8) as in the launches
of one layer, 64 at least (a chunk).  The root mean square over a layer is held to 1.5 times that (few
of its weights are independent).
"""
import ctypes as C
import math

import pytest
import torch

from paper_2108_12430_amd import gwstream as gs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CH = [21, 8, 16, 32, 64, 32, 16, 8, 8, 1]


class BnBwd(C.Structure):
    _fields_ = [(k, C.c_void_p) for k in ("mean", "invstd", "gamma", "beta", "z", "sum_dh", "sum_dhx")] + [("invN", C.c_float)]


class Args(C.Structure):
    _fields_ = [("p", C.c_void_p), ("q", C.c_void_p), ("pbn", BnBwd), ("qbn", BnBwd), ("n", C.c_int), ("Lp", C.c_int),
                ("Lq", C.c_int), ("dw", C.c_void_p)]


@pytest.mark.parametrize("n,W", [(512, 32768), (3, 1040)])
def test_exact_operands(n, W):
    lib = C.CDLL(gs.LIB_PATH)
    size = lib._ZN2gw20wgrad2_scratch_bytesEiPKi
    size.restype = C.c_size_t
    launch = lib._ZN2gw13launch_wgrad2ERA9_KNS_7Wg2ArgsEPvPfPKNS_8F32RangeEiP12ihipStream_t
    Ls = [W, W // 2, W // 4, W // 8, W // 16, W // 8, W // 4, W // 2, W, W]
    g = torch.Generator(device=DEV).manual_seed(5)
    dh = 0.5 + torch.rand(n * 8 * W, device=DEV, generator=g)  # every layer's dh starts here
    x = torch.ones(n * 21 * W, device=DEV)                     # the input, and every z
    zero, one, twenty = (torch.full((64,), v, device=DEV) for v in (0.0, 1.0, 20.0))
    z, o, t = zero.data_ptr(), one.data_ptr(), twenty.data_ptr()
    act = BnBwd(z, o, z, t, 0, 0, 0, 0.0)
    dz = BnBwd(z, o, o, z, x.data_ptr(), z, z, 1.0)
    raw = BnBwd()
    a, grads, lp = (Args * 9)(), [], (C.c_int * 9)()
    for l in range(9):
        in_p = l >= 4  # the layer's input is P
        gin, gout = (x.data_ptr(), raw if l == 0 else act), (dh.data_ptr(), raw if l == 8 else dz)
        (pp, pb), (qp, qb) = (gin, gout) if in_p else (gout, gin)
        lp[l] = Ls[l] if in_p else Ls[l + 1]
        grads.append(torch.full((CH[l] if 4 <= l < 8 else CH[l + 1], CH[l + 1] if 4 <= l < 8 else CH[l], 7), 7.0,
                                device=DEV))
        a[l] = Args(pp, qp, pb, qb, n, lp[l], Ls[l + 1] if in_p else Ls[l], grads[l].data_ptr())
    scratch = torch.empty(size(n, lp), dtype=torch.uint8, device=DEV)
    db = torch.zeros(1, device=DEV)
    assert launch(a, C.c_void_p(scratch.data_ptr()), C.c_void_p(db.data_ptr()), None, 0,
                  gs._stream()) == 0
    for l in range(9):
        co, Li, Lo = CH[l + 1], Ls[l], Ls[l + 1]
        d = dh[: n * co * Lo].view(n, co, Lo).sum(0, dtype=torch.float64)  # [co][Lo]
        exact = torch.empty(co, 7, dtype=torch.float64, device=DEV)
        for j in range(7):
            if 4 <= l < 8:  # output 2 t - 3 + j of input t
                u = 2 * torch.arange(Li, device=DEV) - 3 + j
                exact[:, j] = d[:, u[(u >= 0) & (u < Lo)]].sum(1)
            else:           # input s t - 3 + j of output t
                u = (1 if l == 8 else 2) * torch.arange(Lo, device=DEV) - 3 + j
                exact[:, j] = d[:, (u >= 0) & (u < Li)].sum(1)
        got = grads[l].double()
        want = (exact[None] if 4 <= l < 8 else exact[:, None]).expand_as(got)
        err = ((got - want) / want).square().mean().sqrt().item()
        N = n * lp[l]
        K = max(64, N / (512 if l == 1 or l >= 6 else 256))
        bound = 1.5 * math.hypot(2.0 ** -23 / 6 * K / math.sqrt(N), 2.0 ** -24 / math.sqrt(3))
        assert err <= bound, (l, err, bound)
    assert abs(db.item() / dh[: n * W].sum(dtype=torch.float64).item() - 1) <= 2.0 ** -23
