"""Every form of the matrix-core grouped kernels' epilogue (windows, smallest shifts, PReLU), at channel counts
that fill and do not fill a block of 64, ragged bands and several images per unit, alone and in one
shared launch of plain and PReLU layers, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from workloads import make_gconv_layer
from workloads.generators import prelu_mult_neg
from gpu_util import assert_same, dev

pytestmark = pytest.mark.gpu

# n, h, w, c, gs, stride
SHAPES = [(3, 7, 7, 48, 16, 1), (1, 31, 29, 64, 4, 1), (5, 9, 11, 72, 8, 2), (2, 15, 13, 96, 32, 1), (1, 1, 1, 16, 16, 2),
          (1, 4, 187, 32, 16, 1), (17, 2, 3, 128, 64, 2)]
FORMS = [((0, 127), (2, 9), False), ((0, 127), (1, 9), False), ((-128, 127), (1, 9), False), ((-128, 127), (0, 9), False),
         ((-30, 80), (2, 9), False), ((-128, 127), (2, 9), True), ((-128, 127), (1, 9), True), ((-90, 127), (2, 9), True)]


def _layer(P, shape, f):
    n, h, w, c, gs, stride = shape
    window, shifts, prelu = FORMS[f]
    L = make_gconv_layer(500 + 13 * f + c + 3 * h, n, h, w, c, gs, stride, signed_x=True, act_window=window, shift_range=shifts)
    L.shift[:] += 6 * (np.arange(c) % 3 > 0) * (L.shift > shifts[0])  # most channels not saturated
    neg = prelu_mult_neg(f, L.mult) if prelu else None
    rq = P.Requant(dev(L.bias), dev(L.mult), dev(L.shift), window[0], window[1], dev(neg) if prelu else None)
    want = oracle.gconv3x3(L.x, L.weight, stride, L.bias, L.mult, L.shift, window[0], window[1], mult_neg=neg)
    frag = dev(P.prom_gconv_pack(L.weight)) if f % 2 else None
    return dev(L.x), dev(L.weight), stride, rq, frag, want


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forms(shape):
    import torch
    import paper_2505_03254_amd as P
    layers = [_layer(P, shape, f) for f in range(len(FORMS))]
    for (x, w, stride, rq, frag, want), form in zip(layers, FORMS):
        y = P.prom_gconv3x3(x, w, stride, rq, w_frag=frag)
        assert_same(y.cpu().numpy(), want, f"{shape} {form}")
    ys = [torch.empty(l[5].shape, dtype=torch.int8, device="cuda") for l in layers]
    P.prom_gconv3x3_sequence([(x, w, s, rq, y, frag) for (x, w, s, rq, frag, _), y in zip(layers, ys)])
    torch.cuda.synchronize()
    for y, l, form in zip(ys, layers, FORMS):
        assert_same(y.cpu().numpy(), l[5], f"{shape} {form} in the shared launch")
