"""The tile kernel of the pointwise layers at the sizes where it can go wrong: each of its six tiles (named by the
library, test_every_tile), 1 to 10 k steps (whole and broken groups of four), ragged pixel counts, column tiles that
the channels do not fill, and every form of its epilogue, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from workloads import make_pw_layer
from workloads.generators import prelu_mult_neg
from gpu_util import assert_same, dev

pytestmark = pytest.mark.gpu

# n, h, w, cin, cout
SHAPES = [(1, 1, 1, 64, 256), (1, 9, 9, 128, 256), (3, 7, 5, 192, 208), (1, 13, 17, 320, 512), (1, 5, 7, 448, 1024),
          (1, 3, 11, 576, 272), (16, 14, 14, 512, 1024), (7, 55, 57, 64, 256), (5, 53, 51, 128, 496)]
# window, shift range, PReLU: [0, 127] with and without shifts below 2, [-128, 127] with and without shift 0,
# another window, PReLU in the full window, with shift 0 and in another window
FORMS = [((0, 127), (2, 9), False), ((0, 127), (1, 6), False), ((-128, 127), (1, 9), False), ((-128, 127), (0, 5), False),
         ((-20, 90), (2, 9), False), ((-128, 127), (1, 9), True), ((-128, 127), (0, 4), True), ((-100, 127), (1, 9), True)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("res", [False, True])
def test_tile_kernel(shape, res):
    import torch
    import paper_2505_03254_amd as P
    n, h, w, cin, cout = shape
    forms = FORMS if n * h * w < 2000 else FORMS[::3] + FORMS[5:6]
    for f, (window, shifts, prelu) in enumerate(forms):
        L = make_pw_layer(7000 + 31 * cin + cout + f, n, h, w, cin, cout, signed_x=True, act_window=window,
                          with_residual=True, shift_range=shifts)
        L.bias[::5] *= 100                       # some channels saturate on either side
        L.residual.reshape(-1)[::11] = -128
        L.residual.reshape(-1)[::13] = 127
        neg = prelu_mult_neg(f, L.mult) if prelu else None
        rq = P.Requant(dev(L.bias), dev(L.mult), dev(L.shift), window[0], window[1], dev(neg) if prelu else None)
        r = L.residual if res else None
        want = oracle.pw_conv(L.x, L.weight, L.bias, L.mult, L.shift, window[0], window[1], residual=r, mult_neg=neg)
        x, wp = dev(L.x), dev(P.prom_pack_ternary(L.weight))
        y = dev(L.residual).clone() if res else None   # in place
        for plan in (P.PwPlan(k_outer=1), None):
            got = P.prom_pw_conv_ex(x, wp, cout, rq, dev(r) if res else None, plan=plan)
            assert_same(got.cpu().numpy(), want, f"{shape} {window} {shifts} prelu={prelu} plan={plan}")
        if res:
            P.prom_pw_conv(x, wp, cout, rq, y, y=y)
            torch.cuda.synchronize()
            assert_same(y.cpu().numpy(), want, f"{shape} in place")


# Launched alone: two wavefronts per tile, input channels that fill no whole k step, output channels that fill no
# whole tile; the plan with the k loop innermost is the streaming kernel.
NARROW = [(1, 1, 1, 16, 96), (1, 14, 14, 80, 112), (2, 9, 7, 96, 576), (3, 13, 11, 144, 208), (1, 7, 7, 160, 960),
          (1, 5, 9, 240, 144), (2, 3, 5, 304, 272), (1, 7, 9, 464, 496), (9, 31, 29, 48, 320), (3, 55, 57, 256, 128)]


@pytest.mark.parametrize("shape", NARROW, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("prelu", [False, True])
def test_narrow_layers(shape, prelu):
    import paper_2505_03254_amd as P
    n, h, w, cin, cout = shape
    L = make_pw_layer(9000 + 31 * cin + cout, n, h, w, cin, cout, signed_x=True, act_window=(-128, 127),
                      with_residual=True, shift_range=(0, 9))
    L.bias[::5] *= 100
    neg = prelu_mult_neg(3, L.mult) if prelu else None
    rq = P.Requant(dev(L.bias), dev(L.mult), dev(L.shift), -128, 127, dev(neg) if prelu else None)
    for r in (None, L.residual):
        want = oracle.pw_conv(L.x, L.weight, L.bias, L.mult, L.shift, -128, 127, residual=r, mult_neg=neg)
        x, wp, rd = dev(L.x), dev(P.prom_pack_ternary(L.weight)), None if r is None else dev(r)
        for plan in (None, P.PwPlan(k_outer=-1)):
            got = P.prom_pw_conv_ex(x, wp, cout, rq, rd, plan=plan)
            assert_same(got.cpu().numpy(), want, f"{shape} prelu={prelu} residual={r is not None} plan={plan}")


# The six tiles of the kernel (pixels x channels) at k steps that are no multiple of four, pixels and channels that fill
# no whole tile, input channels that fill the last k step and that do not.
TILES = {(32, 128): [(1, 5, 7, 384, 304), (1, 5, 7, 304, 144)], (32, 256): [(29, 13, 11, 320, 144), (47, 5, 7, 432, 528)],
         (64, 128): [(23, 31, 29, 320, 144), (47, 13, 11, 336, 528)], (64, 256): [(2, 55, 57, 448, 400), (5, 53, 51, 304, 144)],
         (128, 128): [(9, 55, 57, 320, 272), (9, 55, 57, 336, 304)], (128, 256): [(11, 31, 29, 448, 528), (5, 53, 51, 592, 400)]}


@pytest.mark.parametrize("tile,shape", [(t, s) for t in TILES for s in TILES[t]], ids=lambda v: "x".join(map(str, v)))
def test_every_tile(tile, shape):
    import paper_2505_03254_amd as P
    n, h, w, cin, cout = shape
    # [0, 127]; any shift; another window; PReLU in the full window and with shift 0: with the residual every second time
    for f, (window, shifts, prelu) in enumerate([FORMS[0], FORMS[3], FORMS[4], FORMS[5], FORMS[6]]):
        res = f % 2 == 1
        assert P.prom_pw_kernel_query(*shape, residual=res, prelu=prelu) == tile
        L = make_pw_layer(8100 + 31 * cin + cout + f, n, h, w, cin, cout, signed_x=True, act_window=window,
                          with_residual=True, shift_range=shifts)
        L.bias[::5] *= 100
        neg = prelu_mult_neg(f, L.mult) if prelu else None
        rq = P.Requant(dev(L.bias), dev(L.mult), dev(L.shift), window[0], window[1], dev(neg) if prelu else None)
        r = L.residual if res else None
        want = oracle.pw_conv(L.x, L.weight, L.bias, L.mult, L.shift, window[0], window[1], residual=r, mult_neg=neg)
        got = P.prom_pw_conv(dev(L.x), dev(P.prom_pack_ternary(L.weight)), cout, rq, dev(r) if res else None)
        assert_same(got.cpu().numpy(), want, f"{tile} {shape} {window} {shifts} prelu={prelu} residual={res}")


def test_narrow_layers_run_on_the_tile_kernel():
    import paper_2505_03254_amd as P
    for shape in NARROW:
        for res in (False, True):
            for prelu in (False, True):
                assert P.prom_pw_kernel_query(*shape, residual=res, prelu=prelu) is not None, shape
