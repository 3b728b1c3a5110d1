"""Every form of the depthwise and the block kernels' epilogues (windows, smallest shifts, PReLU) at heights that
leave rows over in the kernels' groups of 4 and 8, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from workloads import make_block, make_dw_layer
from workloads.generators import prelu_mult_neg
from gpu_util import assert_same, dev

pytestmark = pytest.mark.gpu

FORMS = [((0, 127), (2, 9), False), ((0, 127), (1, 9), False), ((0, 127), (0, 9), False), ((-128, 127), (1, 9), False),
         ((-128, 127), (0, 9), False), ((-30, 80), (2, 9), False), ((-128, 127), (2, 9), True), ((-128, 127), (1, 9), True),
         ((-90, 127), (2, 9), True)]


def _requant(P, L, window, neg):
    return P.Requant(dev(L.bias), dev(L.mult), dev(L.shift), window[0], window[1], None if neg is None else dev(neg))


def _spread(L, low):
    """Most channels with larger shifts, so that not everything saturates; some keep the smallest."""
    L.shift[:] = np.minimum(L.shift + 5 * (np.arange(L.shift.size) % 4 > 0) * (L.shift > low), 31)


@pytest.mark.parametrize("shape", [(2, 9, 7, 20, 1), (1, 15, 33, 64, 1), (3, 1, 5, 8, 1), (2, 11, 9, 36, 2), (9, 3, 2, 16, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_depthwise_forms(shape):
    import torch
    import paper_2505_03254_amd as P
    n, h, w, c, stride = shape
    layers, wants = [], []
    for f, (window, shifts, prelu) in enumerate(FORMS):
        L = make_dw_layer(900 + f + c, n, h, w, c, stride, signed_x=True, act_window=window, shift_range=shifts)
        _spread(L, shifts[0])
        neg = prelu_mult_neg(f, L.mult) if prelu else None
        wants.append(oracle.dw_conv(L.x, L.weight, stride, L.bias, L.mult, L.shift, window[0], window[1], mult_neg=neg))
        x, wd, rq = dev(L.x), dev(L.weight), _requant(P, L, window, neg)
        assert_same(P.prom_dw_conv(x, wd, stride, rq).cpu().numpy(), wants[-1], f"{shape} {window} {shifts} {prelu}")
        layers.append((x, wd, stride, rq, torch.empty(wants[-1].shape, dtype=torch.int8, device="cuda")))
    P.prom_dw_conv_sequence(layers)
    torch.cuda.synchronize()
    for l, want, form in zip(layers, wants, FORMS):
        assert_same(l[4].cpu().numpy(), want, f"{shape} {form} in the shared launch")


@pytest.mark.parametrize("shape", [(2, 9, 7, 16, 6, 16, 1), (1, 14, 15, 24, 4, 40, 2), (3, 7, 7, 64, 6, 64, 1), (2, 5, 6, 136, 3, 136, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_block_forms(shape):
    import torch
    import paper_2505_03254_amd as P
    n, h, w, cin, t, cout, stride = shape
    for f, (window, shifts, prelu) in enumerate(FORMS):
        B = make_block(700 + f + cin, n, h, w, cin, t, cout, stride, signed_x=True, expand_shift=shifts, dw_shift=shifts,
                       project_shift=(0, 9) if f % 3 == 0 else (1, 9))
        for L, low in ((B.expand, shifts[0]), (B.dw, shifts[0]), (B.project, 0)):
            _spread(L, low)
        e, d, p = B.expand, B.dw, B.project
        pwin = (-128, 127) if f % 2 == 0 else (-100, 99)
        en, dn = (prelu_mult_neg(f, e.mult), prelu_mult_neg(f + 1, d.mult)) if prelu else (None, None)
        if f == 7:
            dn = None  # one of the two layers without a negative-side multiplier
        t1 = oracle.pw_conv(B.x, e.weight, e.bias, e.mult, e.shift, window[0], window[1], mult_neg=en)
        t2 = oracle.dw_conv(t1, d.weight, stride, d.bias, d.mult, d.shift, window[0], window[1], mult_neg=dn)
        want = oracle.pw_conv(t2, p.weight, p.bias, p.mult, p.shift, pwin[0], pwin[1], residual=B.x if B.add_residual else None)
        ws = torch.empty(P.prom_block_workspace_size(n, h, w, cin, cin * t, cout, stride), dtype=torch.int8, device="cuda")
        for path in (P.BLOCK_AUTO, P.BLOCK_PLANES, P.BLOCK_UNFUSED):
            if path == P.BLOCK_PLANES and not P.prom_block_planes_applies(n, h, w, cin, cin * t, cout, stride):
                continue
            y = P.prom_block(dev(B.x), cin * t, cout, stride, dev(P.prom_pack_ternary(e.weight)), _requant(P, e, window, en),
                             dev(d.weight), _requant(P, d, window, dn), dev(P.prom_pack_ternary(p.weight)),
                             _requant(P, p, pwin, None), B.add_residual, ws, path=path)
            assert_same(y.cpu().numpy(), want, f"{shape} {window} {shifts} prelu={prelu} path={path}")


# Windows other than [0, 127] and [-128, 127] with no shift of 0: one-sided, of one value, at either end; shifts of
# exactly 1 and up to 31
OTHER = [((0, 100), (1, 9)), ((-100, 99), (1, 1)), ((1, 127), (2, 31)), ((-128, 126), (1, 31)), ((5, 5), (1, 9)),
         ((-128, -128), (1, 9)), ((127, 127), (1, 9))]


@pytest.mark.parametrize("window,shifts", OTHER, ids=lambda v: "_".join(map(str, v)))
def test_other_windows(window, shifts):
    import torch
    import paper_2505_03254_amd as P
    layers, wants = [], []
    for n, h, w, c, stride in ((2, 9, 7, 20, 1), (1, 5, 6, 8, 1), (2, 11, 9, 36, 2)):
        L = make_dw_layer(1200 + c, n, h, w, c, stride, signed_x=True, act_window=window, shift_range=shifts)
        wants.append(oracle.dw_conv(L.x, L.weight, stride, L.bias, L.mult, L.shift, window[0], window[1]))
        x, wd, rq = dev(L.x), dev(L.weight), _requant(P, L, window, None)
        assert_same(P.prom_dw_conv(x, wd, stride, rq).cpu().numpy(), wants[-1], f"{c} {window} {shifts}")
        layers.append((x, wd, stride, rq, torch.empty(wants[-1].shape, dtype=torch.int8, device="cuda")))
    P.prom_dw_conv_sequence(layers)
    torch.cuda.synchronize()
    for l, want in zip(layers, wants):
        assert_same(l[4].cpu().numpy(), want, f"{window} {shifts} in the shared launch")
    n, h, w, cin, t, cout = 2, 9, 7, 16, 6, 16
    B = make_block(1300, n, h, w, cin, t, cout, 1, signed_x=True, expand_shift=shifts, dw_shift=shifts, project_shift=(1, 9))
    e, d, p = B.expand, B.dw, B.project
    t1 = oracle.pw_conv(B.x, e.weight, e.bias, e.mult, e.shift, window[0], window[1])
    t2 = oracle.dw_conv(t1, d.weight, 1, d.bias, d.mult, d.shift, window[0], window[1])
    want = oracle.pw_conv(t2, p.weight, p.bias, p.mult, p.shift, -128, 127, residual=B.x if B.add_residual else None)
    ws = torch.empty(P.prom_block_workspace_size(n, h, w, cin, cin * t, cout, 1), dtype=torch.int8, device="cuda")
    for path in (P.BLOCK_PLANES, P.BLOCK_UNFUSED):
        y = P.prom_block(dev(B.x), cin * t, cout, 1, dev(P.prom_pack_ternary(e.weight)), _requant(P, e, window, None),
                         dev(d.weight), _requant(P, d, window, None), dev(P.prom_pack_ternary(p.weight)),
                         _requant(P, p, (-128, 127), None), B.add_residual, ws, path=path)
        assert_same(y.cpu().numpy(), want, f"block {window} {shifts} path={path}")
