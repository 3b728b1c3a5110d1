"""The block kernel whose wavefronts own pixel tiles (prom_block with PROM_BLOCK_AUTO where prom_block_tile_applies says
so) against the CPU oracle, every output: every variant of the kernel, ragged tiles in both directions, an odd number of
16-channel planes, output channels that fill no whole lanes, several rounds per workgroup, hidden channels split over
wavefronts, every form of the requantisation, and the edges of the tensors."""
import pytest

import oracle
from gpu_util import assert_same, dev
from test_gpu_dw_forms import FORMS, _requant, _spread
from workloads import make_block
from workloads.generators import prelu_mult_neg

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, h, w, cin, t, cout, stride.  Stride 1, up to 32 output channels: tiles of 8, 6, 4 and 2 rows
    (64, 56, 56, 8, 4, 8, 1), (3, 113, 40, 32, 4, 24, 1), (128, 60, 1, 20, 4, 16, 1), (1, 1, 60, 8, 2, 8, 1),
    # up to 64: tiles of 6, 4 and 2 rows
    (64, 33, 57, 8, 4, 64, 1), (128, 15, 43, 8, 2, 48, 1), (1, 1, 60, 8, 2, 48, 1),
    # stride 2
    (128, 33, 57, 8, 2, 8, 2), (1, 1, 60, 8, 2, 8, 2), (1, 1, 60, 8, 2, 48, 2), (2, 57, 113, 16, 6, 24, 2), (32, 57, 55, 24, 6, 32, 2),
    # skip; 9 planes; 20 and 28 channels; odd sizes; one output column and row in the last tile
    (1, 57, 57, 24, 6, 24, 1), (1, 43, 43, 20, 4, 20, 1), (2, 45, 29, 28, 4, 28, 1), (1, 112, 15, 16, 6, 16, 1), (1, 9, 71, 64, 1, 64, 1),
    # 64 channels in, the hidden channels over several wavefronts
    (2, 28, 28, 32, 6, 32, 1), (1, 56, 56, 16, 3, 64, 2),
]


def _case(P, B, window, prelu, pwin):
    import torch
    e, d, p = B.expand, B.dw, B.project
    en, dn, pn = (prelu_mult_neg(k, l.mult) if prelu else None for k, l in enumerate((e, d, p)))
    t1 = oracle.pw_conv(B.x, e.weight, e.bias, e.mult, e.shift, window[0], window[1], mult_neg=en)
    t2 = oracle.dw_conv(t1, d.weight, B.stride, d.bias, d.mult, d.shift, window[0], window[1], mult_neg=dn)
    want = oracle.pw_conv(t2, p.weight, p.bias, p.mult, p.shift, pwin[0], pwin[1], residual=B.x if B.add_residual else None, mult_neg=pn)
    ws = torch.empty(P.prom_block_workspace_size(B.n, B.h, B.w, B.cin, B.chid, B.cout, B.stride), dtype=torch.int8, device="cuda")
    # the output between guards
    y = torch.full((want.size + 512,), 77, dtype=torch.int8, device="cuda")
    out = y[256:256 + want.size].view(want.shape)
    P.prom_block(dev(B.x), B.chid, B.cout, B.stride, dev(P.prom_pack_ternary(e.weight)), _requant(P, e, window, en),
                 dev(d.weight), _requant(P, d, window, dn), dev(P.prom_pack_ternary(p.weight)), _requant(P, p, pwin, pn),
                 B.add_residual, ws, out)
    torch.cuda.synchronize()
    assert (y[:256] == 77).all() and (y[256 + want.size:] == 77).all()
    assert_same(out.cpu().numpy(), want, f"{B.n}x{B.h}x{B.w} {B.cin}->{B.chid}->{B.cout} stride {B.stride} {window} prelu={prelu}")


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_shapes(shape):
    import paper_2505_03254_amd as P
    n, h, w, cin, t, cout, stride = shape
    assert P.prom_block_tile_applies(n, h, w, cin, cin * t, cout, stride)
    B = make_block(900 + cin + w, n, h, w, cin, t, cout, stride, signed_x=True, expand_shift=(2, 5), dw_shift=(7, 9), project_shift=(2, 5))
    _case(P, B, (0, 127), False, (-128, 127))
    if P.prom_block_tile_applies(n, h, w, cin, cin * t, cout, stride, True) and n < 64:
        _case(P, B, (-128, 127), True, (-128, 127))


def test_every_variant_is_covered():
    import paper_2505_03254_amd as P
    got = {P.prom_block_tile_applies(n, h, w, cin, cin * t, cout, stride) for n, h, w, cin, t, cout, stride in SHAPES}
    assert got == set(range(1, 11)), got


@pytest.mark.parametrize("shape", [(1, 57, 43, 16, 3, 16, 1), (1, 45, 59, 24, 2, 36, 2)], ids=lambda s: "x".join(map(str, s)))
def test_forms(shape):
    import paper_2505_03254_amd as P
    n, h, w, cin, t, cout, stride = shape
    for f, (window, shifts, prelu) in enumerate(FORMS):
        assert P.prom_block_tile_applies(n, h, w, cin, cin * t, cout, stride, prelu)
        B = make_block(1700 + f + cin, n, h, w, cin, t, cout, stride, signed_x=True, expand_shift=shifts, dw_shift=shifts,
                       project_shift=(0, 9) if f % 3 == 0 else (1, 9))
        for L, low in ((B.expand, shifts[0]), (B.dw, shifts[0]), (B.project, 0)):
            _spread(L, low)
        _case(P, B, window, prelu, (-128, 127) if f % 2 == 0 else (-100, 99))


def test_limits():
    import paper_2505_03254_amd as P
    assert P.prom_block_tile_applies(128, 56, 56, 24, 144, 24, 1)
    assert not P.prom_block_tile_applies(128, 56, 56, 24, 136, 24, 1)   # hidden channels not a multiple of 16
    assert not P.prom_block_tile_applies(128, 56, 56, 72, 144, 24, 1)   # more than 64 channels in
    assert not P.prom_block_tile_applies(128, 56, 56, 24, 144, 72, 1)   # or out
    assert not P.prom_block_tile_applies(128, 56, 56, 18, 144, 24, 1)   # no whole dwords
    assert not P.prom_block_tile_applies(128, 7, 7, 32, 192, 32, 1)     # a tile would be half empty
    assert not P.prom_block_tile_applies(64, 1448, 1448, 16, 96, 16, 1)  # 2 GiB
    with pytest.raises(P.PromError):
        P.prom_block_tile_applies(0, 7, 7, 16, 96, 16, 1)
