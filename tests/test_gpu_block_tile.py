"""The block kernel whose wavefronts own pixel tiles against the CPU oracle, every output.  Through PROM_BLOCK_AUTO at
shapes where prom_block_tile_applies says that the library takes it; and with plans of the test's choice: every variant
with and without PReLU over several rounds per workgroup with a ragged last one, the hidden channels split over wavefronts
with a tile count that leaves some of them without a tile, and every form of the requantisation, the same and different
ones in the two layers.  Ragged tiles in both directions, odd numbers of 16-channel planes, output channels that fill no
whole lanes, the skip connection and the edges of the tensors come in all of them."""
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


def _case(P, B, window, prelu, pwin, dw_window=None, path=0):
    """prelu: for all three layers, or one answer for each."""
    import torch
    e, d, p = B.expand, B.dw, B.project
    dw_window = dw_window or window
    which = prelu if isinstance(prelu, tuple) else (prelu,) * 3
    en, dn, pn = (prelu_mult_neg(k, l.mult) if w else None for k, (l, w) in enumerate(zip((e, d, p), which)))
    t1 = oracle.pw_conv(B.x, e.weight, e.bias, e.mult, e.shift, window[0], window[1], mult_neg=en)
    t2 = oracle.dw_conv(t1, d.weight, B.stride, d.bias, d.mult, d.shift, dw_window[0], dw_window[1], mult_neg=dn)
    want = oracle.pw_conv(t2, p.weight, p.bias, p.mult, p.shift, pwin[0], pwin[1], residual=B.x if B.add_residual else None, mult_neg=pn)
    ws = torch.empty(P.prom_block_workspace_size(B.n, B.h, B.w, B.cin, B.chid, B.cout, B.stride), dtype=torch.int8, device="cuda")
    # the output between guards
    y = torch.full((want.size + 512,), 77, dtype=torch.int8, device="cuda")
    out = y[256:256 + want.size].view(want.shape)
    P.prom_block(dev(B.x), B.chid, B.cout, B.stride, dev(P.prom_pack_ternary(e.weight)), _requant(P, e, window, en),
                 dev(d.weight), _requant(P, d, dw_window, dn), dev(P.prom_pack_ternary(p.weight)), _requant(P, p, pwin, pn),
                 B.add_residual, ws, out, path=path)
    torch.cuda.synchronize()
    assert (y[:256] == 77).all() and (y[256 + want.size:] == 77).all()
    assert_same(out.cpu().numpy(), want, f"{B.n}x{B.h}x{B.w} {B.cin}->{B.chid}->{B.cout} stride {B.stride} {window} {dw_window} "
                f"prelu={prelu} path={path:#x}")


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


# the variants by number: stride, rows of a tile, 16-channel tiles of the output, most wavefronts of a workgroup
VARIANTS = [(1, 8, 2, 8), (1, 6, 2, 8), (1, 4, 2, 12), (1, 2, 2, 16), (1, 6, 4, 8), (1, 4, 4, 8), (1, 2, 4, 12),
            (2, 8, 2, 8), (2, 4, 2, 12), (2, 4, 4, 8)]


def _variant(v):
    stride, rows, cot, waves = VARIANTS[v - 1]
    return stride, rows, cot, waves, 14 if stride == 1 else 7


def _in(out, stride, odd):
    """An input size for `out` outputs."""
    return out if stride == 1 else 2 * out - odd


@pytest.mark.parametrize("prelu", [False, True])
@pytest.mark.parametrize("v", range(1, len(VARIANTS) + 1))
def test_rounds(v, prelu):
    """More tiles than wavefronts that can be resident: every workgroup walks over several, the last round is ragged; the
    last tile of an image has one row and three columns.  5 planes and 20 channels, or 3 and 48."""
    import paper_2505_03254_amd as P
    stride, rows, cot, waves, cols = _variant(v)
    n = 256 * waves // 6 + 7
    assert n * 6 > 256 * waves and n * 6 % (256 * waves) != 0
    cin, t = (20, 4) if cot == 2 else (48, 1)
    cout = cin if stride == 1 else cin - 4
    B = make_block(4000 + v, n, _in(2 * rows + 1, stride, 1), _in(cols + 3, stride, 0), cin, t, cout, stride, signed_x=True,
                   expand_shift=(2, 5), dw_shift=(7, 9), project_shift=(2, 5))
    assert B.add_residual == (stride == 1)
    _case(P, B, (-128, 127) if prelu else (0, 127), prelu, (-128, 127), path=P.block_tile_plan(v, 1, waves))


@pytest.mark.parametrize("split", [2, 3, 4, 6])
@pytest.mark.parametrize("v", range(1, len(VARIANTS) + 1))
def test_split(v, split):
    """Hidden channels over wavefronts: 11 planes, 13 tiles, so that the last workgroup has wavefronts without a tile."""
    import paper_2505_03254_amd as P
    stride, rows, cot, waves, cols = _variant(v)
    sums = (rows if stride == 1 else rows // 2) * cot  # KB of partial sums of a wavefront, of 160
    tiles = min(waves, 159 // sums) // split
    assert tiles == 1 or 13 % tiles != 0
    B = make_block(4100 + v, 13, _in(rows - 1, stride, 1), _in(cols - 1, stride, 0), 16, 11, 16 if cot == 2 else 40, stride,
                   signed_x=True, expand_shift=(2, 5), dw_shift=(7, 9), project_shift=(2, 5))
    _case(P, B, (0, 127), False, (-128, 127), path=P.block_tile_plan(v, split, tiles))
    _case(P, B, (-128, 127), True, (-128, 127), path=P.block_tile_plan(v, split, tiles))


# (window, shifts, PReLU) of the expansion and of the depthwise layer
MIXED = [(((0, 127), (1, 9), False), ((0, 127), (2, 9), False)), (((0, 127), (2, 9), False), ((-128, 127), (1, 9), False)),
         (((-30, 80), (2, 9), False), ((0, 127), (2, 9), False)), (((0, 127), (2, 9), False), ((0, 127), (0, 9), False)),
         (((-128, 127), (0, 9), False), ((0, 127), (2, 9), False)), (((-128, 127), (2, 9), True), ((0, 127), (2, 9), False)),
         (((0, 127), (2, 9), False), ((-128, 127), (2, 9), True)), (((-128, 127), (1, 9), True), ((-128, 127), (2, 9), True)),
         (((-128, 127), (2, 9), True), ((-90, 127), (0, 9), True))]


@pytest.mark.parametrize("v", range(1, len(VARIANTS) + 1))
def test_forms_of_every_variant(v):
    import paper_2505_03254_amd as P
    stride, rows, cot, waves, cols = _variant(v)
    for f, (fe, fd) in enumerate([(form, form) for form in FORMS] + MIXED):
        cin, t = (16, 3) if cot == 2 else (48, 1)
        B = make_block(4200 + 20 * v + f, 2, _in(rows + 1, stride, 0), _in(cols + 2, stride, 1), cin, t, cin, stride,
                       signed_x=True, expand_shift=fe[1], dw_shift=fd[1], project_shift=(0, 9) if f % 3 == 0 else (1, 9))
        for L, low in ((B.expand, fe[1][0]), (B.dw, fd[1][0]), (B.project, 0)):
            _spread(L, low)
        _case(P, B, fe[0], (fe[2], fd[2], f % 4 == 1), (-128, 127) if f % 2 == 0 else (-100, 99), dw_window=fd[0],
              path=P.block_tile_plan(v))


def test_plans_that_do_not_exist():
    import paper_2505_03254_amd as P
    B = make_block(4300, 1, 9, 9, 16, 2, 16, 1, signed_x=True)
    for plan in ((8, 0, 0), (11, 0, 0), (1, 5, 0), (1, 2, 1), (1, 1, 9), (4, 0, 17)):  # (two planes cannot be split)
        with pytest.raises(P.PromError) as err:
            _case(P, B, (0, 127), False, (-128, 127), path=P.block_tile_plan(*plan))
        assert err.value.code == -2, plan
    wide = make_block(4301, 1, 9, 9, 72, 2, 16, 1, signed_x=True)
    with pytest.raises(P.PromError) as err:
        _case(P, wide, (0, 127), False, (-128, 127), path=P.BLOCK_TILE)
    assert err.value.code == -2
    for path in (6, 256 + 6, -1, 256):
        with pytest.raises(P.PromError) as err:
            _case(P, B, (0, 127), False, (-128, 127), path=path)
        assert err.value.code == -1, path
