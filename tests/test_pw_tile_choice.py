"""Which kernel a pointwise layer launched alone runs on (prom_pw_kernel_query, on the host alone): the rule between
the streaming kernel and the kernel with the k loop outermost, and the shape of the latter's tiles."""
import os

import pytest


@pytest.fixture(scope="module")
def P():
    import paper_2505_03254_amd as P
    if not os.path.exists(P.library_path()):
        from paper_2505_03254_amd.build import build
        build()
    P.load_library()
    return P


def test_query_names_the_kernel(P):
    # planned for the tile kernel, launched alone on it, and forced either way
    assert P.prom_pw_kernel_query(128, 7, 7, 2048, 1024) is not None
    assert P.prom_pw_kernel_query(1, 14, 14, 64, 384) is not None
    assert P.prom_pw_plan_query(1, 14, 14, 64, 384)["k_outer"] == 0
    for shape in ((128, 7, 7, 2048, 1024), (1, 14, 14, 64, 384)):
        assert P.prom_pw_kernel_query(*shape, plan=P.PwPlan(k_outer=-1)) is None
        tm, tn = P.prom_pw_kernel_query(*shape, plan=P.PwPlan(k_outer=1))
        assert tm in (32, 64, 128) and tn in (128, 256)
    # a plan that names the streaming kernel's shape keeps it, channel counts that are no whole pieces have no choice
    assert P.prom_pw_kernel_query(1, 14, 14, 64, 384, plan=P.PwPlan(tiles_per_wave=4)) is None
    assert P.prom_pw_kernel_query(32, 56, 56, 24, 144) is None
    assert P.prom_pw_kernel_query(1, 14, 14, 64, 388) is None
    with pytest.raises(P.PromError):
        P.prom_pw_kernel_query(1, 4, 4, 72, 32, plan=P.PwPlan(k_outer=1))
    with pytest.raises(P.PromError):
        P.prom_pw_kernel_query(0, 4, 4, 64, 32)


def test_workgroups_alone_leave_the_planned_kernel(P):
    # a layer planned for the tile kernel stays on it; one that is not gets the streaming kernel's workgroups
    assert P.prom_pw_kernel_query(128, 14, 14, 1024, 512, plan=P.PwPlan(workgroups=64)) is not None
    assert P.prom_pw_kernel_query(1, 14, 14, 64, 384, plan=P.PwPlan(workgroups=4)) is None


def test_tile_shapes(P):
    # (8, 2) has too few wavefronts in flight for one or two tiles per compute unit
    for shape in ((107, 14, 14, 512, 320), (96, 14, 14, 160, 384), (128, 14, 14, 1024, 320)):
        assert P.prom_pw_kernel_query(*shape) == (64, 128), shape
    assert P.prom_pw_kernel_query(64, 14, 14, 2048, 320)[1] == 128  # 320 channels are two and a half tiles of 128
    assert P.prom_pw_kernel_query(128, 14, 14, 1024, 512) == (128, 256)
    # a layer that is planned for the tile kernel, or asked for by the caller, gets the shape that the estimate names
    # also where the rule for narrower layers would keep the streaming kernel
    assert P.prom_pw_plan_query(128, 14, 14, 1024, 272)["k_outer"] == 1
    assert P.prom_pw_kernel_query(128, 14, 14, 1024, 272)[1] == 128
    assert P.prom_pw_kernel_query(1, 7, 7, 1024, 64, plan=P.PwPlan(k_outer=1)) == (32, 128)


def test_deep_layers_with_few_pixels_stay(P):
    # as long as the streaming kernel's workgroups all run at a time
    for shape in ((8, 14, 14, 960, 896), (25, 7, 11, 1344, 768), (4, 14, 14, 1024, 512), (1, 32, 64, 1024, 1024)):
        assert P.prom_pw_kernel_query(*shape) is None, shape
    for shape in ((1, 3, 683, 1024, 1024), (32, 14, 14, 1024, 512), (16, 14, 14, 1536, 1024)):
        assert P.prom_pw_kernel_query(*shape) is not None, shape
    # rows that are no whole 64 bytes: from half as many on
    assert P.prom_pw_kernel_query(6, 14, 14, 992, 1024) is not None
    assert P.prom_pw_kernel_query(2, 14, 14, 992, 1024) is None


def test_streams_without_residual_stay(P):
    for shape in ((64, 56, 56, 128, 256), (128, 56, 56, 128, 256), (64, 56, 56, 256, 256), (128, 28, 28, 256, 512),
                  (192, 14, 14, 192, 768)):
        assert P.prom_pw_kernel_query(*shape) is None, shape
        assert P.prom_pw_kernel_query(*shape, prelu=True) is not None, shape
    for shape in ((128, 56, 56, 128, 256), (128, 28, 28, 256, 512), (192, 14, 14, 192, 768)):
        assert P.prom_pw_kernel_query(*shape, residual=True) is not None, shape
    for shape in ((16, 56, 56, 128, 256), (32, 28, 28, 256, 512), (80, 28, 28, 256, 512)):  # few tiles, a full last round
        assert P.prom_pw_kernel_query(*shape) is not None, shape


def test_ragged_channels_with_two_tiles_per_unit(P):
    # 96 -> 576 runs in its own tiles of 128 x 128; how many of 128 x 256 there would be does not matter
    for n in (96, 111, 114, 128, 135, 139, 142):
        assert P.prom_pw_kernel_query(n, 14, 14, 96, 576) is not None, n
    assert P.prom_pw_kernel_query(128, 14, 14, 96, 576) == (128, 128)
    assert P.prom_pw_kernel_query(114, 14, 14, 192, 768, residual=True) is None     # fills its tiles


def test_64_channels_into_ragged_columns_stay_from_12_million_outputs(P):
    for shape in ((128, 28, 28, 64, 160), (122, 28, 28, 64, 224), (86, 28, 28, 64, 288), (90, 28, 28, 64, 336)):
        assert P.prom_pw_kernel_query(*shape) is None, shape
    assert P.prom_pw_kernel_query(77, 28, 28, 64, 208, residual=True) is not None
    assert P.prom_pw_kernel_query(96, 28, 28, 64, 160, residual=True, prelu=True) is None
    for shape in ((32, 28, 28, 64, 160), (64, 28, 28, 64, 160), (73, 28, 28, 64, 208), (96, 28, 28, 64, 256), (96, 28, 28, 48, 112)):
        assert P.prom_pw_kernel_query(*shape) is not None, shape


def test_narrow_outputs_of_6_to_8_k_steps_stay(P):
    for shape in ((64, 56, 56, 512, 256), (30, 56, 56, 352, 384)):
        assert P.prom_pw_kernel_query(*shape) is None, shape
        assert P.prom_pw_kernel_query(*shape, residual=True) is not None, shape
    assert P.prom_pw_kernel_query(64, 28, 28, 512, 256) is not None
    assert P.prom_pw_kernel_query(48, 56, 56, 512, 512) is not None


def test_odd_multiples_of_64_with_a_residual_stay_up_to_two_rounds(P):
    assert P.prom_pw_kernel_query(44, 14, 14, 960, 448, residual=True) is None
    assert P.prom_pw_kernel_query(44, 14, 14, 960, 448) is not None
    assert P.prom_pw_kernel_query(128, 14, 14, 960, 448, residual=True) is not None
