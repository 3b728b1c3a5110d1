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
