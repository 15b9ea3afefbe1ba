"""GPU: which path a transport took, asserted beside its results: that a sweep ran where the grid has a
plan, that it abandoned itself where offsets leave a tile's box, and that a sweep whose tiles run
out of time in its middle is finished with the same values (a wait of 0: a tile abandons at the first
progress it does not find), for every kind of sweep."""
import numpy as np
import pytest

from paper_1807_05117_amd import binding as B

from parity_cases import bl_problem
from test_gpu_sweeps import GRIDS, _inputs, _results, _same

pytestmark = pytest.mark.gpu


def _steps(ctx, prob, vs, dv):
    """the same results from step launches"""
    ctx.bl_kernel_timing_enable(True)
    before = ctx.bl_lddmm_ctx_sweeps()
    ref = _results(ctx, prob, vs, dv)
    assert ctx.bl_lddmm_ctx_sweeps()[1:3] == before[1:3]
    ctx.bl_kernel_timing_enable(False)
    return ref


@pytest.mark.parametrize("n,k", GRIDS + [((160, 160, 160), (8, 8, 8)), ((131, 128, 128), (8, 8, 8)),
                                         ((2000, 1000), (8, 8))])
@pytest.mark.parametrize("newton", [False, True])
def test_a_sweep_runs_where_there_is_a_plan(gpu_lib, n, k, newton):
    """an evaluation with its gradient and two products: three sweeps each way"""
    prob, I0, I1, vs, dv = _inputs(n, k, 2, 1.0)
    ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    got = _results(ctx, prob, vs, dv)
    tiles, *rest = ctx.bl_lddmm_ctx_sweeps()
    ref = _steps(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)
    assert (tiles > 0) == (n not in [(160, 160, 160), (131, 128, 128), (2000, 1000)])
    assert tuple(rest) == ((3, 3, 0, 0, 0, 0) if tiles else (0,) * 6)


@pytest.mark.parametrize("n,k,disp", [((128, 128, 128), (16, 16, 16), 40.0),
                                      ((33, 90, 70), (8, 8, 8), 200.0), ((1024, 40), (8, 8), 700.0)])
@pytest.mark.parametrize("newton", [False, True])
def test_offsets_past_the_box_abandon_both_sweeps(gpu_lib, n, k, disp, newton):
    prob, I0, I1, vs, dv = _inputs(n, k, 4, disp)
    ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    got = _results(ctx, prob, vs, dv)
    tiles, fwd, bwd, left_x, left_y, _, _ = ctx.bl_lddmm_ctx_sweeps()
    ref = _steps(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)
    assert tiles > 0 and fwd > 0 and bwd > 0 and left_x > 0 and left_y > 0


@pytest.mark.parametrize("n,k", [((128, 128, 128), (16, 16, 16)), ((96, 96, 96), (16, 16, 16)),
                                 ((130, 50, 37), (8, 8, 8)), ((300, 200), (16, 16))])
@pytest.mark.parametrize("newton", [False, True])
def test_out_of_time_in_the_middle(gpu_lib, n, k, newton):
    """state and adjoint of a gradient, then the two sweeps of a product"""
    prob, I0, I1, vs, dv = _inputs(n, k, 5, 3.0)
    first = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    first.bl_lddmm_ctx_sweep_wait(0)
    E, g = first.bl_lddmm_ctx_set_velocity(vs)
    m = first.bl_lddmm_ctx_get_field("state", prob.nt)
    seen = first.bl_lddmm_ctx_sweeps()
    first.close()
    assert seen[1:] == (1, 1, 0, 0, 1, 1), seen

    ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    ctx.bl_lddmm_ctx_set_velocity(vs)
    ctx.bl_lddmm_ctx_sweep_wait(0)
    H = ctx.bl_lddmm_ctx_hessvec(dv)
    seen = ctx.bl_lddmm_ctx_sweeps()
    assert seen[1:] == (2, 2, 0, 0, 1, 1), seen
    ctx.bl_lddmm_ctx_sweep_wait(100)
    E0, g0, _, m0, H0, _ = _steps(ctx, prob, vs, dv)
    ctx.close()
    assert E == E0 and np.array_equal(g, g0) and np.array_equal(m, m0) and np.array_equal(H, H0)


def test_waits_outside_the_range_are_refused(gpu_lib):
    prob, I0, I1, vs, dv = _inputs((8, 8, 8), (4, 4, 4), 2, 1.0)
    ctx = B.Ctx(bl_problem(prob), I0, I1)
    for wait in (-1.0, 2e6, float("nan")):
        with pytest.raises(B.BLError) as e:
            ctx.bl_lddmm_ctx_sweep_wait(wait)
        assert e.value.code == B.BL_E_INVALID
    ctx.close()
