"""GPU: what a context learns from an abandoned sweep.  Offsets that leave a tile's box do so in every
sweep of the velocity: its later products are step launches, and after it 1, 2, 4, ... velocities are."""
import numpy as np
import pytest

from paper_1807_05117_amd import binding as B

from parity_cases import bl_problem
from test_gpu_sweeps import _inputs, _results, _same

pytestmark = pytest.mark.gpu

PAST = ((128, 128, 128), (16, 16, 16), 4, 40.0)   # ten voxels per step


@pytest.mark.parametrize("newton", [False, True])
def test_velocity_past_the_box_is_swept_once(gpu_lib, newton):
    prob, I0, I1, vs, dv = _inputs(*PAST)
    near = (vs / 16).astype(np.complex64)
    ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    swept, got = [], []
    for i in range(12):   # sweeps are tried at velocities 0, 2, 5 and 10
        before = ctx.bl_lddmm_ctx_sweeps()
        E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
        after = ctx.bl_lddmm_ctx_sweeps()
        swept.append(after[1] - before[1])
        H = [ctx.bl_lddmm_ctx_hessvec(dv) for _ in range(2)]
        # neither direction is tried again by the products
        assert ctx.bl_lddmm_ctx_sweeps()[1:5] == after[1:5], i
        got.append([np.float64(E), g, *H])
    assert swept == [1, 0, 1, 0, 0, 1, 0, 0, 0, 0, 1, 0]
    tiles, fwd, bwd, left_x, left_y, _, _ = ctx.bl_lddmm_ctx_sweeps()
    assert (fwd, bwd, left_x, left_y) == (4, 4, 4, 4)
    for _ in range(7):   # of the eight that rest
        ctx.bl_lddmm_ctx_set_velocity(near)
    assert ctx.bl_lddmm_ctx_sweeps()[1] == 4
    ctx.bl_lddmm_ctx_set_velocity(near)
    ctx.bl_lddmm_ctx_hessvec(dv)
    assert ctx.bl_lddmm_ctx_sweeps()[1:5] == (6, 6, 4, 4)
    ctx.bl_lddmm_ctx_set_velocity(near)
    assert ctx.bl_lddmm_ctx_sweeps()[1:5] == (7, 7, 4, 4)
    ctx.bl_kernel_timing_enable(True)
    E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
    ref = [np.float64(E), g, *[ctx.bl_lddmm_ctx_hessvec(dv) for _ in range(2)]]
    ctx.close()
    assert all(_same(x, ref) for x in got)


def test_registration_past_the_box(gpu_lib):
    """a whole registration whose first velocities leave the box is that of the step launches"""
    prob, I0, I1, vs, dv = _inputs((96, 96, 96), (8, 8, 8), 2, 60.0)
    opts = B.opts_struct(max_gn=2, max_pcg=3)
    p = bl_problem(prob)
    got = B.bl_lddmm_register(p, I0, I1, vs, opts)
    again = B.bl_lddmm_register(p, I0, I1, vs, opts)   # the cached context, which rests
    srv = B.Server(batched=True, max_slots=1)          # step launches
    rc, v, w, st, _ = srv.wait(srv.submit(p, I0, I1, vs, opts))
    srv.close()
    assert rc == B.BL_OK
    for r in (got, again):
        assert np.array_equal(r[0], v) and np.array_equal(r[1], w) and r[2]["E"] == st["E"]


def test_noalloc_products_past_the_box(gpu_lib):
    prob, I0, I1, vs, dv = _inputs(*PAST)
    p = bl_problem(prob)
    ref = B.bl_lddmm_hessvec(p, I0, I1, vs, dv)
    near = (vs / 16).astype(np.complex64)
    ref_near = B.bl_lddmm_hessvec(p, I0, I1, near, dv)
    for _ in range(4):
        assert np.array_equal(B.bl_lddmm_hessvec_noalloc(p, I0, I1, vs, dv), ref)
    for _ in range(4):
        assert np.array_equal(B.bl_lddmm_hessvec_noalloc(p, I0, I1, near, dv), ref_near)
