"""GPU: an abandoned sweep whose wait for its earlier parts is given up (here after no look at all, a
limit that a working run does not meet) fails the call that waits for it, or the next one after an
enqueued product, as a device error; the context then serves the velocity set again."""
import numpy as np
import pytest

from paper_1807_05117_amd import binding as B

from parity_cases import bl_problem
from test_gpu_sweeps import _inputs

pytestmark = pytest.mark.gpu

# offsets of ten voxels per step: every sweep leaves its tiles' boxes and is abandoned
CASE = ((128, 128, 128), (16, 16, 16), 4, 40.0)
ALL = 2 ** 24


def _device_error(f):
    with pytest.raises(B.BLError) as e:
        f()
    assert e.value.code == B.BL_E_DEVICE and "waited" in str(e.value), e.value


@pytest.mark.parametrize("newton", [False, True])
def test_given_up(gpu_lib, newton):
    prob, I0, I1, vs, dv = _inputs(*CASE)
    ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
    E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
    H = ctx.bl_lddmm_ctx_hessvec(dv)
    ctx.close()
    for gradient in (False, True):
        ctx = B.Ctx(bl_problem(prob, newton=newton), I0, I1)
        ctx.bl_lddmm_ctx_sweep_polls(0)
        _device_error(lambda: ctx.bl_lddmm_ctx_set_velocity(vs, want_gradient=gradient))
        with pytest.raises(B.BLError) as e:   # no velocity: its state is not valid
            ctx.bl_lddmm_ctx_hessvec(dv)
        assert e.value.code == B.BL_E_INVALID
        ctx.bl_lddmm_ctx_sweep_polls(ALL)
        E2, g2 = ctx.bl_lddmm_ctx_set_velocity(vs)
        assert E2 == E and np.array_equal(g2, g)
        assert np.array_equal(ctx.bl_lddmm_ctx_hessvec(dv), H)
        ctx.close()


def test_given_up_in_an_enqueued_product(gpu_lib):
    import torch
    prob, I0, I1, vs, dv = _inputs((96, 96, 96), (16, 16, 16), 4, 3.0)
    s = torch.cuda.current_stream()
    dI0, dI1, dvs, ddv = (torch.from_numpy(x).cuda() for x in (I0, I1, vs, dv))
    ctx = B.Ctx(bl_problem(prob, device=True, stream=s.cuda_stream), dI0, dI1)
    E, g = ctx.bl_lddmm_ctx_set_velocity(dvs)
    H = ctx.bl_lddmm_ctx_hessvec(ddv).clone()
    ctx.bl_lddmm_ctx_sweep_wait(0)
    ctx.bl_lddmm_ctx_sweep_polls(0)
    ctx.bl_lddmm_ctx_hessvec(ddv)
    ctx.bl_lddmm_ctx_sweep_wait(100)
    ctx.bl_lddmm_ctx_sweep_polls(ALL)
    _device_error(lambda: ctx.bl_lddmm_ctx_set_velocity(dvs))
    E2, g2 = ctx.bl_lddmm_ctx_set_velocity(dvs)
    assert E2 == E and torch.equal(g2, g) and torch.equal(ctx.bl_lddmm_ctx_hessvec(ddv), H)
    ctx.close()


def test_polls_outside_the_range_are_refused(gpu_lib):
    prob, I0, I1, vs, dv = _inputs((8, 8, 8), (4, 4, 4), 2, 1.0)
    ctx = B.Ctx(bl_problem(prob), I0, I1)
    for polls in (-1, ALL + 1):
        with pytest.raises(B.BLError) as e:
            ctx.bl_lddmm_ctx_sweep_polls(polls)
        assert e.value.code == B.BL_E_INVALID
    ctx.close()
