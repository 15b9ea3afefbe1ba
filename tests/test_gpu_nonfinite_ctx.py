"""GPU: a context that was given a non-finite velocity reports it and serves the next valid one as if
nothing had been: the flag of the refused call's band outputs is not left for a later call to find."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem

pytestmark = pytest.mark.gpu

MODELS = [{}, dict(nonstationary=True), dict(newton=True), dict(deformation=True),
          dict(precision=B.BL_MIXED)]


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_valid_gradient_after_a_nonfinite_velocity(gpu_lib, model, bad):
    prob = O.Problem(3, (20, 18, 16), (6, 6, 4), 3)
    rng = np.random.default_rng(3)
    I0, I1 = (rng.random(prob.shape).astype(np.float32) for _ in range(2))
    vs = O.project(phantoms.raw_band_velocity(1, 3, prob.k), prob)
    vs = (vs / O.max_displacement_voxels(vs, prob)).astype(np.complex64)
    if model.get("nonstationary"):
        vs = np.stack([vs] * (prob.nt + 1))
    wrong = vs.copy()
    wrong[..., 1, 2] = bad
    ctx = B.Ctx(bl_problem(prob, **model), I0, I1)
    E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
    for gradient in (True, False):
        with pytest.raises(B.BLError) as e:
            ctx.bl_lddmm_ctx_set_velocity(wrong, want_gradient=gradient)
        assert e.value.code == B.BL_E_NONFINITE
        E2, g2 = ctx.bl_lddmm_ctx_set_velocity(vs)
        assert E2 == E and np.array_equal(g2, g)
    ctx.close()
