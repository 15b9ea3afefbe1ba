"""GPU: the setup with its neighbourhoods in LDS (launch shape 4) against the setup that gathers
from global memory (shape 1): bitwise equal energies, states, gradients and products.

Grids that the 64 x 8 x 4 tiles do not divide, several tiles along x, grids smaller than a tile
and its halo (the box wraps more than once), offsets within one voxel per step, within the box,
partly and wholly past it; a velocity per time node."""
import os

import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem

pytestmark = pytest.mark.gpu

NT = 4


def _run(shape, prob, I0, I1, vs, dv, **kw):
    os.environ["BL_LAUNCH_SHAPES"] = f"2,2,2,2,{shape},1,0"
    try:
        ctx = B.Ctx(bl_problem(prob, **kw), I0, I1)
        E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
        out = [np.float64(E), g, ctx.bl_lddmm_ctx_get_field("state", NT),
               ctx.bl_lddmm_ctx_hessvec(dv)]
        ctx.close()
    finally:
        os.environ.pop("BL_LAUNCH_SHAPES", None)
    return out


@pytest.mark.parametrize("n,k", [((128, 24, 20), (16, 8, 8)), ((130, 21, 13), (16, 8, 4)),
                                 ((61, 8, 4), (8, 4, 4)), ((65, 9, 5), (8, 4, 4)),
                                 ((6, 5, 4), (4, 4, 4)), ((200, 17, 30), (8, 8, 8))])
@pytest.mark.parametrize("disp", [2.0, 7.0, 13.0, 100.0])
@pytest.mark.parametrize("nonstationary", [False, True])
def test_setup_forms_agree(gpu_lib, n, k, disp, nonstationary):
    prob = O.Problem(3, n, k, NT)
    rng = np.random.default_rng(1)
    I0 = rng.random(prob.shape, dtype=np.float32)
    I1 = np.roll(I0, 1, axis=-1)
    vs = O.project(phantoms.raw_band_velocity(3, 3, k), prob)
    vs = vs * (disp / O.max_displacement_voxels(vs, prob))
    dv = O.project(phantoms.random_band_direction(4, 3, k), prob)
    if nonstationary:
        vs = np.stack([vs * (1.0 - 0.2 * i) for i in range(NT + 1)])
        dv = np.stack([dv] * (NT + 1))
    args = (prob, I0, I1, vs.astype(np.complex64), dv.astype(np.complex64))
    got = _run(4, *args, nonstationary=nonstationary)
    ref = _run(1, *args, nonstationary=nonstationary)
    assert all(np.array_equal(a, b) for a, b in zip(got, ref))
