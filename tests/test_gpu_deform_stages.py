"""GPU: the deformation method's stage kernels at the edges of their tiles."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem, rel2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [((24, 20, 12), (8, 8, 4)), ((30, 50, 18), (18, 34, 6)),
                                 ((70, 20, 16), (66, 4, 4)), ((50, 44, 40), (40, 36, 32)),
                                 ((20, 100, 12), (4, 96, 8)), ((130, 12, 8), (128, 2, 4))])
def test_stage_kernels_at_tile_edges(gpu_lib, n, k, monkeypatch):
    """the stage kernels' tiles of 16 ky by 32 kx and of 16 x (several, partial, more than five x
    tiles, bands up to 128) against the unfused chain, with that comparison's tolerance"""
    prob = O.Problem(3, n, k, 3)
    rng = np.random.default_rng(2)
    I0, I1 = (np.cumsum(rng.random(prob.shape), axis=-1).astype(np.float32) for _ in range(2))
    vh = O.project(phantoms.raw_band_velocity(4, 3, k), prob)
    vh = (vh * (1.0 / O.max_displacement_voxels(vh, prob))).astype(np.complex64)
    dv = O.project(phantoms.random_band_direction(5, 3, k), prob).astype(np.complex64)
    out = {}
    for flag in ("1", "0"):
        monkeypatch.setenv("BL_DEFORM_FUSED", flag)
        ctx = B.Ctx(bl_problem(prob, deformation=True), I0, I1)
        E, g = ctx.bl_lddmm_ctx_set_velocity(vh)
        out[flag] = (E, g.astype(np.complex128),
                     ctx.bl_lddmm_ctx_hessvec(dv).astype(np.complex128))
        ctx.close()
    (E1, g1, H1), (E0, g0, H0) = out["1"], out["0"]
    assert abs(E1 - E0) <= 1e-6 * E0
    assert rel2(g1, g0) < 2e-6 and rel2(H1, H0) < 2e-6
