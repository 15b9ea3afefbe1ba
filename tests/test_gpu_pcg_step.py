"""GPU: the solver's PCG launches (start of a solve in one launch; the final sums with the next
direction, as one problem takes it) at bands smaller than one block, ragged ones and ones past the
grid of 512 blocks, one PCG step and several.  The cohort server sums and steps in launches of their
own, in the same order: every velocity and statistic is bitwise the same."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,band,max_pcg",
                         [((8, 8), (2, 2), 4), ((16, 16, 16), (2, 2, 2), 1),
                          ((20, 14, 24), (4, 6, 10), 7), ((44, 40, 44), (44, 40, 44), 3)])
def test_pcg_of_one_problem_and_of_a_cohort(gpu_lib, grid, band, max_pcg):
    dim, nt = len(grid), 3
    prob = O.Problem(dim, grid, band, nt)
    rng = np.random.default_rng(11)
    vs = O.project(phantoms.raw_band_velocity(2, dim, band), prob)
    vs *= 1.0 / O.max_displacement_voxels(vs, prob)
    I0 = rng.random(prob.shape).astype(np.float32)
    I1 = O.warp(I0.astype(np.float64), vs, prob).astype(np.float32)
    p = B.make_problem(dim, grid, band, nt)
    opts = B.opts_struct(max_gn=3, max_pcg=max_pcg)
    v, w, st = B.bl_lddmm_register(p, I0, I1, np.zeros(B.band_shape(p), np.complex64), opts)
    srv = B.Server(batched=True, max_slots=2)
    rc, v2, w2, st2, _ = srv.wait(srv.submit(p, I0, I1, opts=opts))
    srv.close()
    assert rc == B.BL_OK and st["hessvecs"] > 0
    assert np.array_equal(v, v2) and np.array_equal(w, w2)
    for k in ("status", "gn_iters", "hessvecs", "pcg_total", "E", "pcg_iters", "eps"):
        assert st[k] == st2[k], (k, st[k], st2[k])
