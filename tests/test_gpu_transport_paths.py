"""GPU: the transports' two index paths.  A wavefront whose offsets all stay below a period
wraps its taps by unsigned minima, any other one takes the general wrap; blocks cover 256
entries of the flattened plane whatever the row length.  Velocities around a whole period
(some lanes below it, some past it), of several periods and of the opposite sign, on grids whose
rows and planes no block divides, against the oracle.

Tolerance: the offsets are FP32 values of up to 3 n voxels with a relative error of about 1e-6
(transform sums and Heun average), i.e. below 1e-4 voxels on these grids, and a d-linear
interpolation moves by at most the image's range per voxel."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem, grad_error

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.mark.parametrize("n,k", [((30, 26), (8, 6)), ((4, 5, 7), (4, 4, 4)), ((33, 9, 11), (8, 4, 4)),
                                 ((70, 10, 6), (8, 4, 4))])
@pytest.mark.parametrize("periods", [0.0, 1.0, -1.0, 2.6])
def test_offsets_past_a_period(gpu_lib, n, k, periods):
    dim = len(n)
    prob = O.Problem(dim, n, k, 2)
    rng = np.random.default_rng(3)
    I0 = sum(np.cos(2 * np.pi * (i / m + rng.random())) for i, m in
             zip(np.indices(prob.shape), prob.shape)).astype(np.float32)
    vs = O.project(phantoms.raw_band_velocity(1, dim, k), prob)
    vs *= 0.4 * prob.nt / O.max_displacement_voxels(vs, prob)
    # a constant part of `periods` whole periods per step along every axis
    for j in range(dim):
        vs[j][tuple(K // 2 for K in prob.bshape)] += periods * prob.nt * n[j] / prob.nref
    vs = vs.astype(np.complex64)
    p = bl_problem(prob)
    ref = O.warp(I0.astype(np.float64), vs, prob)
    m1 = B.bl_lddmm_warp(p, I0, vs)
    err = np.abs(m1 - ref).max() / np.abs(I0).max()
    I1 = np.roll(I0, 1, axis=0)
    g, E = B.bl_lddmm_gradient(p, I0, I1, vs)
    st = O.evaluate(vs, I0.astype(np.float64), I1.astype(np.float64), prob)
    ge = grad_error(g, O.gradient(st), prob, vs)
    print(n, periods, "m(1) %.1e gradient %.1e" % (err, ge), flush=True)
    assert err < TOL
    assert ge < TOL
