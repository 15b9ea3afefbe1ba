"""GPU: the transforms on the matrix cores at the edges of their tiles of 16 (columns, rows, kz, ky
and kx that no tile divides, one coefficient, the widest bands, the bands past 128 that take the
vector kernels), 2D and 3D.

Against the FP64 sums: an FP32 sum of K terms rounds K times, each time by at most 2^-24 of a
partial sum, so the relative error in the 2-norm stays below (K + 6) 2^-24 with K the terms of all
stages (six more for the twiddles, the products and the z stages' sums and differences)."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem, rel2

pytestmark = pytest.mark.gpu

SHAPES = [((20, 12, 9), (2, 2, 2)), ((33, 40, 17), (16, 18, 16)), ((48, 20, 70), (34, 16, 34)),
          ((24, 150, 12), (8, 132, 4)), ((150, 24, 12), (132, 8, 4)), ((12, 10, 140), (4, 4, 128)),
          ((13, 10, 100), (4, 4, 66)), ((16, 18, 101), (10, 6, 98)), ((270, 9, 6), (6, 4, 4)),
          ((70, 130), (32, 66)), ((5, 4), (4, 2)), ((257, 31), (128, 30))]


@pytest.mark.parametrize("n,k", SHAPES)
def test_transforms_at_tile_edges(gpu_lib, n, k):
    dim = len(n)
    prob = O.Problem(dim, n, k, 3)
    p = bl_problem(prob)
    vh = O.project(phantoms.raw_band_velocity(6, dim, k), prob).astype(np.complex64)
    grid = B.bl_band_to_grid(p, vh)
    for c in range(dim):
        ref = O.iota(vh[c].astype(np.complex128), prob)
        assert rel2(grid[c], ref) < (sum(k) + 6) * 2.0 ** -24, c
    f = np.random.default_rng(5).standard_normal((2,) + prob.shape).astype(np.float32)
    band = B.bl_grid_to_band(p, f)
    for c in range(2):
        ref = O.pi_(f[c].astype(np.float64), prob)
        assert rel2(band[c], ref) < (sum(n) + 6) * 2.0 ** -24, c
