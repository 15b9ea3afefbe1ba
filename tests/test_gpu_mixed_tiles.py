"""GPU: the mixed-precision z stages at the edges of their tiles (32 or 64 columns, 32 planes, 16
planes a step, every count of kz fragments), 2D and 3D.

Against the FP64 sums.  A BF16 number keeps 8 bits, so |lo| <= 2^-9 |x| and the rest after lo is
below 2^-18 |x|: with the dropped lo*lo term a product is off by at most 3 2^-18 of itself.  In the
2-norm the errors of all terms of one sign add up to at most sqrt(K) times that for the K = kz
orthogonal rows of iota, and sqrt(nz) times for pi of noise (whose sums keep kz / nz of its square).
The FP32 stages and sums add 2^-24 for each term, as in the plain form."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem, rel2

pytestmark = pytest.mark.gpu

SHAPES = [((5, 7, 4), (2, 2, 2)), ((9, 7, 33), (4, 4, 16)), ((13, 5, 64), (4, 4, 30)),
          ((11, 17, 47), (4, 6, 34)), ((8, 16, 130), (4, 4, 48)), ((13, 11, 97), (4, 4, 66)),
          ((6, 11, 96), (4, 4, 82)), ((21, 5, 128), (4, 2, 98)), ((7, 19, 140), (4, 4, 128)),
          ((160, 192, 40), (8, 8, 40)), ((31, 33), (8, 8))]


@pytest.mark.parametrize("n,k", SHAPES)
def test_mixed_transforms_at_tile_edges(gpu_lib, n, k):
    dim = len(n)
    prob = O.Problem(dim, n, k, 3)
    p = bl_problem(prob, precision=B.BL_MIXED)
    vh = O.project(phantoms.raw_band_velocity(6, dim, k), prob).astype(np.complex64)
    grid = B.bl_band_to_grid(p, vh)
    for c in range(dim):
        ref = O.iota(vh[c].astype(np.complex128), prob)
        assert rel2(grid[c], ref) < 3 * 2.0 ** -18 * np.sqrt(k[-1]) + (sum(k) + 6) * 2.0 ** -24, c
    f = np.random.default_rng(5).standard_normal((2,) + prob.shape).astype(np.float32)
    band = B.bl_grid_to_band(p, f)
    for c in range(2):
        ref = O.pi_(f[c].astype(np.float64), prob)
        assert rel2(band[c], ref) < 3 * 2.0 ** -18 * np.sqrt(n[-1]) + (sum(n) + 6) * 2.0 ** -24, c
