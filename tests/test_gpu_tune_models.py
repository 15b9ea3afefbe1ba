"""GPU: launch shapes remembered for a grid by a stationary and by a non-stationary context do not
meet: the setup of a non-stationary velocity (one launch for all steps, its form fixed by the tiles of
all of them) is neither taken from a stationary context's timing nor remembered for one."""
import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem

pytestmark = pytest.mark.gpu

SETUP = 4   # the setup's place in a remembered line


@pytest.mark.parametrize("stationary_first", [False, True])
def test_models_do_not_share_the_setup_shape(gpu_lib, stationary_first, tmp_path, monkeypatch):
    # 100 tiles of 64 x 8 x 4 voxels a step: below 512 for one step, above it for eight
    prob = O.Problem(3, (40, 40, 80), (6, 6, 6), 8)
    cache = tmp_path / "shapes.txt"
    monkeypatch.setenv("BL_TUNE_CACHE", str(cache))
    for name in ("BL_TRANSPORT_ZV", "BL_LAUNCH_SHAPES"):
        monkeypatch.delenv(name, raising=False)
    B.load().bl_lddmm_tune_reload()
    rng = np.random.default_rng(0)
    I0 = rng.random(prob.shape).astype(np.float32)
    vs = O.project(phantoms.raw_band_velocity(1, 3, prob.k), prob)
    vs = (vs / O.max_displacement_voxels(vs, prob)).astype(np.complex64)
    lines = {}
    try:
        for nonstationary in (not stationary_first, stationary_first):
            ctx = B.Ctx(bl_problem(prob, nonstationary=nonstationary), I0, I0)
            ctx.bl_lddmm_ctx_set_velocity(np.stack([vs] * (prob.nt + 1)) if nonstationary else vs)
            ctx.close()
            new = [x for x in cache.read_text().splitlines() if x not in lines.values()]
            assert len(new) == 1, (nonstationary, new)   # each model times and remembers its own
            lines[nonstationary] = new[0]
    finally:
        monkeypatch.undo()
        B.load().bl_lddmm_tune_reload()
    shapes = {ns: [int(x) for x in line.split(":")[1].split()] for ns, line in lines.items()}
    assert shapes[True][SETUP] == 4      # by rule: 800 tiles
    assert lines[True].split(":")[0] != lines[False].split(":")[0]
