"""GPU: which settings of the launch shapes keep the transports in step launches: those that force a
shape, not those that only keep the defaults without timing."""
import pytest

from paper_1807_05117_amd import binding as B

from parity_cases import bl_problem
from test_gpu_sweeps import _inputs, _results, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,value,forced", [
    ("BL_TRANSPORT_ZV", "0", False), ("BL_TRANSPORT_ZV", "3", False), ("BL_TRANSPORT_ZV", "4", True),
    ("BL_LAUNCH_SHAPES", "2,2,2,2,4,1,0", True), ("BL_LAUNCH_SHAPES", "2,2", False)])
def test_only_forced_shapes_keep_to_steps(gpu_lib, name, value, forced, monkeypatch):
    prob, I0, I1, vs, dv = _inputs((64, 60, 62), (8, 8, 8), 3, 2.0)
    ref = _results(B.Ctx(bl_problem(prob), I0, I1), prob, vs, dv)
    monkeypatch.setenv(name, value)
    ctx = B.Ctx(bl_problem(prob), I0, I1)
    got = _results(ctx, prob, vs, dv)
    fwd, bwd = ctx.bl_lddmm_ctx_sweeps()[1:3]
    ctx.close()
    assert _same(got, ref)
    assert (fwd, bwd) == ((0, 0) if forced else (3, 3))
