"""GPU: allocation-free products beside another stream's additions, whose blocks hold the compute units
that sweeps wait for: each call has a context of its own, and the calls rest from sweeps all the same."""
import numpy as np
import pytest

from paper_1807_05117_amd import binding as B

from parity_cases import bl_problem
from test_gpu_sweeps import _inputs

pytestmark = pytest.mark.gpu


def test_noalloc_products_beside_other_work_rest_from_sweeps(gpu_lib):
    import torch
    calls = 16
    prob, I0, I1, vs, dv = _inputs((128, 128, 128), (16, 16, 16), 5, 3.0)
    p, other = bl_problem(prob), torch.cuda.Stream()
    ref = B.bl_lddmm_hessvec_noalloc(p, I0, I1, vs, dv)
    with torch.cuda.stream(other):
        x = torch.zeros(1 << 28, device="cuda")
        x.add_(1)   # 0.4 ms
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        with torch.cuda.stream(other):
            for _ in range(400):
                x.add_(1)
        got = [B.bl_lddmm_hessvec_noalloc(p, I0, I1, vs, dv) for _ in range(calls)]
        busy = not other.query()
        torch.cuda.synchronize()
    assert busy   # until the last call
    swept = sum("k_sweep" in e.name for e in prof.events())
    # without rests three each; if all are late, the 1st and 2nd call have three, the 3rd two, the
    # 5th, 8th and 13th one
    assert 0 < swept < 3 * calls, swept
    assert all(np.array_equal(h, ref) for h in got)
