"""GPU: a transport's time steps in one launch (tiles resident on the device, taps in registers)
against the same steps launched one by one, which per-kernel timing selects: bitwise equal
energies, states, gradients and products.

The grids are chosen where the tiling can go wrong: rows that are no multiple of the 16-byte
loads, planes and rows that no tile divides, one tile for the whole grid, tiles that span one
axis, two dimensions; offsets that leave a tile's box (the sweep is abandoned and finished
through tickets); few time steps; several threads whose sweeps compete for the device; graph
replays."""
import threading

import numpy as np
import pytest

import oracle as O
from paper_1807_05117_amd import binding as B
from paper_1807_05117_amd import phantoms

from parity_cases import bl_problem

pytestmark = pytest.mark.gpu


def _inputs(n, k, nt, disp, seed=0):
    dim = len(n)
    prob = O.Problem(dim, n, k, nt)
    rng = np.random.default_rng(seed)
    I0 = sum(np.cos(2 * np.pi * (2 * i / m + rng.random())) for i, m in
             zip(np.indices(prob.shape), prob.shape)).astype(np.float32)
    I0 += 0.1 * rng.random(prob.shape, dtype=np.float32)
    vs = O.project(phantoms.raw_band_velocity(seed, dim, k), prob)
    vs = (vs * (disp / O.max_displacement_voxels(vs, prob))).astype(np.complex64)
    dv = O.project(phantoms.random_band_direction(seed + 1, dim, k), prob)
    dv = (dv / np.abs(dv).max()).astype(np.complex64)
    return prob, I0, np.roll(I0, 1, axis=-1), vs, dv


def _results(ctx, prob, vs, dv):
    E, g = ctx.bl_lddmm_ctx_set_velocity(vs)
    m = [ctx.bl_lddmm_ctx_get_field("state", i) for i in (1, prob.nt)]
    return [np.float64(E), g, *m, ctx.bl_lddmm_ctx_hessvec(dv), ctx.bl_lddmm_ctx_hessvec(dv)]


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


GRIDS = [((128, 128, 128), (16, 16, 16)), ((96, 96, 96), (16, 16, 16)), ((40, 48, 40), (10, 12, 10)),
         ((33, 21, 13), (8, 8, 4)), ((130, 50, 37), (8, 8, 8)), ((20, 4, 4), (8, 4, 4)),
         ((10, 70, 6), (4, 8, 4)), ((12, 6, 90), (4, 4, 8)), ((8, 8, 8), (4, 4, 4)),
         ((1000, 5, 8), (8, 4, 4)), ((64, 64), (16, 16)), ((31, 45), (8, 8)), ((300, 200), (16, 16)),
         ((1024, 40), (8, 8)), ((4, 4), (4, 4))]


@pytest.mark.parametrize("n,k", GRIDS)
@pytest.mark.parametrize("nt,disp", [(4, 3.0), (1, 1.0), (2, 2.0)])
def test_sweeps_equal_steps(gpu_lib, n, k, nt, disp):
    prob, I0, I1, vs, dv = _inputs(n, k, nt, disp)
    ctx = B.Ctx(bl_problem(prob), I0, I1)
    got = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(True)
    ref = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(False)
    again = _results(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)
    assert _same(again, ref)


@pytest.mark.parametrize("n,k", [((128, 128, 128), (16, 16, 16)), ((33, 90, 70), (8, 8, 8)),
                                 ((300, 200), (16, 16))])
@pytest.mark.parametrize("disp", [40.0, 200.0])
def test_offsets_past_the_box(gpu_lib, n, k, disp):
    """many voxels per step: some or all tiles' boxes do not fit, the sweep is finished by tickets"""
    prob, I0, I1, vs, dv = _inputs(n, k, 4, disp)
    ctx = B.Ctx(bl_problem(prob), I0, I1)
    got = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(True)
    ref = _results(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)


def test_first_sweeps_of_a_shape_past_the_box(gpu_lib):
    """the first launches of a kernel start their workgroups late: a tile that abandons the sweep at
    once must not show progress to tiles that have not noticed"""
    for i, n in enumerate([(130, 50, 37), (127, 49, 40), (90, 77, 30), (60, 100, 41), (34, 120, 80)]):
        prob, I0, I1, vs, dv = _inputs(n, (8, 8, 8), 3, 60.0, i)
        ctx = B.Ctx(bl_problem(prob), I0, I1)
        got = _results(ctx, prob, vs, dv)
        ctx.bl_kernel_timing_enable(True)
        ref = _results(ctx, prob, vs, dv)
        ctx.close()
        assert _same(got, ref), n


@pytest.mark.parametrize("newton", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
def test_models(gpu_lib, newton, mixed):
    prob, I0, I1, vs, dv = _inputs((40, 48, 40), (10, 12, 10), 5, 3.0)
    p = bl_problem(prob, precision=B.BL_MIXED if mixed else B.BL_FP32, newton=newton)
    ctx = B.Ctx(p, I0, I1)
    got = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(True)
    ref = _results(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)


def test_threads_compete_for_the_device(gpu_lib):
    """several contexts at once, each on its own stream: they run as steps, or as sweeps that others
    disturb and that are then finished by tickets; every result is the sequential one"""
    cases = [_inputs(n, k, 6, 3.0, seed) for seed, (n, k) in enumerate(
        [((128, 128, 128), (16, 16, 16)), ((96, 96, 96), (16, 16, 16)), ((64, 60, 62), (8, 8, 8)),
         ((130, 50, 37), (8, 8, 8))])]
    ctxs = [B.Ctx(bl_problem(c[0]), c[1], c[2]) for c in cases]
    ref = [_results(x, c[0], c[3], c[4]) for x, c in zip(ctxs, cases)]
    bad, start = [], threading.Barrier(len(cases))

    def work(i):
        start.wait()
        for _ in range(10):
            if not _same(_results(ctxs[i], cases[i][0], cases[i][3], cases[i][4]), ref[i]):
                bad.append(i)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    [t.start() for t in ts]
    [t.join() for t in ts]
    [x.close() for x in ctxs]
    assert not bad


def test_graph_replays(gpu_lib):
    """a captured product replayed with eager products and synchronisations between"""
    import torch

    prob, I0, I1, vs, dv = _inputs((64, 60, 62), (8, 8, 8), 5, 3.0)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        tI0, tI1, tv, tdv = (torch.from_numpy(x).cuda() for x in (I0, I1, vs, dv))
        other = torch.roll(tdv, 1, dims=0).contiguous()
        ctx = B.Ctx(bl_problem(prob, device=True, stream=s.cuda_stream), tI0, tI1)
        ctx.bl_lddmm_ctx_set_velocity(tv)
        ref = ctx.bl_lddmm_ctx_hessvec(tdv).clone()
        src, out = tdv.clone(), torch.empty_like(tdv)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            ctx.bl_lddmm_ctx_hessvec(src, out)
        for i in range(4):
            out.zero_()
            graph.replay()
            s.synchronize()
            assert torch.equal(out, ref), i
            eager = ctx.bl_lddmm_ctx_hessvec(other)
            s.synchronize()
            assert torch.isfinite(torch.view_as_real(eager)).all()
        ctx.close()


@pytest.mark.parametrize("n,k", [((128, 128, 128), (16, 16, 16)), ((33, 21, 13), (8, 8, 4)),
                                 ((130, 50, 37), (8, 8, 8)), ((8, 8, 8), (4, 4, 4)), ((96, 40), (8, 8)),
                                 ((300, 200), (16, 16))])
@pytest.mark.parametrize("nt,disp", [(4, 3.0), (1, 1.0), (3, 60.0)])
def test_newton_products(gpu_lib, n, k, nt, disp):
    """the Newton product's sweeps (at 60 voxels finished by tickets) against its steps"""
    prob, I0, I1, vs, dv = _inputs(n, k, nt, disp)
    ctx = B.Ctx(bl_problem(prob, newton=True), I0, I1)
    got = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(True)
    ref = _results(ctx, prob, vs, dv)
    ctx.bl_kernel_timing_enable(False)
    again = _results(ctx, prob, vs, dv)
    ctx.close()
    assert _same(got, ref)
    assert _same(again, ref)
