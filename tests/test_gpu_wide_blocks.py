"""The fused stage in blocks of 256 cells, on small meshes: last blocks of one to
four groups, whole and cut off; walls, inflow and transmissive sides; one
variable; every scheme; the positivity fallback.  Against the FP64 oracle's march
(1e-5 normwise per variable, FP32 reconstruction and fluxes; where FP32 selects or
falls back otherwise than FP64 within a step, as at the strong shock with CTENOZ,
the separate kernels leave the oracle as well and no such bound holds) and against
blocks of 64 cells, whose results are the same to the bit: a cell sums its faces
in one order and a face's flux is rounded in one way whatever the blocks are."""
import numpy as np
import pytest

import oracle as O
from paper_2312_17042_amd import cteno as T
from paper_2312_17042_amd import workloads as W

pytestmark = pytest.mark.gpu
STEPS = 5


@pytest.fixture(scope="module")
def ctx():
    c = T.Context(0)
    yield c
    c.close()


def relerr(g, o):
    return max(np.abs(g[v] - o[v]).max() / np.abs(o[v]).max() for v in range(o.shape[0]))


def march(ctx, mesh, u0, block, kw, reorder=1):
    ctx.set_stage_block(block)
    try:
        m = T.Mesh.from_workload(ctx, mesh, precision=T.MIXED, reorder=reorder, **kw)
    finally:
        ctx.set_stage_block(0)
    s = T.Solution(m, u0)
    ends = []
    for graph in (True, False):
        s.set(u0, 0.0)
        assert s.solve(max_steps=STEPS, cfl=0.3, precision=T.MIXED, use_graph=graph) == STEPS
        ends.append(s.download())
    assert np.array_equal(ends[0][0], ends[1][0]) and ends[0][1] == ends[1][1]
    s.set(u0, 0.0)
    for stage in range(3):
        s.rk_stage(stage, 1e-4, T.MIXED)
    out = m.stage_block(), ends[0][0], ends[0][1], s.download()[0], s.fallbacks()
    s.close()
    m.close()
    return out


def check(ctx, mesh, u0, kw, reorder=1):
    block, u, t, stages, fallbacks = march(ctx, mesh, u0, 256, kw, reorder)
    assert block == 256
    uo, so, to = O.Oracle.from_mesh(mesh, **kw).solve(u0, 1e30, cfl=0.3, max_steps=STEPS)
    ctx.set_fused_stage(False)
    try:
        separate = march(ctx, mesh, u0, 256, kw, reorder)
    finally:
        ctx.set_fused_stage(True)
    assert so == STEPS and fallbacks == separate[4]
    if relerr(separate[1], uo) < 1e-5:
        assert relerr(u, uo) < 1e-5 and abs(t - to) < 1e-5 * to
    else:
        assert kw["positivity"] and kw["scheme"] == O.CTENOZ
    small = march(ctx, mesh, u0, 64, kw, reorder)
    assert small[0] == 64 and small[2] == t and small[4] == fallbacks
    assert np.array_equal(small[1], u) and np.array_equal(small[3], stages)


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("problem", ["vortex", "advection"])
@pytest.mark.parametrize("nx,ny", [(8, 8), (8, 16), (12, 8), (9, 7), (15, 11), (16, 16), (19, 17), (23, 21)])
def test_last_blocks(ctx, degree, problem, nx, ny):
    if problem == "vortex":
        mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
        u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
        kw = dict(physics=O.EULER, scheme=O.CTENOZ, degree=degree, lambda1_prime=1e4)
    else:
        mesh = W.split_jitter_mesh(nx, ny, (0.0, 1.0, 0.0, 1.0), seed=31)
        u0 = W.cell_average(mesh, W.advection_sine(0.0), n=4)
        kw = dict(physics=O.ADVECTION, scheme=O.CTENO, degree=degree, lambda1_prime=1e15, ax=1.0, ay=-0.5)
    check(ctx, mesh, u0, kw)


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("case", ["sod", "shock_density", "dmr"])
@pytest.mark.parametrize("scheme", [O.CTENO, O.CTENOZ, O.CWENO, O.TENO])
def test_boundaries_schemes_and_fallback(ctx, degree, case, scheme):
    if case == "sod":
        mesh, u0 = W.sod_case(45, 11, seed=3, prescribed=True)
    elif case == "shock_density":
        mesh, u0 = W.shock_density_case(40, 9, seed=12, quad=3)
    else:
        mesh, u0 = W.dmr_case(44, 11, seed=13, quad=3)
    check(ctx, mesh, u0, dict(physics=O.EULER, scheme=scheme, degree=degree, positivity=1,
                              lambda1_prime=1e4 if scheme == O.CTENOZ else 1e15))


@pytest.mark.parametrize("gamma_form,scheme", [(O.GAMMA_LAMBDA, O.CTENO), (O.GAMMA_SCALED, O.CTENOZ)])
def test_gamma_forms(ctx, gamma_form, scheme):
    mesh = W.split_jitter_mesh(15, 11, (0.0, 10.0, 0.0, 10.0), seed=31)
    u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
    check(ctx, mesh, u0, dict(physics=O.EULER, scheme=scheme, degree=3, lambda1_prime=1e4, gamma_form=gamma_form))


def test_row_by_row_numbering(ctx):
    mesh = W.split_jitter_mesh(24, 23, (0.0, 10.0, 0.0, 10.0), seed=31)
    u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
    check(ctx, mesh, u0, dict(physics=O.EULER, scheme=O.CTENOZ, degree=3, lambda1_prime=1e4), reorder=0)


@pytest.mark.parametrize("nx,ny,scatter,mixed,fp64", [(781, 769, False, 256, 64), (774, 774, False, 64, 64),
                                                      (781, 769, True, 0, 0)])
def test_block_by_size(ctx, nx, ny, scatter, mixed, fp64):
    """1,201,178 cells and 1,198,152, on both sides of the line; a scattered
    numbering runs the separate kernels."""
    mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
    if scatter:
        mesh.tri = np.ascontiguousarray(mesh.tri[np.random.default_rng(7).permutation(mesh.n_cells)])
    m = T.Mesh.from_workload(ctx, mesh, precision=T.BOTH, reorder=0 if scatter else 1, degree=2)
    assert m.stage_block(T.MIXED) == mixed and m.stage_block(T.FP64) == fp64
    m.close()
    if not scatter:
        m = T.Mesh.from_workload(ctx, mesh, precision=T.MIXED, variables=T.CHARACTERISTIC, degree=2)
        assert m.stage_block(T.MIXED) == 64
        m.close()


def test_other_sizes_are_refused(ctx):
    for cells in (1, 63, 128, 512, -1):
        with pytest.raises(T.CtenoError) as e:
            ctx.set_stage_block(cells)
        assert e.value.status == T.ERR_INVALID
