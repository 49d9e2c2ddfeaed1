"""Degree 2 and 3 kernels at the edges of their 64-cell groups: the last group
full, one square over and one short; and a caller numbering that scatters
neighbours, so that a group's neighbour list takes several rounds to load and
most faces lead to other groups.  Against the FP64 oracle, 1e-12 normwise per
variable in FP64 (round-off of the same arithmetic in another order), 1e-5 in
mixed precision (FP32 reconstruction and fluxes).  Large mixed meshes, whose fused
stage runs in blocks of four groups, at last blocks of one, three and four
groups and with a numbering too scattered for them, against the separate
kernels, which the other tests hold to the oracle: 1e-6, some FP32 roundings of
the fluxes over two steps."""
import numpy as np
import pytest

import oracle as O
from paper_2312_17042_amd import cteno as T
from paper_2312_17042_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = T.Context(0)
    yield c
    c.close()


def relerr(g, o):
    return max(np.abs(g[v] - o[v]).max() / np.abs(o[v]).max() for v in range(o.shape[0]))


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("problem", ["vortex", "advection"])
@pytest.mark.parametrize("nx,ny,scatter", [(8, 16, False), (9, 7, False), (13, 5, False), (24, 23, True)])
def test_group_edges(ctx, degree, problem, nx, ny, scatter):
    if problem == "vortex":
        mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
        u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
        kw = dict(physics=O.EULER, scheme=O.CTENOZ, degree=degree, lambda1_prime=1e4)
    else:
        mesh = W.split_jitter_mesh(nx, ny, (0.0, 1.0, 0.0, 1.0), seed=31)
        u0 = W.cell_average(mesh, W.advection_sine(0.0), n=4)
        kw = dict(physics=O.ADVECTION, scheme=O.CTENO, degree=degree, lambda1_prime=1e15, ax=1.0, ay=1.0)
    if scatter:
        order = np.random.default_rng(7).permutation(mesh.n_cells)
        mesh.tri = np.ascontiguousarray(mesh.tri[order])
        u0 = np.ascontiguousarray(u0[:, order])
    o = O.Oracle.from_mesh(mesh, **kw)
    steps = 5
    uo, so, _ = o.solve(u0, 1e30, cfl=0.3, max_steps=steps)
    ro = o.residual(u0)
    m = T.Mesh.from_workload(ctx, mesh, precision=T.BOTH, reorder=0, **kw)
    for prec, tol in ((T.FP64, 1e-12), (T.MIXED, 1e-5)):
        s = T.Solution(m, u0)
        if prec == T.FP64:
            assert relerr(s.residual(prec).cpu().numpy(), ro) < 1e-12
        for graph in (True, False):
            s.set(u0, 0.0)
            assert s.solve(max_steps=steps, cfl=0.3, precision=prec, use_graph=graph) == so == steps
            assert relerr(s.download()[0], uo) < tol
        s.close()
    m.close()


@pytest.mark.parametrize("nx,ny,scatter", [(781, 769, False), (800, 751, False), (800, 752, False), (781, 769, True)])
def test_wide_blocks(ctx, nx, ny, scatter):
    mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
    u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=2)
    if scatter:
        order = np.random.default_rng(7).permutation(mesh.n_cells)
        mesh.tri = np.ascontiguousarray(mesh.tri[order])
        u0 = np.ascontiguousarray(u0[:, order])
    m = T.Mesh.from_workload(ctx, mesh, precision=T.MIXED, reorder=0 if scatter else 1, physics=O.EULER,
                             scheme=O.CTENOZ, degree=3, lambda1_prime=1e4)
    s = T.Solution(m, u0)
    got = []
    try:
        for fused in (False, True):
            ctx.set_fused_stage(fused)
            s.set(u0, 0.0)
            assert s.solve(max_steps=2, cfl=0.3, precision=T.MIXED) == 2
            got.append(s.download()[0])
    finally:
        ctx.set_fused_stage(True)
        s.close()
        m.close()
    assert relerr(got[1], got[0]) < 1e-6
