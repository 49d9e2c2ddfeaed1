"""Which kernels a stage of degree 2 and 3 runs: numberings that scatter
neighbours, where more than half of the faces lead to other blocks, take the
separate kernels (the same results to the bit as with the fused stage switched
off); both kinds against the FP64 oracle, 1e-12 normwise in FP64 and 1e-5 in mixed
precision."""
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


def shuffled(mesh, u0, reach):
    """The cells within `reach` places of where they were, or anywhere."""
    rng, n = np.random.default_rng(7), mesh.n_cells
    order = rng.permutation(n) if reach is None else np.argsort(np.arange(n) + rng.uniform(0, reach, n), kind="stable")
    mesh.tri = np.ascontiguousarray(mesh.tri[order])
    return np.ascontiguousarray(u0[:, order])


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("variables", [T.CONSERVED, T.CHARACTERISTIC])
@pytest.mark.parametrize("reach", [200, None])
def test_scattered_numberings_take_the_separate_kernels(ctx, degree, variables, reach):
    mesh, u0 = W.shock_density_case(60, 12, seed=12, quad=3)
    u0 = shuffled(mesh, u0, reach)
    kw = dict(physics=O.EULER, scheme=O.CTENO, degree=degree, lambda1_prime=1e15, variables=variables, positivity=1)
    uo, so, _ = O.Oracle.from_mesh(mesh, **kw).solve(u0, 1e30, cfl=0.3, max_steps=5)
    m = T.Mesh.from_workload(ctx, mesh, precision=T.BOTH, reorder=0, **kw)
    s = T.Solution(m, u0)
    try:
        for prec, tol in ((T.FP64, 1e-12), (T.MIXED, 1e-5)):
            got = []
            for fused in (True, False):
                ctx.set_fused_stage(fused)
                s.set(u0, 0.0)
                assert s.solve(max_steps=5, cfl=0.3, precision=prec) == so == 5
                got.append(s.download()[0])
                assert relerr(got[-1], uo) < tol
            # (FP64 with characteristic variables: from 2.75 such faces a cell on)
            if prec == T.MIXED or variables == T.CONSERVED or reach is None:
                assert np.array_equal(got[0], got[1])
    finally:
        ctx.set_fused_stage(True)
        s.close()
        m.close()


@pytest.mark.parametrize("problem,degree,n", [("advection", 2, 380), ("advection", 3, 274), ("vortex", 2, 350),
                                              ("vortex", 3, 264)])
def test_streams_that_the_cache_keeps(ctx, problem, degree, n):
    """Meshes whose pseudo-inverse streams are loaded through the caches in both
    precisions: face values of sampled cells against the oracle (1e-12; mixed with
    the selections of FP64 5e-6), and the fused stage against the separate kernels
    over two steps (1e-12; mixed 1e-6, some FP32 roundings of the fluxes)."""
    if problem == "vortex":
        mesh = W.split_jitter_mesh(n, n, (0.0, 10.0, 0.0, 10.0), seed=31)
        u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=2)
        kw = dict(physics=O.EULER, scheme=O.CTENOZ, degree=degree, lambda1_prime=1e4)
    else:
        mesh = W.split_jitter_mesh(n, n, (0.0, 1.0, 0.0, 1.0), seed=31)
        u0 = W.cell_average(mesh, W.advection_sine(0.0), n=2)
        kw = dict(physics=O.ADVECTION, scheme=O.CTENO, degree=degree, lambda1_prime=1e15, ax=1.0, ay=1.0)
    cells = np.unique(np.r_[np.arange(70), np.random.default_rng(5).integers(0, mesh.n_cells, 400),
                            np.arange(mesh.n_cells - 70, mesh.n_cells)])
    values, selected = O.Oracle.from_mesh(mesh, **kw).reconstruct_cells(u0, cells)
    m = T.Mesh.from_workload(ctx, mesh, precision=T.BOTH, **kw)
    s = T.Solution(m, u0)
    try:
        fv, own = s.reconstruct(T.FP64)
        assert np.array_equal(own.cpu().numpy()[cells], selected)
        for got, tol in ((fv, 1e-12), (s.reconstruct(T.MIXED, forced=own.cpu().numpy())[0], 5e-6)):
            got = got.cpu().numpy()[cells].reshape(-1, m.nv)
            assert relerr(got.T, values.reshape(-1, m.nv).T) < tol
        for prec, tol in ((T.FP64, 1e-12), (T.MIXED, 1e-6)):
            ends = []
            for fused in (True, False):
                ctx.set_fused_stage(fused)
                s.set(u0, 0.0)
                assert s.solve(max_steps=2, cfl=0.3, precision=prec) == 2
                ends.append(s.download()[0])
            assert relerr(ends[0], ends[1]) < tol
    finally:
        ctx.set_fused_stage(True)
        s.close()
        m.close()
