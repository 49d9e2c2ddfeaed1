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
