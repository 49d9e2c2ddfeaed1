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
import math

import numpy as np
import pytest
import torch

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


def gauss_basis(r):
    """The degree-r basis (monomials less their means over the reference
    triangle) at the faces' Gauss points, [3][N_q][K]."""
    ex = [(d - k, k) for d in range(1, r + 1) for k in range(d + 1)]
    mean = [2.0 * math.factorial(a) * math.factorial(b) / math.factorial(a + b + 2) for a, b in ex]
    g = 0.5 * (np.polynomial.legendre.leggauss((r + 2) // 2)[0] + 1.0)
    v = np.array([[0.0, 0.0], [1.0, 0.0], [0.0, 1.0]])
    x = v[:, None] + g[:, None] * (np.roll(v, -1, 0) - v)[:, None]
    return np.stack([x[..., 0] ** a * x[..., 1] ** b - m for (a, b), m in zip(ex, mean)], -1)


@pytest.mark.parametrize("degree", [4, 5, 6])
@pytest.mark.parametrize("nx,ny,scatter", [(16, 12, False), (12, 11, False), (15, 9, False), (24, 23, True)])
def test_high_order_products(ctx, degree, nx, ny, scatter):
    """Degree 4 to 6 with the last 16 cells of a wave full and cut off: each
    polynomial in turn, selected by force, against its products with the mesh's
    own pseudo-inverses, within the rounding bound of sums of that length."""
    mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
    u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
    if scatter:
        order = np.random.default_rng(7).permutation(mesh.n_cells)
        mesh.tri = np.ascontiguousarray(mesh.tri[order])
        u0 = np.ascontiguousarray(u0[:, order])
    m = T.Mesh.from_workload(ctx, mesh, precision=T.BOTH, physics=O.EULER, scheme=O.TENO, degree=degree,
                             lambda1_prime=1e4)
    s = T.Solution(m, u0)
    cen, dr, dn = m.stencils()
    B = gauss_basis(degree)
    N = mesh.n_cells
    for prec, eps in ((T.FP64, 2.0**-53), (T.MIXED, 2.0**-24)):
        Pc, Pd = m.pinv(np.arange(N), prec)
        for bit in range(4):
            P, st = (Pc, cen) if bit == 0 else (Pd[:, bit - 1], dr[:, bit - 1])
            d = np.where(st[:, None] >= 0, u0.T[np.maximum(st, 0)].transpose(0, 2, 1) - u0.T[:, :, None], 0.0)
            b = B[..., :P.shape[1]]
            want = u0.T[:, None, None] + np.einsum("fqk,nkj,nvj->nfqv", b, P, d)
            mag = np.einsum("fqk,nkj,nvj->nfqv", np.abs(b), np.abs(P), np.abs(d))
            on = np.ones(N, bool) if bit == 0 else dn[:, bit - 1] > 0
            assert on.any()
            forced = np.full((N, 4), 1 << bit, np.uint8)
            got = s.reconstruct(prec, forced=forced)[0].cpu().numpy()
            bound = 2 * (P.shape[1] + P.shape[2] + 6) * eps * mag + 2 * eps * np.abs(want)
            assert (np.abs(got - want) <= bound)[on].all(), (prec, bit)
    s.close()
    m.close()


@pytest.mark.parametrize("nx,ny", [(8, 16), (13, 5)])
@pytest.mark.parametrize("problem", ["vortex", "advection"])
@pytest.mark.parametrize("prec", [T.FP64, T.MIXED])
def test_face_values_at_any_alignment(ctx, problem, nx, ny, prec):
    """A caller's face values that start at any element of an array give the
    fluxes of the same values in an array of their own."""
    mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
    if problem == "vortex":
        u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=4)
        kw = dict(physics=O.EULER, scheme=O.CTENOZ, degree=3, lambda1_prime=1e4)
    else:
        u0 = W.cell_average(mesh, W.advection_sine(0.0), n=4)
        kw = dict(physics=O.ADVECTION, scheme=O.CTENO, degree=3, lambda1_prime=1e15, ax=1.0, ay=1.0)
    m = T.Mesh.from_workload(ctx, mesh, precision=prec, **kw)
    s = T.Solution(m, u0)
    values, selected = s.reconstruct(prec)
    assert torch.equal(s.reconstruct(prec, forced=selected.cpu().numpy())[0], values)
    want = T.flux(m, values, prec)
    for off in (1, 2, 3):
        buf = torch.zeros(values.numel() + off, dtype=values.dtype, device=values.device)
        view = buf[off:].view(values.shape)
        view.copy_(values)
        assert torch.equal(T.flux(m, view, prec), want)
        out = torch.zeros(want.numel() + off, dtype=want.dtype, device=want.device)
        assert torch.equal(T.flux(m, values, prec, out=out[off:].view(want.shape)), want)
    s.close()
    m.close()


@pytest.mark.parametrize("nx", [361, 363, 724, 725])
@pytest.mark.parametrize("pinned", [False, True])
def test_large_state_transfers(ctx, nx, pinned):
    """States on both sides of the sizes from which transfers are staged, with
    ragged last chunks, come back bit for bit."""
    mesh = W.split_jitter_mesh(nx, nx, (0.0, 1.0, 0.0, 1.0), seed=31)
    rng = np.random.default_rng(3)
    u = [rng.standard_normal((4, mesh.n_cells)) for _ in range(2)]
    m = T.Mesh.from_workload(ctx, mesh, precision=T.FP64, physics=O.EULER, scheme=O.CTENO, degree=2,
                             lambda1_prime=1e15)
    s = T.Solution(m, u[0])
    assert np.array_equal(s.download()[0], u[0])
    s.set(torch.from_numpy(u[1]).pin_memory().numpy() if pinned else u[1], 0.5)
    got, t = s.download()
    assert t == 0.5 and np.array_equal(got, u[1])
    s.close()
    m.close()
