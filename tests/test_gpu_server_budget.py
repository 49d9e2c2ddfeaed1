"""What a served request allocates on the device, from its upload to its
result, stays within what the server counts against its budget: both degrees,
Morton order and a caller's scattered numbering (longest neighbour lists),
small and ragged meshes."""
import numpy as np
import pytest

from paper_2312_17042_amd import cteno as T
from paper_2312_17042_amd import workloads as W

pytestmark = pytest.mark.gpu


class CountingAllocator(T.TorchAllocator):
    def __init__(self, device, stream):
        super().__init__(device, stream)
        self.live = self.peak = 0
        sizes, alloc, free = {}, self.alloc_fn, self.free_fn

        def counted(nbytes, user):
            p = alloc(nbytes, user)
            if p:
                sizes[p] = nbytes
                self.live += nbytes
                self.peak = max(self.peak, self.live)
            return p

        def released(ptr, user):
            self.live -= sizes.pop(ptr)
            free(ptr, user)

        self.keep = (alloc, free)
        self.alloc_fn, self.free_fn = T._ALLOC_FN(counted), T._FREE_FN(released)


@pytest.mark.parametrize("degree", [2, 3])
@pytest.mark.parametrize("nx,ny,scatter", [(12, 12, False), (12, 12, True), (61, 53, True), (128, 64, False),
                                           (128, 64, True)])
def test_upload_stays_within_its_reservation(monkeypatch, degree, nx, ny, scatter):
    mesh = W.split_jitter_mesh(nx, ny, (0.0, 10.0, 0.0, 10.0), seed=31)
    u0 = W.cell_average(mesh, W.isentropic_vortex(0.0, 3.0, (5.0, 5.0), (10.0, 10.0)), n=2)
    if scatter:
        order = np.random.default_rng(7).permutation(mesh.n_cells)
        mesh.tri = np.ascontiguousarray(mesh.tri[order])
        u0 = np.ascontiguousarray(u0[:, order])
    monkeypatch.setattr(T, "TorchAllocator", CountingAllocator)
    ctx = T.Context(0)
    srv = T.Server(ctx, T.make_scheme(degree=degree, precision=T.MIXED, reorder=0 if scatter else 1),
                   budget_bytes=1 << 28, max_slots=2)
    base = ctx.allocator.live
    ctx.allocator.peak = base
    t = srv.submit(mesh, u0, n_steps=3)
    srv.drain()
    state, u, steps, _ = srv.poll(t, take=True)
    assert state == T.REQ_DONE and steps == 3 and np.isfinite(u).all()
    assert 0 < ctx.allocator.peak - base <= srv.stats()["peak_bytes"]
    srv.close()
    ctx.close()
