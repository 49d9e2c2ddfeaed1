"""The C entry points' host code on a stand-in for the HIP runtime
(host/hip_standin.cpp: device memory in host memory, kernels that do nothing):
what is allocated, captured, launched and copied, and in which order.  Each
test runs in a process of its own, which loads the stand-in before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PRELUDE = """
import ctypes as C, os, sys
sys.path.insert(0, {root!r})
standin = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
standin.standin_count.restype = C.c_int64
count = lambda what: standin.standin_count(what.encode())
standin.standin_caller()
import numpy as np
from paper_2312_17042_amd import cteno as T, workloads as W
L = T.lib()

def ok(rc, want=T.OK):
    assert rc == want, (rc, L.cteno_last_error())

def context(stream=None):
    h = C.c_void_p()
    ok(L.cteno_ctx_create(0, C.c_void_p(stream), None, None, None, C.byref(h)))
    return h

def upload(ctx, m, scheme):
    h, d = C.c_void_p(), T.mesh_desc(m.xy, m.tri, m.box, m.bc)
    ok(L.cteno_mesh_upload(ctx, C.byref(d), C.byref(scheme), C.byref(h)))
    return h

def solution(ctx, mesh, u):
    h = C.c_void_p()
    ok(L.cteno_sol_create(ctx, mesh, T._np_ptr(u), 0.0, C.byref(h)))
    return h
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """Runs a script on the stand-in."""
    so = str(tmp_path_factory.mktemp("standin") / "libhip_standin.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-isystem",
                    os.path.join(ROCM, "include"), os.path.join(HERE, "host", "hip_standin.cpp"), "-o", so], check=True)

    def run(script, *args, timeout=120):
        code = PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(script) + "\nprint('done', flush=True)\nos._exit(0)\n"
        r = subprocess.run([sys.executable, "-c", code, *map(str, args)], capture_output=True, text=True,
                           timeout=timeout)
        assert r.returncode == 0 and r.stdout.endswith("done\n"), r.stdout + r.stderr

    return run


@pytest.mark.parametrize("degree,requests", [(2, 176), (3, 120)])
def test_server_runs_every_solve_that_the_budget_admits(host, degree, requests):
    """Solves of whole 256-cell blocks, as many as the device budget holds, all
    run at once: the batched grid covers them."""
    host("""
    degree, n = map(int, sys.argv[1:])
    m = W.split_jitter_mesh(128, 64, (0.0, 10.0, 0.0, 5.0), seed=5)
    u = np.ascontiguousarray(np.tile([[1.0], [0.5], [0.0], [3.0]], (1, m.n_cells)))
    scheme = T.make_scheme(degree=degree, precision=T.MIXED)
    ctx = context()
    import time
    def server(budget, slots):
        h = C.c_void_p()
        ok(L.cteno_server_create(ctx, C.byref(scheme), budget, slots, C.byref(h)))
        return h
    def submit(sv):
        d, t = T.mesh_desc(m.xy, m.tri, m.box, m.bc), C.c_uint64()
        ok(L.cteno_server_submit(sv, C.byref(d), T._np_ptr(u), 1 << 30, 0.3, C.byref(t)))
        return t.value
    def stats(sv):
        s = T.ServerStats()
        ok(L.cteno_server_get_stats(sv, C.byref(s)))
        return s
    def wait(sv, tickets, what):
        info = T.RequestInfo()
        for _ in range(6000):
            s = stats(sv)
            for t in tickets:
                ok(L.cteno_server_request_info(sv, t, C.byref(info)))
                if info.state == T.REQ_FAILED:
                    ok(L.cteno_server_poll(sv, t, None, None, None, None))
            if what(s):
                return s
            time.sleep(0.01)
        raise SystemExit(f"{s.active} of {len(tickets)} solves run")
    one = server(1 << 30, 1)
    s = wait(one, [submit(one)], lambda s: s.active == 1)
    resident, reserve = s.bytes_in_use, s.peak_bytes
    assert resident < reserve
    many = server((n - 1) * resident + reserve, n)
    tickets = [submit(many) for _ in range(n)]
    s = wait(many, tickets, lambda s: s.active == n)
    # ticks with all of them do not stop the server
    wait(many, tickets, lambda t: t.active == n and t.ticks > s.ticks + 8)
    """, degree, requests)


@pytest.mark.parametrize("steps,captures", [(1, 1), (3, 1), (4, 1), (5, 2), (16, 1), (18, 2), (40, 1)])
def test_march_captures_before_it_launches(host, steps, captures):
    """The graphs that a march needs are captured before its first step: when one
    cannot be made the call fails with nothing launched, and the next call marches."""
    host("""
    steps, captures = map(int, sys.argv[1:])
    m = W.split_jitter_mesh(16, 16, (0.0, 10.0, 0.0, 10.0), seed=5)
    u = np.ascontiguousarray(np.tile([[1.0], [0.5], [0.0], [3.0]], (1, m.n_cells)))
    ctx = context()
    mesh = upload(ctx, m, T.make_scheme(degree=3, precision=T.BOTH))
    for prec in (T.FP64, T.MIXED):
        for failing in range(1, captures + 1):
            sol, n = solution(ctx, mesh, u), C.c_int64(-7)
            march = lambda: L.cteno_solve(ctx, mesh, sol, prec, 1e30, steps, 0.3, 1, C.byref(n))
            launched, made = count("graph_launch"), count("instantiate")
            kernels, events = count("kernel"), count("event_alive")
            standin.standin_fail_instantiate(failing)
            ok(march(), T.ERR_DEVICE)
            assert count("graph_launch") == launched and count("kernel") == kernels and n.value == -7
            assert count("graph_alive") == 0 and count("event_alive") == events
            ok(march())
            assert count("graph_launch") - launched == steps // 4 + steps % 4
            # (the one that failed is made again, those before it are kept)
            assert count("instantiate") - made == captures + 1 and count("graph_alive") == 0
            L.cteno_sol_destroy(sol)
    """, steps, captures)


@pytest.mark.parametrize("stream,staged", [(None, True), (1, True), (2, False)])
def test_staged_transfers_keep_the_caller_s_stream(host, stream, staged):
    """Large states are staged by several threads, except on the per-thread
    stream (2), whose handle means another stream in each of them: there every
    copy comes from the calling thread.  (1: the legacy null stream.)"""
    host("""
    stream, staged = eval(sys.argv[1]), eval(sys.argv[2])
    m = W.split_jitter_mesh(820, 660, (0.0, 10.0, 0.0, 10.0), seed=5)    # 34.6 MB of Euler states
    u = np.random.default_rng(1).random((4, m.n_cells)) + 1.0
    ctx = context(stream)
    mesh = upload(ctx, m, T.make_scheme(degree=2, precision=T.MIXED))
    sol = solution(ctx, mesh, u)
    got, t = np.empty_like(u), C.c_double()
    before = count("foreign_copy")
    for k in range(4):
        ok(L.cteno_sol_set(sol, T._np_ptr(u), 0.25))
        ok(L.cteno_sol_download(sol, T._np_ptr(got), C.byref(t)))
        assert t.value == 0.25
    assert (count("foreign_copy") > before) == staged
    """, stream, staged, timeout=240)


@pytest.mark.parametrize("degree", [2, 3, 4])
@pytest.mark.parametrize("precision", ["FP64", "MIXED"])
def test_stages_after_a_reconstruction_allocate_nothing(host, degree, precision):
    """A program that has reconstructed once may capture its RK stages."""
    host("""
    degree, prec = int(sys.argv[1]), getattr(T, sys.argv[2])
    m = W.split_jitter_mesh(20, 16, (0.0, 10.0, 0.0, 10.0), seed=5)
    u = np.ascontiguousarray(np.tile([[1.0], [0.5], [0.0], [3.0]], (1, m.n_cells)))
    ctx = context()
    for fused in (1, 0):
        ok(L.cteno_ctx_set_fused_stage(ctx, fused))
        mesh = upload(ctx, m, T.make_scheme(degree=degree, precision=T.BOTH))
        sol = solution(ctx, mesh, u)
        values = np.empty((m.n_cells, 3, 4, 4))
        ok(L.cteno_reconstruct(ctx, mesh, sol, prec, T._np_ptr(values), None, None))
        ok(L.cteno_ctx_set_fused_stage(ctx, 1))
        before = count("malloc")
        for stage in range(3):
            ok(L.cteno_rk_stage(ctx, mesh, sol, prec, stage, 1e-3))
        assert count("malloc") == before
    """, degree, precision)


def test_staging_is_made_when_transfers_pay_for_it(host):
    """A program that takes one smaller state back makes no pinned buffers; they
    come with the transfer that completes 32 MB, once, and bounded."""
    host("""
    m = W.split_jitter_mesh(520, 350, (0.0, 10.0, 0.0, 10.0), seed=5)     # 11.6 MB of Euler states
    u = np.random.default_rng(1).random((4, m.n_cells)) + 1.0
    got, t = np.empty_like(u), C.c_double()
    ctx = context()
    mesh = upload(ctx, m, T.make_scheme(degree=2, precision=T.MIXED))
    sol = solution(ctx, mesh, u)
    before, made = count("pinned"), []
    for k in range(5):
        ok(L.cteno_sol_set(sol, T._np_ptr(u), 0.0))
        ok(L.cteno_sol_download(sol, T._np_ptr(got), C.byref(t)))
        made.append(count("pinned") - before)
    assert made == [0, 0, 1, 1, 1], made
    """)


def test_long_neighbour_lists_are_accepted(host):
    """Lists of more than 2^31 cells in all (some 120M cells of degree 3 in a
    numbering that scatters every stencil), which a slot table had no limit for."""
    host("""
    m = W.split_jitter_mesh(15, 10, (0.0, 10.0, 0.0, 10.0), seed=5)      # five groups
    ctx = context()
    for each, want in (((1 << 29) - 1, T.OK), ((1 << 30) - 1, T.ERR_INVALID)):
        standin.standin_fill(C.c_size_t(5 * 4), C.c_int32(each))         # the groups' lengths
        d, h, scheme = T.mesh_desc(m.xy, m.tri, m.box, m.bc), C.c_void_p(), T.make_scheme(degree=3, reorder=0)
        ok(L.cteno_mesh_upload(ctx, C.byref(d), C.byref(scheme), C.byref(h)), want)
        if want == T.OK:
            L.cteno_mesh_destroy(h)
    """)
