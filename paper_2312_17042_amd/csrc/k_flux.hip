// Flux / residual / RK stage kernels, step control, the batched serving
// kernels, layout conversions and utilities; the reconstruction dispatch.
#include "recon_quad.h"

#include <mutex>

namespace cteno {

hipError_t launch_reconstruct(const DeviceMesh &m, bool fp32, const double *U, void *FV, uint8_t *delta, int dmode,
                              const int *done, hipStream_t st, unsigned long long *fb_count, bool stage) {
    if (m.r >= 4)
        return fp32 ? reconstruct_hi<float>(m, U, FV, delta, dmode, done, st, fb_count)
                    : reconstruct_hi<double>(m, U, FV, delta, dmode, done, st, fb_count);
    return fp32 ? reconstruct_lo<float>(m, U, FV, delta, dmode, done, st, fb_count, stage)
                : reconstruct_lo<double>(m, U, FV, delta, dmode, done, st, fb_count, stage);
}

// Fluxes, residual (MODE 1) or RK stage (MODE 2) of cell i from all cells' face
// values, a quad of lanes per cell: a lane per face, then per variable.  Returns
// the CFL bound of the new state when requested, else +inf.  All lanes of a block
// call it (live: the cell exists).  A lane per cell took its faces one after the
// other, with 64 rows under each load: 9.5k cells of three Gauss points in FP64
// 12.6 us, now 5.4; 215k cells 45.7, now 39.7 (165 MB).  At 8M cells in mixed
// precision 492, now 405 us; in FP64 the fourth lane's repeated face shows in an RK
// stage (822, now 904; residual 765, 758; face fluxes 1183, 755).  What is left at
// large sizes are the neighbours' face values, read from memory in rows of their own.
template <typename real, int NV, int PHYS, int MODE, int NQ>
__device__ __forceinline__ double flux_quad(const FluxArgs<real> a, const FluxPtrs<real> ptr, int64_t i, bool live) {
    const int q = threadIdx.x & 3, f = q < 2 ? q : 2, v = NV == 4 ? q : 0;
    double u0 = 0.0, us = 0.0;
    if (MODE == 2) {
        us = ptr.Us[i * NV + v];
        if (a.stage) u0 = ptr.Un[i * NV + v];
    }
    const double ar = MODE == 0 ? 1.0 : ptr.area[i];
    real nx, ny, len, own[NQ][NV], oth[NQ][NV];
    uint32_t code;
    face_record<real>(ptr.fr, i, f, nx, ny, len, code);
    load_row<real, NQ * NV>(ptr.FV + (i * 3 + f) * NQ * NV, &own[0][0]);
    bool owner = true, wallf = false, bad = false;
    if (code & kNbBoundary) {
        wallf = boundary_state<real, NV, PHYS, MODE, NQ>(a, ptr.dt_ptr, code, own, oth);
    } else {
        owner = (code & kNbOwner) != 0;
        const int64_t j = code & kNbIndexMask;
        load_row<real, NQ * NV>(ptr.FV + (j * 3 + ((code >> 28) & 3)) * NQ * NV, &oth[0][0]);
    }
    double term[NV];
    face_term<real, NV, PHYS, NQ>(a, own, oth, owner, wallf, nx, ny, len, term, bad);
    if (bad && live && ptr.nonphys) atomicOr(ptr.nonphys, 1);
    if (MODE == 0) {
        if (live && q < 3) {
            real row[NV];
#pragma unroll
            for (int w = 0; w < NV; ++w) row[w] = (real)term[w];
            store_row<real, NV>(ptr.flux_out + (i * 3 + f) * NV, row);
        }
        return INFINITY;
    }
    double acc = 0.0;
    acc += quad_take<0>(term, v);
    acc += quad_take<1>(term, v);
    acc += quad_take<2>(term, v);
    if (MODE == 1) {
        if (live && q < NV) ptr.resid[i * NV + v] = -acc / ar;
        return INFINITY;
    }
    const double dt = ptr.dt_ptr ? *ptr.dt_ptr : a.dt_value;
    const double un = rk_value(a.stage, u0, us, dt * (-acc / ar));
    if (live && q < NV) ptr.Uout[i * NV + v] = un;
    if (!ptr.want_dt) return INFINITY;
    double u4[NV], nrm[3][3];
    quad_state<NV>(un, u4);
    const double n[3] = {(double)nx, (double)ny, (double)len};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        nrm[0][k] = quad_bcast<0>(n[k]);
        nrm[1][k] = quad_bcast<1>(n[k]);
        nrm[2][k] = quad_bcast<2>(n[k]);
    }
    const double dtc = cell_dt_bound<NV, PHYS>(u4, nrm, ar, a.gamma64, (double)a.ax, (double)a.ay);
    return live ? dtc : INFINITY;
}

template <typename real, int NV, int PHYS, int MODE, int NQ>
__global__ __launch_bounds__(256) void k_flux(const FluxArgs<real> a) {
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * 64 + (threadIdx.x >> 2);
    if (a.ctrl && a.ctrl->done) return;        // uniform across the grid
    const FluxPtrs<real> ptr{a.FV, a.fr, a.area, a.Un, a.Us, a.Uout, a.dt_ptr, a.flux_out, a.resid, a.nonphys,
                             a.dt_part != nullptr};
    const double dtc = flux_quad<real, NV, PHYS, MODE, NQ>(a, ptr, i, i < a.N);
    if (MODE == 2 && a.dt_part) {
        const double bm = block_min(dtc);
        if (threadIdx.x == 0) a.dt_part[blockIdx.x] = bm;
    }
}

template <typename real, int NV, int PHYS>
static hipError_t flux_t(const DeviceMesh &m, const FluxLaunch &f, hipStream_t st) {
    FluxArgs<real> a;
    fill_flux_args<real>(m, f, a);
    const unsigned grid = (unsigned)m.groups();
#define FX_LAUNCH(NQ)                                                                                         \
    switch (f.mode) {                                                                                         \
        case 0: hipLaunchKernelGGL((k_flux<real, NV, PHYS, 0, NQ>), dim3(grid), dim3(256), 0, st, a); break; \
        case 1: hipLaunchKernelGGL((k_flux<real, NV, PHYS, 1, NQ>), dim3(grid), dim3(256), 0, st, a); break; \
        default: hipLaunchKernelGGL((k_flux<real, NV, PHYS, 2, NQ>), dim3(grid), dim3(256), 0, st, a); break; \
    }
    switch (m.tab.Nq) {
        case 2: FX_LAUNCH(2); break;
        case 3: FX_LAUNCH(3); break;
        case 4: FX_LAUNCH(4); break;
        default: return hipErrorInvalidValue;
    }
#undef FX_LAUNCH
    return hipGetLastError();
}

hipError_t launch_stage(const DeviceMesh &m, bool fp32, const FluxLaunch &f, const int *done, int part,
                        hipStream_t st, unsigned long long *fb_count) {
    return fp32 ? stage_fused<float>(m, f, done, part, st, fb_count)
                : stage_fused<double>(m, f, done, part, st, fb_count);
}

hipError_t launch_flux(const DeviceMesh &m, bool fp32, const FluxLaunch &f, hipStream_t st) {
    if (m.physics == CTENO_EULER)
        return fp32 ? flux_t<float, 4, CTENO_EULER>(m, f, st) : flux_t<double, 4, CTENO_EULER>(m, f, st);
    return fp32 ? flux_t<float, 1, CTENO_ADVECTION>(m, f, st) : flux_t<double, 1, CTENO_ADVECTION>(m, f, st);
}

// ===========================================================================
// time-step control
// ===========================================================================

template <typename real, int NV, int PHYS>
__global__ __launch_bounds__(256) void k_dt_partials(int64_t N, const double *U, const real *fr, const double *area,
                                                     double gamma, double ax, double ay, double *part) {
    double dtc = INFINITY;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (int64_t)gridDim.x * 256) {
        double u[NV], nrm[3][3];
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = U[i * NV + v];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            real nx, ny, len;
            uint32_t code;
            face_record<real>(fr, i, f, nx, ny, len, code);
            nrm[f][0] = nx; nrm[f][1] = ny; nrm[f][2] = len;
        }
        dtc = fmin(dtc, cell_dt_bound<NV, PHYS>(u, nrm, area[i], gamma, ax, ay));
    }
    const double bm = block_min(dtc);
    if (threadIdx.x == 0) part[blockIdx.x] = bm;
}

hipError_t launch_dt_partials(const DeviceMesh &m, bool fp32, const double *U, double *part, int64_t n_part,
                              hipStream_t st) {
    const unsigned grid = (unsigned)n_part;
    const bool f32 = (fp32 && m.fr32) || m.fr64 == nullptr;
    if (m.physics == CTENO_EULER) {
        if (f32) hipLaunchKernelGGL((k_dt_partials<float, 4, CTENO_EULER>), dim3(grid), dim3(256), 0, st, m.N, U,
                                    m.fr32, m.area, m.gamma, m.ax, m.ay, part);
        else hipLaunchKernelGGL((k_dt_partials<double, 4, CTENO_EULER>), dim3(grid), dim3(256), 0, st, m.N, U,
                                m.fr64, m.area, m.gamma, m.ax, m.ay, part);
    } else {
        if (f32) hipLaunchKernelGGL((k_dt_partials<float, 1, CTENO_ADVECTION>), dim3(grid), dim3(256), 0, st, m.N, U,
                                    m.fr32, m.area, m.gamma, m.ax, m.ay, part);
        else hipLaunchKernelGGL((k_dt_partials<double, 1, CTENO_ADVECTION>), dim3(grid), dim3(256), 0, st, m.N, U,
                                m.fr64, m.area, m.gamma, m.ax, m.ay, part);
    }
    return hipGetLastError();
}

// Commits the pending step (t <- t_next), then decides the next one exactly
// as: stop when t >= t_final or the step budget is used; dt = cfl * bound;
// clip the last step onto t_final.
__device__ void control_logic(Ctrl *c, double bound, int commit_only) {
    if (c->pending) {
        c->t = c->t_next;
        c->step += 1;
        c->pending = 0;
    }
    if (commit_only || c->done) return;
    if (c->nonphysical || !(c->t < c->t_final) || c->step >= c->max_steps) {
        c->done = 1;
        return;
    }
    double dt = c->cfl * bound;
    double tn = c->t + dt;
    if (dt >= c->t_final - c->t) {
        dt = c->t_final - c->t;
        tn = c->t_final;
    }
    if (!(dt > 0.0)) {
        c->done = 1;
        c->nonphysical = 1;
        return;
    }
    c->dt = dt;
    c->t_next = tn;
    c->pending = 1;
}

// minimum of part[0..n) over the block (valid in thread 0)
__device__ __forceinline__ double block_min_array(const double *part, int64_t n, bool reduce) {
    __shared__ double red[16];
    double v = INFINITY;
    if (reduce)
        for (int64_t k = threadIdx.x; k < n; k += blockDim.x) v = fmin(v, part[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double bound = INFINITY;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) bound = fmin(bound, red[k]);
    return bound;
}

// Step control of one march, one block: the bound is the minimum of the
// per-block minima left by the last stage (or by k_dt_partials).
__global__ __launch_bounds__(1024) void k_control(Ctrl *c, const double *part, int64_t n_part, int commit_only) {
    const bool reduce = !commit_only && !c->done;
    const double bound = block_min_array(part, n_part, reduce);
    if (threadIdx.x == 0) control_logic(c, bound, commit_only);
}

hipError_t launch_control(Ctrl *ctrl, const double *part, int64_t n_part, int commit_only, hipStream_t st) {
    hipLaunchKernelGGL(k_control, dim3(1), dim3(1024), 0, st, ctrl, part, n_part, commit_only);
    return hipGetLastError();
}

// ===========================================================================
// batched serving kernels: one launch covers every active solve (slot)
// ===========================================================================

// slot of global block b: slots hold consecutive block ranges in table order
// (binary search for the first range that ends past b)
__device__ __forceinline__ int find_slot(const BatchSlot *tab, int n, int64_t b) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tab[mid].block0 + tab[mid].nblocks > b) hi = mid;
        else lo = mid + 1;
    }
    return lo < n && b >= tab[lo].block0 ? lo : -1;
}

template <int R, int SCHEME, int GFORM>
__global__ __launch_bounds__(256) void k_reconstruct_batch(const ReconArgs<float> a, const BatchSlot *tab,
                                                           const int *n_slots, int stage) {
    const int64_t b = blockIdx.x >> 2;        // four groups of 64 cells per table block
    const int s = find_slot(tab, *n_slots, b);
    if (s < 0) return;                        // uniform across the block
    const BatchSlot &t = tab[s];
    if (t.ctrl->done) return;
    const int64_t i = (b - t.block0) * 256 + (blockIdx.x & 3) * 64 + (threadIdx.x >> 2);
    if ((i & ~int64_t(63)) >= t.N) return;    // a group past the padded cells: whole blocks
    const int q = threadIdx.x & 3;
    const ReconPtrs<float> ptr{t.U[stage], t.lslot, t.desc, t.hlist, t.flags, t.P, nullptr, nullptr,
                               &t.ctrl->fallbacks, nullptr};
    extern __shared__ __align__(16) double rows[];
    double U0;
    float out[3][2];
    recon_quad<float, R, 4, SCHEME, GFORM, 0, 0, true>(a, ptr, rows, i, threadIdx.x, i < t.N, [] {}, U0, out);
    if (i >= t.N) return;
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g) t.FV[((i * 3 + f) * 2 + g) * 4 + q] = out[f][g];
}

// four blocks of 64 cells per table block, as the reconstruction
__global__ __launch_bounds__(256) void k_flux_batch(const FluxArgs<float> a, const BatchSlot *tab, const int *n_slots) {
    const int64_t b = blockIdx.x >> 2;
    const int s = find_slot(tab, *n_slots, b);
    if (s < 0) return;
    const BatchSlot &t = tab[s];
    if (t.ctrl->done) return;                 // uniform across the block
    const int stage = a.stage;
    const int64_t local = 4 * (b - t.block0) + (blockIdx.x & 3);
    const FluxPtrs<float> ptr{t.FV, t.fr, t.area, t.U[0], t.U[stage], stage == 2 ? t.U[0] : t.U[stage + 1],
                              &t.ctrl->dt, nullptr, nullptr, &t.ctrl->nonphysical, stage == 2};
    double dtc = INFINITY;
    if (local * 64 < t.N) {                   // uniform
        const int64_t i = local * 64 + (threadIdx.x >> 2);
        dtc = flux_quad<float, 4, CTENO_EULER, 2, 2>(a, ptr, i, i < t.N);
    }
    if (stage == 2) {
        const double bm = block_min(dtc);
        if (threadIdx.x == 0) t.dt_part[local] = bm;
    }
}

__global__ __launch_bounds__(1024) void k_control_batch(const BatchSlot *tab, const int *n_slots) {
    if ((int)blockIdx.x >= *n_slots) return;
    const BatchSlot &t = tab[blockIdx.x];
    const bool reduce = !t.ctrl->done;
    const double bound = block_min_array(t.dt_part, 4 * t.nblocks, reduce);
    if (threadIdx.x == 0) control_logic(t.ctrl, bound, 0);
}

template <int R>
static hipError_t batch_step_r(const DeviceMesh &proto, const BatchSlot *tab, const int *n_slots, int max_slots,
                               int64_t max_blocks, hipStream_t st) {
    ReconArgs<float> ra;
    fill_recon_constants<float>(proto, ra);
    if (!ra.tab) return hipErrorInvalidValue;
    const dim3 rgrid((unsigned)(4 * max_blocks));
    FluxArgs<float> fa{};
    std::memset(&fa, 0, sizeof fa);
    fa.gamma = (float)proto.gamma; fa.ax = (float)proto.ax; fa.ay = (float)proto.ay; fa.gamma64 = proto.gamma;
    fa.gw[0] = fa.gw[1] = 0.5f;
    fa.gw[2] = fa.gw[3] = 0.0f;
    hipLaunchKernelGGL(k_control_batch, dim3(max_slots), dim3(1024), 0, st, tab, n_slots);
    for (int stage = 0; stage < 3; ++stage) {
        if (proto.scheme == CTENO_SCHEME_CTENOZ && proto.gamma_form == CTENO_GAMMA_SCALED)
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_CTENOZ, CTENO_GAMMA_SCALED>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        else if (proto.scheme == CTENO_SCHEME_CTENOZ)
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_CTENOZ, CTENO_GAMMA_PAPER>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        else if (proto.scheme == CTENO_SCHEME_CWENO)
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_CWENO, CTENO_GAMMA_PAPER>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        else if (proto.scheme == CTENO_SCHEME_TENO)
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_TENO, CTENO_GAMMA_PAPER>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        else if (proto.gamma_form == CTENO_GAMMA_LAMBDA)
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_CTENO, CTENO_GAMMA_LAMBDA>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        else
            hipLaunchKernelGGL((k_reconstruct_batch<R, CTENO_SCHEME_CTENO, CTENO_GAMMA_PAPER>), rgrid,
                               dim3(256), proto.row_bytes(), st, ra, tab, n_slots, stage);
        fa.stage = stage;
        hipLaunchKernelGGL(k_flux_batch, rgrid, dim3(256), 0, st, fa, tab, n_slots);
    }
    return hipGetLastError();
}

hipError_t launch_batch_step(const DeviceMesh &proto, const BatchSlot *tab, const int *n_slots, int max_slots,
                             int64_t max_blocks, hipStream_t st) {
    if (proto.nv != 4 || proto.physics != CTENO_EULER) return hipErrorInvalidValue;
    switch (proto.r) {
        case 2: return batch_step_r<2>(proto, tab, n_slots, max_slots, max_blocks, st);
        case 3: return batch_step_r<3>(proto, tab, n_slots, max_slots, max_blocks, st);
        default: return hipErrorInvalidValue;
    }
}

// ===========================================================================
// layout conversions and utilities
// ===========================================================================

__global__ void k_user_to_state(int64_t N, int nv, const int32_t *perm, const double *user, double *state) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int64_t u = perm[k];
    for (int v = 0; v < nv; ++v) state[k * nv + v] = user[(int64_t)v * N + u];
}
__global__ void k_state_to_user(int64_t N, int nv, const int32_t *perm, const double *state, double *user) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int64_t u = perm[k];
    for (int v = 0; v < nv; ++v) user[(int64_t)v * N + u] = state[k * nv + v];
}
// Rows of `width` units, internal row k <-> caller row perm[k] (TO_USER: to the
// caller's).  Lanes run over the units of consecutive internal rows, so both
// sides are touched in whole rows.  A lane per row touched 64 rows with each
// load: face values of 49k cells at degree 5 in FP32 (144 B rows) 16.6 us, now
// 5.5.
template <typename T, bool TO_USER>
__global__ __launch_bounds__(256) void k_copy_rows(int64_t N, unsigned width, const int32_t *perm, const T *src, T *dst) {
    const int64_t k0 = (int64_t)blockIdx.x * 64;
    const unsigned n = (unsigned)min((int64_t)64, N - k0) * width;
    for (unsigned t = threadIdx.x; t < n; t += 256) {
        const unsigned r = t / width;
        const int64_t k = (k0 + r) * width + (t - r * width), u = (int64_t)perm[k0 + r] * width + (t - r * width);
        if (TO_USER) dst[u] = src[k];
        else dst[k] = src[u];
    }
}

static unsigned grid_for(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_user_to_state(const DeviceMesh &m, const double *user, double *state, hipStream_t st) {
    hipLaunchKernelGGL(k_user_to_state, dim3(grid_for(m.N)), dim3(256), 0, st, m.N, m.nv, m.perm, user, state);
    return hipGetLastError();
}
hipError_t launch_state_to_user(const DeviceMesh &m, const double *state, double *user, hipStream_t st) {
    hipLaunchKernelGGL(k_state_to_user, dim3(grid_for(m.N)), dim3(256), 0, st, m.N, m.nv, m.perm, state, user);
    return hipGetLastError();
}
// rows of `bytes` bytes in the widest unit that divides them and that both
// pointers are aligned to (the caller's may be a view of a larger array)
template <bool TO_USER>
static hipError_t copy_rows(const DeviceMesh &m, size_t bytes, const void *src, void *dst, hipStream_t st) {
    const dim3 grid((unsigned)((m.N + 63) / 64)), block(256);
    const size_t a = bytes | (size_t)(uintptr_t)src | (size_t)(uintptr_t)dst;
#define CR_LAUNCH(T)                                                                                              \
    hipLaunchKernelGGL((k_copy_rows<T, TO_USER>), grid, block, 0, st, m.N, (unsigned)(bytes / sizeof(T)), m.perm, \
                       (const T *)src, (T *)dst)
    if (a % 16 == 0) CR_LAUNCH(uint4);
    else if (a % 8 == 0) CR_LAUNCH(uint2);
    else if (a % 4 == 0) CR_LAUNCH(uint32_t);
    else CR_LAUNCH(uint8_t);
#undef CR_LAUNCH
    return hipGetLastError();
}
hipError_t launch_fv_to_user(const DeviceMesh &m, bool fp32, const void *fv, void *user, hipStream_t st) {
    return copy_rows<true>(m, (size_t)3 * m.tab.Nq * m.nv * (fp32 ? 4 : 8), fv, user, st);
}
hipError_t launch_fv_from_user(const DeviceMesh &m, bool fp32, const void *user, void *fv, hipStream_t st) {
    return copy_rows<false>(m, (size_t)3 * m.tab.Nq * m.nv * (fp32 ? 4 : 8), user, fv, st);
}
hipError_t launch_flux_to_user(const DeviceMesh &m, bool fp32, const void *fo, void *user, hipStream_t st) {
    return copy_rows<true>(m, (size_t)3 * m.nv * (fp32 ? 4 : 8), fo, user, st);
}
hipError_t launch_delta_to_user(const DeviceMesh &m, const uint8_t *d, uint8_t *user, hipStream_t st) {
    return copy_rows<true>(m, (size_t)m.delta_bytes(), d, user, st);
}
hipError_t launch_delta_from_user(const DeviceMesh &m, const uint8_t *user, uint8_t *d, hipStream_t st) {
    return copy_rows<false>(m, (size_t)m.delta_bytes(), user, d, st);
}

__global__ void k_count_diff(int64_t n, const uint8_t *a, const uint8_t *b, unsigned long long *count) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long c = (k < n && a[k] != b[k]) ? 1ull : 0ull;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}
hipError_t launch_count_diff(const DeviceMesh &m, const uint8_t *a, const uint8_t *b, unsigned long long *count,
                             hipStream_t st) {
    const int64_t n = m.N * m.delta_bytes();
    hipLaunchKernelGGL(k_count_diff, dim3(grid_for(n)), dim3(256), 0, st, n, a, b, count);
    return hipGetLastError();
}

__global__ void k_fill_u64(unsigned long long *p, unsigned long long v, size_t n) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = v;
}
hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for((int64_t)n)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n) {
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = v;
}
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for((int64_t)n)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

__global__ void k_copy16(uint4 *dst, const uint4 *src, size_t n) {
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        dst[k] = src[k];
}
hipError_t launch_copy16(void *dst, const void *src, size_t n16, hipStream_t st) {
    unsigned grid = (unsigned)std::min<size_t>((n16 + 255) / 256, 256 * 64);
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy16, dim3(grid), dim3(256), 0, st, (uint4 *)dst, (const uint4 *)src, n16);
    return hipGetLastError();
}

// ===========================================================================
// fixed device scratch of the allocation-free entry point
// ===========================================================================

// One static buffer per device for callers that cannot allocate device
// memory (cteno_flux_noalloc): the internal-order face-point values, face
// fluxes and the non-physical flag of one call.  Host code must use the
// address that hipGetSymbolAddress returns for the device, never the
// array's name, which on the host is only a stand-in.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;     // the device must be current
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void *scratch_device_ptr(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_ptr[device];
}

// the cell of slot j of cell i, from the row-number table
template <int R>
__device__ __forceinline__ int32_t row_cell(const uint16_t *lslot, const int2 *desc, const int32_t *hlist,
                                            int64_t i, int j) {
    const int r = lslot[lslot_index<R>(i, j)];
    return r < 64 ? (int32_t)((i & ~int64_t(63)) + r) : hlist[desc[i >> 6].x + (r - 64)];
}
// RL: the degree, 0 for the slot table and for one variable above degree 3
template <int RL>
__global__ void k_gather_entries(int n, const int32_t *idx, int E, int VW, const double *s64, const float *s32,
                                 const int32_t *si, double *dst) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * E) return;
    const int a = (int)(t / E), e = (int)(t % E);
    size_t src;
    if constexpr (RL == 0) src = avix(idx[a], e, E, VW);
    else if constexpr (RL <= 3) src = quad_index_entry<RL>(idx[a], e, VW);
    else src = ho_index<RL>(idx[a], e / HoRows<RL>::C, e % HoRows<RL>::C, VW);
    dst[t] = s64 ? s64[src] : (s32 ? (double)s32[src] : (double)si[src]);
}
template <int R>
__global__ void k_gather_cells(int n, const int32_t *idx, int SP, const uint16_t *lslot, const int2 *desc,
                               const int32_t *hlist, double *dst) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * SP) return;
    dst[t] = (double)row_cell<R>(lslot, desc, hlist, idx[t / SP], (int)(t % SP));
}
hipError_t launch_gather_entries(const DeviceMesh &m, int n, const int32_t *idx, int E, const double *src64,
                                 const float *src32, const int32_t *srci, double *dst, hipStream_t st) {
    const int VW = src64 ? 2 : 4;
    const dim3 grid(grid_for((int64_t)n * E)), block(256);
#define GE_LAUNCH(RL) \
    hipLaunchKernelGGL((k_gather_entries<RL>), grid, block, 0, st, n, idx, E, VW, src64, src32, srci, dst)
    if (!src64 && !src32 && !srci) {
        if (m.r == 2) hipLaunchKernelGGL(k_gather_cells<2>, grid, block, 0, st, n, idx, E, m.lslot, m.desc, m.hlist, dst);
        else hipLaunchKernelGGL(k_gather_cells<3>, grid, block, 0, st, n, idx, E, m.lslot, m.desc, m.hlist, dst);
    } else if (srci || (m.r >= 4 && m.nv == 1)) GE_LAUNCH(0);
    else if (m.r == 2) GE_LAUNCH(2);
    else if (m.r == 3) GE_LAUNCH(3);
    else if (m.r == 4) GE_LAUNCH(4);
    else if (m.r == 5) GE_LAUNCH(5);
    else GE_LAUNCH(6);
#undef GE_LAUNCH
    return hipGetLastError();
}

// ===========================================================================
// neighbour lists of the 64-cell groups
// ===========================================================================

// The cells outside group blockIdx.x that its stencils reach, each once and
// ascending, in LDS; returns their number.  Bitonic sort of the group's
// outside entries (padded with INT_MAX to a power of two), then the first of
// each run moves to its rank.
constexpr int kHaloSort = 2048;           // >= 64 cells x 18 slots
__device__ __forceinline__ int group_halo(const int32_t *slot, int SP, int (&key)[kHaloSort],
                                          int (&uniq)[kHaloSort]) {
    __shared__ int cnt;
    __shared__ int wsum[4];
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    if (threadIdx.x == 0) cnt = 0;
    for (int k = threadIdx.x; k < kHaloSort; k += 256) key[k] = 0x7FFFFFFF;
    __syncthreads();
    for (int k = threadIdx.x; k < 64 * SP; k += 256) {
        const int m = slot[avix(i0 + (k & 63), k >> 6, SP, 4)];
        if ((m >> 6) != (int)blockIdx.x) key[atomicAdd(&cnt, 1)] = m;
    }
    __syncthreads();
    int n2 = 64;
    while (n2 < cnt) n2 *= 2;
    for (int len = 2; len <= n2; len *= 2)
        for (int st = len / 2; st > 0; st /= 2) {
            for (int p = threadIdx.x; p < n2 / 2; p += 256) {
                const int a = 2 * p - (p & (st - 1)), b = a + st;
                const int x = key[a], y = key[b];
                if ((x > y) == ((a & len) == 0)) { key[a] = y; key[b] = x; }
            }
            __syncthreads();
        }
    // ranks of the first of each run: a contiguous share per thread
    const int per = n2 < 256 ? 1 : n2 / 256, k0 = threadIdx.x * per;
    int c = 0;
    for (int k = k0; k < k0 + per && k < cnt; ++k) c += k == 0 || key[k] != key[k - 1];
    int s = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(s, o, 64);
        if ((threadIdx.x & 63) >= (unsigned)o) s += y;
    }
    if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    int rank = s - c, total = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < (int)(threadIdx.x >> 6)) rank += wsum[w];
        total += wsum[w];
    }
    for (int k = k0; k < k0 + per && k < cnt; ++k)
        if (k == 0 || key[k] != key[k - 1]) uniq[rank++] = key[k];
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(256) void k_halo_counts(const int32_t *slot, int SP, int32_t *len) {
    __shared__ int key[kHaloSort], uniq[kHaloSort];
    const int n = group_halo(slot, SP, key, uniq);
    if (threadIdx.x == 0) len[blockIdx.x] = n;
}
template <int R>
__global__ __launch_bounds__(256) void k_halo_lists(const int32_t *slot, int SP, const int2 *desc,
                                                    int32_t *hlist, uint16_t *lslot) {
    __shared__ int key[kHaloSort], uniq[kHaloSort];
    const int n = group_halo(slot, SP, key, uniq);
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    for (int k = threadIdx.x; k < n; k += 256) hlist[desc[blockIdx.x].x + k] = uniq[k];
    for (int k = threadIdx.x; k < 64 * 4 * QuadDims<R>::SK; k += 256) {
        const int64_t i = i0 + (k & 63);
        const int j = k >> 6, m = j < SP ? slot[avix(i, j, SP, 4)] : (int)i;     // pads: the cell itself
        int row = m & 63;
        if ((m >> 6) != (int)blockIdx.x) {
            int lo = 0, hi = n - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (uniq[mid] < m) lo = mid + 1;
                else hi = mid;
            }
            row = 64 + lo;
        }
        lslot[lslot_index<R>(i, j)] = (uint16_t)row;
    }
}
hipError_t launch_halo_counts(const DeviceMesh &m, int32_t *len, hipStream_t st) {
    if (m.r > 3 || 64 * m.SP > kHaloSort) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_halo_counts, dim3((unsigned)m.groups()), dim3(256), 0, st, m.slot, m.SP, len);
    return hipGetLastError();
}
hipError_t launch_halo_lists(const DeviceMesh &m, hipStream_t st) {
    if (m.r > 3 || 64 * m.SP > kHaloSort) return hipErrorInvalidValue;
    const dim3 grid((unsigned)m.groups());
    if (m.r == 2)
        hipLaunchKernelGGL(k_halo_lists<2>, grid, dim3(256), 0, st, m.slot, m.SP, m.desc, m.hlist, m.lslot);
    else
        hipLaunchKernelGGL(k_halo_lists<3>, grid, dim3(256), 0, st, m.slot, m.SP, m.desc, m.hlist, m.lslot);
    return hipGetLastError();
}

// ===========================================================================
// block data of the fused stage
// ===========================================================================

// the arrays of a DeviceMesh that these kernels read and write
struct BlockMesh {
    int64_t N, Np;
    const float *fr32;
    const double *fr64, *area;
    bool f32;
    StageLists l;
    BlockMesh(const DeviceMesh &m, bool fp32)
        : N(m.N), Np(m.Np), fr32(m.fr32), fr64(m.fr64), area(m.area), f32(fp32), l(m.lists[fp32]) {}
};

// the neighbour code of face f of cell i, from either kind of face record
__device__ __forceinline__ uint32_t face_code(const BlockMesh &m, int64_t i, int f) {
    if (m.fr32) return (uint32_t)__float_as_int(m.fr32[avix(i, 4 * f + 3, 12, 4)]);
    return (uint32_t)__double_as_longlong(m.fr64[avix(i, 4 * f + 3, 12, 2)]);
}
// record k of a list: normal and length of face f of cell i, and a code
__device__ __forceinline__ void put_record(const BlockMesh &m, void *rec, int64_t k, int64_t i, int f, uint32_t code) {
    if (m.f32) {
        float *r = (float *)rec + 4 * k;
        for (int e = 0; e < 3; ++e) r[e] = m.fr32[avix(i, 4 * f + e, 12, 4)];
        r[3] = __int_as_float((int)code);
    } else {
        double *r = (double *)rec + 4 * k;
        for (int e = 0; e < 3; ++e) r[e] = m.fr64[avix(i, 4 * f + e, 12, 2)];
        r[3] = __longlong_as_double((long long)code);
    }
}

// exclusive sum over a wave and the total
__device__ __forceinline__ int wave_scan(int x, int &total) {
    int s = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(s, o, 64);
        if ((int)(threadIdx.x & 63) >= o) s += y;
    }
    total = __shfl(s, 63, 64);
    return s - x;
}

// a cell's listed faces and its faces to other blocks of `bc` cells, as bit masks
__device__ __forceinline__ void cell_faces(const BlockMesh &m, int64_t i, int bc, uint32_t (&code)[3], int &listed,
                                           int &cross) {
    listed = cross = 0;
    if (i >= m.N) return;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        code[f] = face_code(m, i, f);
        if (code[f] & kNbBoundary) listed |= 1 << f;
        else if ((int64_t)(code[f] & kNbIndexMask) / bc != i / bc) cross |= 1 << f;
        else if (code[f] & kNbOwner) listed |= 1 << f;
    }
}

// one wave per group
__global__ __launch_bounds__(256) void k_block_counts(const BlockMesh m, const BlockCounts c) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, g = i >> 6;
    if (i >= m.Np) return;                    // whole waves
    uint32_t code[3];
    int listed, cross, cross256, nf, nx, ns, n256;
    cell_faces(m, i, 256, code, listed, cross256);
    cell_faces(m, i, m.l.bc, code, listed, cross);
    (void)wave_scan(__popc(listed), nf);
    (void)wave_scan(cross ? 1 : 0, nx);
    (void)wave_scan(__popc(cross), ns);
    (void)wave_scan(cross256 ? 1 : 0, n256);
    if ((threadIdx.x & 63) == 0) {
        c.faces[g] = nf;
        c.cross[g] = nx;
        c.sides[g] = ns;
        if (n256) atomicAdd(c.cross256, n256);
    }
}
hipError_t launch_block_counts(const DeviceMesh &m, bool f32, const BlockCounts &c, hipStream_t st) {
    hipLaunchKernelGGL(k_block_counts, dim3(grid_for(m.Np)), dim3(256), 0, st, BlockMesh(m, f32), c);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_block_lists(const BlockMesh m, const BlockCounts base) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, g = i >> 6;
    if (i >= m.Np) return;                    // whole waves
    uint32_t code[3];
    int listed, cross, total;
    cell_faces(m, i, m.l.bc, code, listed, cross);
    int64_t k = base.faces[g] + wave_scan(__popc(listed), total);
    const int64_t t = base.cross[g] + wave_scan(cross ? 1 : 0, total);
    const uint32_t s0 = (uint32_t)(base.sides[g] + wave_scan(__popc(cross), total));
    const uint32_t id = cross ? s0 | ((uint32_t)cross << 28) : 0u;
    m.l.xid[i] = id;
    if (i >= m.N) return;
    const uint32_t lm = (uint32_t)m.l.bc - 1u;
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        if (!((listed >> f) & 1)) continue;
        uint32_t bf = ((uint32_t)i & lm) | ((uint32_t)f << 8);
        if (code[f] & kNbBoundary) bf |= kBfBoundary | ((code[f] & 3u) << 10);
        else bf |= (code[f] & lm) << 10 | ((code[f] >> 28) & 3u) << 18;
        put_record(m, m.l.frec, k++, i, f, bf);
    }
    if (cross) {
        m.l.xcells[t] = make_int2((int)i, (int)id);
        m.l.xarea[t] = m.area[i];
    }
}
// one thread per cross cell: its side records (every cell's first side is known)
__global__ __launch_bounds__(256) void k_side_records(const BlockMesh m) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m.l.n_cross) return;
    const int64_t i = m.l.xcells[t].x;
    const uint32_t id = m.l.xid[i];
    int64_t s = id & kNbIndexMask;
    for (int f = 0; f < 3; ++f) {
        if (!((id >> (28 + f)) & 1)) continue;
        const uint32_t code = face_code(m, i, f), idj = m.l.xid[code & kNbIndexMask];
        const int gf = (int)((code >> 28) & 3u);
        const uint32_t other = (idj & kNbIndexMask) + __popc((idj >> 28) & ((1u << gf) - 1u));
        const bool fb = (int64_t)(code & kNbIndexMask) / 256 != i / 256;
        put_record(m, m.l.xrec, s++, i, f, other | (code & kNbOwner) | (fb ? kSideFar : 0u));
    }
}
hipError_t launch_block_lists(const DeviceMesh &m, bool f32, const BlockCounts &base, hipStream_t st) {
    const BlockMesh b(m, f32);
    hipLaunchKernelGGL(k_block_lists, dim3(grid_for(m.Np)), dim3(256), 0, st, b, base);
    if (b.l.n_cross) hipLaunchKernelGGL(k_side_records, dim3(grid_for(b.l.n_cross)), dim3(256), 0, st, b);
    return hipGetLastError();
}

}  // namespace cteno
