// Fused SSP-RK3 stage of degree 2 and 3 for one arithmetic type;
// instantiated per type by k_stage_f32.hip and k_stage_f64.hip.
//
// Part 0 (k_stage), a quad of lanes per cell, a group of 64 cells per block:
// the reconstruction of the group's cells (sec. 2.1-2.6) goes to LDS; after a
// block barrier the lanes take the group's listed faces -- its boundary faces
// and the faces between two of its cells -- one Gauss point each, and leave
// the face's flux (sec. 2.7) in LDS for both of its cells, with opposite
// signs; after a second barrier each cell sums its faces and applies its RK
// stage, a lane per variable.  The values of a face to another group go to
// memory, at the place of that side of the face, and k_stage_cross (part 1)
// adds these faces to their cells' states.  The two cells of a face see
// bitwise opposite terms, so the update stays conservative to FP64 round-off
// without atomics.  Face values of faces inside a group never leave the chip.
#pragma once
#include "recon_quad.h"

namespace cteno {

// record k of the blocks' listed faces, or side k
__device__ __forceinline__ void packed_face(const float *rec, int64_t k, float &nx, float &ny, float &len,
                                            uint32_t &code) {
    const float4 r = reinterpret_cast<const float4 *>(rec)[k];
    nx = r.x; ny = r.y; len = r.z;
    code = (uint32_t)__float_as_int(r.w);
}
__device__ __forceinline__ void packed_face(const double *rec, int64_t k, double &nx, double &ny, double &len,
                                            uint32_t &code) {
    const double2 *b = reinterpret_cast<const double2 *>(rec) + 2 * k;
    const double2 r0 = b[0], r1 = b[1];
    nx = r0.x; ny = r0.y; len = r1.x;
    code = (uint32_t)__double_as_longlong(r1.y);
}

// Gauss point g of a listed face of the block that starts at cell i0: its
// lane pair leaves the face's terms for both of its cells in lterm, the first
// lane the owner's, the second the other cell's, its exact negation.  True for a
// non-physical state.
template <typename real, int NV, int PHYS>
__device__ __forceinline__ bool listed_face(const FluxArgs<real> fa, double dt, int64_t i0, int g, real nx, real ny,
                                            real len, uint32_t code, const real *lfv, real *lterm) {
    constexpr int NQ = 2;
    const int own = ((code & 255u) * 3 + ((code >> 8) & 3u)) * NQ * NV;
    const int oth = (((code >> 10) & 255u) * 3 + ((code >> 18) & 3u)) * NQ * NV;
    real A[NV], B[NV], F[NV];
    load_row<real, NV>(lfv + own + g * NV, A);
    bool wallf = false, bad = false;
    if (code & kBfBoundary)
        wallf = boundary_point<real, NV, PHYS>(fa, dt, i0 + (code & 255u), (code >> 8) & 3u, (code >> 10) & 3u, g, A, B);
    else
        load_row<real, NV>(lfv + oth + (NQ - 1 - g) * NV, B);
    if (PHYS == CTENO_EULER) {
        if (wallf) bad = !wall_flux<real>(fa.gamma, A, nx, ny, F);
        else bad = !hllc<real, std::is_same<real, float>::value ? 0 : -1>(fa.gamma, A, B, nx, ny, F);
    } else {
        const real an = fa.ax * nx + fa.ay * ny;
        F[0] = an * (an >= 0 ? A[0] : B[0]);
    }
    real term[NV];
#pragma unroll
    for (int w = 0; w < NV; ++w) {
        const real Fo = pair_swap(F[w]);
        real sum = 0;
        sum += fa.gw[0] * (g ? Fo : F[w]);
        sum += fa.gw[1] * (g ? F[w] : Fo);
        const real t = len * sum;
        term[w] = g ? -t : t;
    }
    if (!g) store_row<real, NV>(lterm + own / NQ, term);
    else if (!(code & kBfBoundary)) store_row<real, NV>(lterm + oth / NQ, term);
    return bad;
}

// The registers are held to five waves per SIMD in FP32 and four in FP64; FP64
// with characteristic variables would spill at four (128 B a lane) and runs three
template <typename real, int R, int NV, int SCHEME, int GFORM, int VARS, int PHYS, bool NT>
__global__ __launch_bounds__(256, (std::is_same<real, double>::value ? (VARS ? 3 : 4) : 5))
void k_stage(const ReconArgs<real> ra, const ReconPtrs<real> rp, const FluxArgs<real> fa) {
    constexpr int NQ = 2, ROW = 3 * NQ * NV;
    constexpr bool F32 = std::is_same<real, float>::value;
    extern __shared__ __align__(16) double rows[];       // the averages that the group reaches
    __shared__ __align__(16) real lfv[64 * ROW];         // the group's face-point values
    __shared__ __align__(16) real lterm[64 * 3 * NV];    // outward face fluxes of its cells
    const int64_t grp = xcd_block(blockIdx.x, gridDim.x);
    const int cl = threadIdx.x >> 2, q = threadIdx.x & 3, v = NV == 4 ? q : 0;
    const int64_t i = grp * 64 + cl;
    const bool live = i < fa.N;
    const double dtp = *(fa.dt_ptr ? fa.dt_ptr : fa.area), dt = fa.dt_ptr ? dtp : fa.dt_value;
    // requested behind the products: the update's operands and the lane's first
    // listed face
    double un0, ar, U0;
    uint32_t xid, code;
    real nx, ny, len, out[3][NQ];
    const int2 fd = fa.fdesc[grp];
    const int f0 = fd.x, nf = fd.y;
    auto mid = [&] {
        un0 = fa.stage ? fa.Un[i * NV + v] : 0.0;        // (stage 0 does not use it)
        ar = fa.area[i];
        xid = fa.xid[i];
        // (a place past the list reads the list's last entry)
        packed_face(fa.frec, f0 + max(min((int)(threadIdx.x >> 1), nf - 1), 0), nx, ny, len, code);
    };
    if (!recon_quad<real, R, NV, SCHEME, GFORM, 0, VARS, NT>(ra, rp, rows, i, threadIdx.x, live, mid, U0, out)) return;
    const int xmask = xid >> 28;                         // the cell's faces to other groups
    if (q < NV) {
#pragma unroll
        for (int f = 0; f < 3; ++f) {
#pragma unroll
            for (int g = 0; g < NQ; ++g) lfv[cl * ROW + (f * NQ + g) * NV + v] = out[f][g];
            if (!F32) lterm[(cl * 3 + f) * NV + v] = 0;  // stays for the faces to other groups
        }
        if (xmask) {
            // only the values of these leave the chip
            int64_t s = xid & kNbIndexMask;
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if ((xmask >> f) & 1) {
#pragma unroll
                    for (int g = 0; g < NQ; ++g) const_cast<real *>(fa.FV)[(s * NQ + g) * NV + v] = out[f][g];
                    ++s;
                }
        }
    }
    __syncthreads();
    // the listed faces, a lane per face and Gauss point (lane pairs share a face)
    bool bad = false;
    for (int k = threadIdx.x; k < 2 * nf; k += 256) {
        if (k >= 256) packed_face(fa.frec, f0 + (k >> 1), nx, ny, len, code);
        bad |= listed_face<real, NV, PHYS>(fa, dt, grp * 64, k & 1, nx, ny, len, code, lfv, lterm);
    }
    if (bad && fa.nonphys) atomicOr(fa.nonphys, 1);
    __syncthreads();
    double dtc = INFINITY;
    double acc = 0.0;
#pragma unroll
    for (int f = 0; f < 3; ++f) acc += (double)lterm[(cl * 3 + f) * NV + v];
    const double un = rk_value(fa.stage, un0, U0, dt * (-acc / ar));
    if (live && q < NV) {
        if (!F32 || !xmask) {
            // (FP64: a cross cell's state without its faces to other groups)
            fa.Uout[i * NV + v] = un;
        } else {
            // FP32: part 1 sums a cross cell's faces; the terms of those inside
            // the group (at most two) go to the places of its first side
            int64_t k = 2 * (int64_t)(xid & kNbIndexMask);
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if (!((xmask >> f) & 1)) fa.xterm[k++ * NV + v] = lterm[(cl * 3 + f) * NV + v];
        }
    }
    if (fa.dt_part) {
        // the CFL bound of the new state
        double u4[NV], nrm[3][3];
        quad_state<NV>(un, u4);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            real fx, fy, fl;
            uint32_t fc;
            face_record<real>(fa.fr, i, f, fx, fy, fl, fc);
            nrm[f][0] = (double)fx; nrm[f][1] = (double)fy; nrm[f][2] = (double)fl;
        }
        if (live && !xmask) dtc = cell_dt_bound<NV, PHYS>(u4, nrm, ar, fa.gamma64, (double)fa.ax, (double)fa.ay);
        const double bm = block_min(dtc);
        if (threadIdx.x == 0) fa.dt_part[fa.part_off + blockIdx.x] = bm;
    }
}

// part 0 in FP32 for large meshes: blocks of 256 cells, their four groups one
// after the other.  The next group's list, averages, row numbers and stream are
// requested when the products have used this group's, so they are in flight
// during the selection and the face values; the faces between the block's
// groups stay on the chip, which leaves part 1 half the sides.  On 8M cells at
// degree 3 this takes 1463 + 82 us, blocks of 64 cells 1455 + 273.  It moves 7.6
// GB, 5.1 TB/s; a wave waits 38 % of its cycles for memory, LDS and barriers and
// 37 % for the matrix and vector units.  Three waves per SIMD; at four the stream
// spills (1728 us).
template <int R, int NV, int SCHEME, int GFORM, int PHYS>
__global__ __launch_bounds__(256, 3)
void k_stage_wide(const ReconArgs<float> ra, const ReconPtrs<float> rp, const FluxArgs<float> fa, int row_doubles) {
    using real = float;
    constexpr int NQ = 2, ROW = 3 * NQ * NV, K = QuadDims<R>::K;
    // two groups' averages, row_doubles apart; after the last group the face
    // fluxes of the block's cells
    extern __shared__ __align__(16) double rows[];
    real *const lterm = reinterpret_cast<real *>(rows);  // [256][3][NV]
    __shared__ __align__(16) real lfv[256 * ROW];        // the block's face-point values
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int t = threadIdx.x, cl = t >> 2, lane = t & 63, q = t & 3, v = NV == 4 ? q : 0;
    const int64_t g0 = blk * 4;
    const int ng = (int)min((int64_t)4, (fa.Np >> 6) - g0);
    const double dtp = *(fa.dt_ptr ? fa.dt_ptr : fa.area), dt = fa.dt_ptr ? dtp : fa.dt_value;
    const int2 fd = fa.fdesc[blk];
    int2 desc[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) desc[p] = rp.desc[g0 + min(p, ng - 1)];
    const int stop = *(rp.done ? rp.done : &rp.desc->x);
    if (rp.done && stop) return;
    GroupRows<NV> gr;
    QuadStream<real, R, true> qs;
    double U0, Un0;
    int fl, fln;
    uint32_t xid, xidn;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    auto request = [&](int p) {          // group p's data
        const int64_t g = g0 + p, i = g * 64 + cl, tile = g * 4 + wave;
        Un0 = rp.U[i * NV + v];
        fln = rp.flags[i] & 7;
        xidn = fa.xid[i];
        qs.request_ids(rp.lslot, tile, lane);
        qs.request(rp.P, tile, lane);
    };
    float ao[K], ad[3][2];
    auto products = [&](int p, const int2 &d) {
        double *rw = rows + (p & 1) * row_doubles;
        U0 = Un0;
        fl = fln;
        xid = xidn;
        gr.store(rw, rp.U, rp.hlist, d, t, v, U0);
        __syncthreads();
        qs.template products<NV>(rp.P, (g0 + p) * 4 + wave, rw, lane, v, U0, ao, ad);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto finish = [&](int p) {
        const int64_t i = (g0 + p) * 64 + cl;
        real out[3][NQ];
        recon_finish<real, R, NV, SCHEME, GFORM, 0, 0>(ra, rp, i, q, i < fa.N, U0, fl, ao, ad, out);
        const int xmask = i < fa.N ? xid >> 28 : 0, c = p * 64 + cl;
        if (q < NV) {
#pragma unroll
            for (int f = 0; f < 3; ++f) {
#pragma unroll
                for (int g = 0; g < NQ; ++g) lfv[c * ROW + (f * NQ + g) * NV + v] = out[f][g];
            }
            if (xmask) {
                int64_t s = xid & kNbIndexMask;
#pragma unroll
                for (int f = 0; f < 3; ++f)
                    if ((xmask >> f) & 1) {
#pragma unroll
                        for (int g = 0; g < NQ; ++g) const_cast<real *>(fa.FV)[(s * NQ + g) * NV + v] = out[f][g];
                        ++s;
                    }
            }
        }
    };
    // (requested in the loop's order: a wait in it counts what lies behind on
    // every way to it)
    gr.list(rp.hlist, desc[0], t);
    gr.averages(rp.U, v);
    gr.list(rp.hlist, desc[1], t);
    request(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
    for (int p = 0; p + 1 < ng; ++p) {
        products(p, p == 0 ? desc[0] : p == 1 ? desc[1] : desc[2]);
        gr.averages(rp.U, v);            // group p + 1's, from the list requested a group ago
        gr.list(rp.hlist, p == 0 ? desc[2] : desc[3], t);
        request(p + 1);
        __builtin_amdgcn_sched_barrier(0);
        finish(p);
    }
    products(ng - 1, desc[3]);           // (desc past the block repeat its last group's)
    float nx, ny, len;
    uint32_t code;
    packed_face(fa.frec, fd.x + max(min(t >> 1, fd.y - 1), 0), nx, ny, len, code);
    __builtin_amdgcn_sched_barrier(0);
    finish(ng - 1);
    __syncthreads();                     // the values are there, and the averages done with
    for (int k = t; k < 256 * 3 * NV; k += 256) lterm[k] = 0;     // stays for the faces to other blocks
    __syncthreads();
    // the update's operands come during the fluxes
    double us[4], un0[4], ar[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int64_t i = (g0 + min(p, ng - 1)) * 64 + cl;
        us[p] = rp.U[i * NV + v];
        un0[p] = fa.stage ? fa.Un[i * NV + v] : 0.0;
        ar[p] = fa.area[i];
    }
    bool bad = false;
#pragma unroll 1
    for (int k = t; k < 2 * fd.y; k += 256) {
        const float cx = nx, cy = ny, cn = len;
        const uint32_t cc = code;
        if (k + 256 < 2 * fd.y) packed_face(fa.frec, fd.x + ((k + 256) >> 1), nx, ny, len, code);
        bad |= listed_face<real, NV, PHYS>(fa, dt, blk * 256, k & 1, cx, cy, cn, cc, lfv, lterm);
    }
    if (bad && fa.nonphys) atomicOr(fa.nonphys, 1);
    __syncthreads();
    double dtc = INFINITY;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int64_t i = (g0 + p) * 64 + cl;
        const int c = p * 64 + cl;
        double acc = 0.0;
#pragma unroll
        for (int f = 0; f < 3; ++f) acc += (double)lterm[(c * 3 + f) * NV + v];
        // (a cross cell's state without its faces to other blocks)
        const double un = rk_value(fa.stage, un0[p], us[p], dt * (-acc / ar[p]));
        const bool live = i < fa.N;
        if (live && q < NV) fa.Uout[i * NV + v] = un;
        if (fa.dt_part && p < ng) {      // uniform
            double u4[NV], nrm[3][3];
            quad_state<NV>(un, u4);
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                real fx, fy, fn;
                uint32_t fc;
                face_record<real>(fa.fr, i, f, fx, fy, fn, fc);
                nrm[f][0] = (double)fx; nrm[f][1] = (double)fy; nrm[f][2] = (double)fn;
            }
            if (live && !(fa.xid[i] >> 28))
                dtc = fmin(dtc, cell_dt_bound<NV, PHYS>(u4, nrm, ar[p], fa.gamma64, (double)fa.ax, (double)fa.ay));
        }
    }
    if (fa.dt_part) {
        const double bm = block_min(dtc);
        if (t == 0) fa.dt_part[fa.part_off + blockIdx.x] = bm;
    }
}

// part 1: a quad of lanes per cross cell, ascending: the faces to other groups
// from both sides' stored values.  Lane q takes Gauss point q % 2 of the cell's
// side q / 2 (a cell has 1.3 on average; a third is a second round), then
// variable q.  (A lane per cell ran up to six fluxes one after the other: 10.3
// us on 16k cells in FP64, now 5.4.)
// They are added to the state that part 0 left.  FP32 rounds face values of the
// state at 1e-8 of it, so the order of the state's own sums shows in a march: in
// FP32 a cell's faces are summed in one order whatever the blocks are -- those
// inside its 256-cell block, then those to other blocks.  In blocks of 64 cells
// (SUM) that takes the faces inside the block from where part 0 left them, and
// the RK stage here.
template <typename real, int NV, int PHYS, bool SUM>
__global__ __launch_bounds__(256) void k_stage_cross(const FluxArgs<real> fa, int64_t n_blocks) {
    constexpr int NQ = 2;
    constexpr bool F32 = std::is_same<real, float>::value;
    const int64_t t = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2);
    const int q = threadIdx.x & 3, v = NV == 4 ? q : 0, g = q & 1;
    if (fa.ctrl && fa.ctrl->done) return;      // uniform across the grid
    const bool live = t < fa.n_cross;
    const int64_t tl = live ? t : fa.n_cross - 1;
    const int2 xc = fa.xcells[tl];
    const int64_t i = xc.x;
    const double ar = fa.xarea[tl];
    const int xmask = (int)((uint32_t)xc.y >> 28), ns = __popc(xmask);
    const int64_t s0 = (uint32_t)xc.y & kNbIndexMask;
    double us, un0 = 0.0;
    real inside[2];
    if constexpr (SUM) {
        us = fa.Us[i * NV + v];
        if (fa.stage) un0 = fa.Un[i * NV + v];
#pragma unroll
        for (int r = 0; r < 2; ++r) inside[r] = fa.xterm[(2 * s0 + r) * NV + v];     // (as many as 3 - ns count)
    } else {
        us = fa.Uout[i * NV + v];
    }
    real side[3] = {0, 0, 0};
    int far[3] = {0, 0, 0};
    const double dt = fa.dt_ptr ? *fa.dt_ptr : fa.dt_value;
    bool bad = false;
#pragma unroll 1
    for (int k0 = 0; k0 < 3; k0 += 2) {
        if (k0 > 0 && !__any(ns > k0)) break;
        const int k = k0 + (q >> 1);
        const bool on = k < ns;
        const int64_t s = s0 + (on ? k : 0);
        real nx, ny, len;
        uint32_t code;
        packed_face(fa.xrec, s, nx, ny, len, code);
        // both cells of a face evaluate F(owner side, other side; owner
        // normal) at the owner's points, so their terms are exact negatives
        const bool owner = (code & kNbOwner) != 0;
        const int64_t so = code & kNbIndexMask;
        const int fr = (int)((code & kSideFar) != 0);
        real A[NV], B[NV], F[NV], term[NV];
        load_row<real, NV>(fa.FV + ((owner ? s : so) * NQ + g) * NV, A);
        load_row<real, NV>(fa.FV + ((owner ? so : s) * NQ + (NQ - 1 - g)) * NV, B);
        const real fx = owner ? nx : -nx, fy = owner ? ny : -ny;
        if (PHYS == CTENO_EULER) {
            bad |= !hllc<real, F32 ? 2 : -1>(fa.gamma, A, B, fx, fy, F, fr && g) && on;
        } else {
            const real an = fa.ax * fx + fa.ay * fy;
            F[0] = an * (an >= 0 ? A[0] : B[0]);
        }
#pragma unroll
        for (int w = 0; w < NV; ++w) {
            const real Fo = pair_swap(F[w]);
            real sum = 0;
            sum += fa.gw[0] * (g ? Fo : F[w]);
            sum += fa.gw[1] * (g ? F[w] : Fo);
            const real x = len * sum;
            term[w] = owner ? x : -x;
        }
        const real t0 = quad_take<0>(term, v), t1 = quad_take<2>(term, v);
        const int b0 = quad_bcast_dyn(0, fr), b1 = quad_bcast_dyn(2, fr);
        if (k0 == 0) {
            side[0] = t0; far[0] = b0;
            side[1] = t1; far[1] = b1;
        } else {
            side[2] = t0; far[2] = b0;
        }
    }
    if (bad && live && fa.nonphys) atomicOr(fa.nonphys, 1);
    double un, acc = 0.0;
    if constexpr (SUM) {
        // the cell's faces in order, the far ones apart
        double accf = 0.0;
        int ks = 0, ki = 0;
        bool anyfar = false;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            if ((xmask >> f) & 1) {
                const double x = (double)(ks == 0 ? side[0] : ks == 1 ? side[1] : side[2]);
                const bool fb = (ks == 0 ? far[0] : ks == 1 ? far[1] : far[2]) != 0;
                if (fb) accf += x;
                else acc += x;
                anyfar |= fb;
                ++ks;
            } else {
                acc += (double)(ki == 0 ? inside[0] : inside[1]);
                ++ki;
            }
        }
        un = rk_value(fa.stage, un0, us, dt * (-acc / ar));
        if (anyfar) un = un + rk_weight(fa.stage) * (dt * (-accf / ar));
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < ns) acc += (double)side[k];
        un = us + rk_weight(fa.stage) * (dt * (-acc / ar));
    }
    if (live && q < NV) fa.Uout[i * NV + v] = un;
    if (fa.dt_part) {
        double u4[NV], nrm[3][3];
        quad_state<NV>(un, u4);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            real nx, ny, len;
            uint32_t code;
            face_record<real>(fa.fr, i, f, nx, ny, len, code);
            nrm[f][0] = (double)nx; nrm[f][1] = (double)ny; nrm[f][2] = (double)len;
        }
        double dtc = INFINITY;
        if (live) dtc = cell_dt_bound<NV, PHYS>(u4, nrm, ar, fa.gamma64, (double)fa.ax, (double)fa.ay);
        // with a share of part 0's minima, so that the step control has only
        // these blocks' to reduce
        const int64_t per = (n_blocks + gridDim.x - 1) / gridDim.x;
        const int64_t p1 = min(n_blocks, per * (blockIdx.x + 1));
        for (int64_t p = per * blockIdx.x + threadIdx.x; p < p1; p += 256) dtc = fmin(dtc, fa.dt_part[fa.part_off + p]);
        const double bm = block_min(dtc);
        if (threadIdx.x == 0) fa.dt_part[blockIdx.x] = bm;
    }
}

template <typename real, int R, int NV, int VARS, int PHYS>
static void stage_launch(const DeviceMesh &m, const ReconArgs<real> &ra, const ReconPtrs<real> &rp,
                         const FluxArgs<real> &fa, hipStream_t st) {
    constexpr bool F32 = std::is_same<real, float>::value;
    const unsigned grid = (unsigned)m.stage_blocks(F32);
#define ST_LAUNCH(SCH, GF)                                                                                        \
    do {                                                                                                          \
        if constexpr (F32 && !VARS)                                                                               \
            if (m.lists[1].bc == 256) {                                                                           \
                hipLaunchKernelGGL((k_stage_wide<R, NV, SCH, GF, PHYS>), dim3(grid), dim3(256),                   \
                                   std::max(2 * m.row_bytes(), 256 * 3 * NV * sizeof(float)), st, ra, rp, fa,     \
                                   (int)(m.row_bytes() / 8));                                                     \
                break;                                                                                            \
            }                                                                                                     \
        if (m.stream_nontemporal(F32))                                                                            \
            hipLaunchKernelGGL((k_stage<real, R, NV, SCH, GF, VARS, PHYS, true>), dim3(grid), dim3(256),          \
                               m.row_bytes(), st, ra, rp, fa);                                                    \
        else                                                                                                      \
            hipLaunchKernelGGL((k_stage<real, R, NV, SCH, GF, VARS, PHYS, false>), dim3(grid), dim3(256),         \
                               m.row_bytes(), st, ra, rp, fa);                                                    \
    } while (0)
    if (m.scheme == CTENO_SCHEME_CTENOZ && m.gamma_form == CTENO_GAMMA_SCALED) ST_LAUNCH(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_SCALED);
    else if (m.scheme == CTENO_SCHEME_CTENOZ) ST_LAUNCH(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_PAPER);
    else if (m.scheme == CTENO_SCHEME_CWENO) ST_LAUNCH(CTENO_SCHEME_CWENO, CTENO_GAMMA_PAPER);
    else if (m.scheme == CTENO_SCHEME_TENO) ST_LAUNCH(CTENO_SCHEME_TENO, CTENO_GAMMA_PAPER);
    else if (m.gamma_form == CTENO_GAMMA_LAMBDA) ST_LAUNCH(CTENO_SCHEME_CTENO, CTENO_GAMMA_LAMBDA);
    else ST_LAUNCH(CTENO_SCHEME_CTENO, CTENO_GAMMA_PAPER);
#undef ST_LAUNCH
}

template <typename real, int R, int NV, int PHYS>
static hipError_t stage_t(const DeviceMesh &m, const FluxLaunch &f, const int *done, hipStream_t st,
                          unsigned long long *fb_count) {
    if (m.E != QuadDims<R>::E || m.SP != QuadDims<R>::SP) return hipErrorInvalidValue;
    ReconArgs<real> ra;
    fill_recon_constants<real>(m, ra);
    ReconPtrs<real> rp{};
    rp.U = f.Us;
    rp.lslot = m.lslot;
    rp.desc = m.desc;
    rp.hlist = m.hlist;
    rp.flags = m.flags;
    if constexpr (std::is_same<real, double>::value) { rp.P = m.P64; rp.fr = m.fr64; }
    else { rp.P = m.P32; rp.fr = m.fr32; }
    rp.fb = fb_count;
    rp.done = done;
    FluxArgs<real> fa;
    fill_flux_args<real>(m, f, fa);
    if (!rp.P || !rp.fr || !ra.tab || !fa.fdesc || !fa.frec || !fa.xid || !rp.lslot || !rp.desc || !rp.hlist) return hipErrorInvalidValue;
    if (m.vars == CTENO_VARS_CHARACTERISTIC) {
        if constexpr (NV == 4) stage_launch<real, R, NV, 1, PHYS>(m, ra, rp, fa, st);
        else return hipErrorInvalidValue;
    } else {
        stage_launch<real, R, NV, 0, PHYS>(m, ra, rp, fa, st);
    }
    return hipGetLastError();
}

template <typename real>
hipError_t stage_fused(const DeviceMesh &m, const FluxLaunch &f, const int *done, int part, hipStream_t st,
                       unsigned long long *fb_count) {
    constexpr bool F32 = std::is_same<real, float>::value;
    const StageLists &l = m.lists[F32];
    if (f.mode != 2 || m.r > 3 || m.tab.Nq != 2 || !l.fused || !f.FV) return hipErrorInvalidValue;
    const bool sum = F32 && l.bc == 64;
    if (l.n_cross && (!l.xcells || !l.xarea || !l.xrec || (sum && !f.xterm))) return hipErrorInvalidValue;
    if (part == 1) {
        if (l.n_cross == 0) return hipSuccess;
        FluxArgs<real> fa;
        fill_flux_args<real>(m, f, fa);
        const dim3 grid((unsigned)l.cross_blocks()), block(256);
        const int64_t nb = m.stage_blocks(F32);
        if (m.physics == CTENO_EULER) {
            if (sum) hipLaunchKernelGGL((k_stage_cross<real, 4, CTENO_EULER, F32>), grid, block, 0, st, fa, nb);
            else hipLaunchKernelGGL((k_stage_cross<real, 4, CTENO_EULER, false>), grid, block, 0, st, fa, nb);
        } else {
            if (sum) hipLaunchKernelGGL((k_stage_cross<real, 1, CTENO_ADVECTION, F32>), grid, block, 0, st, fa, nb);
            else hipLaunchKernelGGL((k_stage_cross<real, 1, CTENO_ADVECTION, false>), grid, block, 0, st, fa, nb);
        }
        return hipGetLastError();
    }
    if (m.physics == CTENO_EULER) {
        if (m.nv != 4) return hipErrorInvalidValue;
        return m.r == 2 ? stage_t<real, 2, 4, CTENO_EULER>(m, f, done, st, fb_count)
                        : stage_t<real, 3, 4, CTENO_EULER>(m, f, done, st, fb_count);
    }
    if (m.nv != 1) return hipErrorInvalidValue;
    return m.r == 2 ? stage_t<real, 2, 1, CTENO_ADVECTION>(m, f, done, st, fb_count)
                    : stage_t<real, 3, 1, CTENO_ADVECTION>(m, f, done, st, fb_count);
}

}  // namespace cteno
