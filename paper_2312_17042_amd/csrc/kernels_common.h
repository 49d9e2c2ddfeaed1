// Device helpers shared by the kernel translation units of the CTENO/CTENOZ
// library: vector loads, face records, the XCD-aware block order, TENO-type
// selections, CWENO weights, HLLC and wall fluxes, boundary states, a face's
// flux term, RK stage values and the CFL bound.
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstring>
#include <cmath>
#include <type_traits>
#include <utility>

#include "kernels.h"

namespace cteno {

// ===========================================================================
// small helpers
// ===========================================================================

template <typename real> struct Vec;
template <> struct Vec<float> { using T = float4; static constexpr int W = 4; };
template <> struct Vec<double> { using T = double2; static constexpr int W = 2; };

__device__ __forceinline__ float comp(const float4 &v, int c) { return c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w; }
__device__ __forceinline__ double comp(const double2 &v, int c) { return c == 0 ? v.x : v.y; }

// Division, reciprocal and square root in the working precision.  FP64 keeps
// the IEEE operations (the fluxes multiply by an IEEE reciprocal where
// several quotients share a denominator: one more rounding).  FP32 takes the
// hardware reciprocal and square root (about 1 ulp each): a few ulps beside
// the correctly rounded sequences, at a fraction of their instruction count.
__device__ __forceinline__ float fdiv(float x, float y) { return x * __builtin_amdgcn_rcpf(y); }
__device__ __forceinline__ double fdiv(double x, double y) { return x / y; }
__device__ __forceinline__ float frcp(float y) { return __builtin_amdgcn_rcpf(y); }
__device__ __forceinline__ double frcp(double y) { return 1.0 / y; }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fsqrt(double x) { return sqrt(x); }

// Pressure of a conserved Euler state (rho, m_x, m_y, E).  The positivity
// fallback of the reconstructions and the admissibility test of the fluxes
// evaluate it with this one sequence of roundings (contraction into fused
// operations is off here), so a face state that the fallback accepts is
// accepted by the flux: two formulas could disagree on a state whose
// pressure is within rounding of zero, which FP32 meets in strong shocks.
template <typename real>
__device__ __forceinline__ real euler_pressure(real g, real r, real mx, real my, real E) {
#pragma clang fp contract(off)
    const real q = (real)0.5 * (mx * mx + my * my);
    real ke;
    if constexpr (std::is_same<real, float>::value) ke = q * __builtin_amdgcn_rcpf(r);
    else ke = q / r;
    return (g - 1) * (E - ke);
}

// n consecutive reals from/to an aligned address with the widest vector the
// row size allows (16 bytes, else 8 bytes)
template <typename real, int n>
__device__ __forceinline__ void load_row(const real *__restrict__ p, real *out) {
    if constexpr ((n * sizeof(real)) % 16 == 0) {
        using V = typename Vec<real>::T;
        constexpr int W = Vec<real>::W;
#pragma unroll
        for (int k = 0; k < n / W; ++k) {
            const V v = reinterpret_cast<const V *>(p)[k];
#pragma unroll
            for (int c = 0; c < W; ++c) out[k * W + c] = comp(v, c);
        }
    } else if constexpr (std::is_same<real, float>::value && n % 2 == 0) {
#pragma unroll
        for (int k = 0; k < n / 2; ++k) {
            const float2 v = reinterpret_cast<const float2 *>(p)[k];
            out[2 * k] = v.x;
            out[2 * k + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int k = 0; k < n; ++k) out[k] = p[k];
    }
}
template <typename real, int n>
__device__ __forceinline__ void store_row(real *__restrict__ p, const real *in) {
    if constexpr ((n * sizeof(real)) % 16 == 0) {
        if constexpr (std::is_same<real, float>::value) {
#pragma unroll
            for (int k = 0; k < n / 4; ++k)
                reinterpret_cast<float4 *>(p)[k] = make_float4(in[4 * k], in[4 * k + 1], in[4 * k + 2], in[4 * k + 3]);
        } else {
#pragma unroll
            for (int k = 0; k < n / 2; ++k) reinterpret_cast<double2 *>(p)[k] = make_double2(in[2 * k], in[2 * k + 1]);
        }
    } else if constexpr (std::is_same<real, float>::value && n % 2 == 0) {
#pragma unroll
        for (int k = 0; k < n / 2; ++k) reinterpret_cast<float2 *>(p)[k] = make_float2(in[2 * k], in[2 * k + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < n; ++k) p[k] = in[k];
    }
}

// face record of local face f: unit normal, length, neighbour code
template <typename real>
__device__ __forceinline__ void face_record(const real *fr, int64_t i, int f, real &nx, real &ny, real &len,
                                            uint32_t &code) {
    if constexpr (std::is_same<real, float>::value) {
        const float4 r = reinterpret_cast<const float4 *>(fr)[(size_t)(i >> 6) * 3 * 64 + f * 64 + (i & 63)];
        nx = r.x; ny = r.y; len = r.z;
        code = (uint32_t)__float_as_int(r.w);
    } else {
        const double2 *b = reinterpret_cast<const double2 *>(fr) + (size_t)(i >> 6) * 6 * 64 + (i & 63);
        const double2 r0 = b[(2 * f) * 64], r1 = b[(2 * f + 1) * 64];
        nx = r0.x; ny = r0.y; len = r1.x;
        code = (uint32_t)__double_as_longlong(r1.y);
    }
}

// Work-groups are dispatched round-robin over the 8 XCDs; remap them so that
// each XCD (and its L2) works on one contiguous range of cells, which keeps
// the neighbour gathers of adjacent blocks in the same L2.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
    if (nb < 8) return b;
    const int64_t per = nb / 8, rem = nb % 8;
    const int64_t x = b % 8, pos = b / 8;
    return x < rem ? x * (per + 1) + pos : rem * (per + 1) + (x - rem) * per + pos;
}

// ===========================================================================
// reconstruction
// ===========================================================================

template <typename real>
__device__ __forceinline__ real pow6(real x) {
    const real x2 = x * x;
    return x2 * x2 * x2;
}

// TENO selection bits for one variable: bit 0 central, bit 1+s directional s.
// FP64 follows Algorithms 1/2 literally; FP32 evaluates the same chi_s
// through ratios that cannot overflow (gamma_s reaches 1e72 in FP64 terms).
template <typename real, int SCHEME, int GFORM>
__device__ __forceinline__ int teno_bits(const real si[4], int adm, int st, real lam1, real lams, real lratio,
                                         real ct, real eps) {
    int bits = 0;
    if constexpr (std::is_same<real, double>::value) {
        double g[4], sum = 0.0;
        if (SCHEME == CTENO_SCHEME_CTENO) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double lam = s == 0 ? (double)lam1 : (double)lams;
                g[s] = (GFORM == CTENO_GAMMA_LAMBDA ? lam : 1.0) / pow6(si[s] + eps);
            }
        } else {
            double tsum = 0.0;
#pragma unroll
            for (int s = 1; s < 4; ++s) if ((adm >> s) & 1) tsum += fabs(si[s] - si[0]);
            const double tau = pow6(tsum / (st - 1));
#pragma unroll
            for (int s = 0; s < 4; ++s)
                g[s] = 1.0 + (GFORM == CTENO_GAMMA_SCALED ? tau / pow6(si[s] + eps) : tau / (si[s] + eps));
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) if ((adm >> s) & 1) sum += g[s];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if ((adm >> s) & 1) {
                const double chi = g[s] / sum;
                if (!(chi < ct)) bits |= 1 << s;
            }
    } else {
        // chi_s < C_T is decided as num_s < C_T sum_t num_t (sum > 0), with
        // one reciprocal per stencil and no division
        float e[4], re[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            e[s] = si[s] + eps;
            re[s] = frcp(e[s]);
        }
        if (SCHEME == CTENO_SCHEME_CTENO) {
            // chi_s = 1 / den_s, den_s = sum_t (lambda_t / lambda_s) (e_s / e_t)^6
            const float ilratio = frcp(lratio);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (!((adm >> s) & 1)) continue;
                float den = 0.0f;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (!((adm >> t) & 1)) continue;
                    float lr = 1.0f;
                    if (GFORM == CTENO_GAMMA_LAMBDA && s != t) lr = (t == 0) ? lratio : (s == 0 ? ilratio : 1.0f);
                    den += lr * pow6(e[s] * re[t]);
                }
                if (!(ct * den > 1.0f)) bits |= 1 << s;
            }
        } else {
            float tsum = 0.0f, emin = e[0], remin = re[0];
#pragma unroll
            for (int s = 1; s < 4; ++s)
                if ((adm >> s) & 1) {
                    tsum += fabsf(e[s] - e[0]);
                    emin = fminf(emin, e[s]);
                    remin = fmaxf(remin, re[s]);
                }
            const float mean = tsum * (st == 2 ? 1.0f : st == 3 ? 0.5f : 1.0f / 3.0f);
            float num[4], sum = 0.0f;
            if constexpr (GFORM == CTENO_GAMMA_SCALED) {
                // gamma_s = 1 + X^6 w_s^6 with X = mean |SI_s - SI_1| / emin
                const float X = mean * remin;
                if (X <= 1e5f) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) num[s] = 1.0f + pow6(X * (emin * re[s]));
                } else {
                    const float iX6 = pow6(frcp(X));
#pragma unroll
                    for (int s = 0; s < 4; ++s) num[s] = iX6 + pow6(emin * re[s]);
                }
            } else {
                const float tau = pow6(mean);
                const float G = tau * remin;       // gamma_s = 1 + G w_s, w_s = emin / e_s in (0, 1]
                if (G <= 1e30f) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) num[s] = 1.0f + G * (emin * re[s]);
                } else {
                    const float iG = frcp(G);
#pragma unroll
                    for (int s = 0; s < 4; ++s) num[s] = iG + emin * re[s];
                }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) if ((adm >> s) & 1) sum += num[s];
            const float lim = ct * sum;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if ((adm >> s) & 1) {
                    if (!(num[s] < lim)) bits |= 1 << s;
                }
        }
    }
    return bits;
}

// CWENO nonlinear weights (sec. 2.2-2.3: the WENO weights with exponent 4 and
// the linear weights of eq. e18) of the admissible stencils.  FP64 follows
// the formula; FP32 evaluates w_s = 1 / sum_t (lambda_t / lambda_s)
// (e_s / e_t)^4, e = SI + eps, which cannot overflow into a NaN.
template <typename real>
__device__ __forceinline__ void cweno_weights(const real si[4], int adm, real lams, real lam1, real lratio, real eps,
                                              real w[4]) {
    if constexpr (std::is_same<real, double>::value) {
        double g[4], sum = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double e = si[s] + eps, e2 = e * e;
            g[s] = ((adm >> s) & 1) ? (s == 0 ? lam1 : lams) / (e2 * e2) : 0.0;
            sum += g[s];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) w[s] = g[s] / sum;
    } else {
        float e[4], re[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            e[s] = si[s] + eps;
            re[s] = frcp(e[s]);
        }
        const float ilratio = frcp(lratio);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            float den = 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (!((adm >> t) & 1)) continue;
                const float lr = (s == t) ? 1.0f : (t == 0 ? lratio : (s == 0 ? ilratio : 1.0f));
                const float q = e[s] * re[t], q2 = q * q;
                den += lr * (q2 * q2);
            }
            w[s] = ((adm >> s) & 1) ? frcp(den) : 0.0f;
        }
    }
}

template <int R>
struct HoDims {
    static constexpr int K = (R + 1) * (R + 2) / 2 - 1;
    static constexpr int RD = (R + 1) / 2;
    static constexpr int KD = (RD + 1) * (RD + 2) / 2 - 1;
    static constexpr int MD = 2 * KD;
    static constexpr int M = 2 * K;
    // variable groups (degrees 4 and 5): the slots are the M central cells,
    // each directional stencil's members contiguous, their stencil in the
    // slot entry; else three groups of M_d slots
    static constexpr bool VARG = M < 3 * MD;
    static constexpr int S = VARG ? M : 3 * MD;
    static constexpr int SP = (S + 3) / 4 * 4;
    static constexpr int EPS = (K + KD + 3) / 4 * 4;
    static constexpr int E = S * EPS;
    static constexpr int NQ = (R + 2) / 2;
    static_assert(S >= 2 * K, "the directional groups must hold the central stencil");
    static_assert(S <= 64, "one lane per least-squares row");
};

// ===========================================================================
// fluxes, residual, Runge-Kutta
// ===========================================================================

// HLLC with Roe-averaged signal speeds (sec. 2.7), in the face-normal frame
// (u normal, w tangential velocity); F returned in the global frame.  In FP32
// the sum H_l + H_r D of the Roe average is contracted by hand: ALT 0 leaves H_l
// unrounded in it, 2 H_r D where `alt` is set and else H_l; 3 is 0 with the other
// product of u_r unrounded.  An FP32 face value of the state rounds at 1e-8 of
// it, so a march repeats its results bit for bit, whatever the blocks are, only
// if each face keeps its own contraction.
template <typename real, int ALT = -1>
__device__ __forceinline__ bool hllc(real g, const real *UL, const real *UR, real nx, real ny, real *F,
                                     bool alt = false) {
    // one reciprocal per denominator, shared by the quotients over it
    const real rl = UL[0], rr = UR[0];
    const real irl = frcp(rl), irr = frcp(rr);
    const real ul = (UL[1] * nx + UL[2] * ny) * irl, wl = (-UL[1] * ny + UL[2] * nx) * irl;
    real mr;
    if constexpr (ALT == 3) mr = __builtin_fmaf(UR[2], ny, UR[1] * nx);
    else mr = UR[1] * nx + UR[2] * ny;
    const real ur = mr * irr, wr = (-UR[1] * ny + UR[2] * nx) * irr;
    const real El = UL[3], Er = UR[3];
    const real h = (real)0.5;
    const real pl = euler_pressure(g, rl, UL[1], UL[2], El);
    const real pr = euler_pressure(g, rr, UR[1], UR[2], Er);
    const bool ok = rl > 0 && rr > 0 && pl > 0 && pr > 0;
    const real cl = fsqrt((g * pl) * irl), cr = fsqrt((g * pr) * irr);
    const real Hl = (El + pl) * irl, Hr = (Er + pr) * irr;
    const real D = fsqrt(rr * irl);
    const real iD = frcp(1 + D);
    const real ut = (ul + ur * D) * iD;
    const real wt = (wl + wr * D) * iD;
    real Hs;
    if constexpr (ALT < 0) {
        Hs = Hl + Hr * D;
    } else {
        const real h0 = __builtin_fmaf(irl, El + pl, Hr * D), h1 = __builtin_fmaf(Hr, D, Hl);
        Hs = ALT == 2 && alt ? h1 : h0;
    }
    const real Ht = Hs * iD;
    const real ct = fsqrt((g - 1) * (Ht - h * (ut * ut + wt * wt)));
    const real SL = fmin(ul - cl, ut - ct);
    const real SR = fmax(ur + cr, ut + ct);
    const real SM = fdiv(rr * ur * (SR - ur) - rl * ul * (SL - ul) + pl - pr, rr * (SR - ur) - rl * (SL - ul));
    const real ps = rl * (ul - SL) * (ul - SM) + pl;
    real Fn[4];
    if (SL > 0) {
        Fn[0] = rl * ul; Fn[1] = rl * ul * ul + pl; Fn[2] = rl * ul * wl; Fn[3] = ul * (El + pl);
    } else if (0 < SM) {
        const real id = frcp(SL - SM);
        const real Us0 = (rl * (SL - ul)) * id;
        const real Us1 = ((SL - ul) * rl * ul + ps - pl) * id;
        const real Us2 = ((SL - ul) * rl * wl) * id;
        const real Us3 = ((SL - ul) * El - pl * ul + ps * SM) * id;
        Fn[0] = rl * ul + SL * (Us0 - rl);
        Fn[1] = (rl * ul * ul + pl) + SL * (Us1 - rl * ul);
        Fn[2] = rl * ul * wl + SL * (Us2 - rl * wl);
        Fn[3] = ul * (El + pl) + SL * (Us3 - El);
    } else if (0 < SR) {
        const real id = frcp(SR - SM);
        const real Us0 = (rr * (SR - ur)) * id;
        const real Us1 = ((SR - ur) * rr * ur + ps - pr) * id;
        const real Us2 = ((SR - ur) * rr * wr) * id;
        const real Us3 = ((SR - ur) * Er - pr * ur + ps * SM) * id;
        Fn[0] = rr * ur + SR * (Us0 - rr);
        Fn[1] = (rr * ur * ur + pr) + SR * (Us1 - rr * ur);
        Fn[2] = rr * ur * wr + SR * (Us2 - rr * wr);
        Fn[3] = ur * (Er + pr) + SR * (Us3 - Er);
    } else {
        Fn[0] = rr * ur; Fn[1] = rr * ur * ur + pr; Fn[2] = rr * ur * wr; Fn[3] = ur * (Er + pr);
    }
    F[0] = Fn[0];
    F[1] = Fn[1] * nx - Fn[2] * ny;
    F[2] = Fn[1] * ny + Fn[2] * nx;
    F[3] = Fn[3];
    return ok;
}

// HLLC through a wall, i.e. against the mirror image of the inside state:
// the Roe-averaged normal velocity and the contact speed are zero, so the
// flux is the star pressure on the normal, p* = p + rho u_n (u_n - S_L),
// with S_L = min(u_n - c, -c~) and c~^2 = (gamma - 1)(H - w^2 / 2).  Written
// out, the mass and energy fluxes through the wall are exactly zero in
// either precision (the star-region formulas leave a rounding residue).
template <typename real>
__device__ __forceinline__ bool wall_flux(real g, const real *UL, real nx, real ny, real *F) {
    const real r = UL[0];
    const real ir = frcp(r);
    const real u = (UL[1] * nx + UL[2] * ny) * ir, w = (-UL[1] * ny + UL[2] * nx) * ir;
    const real E = UL[3];
    const real p = euler_pressure(g, r, UL[1], UL[2], E);
    const bool ok = r > 0 && p > 0;
    const real c = fsqrt((g * p) * ir);
    const real H = (E + p) * ir;
    const real ct = fsqrt((g - 1) * (H - (real)0.5 * w * w));
    const real SL = fmin(u - c, -ct);
    const real ps = r * (u - SL) * u + p;
    F[0] = 0;
    F[1] = ps * nx;
    F[2] = ps * ny;
    F[3] = 0;
    return ok;
}

template <typename real>
struct FluxArgs {
    int64_t N, Np;
    const real *FV;
    const real *fr;         // face records (nx, ny, |A|, code), vector-tiled
    const double *area;
    const double *Un, *Us;
    double *Uout;
    const double *dt_ptr;
    double dt_value;
    real *flux_out;
    double *resid;
    Ctrl *ctrl;             // time march: done flag and time (may be null)
    int *nonphys;           // set when a face state is non-physical (may be null)
    double *dt_part;
    real gamma, ax, ay;
    real gw[4];             // Gauss weights on [0, 1]
    double gamma64;
    int stage;
    // prescribed-state (inflow) boundary faces
    const double *bface;    // [n_inflow][4]: first vertex (x, y) and edge vector of each inflow face
    double bst[2][4];       // outside states behind / ahead of the moving line (conserved variables)
    double bline[3];        // the line x = bline[0] + bline[1] y + bline[2] t
    double gq[4];           // Gauss nodes on [0, 1]
    double t_base;          // time of the stage input when tctrl is null
    const Ctrl *tctrl;      // time march: the stage input's time is tctrl->t, its step *dt_ptr
    // fused stage (StageLists)
    const int2 *fdesc;      // per block its first listed face and their number
    const real *frec;       // records of the blocks' listed faces
    const uint32_t *xid;    // [Np] first side | the faces to other blocks << 28
    const int2 *xcells;     // cross cells and their xid
    const double *xarea;
    const real *xrec;       // [n_sides] side records
    real *xterm;            // [2 n_sides][NV] a cross cell's terms from faces inside its group, at its first side
    int64_t n_cross;
    int64_t part_off;       // the first kernel's minima in dt_part, behind the second kernel's
};

// the launch arguments of a flux / residual / RK stage (MODE f.mode)
template <typename real>
inline void fill_flux_args(const DeviceMesh &m, const FluxLaunch &f, FluxArgs<real> &a) {
    a = FluxArgs<real>{};
    a.N = m.N;
    a.Np = m.Np;
    a.FV = (const real *)f.FV;
    if constexpr (std::is_same<real, double>::value) a.fr = m.fr64;
    else a.fr = m.fr32;
    a.area = m.area;
    a.Un = f.Un; a.Us = f.Us; a.Uout = f.Uout;
    a.dt_ptr = f.dt_ptr; a.dt_value = f.dt_value;
    a.flux_out = (real *)f.flux_out;
    a.resid = f.resid;
    a.ctrl = f.ctrl;
    a.nonphys = f.nonphys ? f.nonphys : (f.ctrl ? &f.ctrl->nonphysical : nullptr);
    a.dt_part = f.dt_part;
    a.gamma = (real)m.gamma; a.ax = (real)m.ax; a.ay = (real)m.ay;
    a.gamma64 = m.gamma;
    a.stage = f.mode == 2 ? f.stage : 0;
    for (int q = 0; q < 4; ++q) a.gw[q] = q < m.tab.Nq ? (real)m.tab.gw[q] : (real)0;
    a.bface = m.bface;
    for (int k = 0; k < 2; ++k)
        for (int v = 0; v < 4; ++v) a.bst[k][v] = m.bst[k][v];
    for (int k = 0; k < 3; ++k) a.bline[k] = m.bline[k];
    for (int q = 0; q < 4; ++q) a.gq[q] = q < m.tab.Nq ? m.tab.gq[q] : 0.0;
    a.t_base = f.t_base;
    a.tctrl = f.ctrl && f.dt_ptr ? f.ctrl : nullptr;
    const StageLists &l = m.lists[std::is_same<real, float>::value ? 1 : 0];
    a.fdesc = l.fdesc;
    a.frec = (const real *)l.frec;
    a.xid = l.xid;
    a.xcells = l.xcells;
    a.n_cross = l.n_cross;
    a.xarea = l.xarea;
    a.xrec = (const real *)l.xrec;
    a.xterm = (real *)f.xterm;
    a.part_off = l.cross_blocks();     // (no cross cells: the first kernel's minima are the last)
}

template <int NV, int PHYS>
__device__ __forceinline__ double cell_dt_bound(const double *U, const double nrm[3][3], double area, double gamma,
                                                double ax, double ay) {
    double sum = 0.0;
    if (PHYS == CTENO_EULER) {
        const double rho = U[0], u = U[1] / rho, v = U[2] / rho;
        const double p = (gamma - 1.0) * (U[3] - 0.5 * rho * (u * u + v * v));
        const double c = sqrt(gamma * p / rho);
#pragma unroll
        for (int f = 0; f < 3; ++f) sum += nrm[f][2] * (fabs(u * nrm[f][0] + v * nrm[f][1]) + c);
    } else {
#pragma unroll
        for (int f = 0; f < 3; ++f) sum += nrm[f][2] * fabs(ax * nrm[f][0] + ay * nrm[f][1]);
    }
    return 2.0 * area / sum;
}

// minimum over the block (all threads call it; result valid in thread 0)
__device__ __forceinline__ double block_min(double v) {
    __shared__ double red[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    double r = INFINITY;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r = fmin(r, red[k]);
    return r;
}

// per-mesh arrays of one flux / residual / RK launch (constants stay in FluxArgs)
template <typename real>
struct FluxPtrs {
    const real *FV;
    const real *fr;
    const double *area;
    const double *Un, *Us;
    double *Uout;
    const double *dt_ptr;
    real *flux_out;
    double *resid;
    int *nonphys;           // set when a face state is non-physical (may be null)
    bool want_dt;
};

// Outside values of a boundary face at its Gauss points, oth[NQ-1-q]
// paired with ownf[q]: a prescribed (inflow) state on the Gauss point's side
// of the moving line at the stage time (t, t + dt, t + dt/2 for the three
// stages), or the inside state (transmissive).  Returns true for a wall of
// the Euler equations, whose flux comes in closed form from the inside state.
template <typename real, int NV, int PHYS, int MODE, int NQ>
__device__ __forceinline__ bool boundary_state(const FluxArgs<real> a, const double *dt_ptr, uint32_t code,
                                               const real (&ownf)[NQ][NV], real (&oth)[NQ][NV]) {
    const uint32_t kind = code & 3u;
    if (PHYS == CTENO_EULER && kind == CTENO_WALL) return true;
    if (kind == CTENO_INFLOW) {
        const double *e = a.bface + 4 * (int64_t)((code >> 2) & kNbInflowMask);
        const double t0 = a.tctrl ? a.tctrl->t : a.t_base;
        const double dts = MODE == 2 ? (dt_ptr ? *dt_ptr : a.dt_value) : 0.0;
        const double ts = t0 + (a.stage == 1 ? dts : a.stage == 2 ? 0.5 * dts : 0.0);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double px = e[0] + a.gq[q] * e[2], py = e[1] + a.gq[q] * e[3];
            const int side = px < a.bline[0] + a.bline[1] * py + a.bline[2] * ts ? 0 : 1;
#pragma unroll
            for (int v = 0; v < NV; ++v) oth[NQ - 1 - q][v] = (real)a.bst[side][v];
        }
    } else {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int v = 0; v < NV; ++v) oth[NQ - 1 - q][v] = ownf[q][v];
    }
    return false;
}

// boundary_state for one Gauss point g of local face f of cell i, in an RK
// stage: the inside state A, the outside state in B
template <typename real, int NV, int PHYS>
__device__ __forceinline__ bool boundary_point(const FluxArgs<real> a, double dt, int64_t i, int f, uint32_t kind,
                                               int g, const real (&A)[NV], real (&B)[NV]) {
    if (PHYS == CTENO_EULER && kind == CTENO_WALL) return true;
    if (kind == CTENO_INFLOW) {
        real nx, ny, len;
        uint32_t code;
        face_record<real>(a.fr, i, f, nx, ny, len, code);
        const double *e = a.bface + 4 * (int64_t)((code >> 2) & kNbInflowMask);
        const double t0 = a.tctrl ? a.tctrl->t : a.t_base;
        const double ts = t0 + (a.stage == 1 ? dt : a.stage == 2 ? 0.5 * dt : 0.0);
        const double gq = g ? a.gq[1] : a.gq[0];
        const double px = e[0] + gq * e[2], py = e[1] + gq * e[3];
        const bool behind = px < a.bline[0] + a.bline[1] * py + a.bline[2] * ts;
#pragma unroll
        for (int v = 0; v < NV; ++v) B[v] = (real)(behind ? a.bst[0][v] : a.bst[1][v]);
    } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) B[v] = A[v];
    }
    return false;
}

// A cell's outward flux through one face, |A| sum_q w_q F_q, with its sign.
// Both cells of a face evaluate F(owner side, other side; owner normal) at
// the owner's Gauss points in the owner's order, so the two terms are
// bitwise negatives of each other.
template <typename real, int NV, int PHYS, int NQ>
__device__ __forceinline__ void face_term(const FluxArgs<real> a, const real (&ownf)[NQ][NV],
                                          const real (&oth)[NQ][NV], bool owner, bool wallf, real nx, real ny,
                                          real len, double (&term)[NV], bool &bad) {
    const real fx = owner ? nx : -nx, fy = owner ? ny : -ny;
    real sumF[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) sumF[v] = 0;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        real A[NV], B[NV], F[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            A[v] = owner ? ownf[q][v] : oth[q][v];
            B[v] = owner ? oth[NQ - 1 - q][v] : ownf[NQ - 1 - q][v];
        }
        if (PHYS == CTENO_EULER) {
            if (wallf) bad |= !wall_flux<real>(a.gamma, A, fx, fy, F);
            else bad |= !hllc<real, std::is_same<real, float>::value ? 3 : -1>(a.gamma, A, B, fx, fy, F);
        } else {
            const real an = a.ax * fx + a.ay * fy;
            F[0] = an * (an >= 0 ? A[0] : B[0]);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) sumF[v] += a.gw[q] * F[v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const double val = (double)(len * sumF[v]);
        term[v] = owner ? val : -val;
    }
}

// SSP-RK3 stage value from U^n, the stage input and dt times the residual
__device__ __forceinline__ double rk_value(int stage, double u0, double us, double dtR) {
    if (stage == 0) return us + dtR;
    if (stage == 1) return 0.75 * u0 + 0.25 * (us + dtR);
    return (1.0 / 3.0) * u0 + (2.0 / 3.0) * (us + dtR);
}
// the weight of dt times the residual in rk_value
__device__ __forceinline__ double rk_weight(int stage) { return stage == 0 ? 1.0 : stage == 1 ? 0.25 : 2.0 / 3.0; }

}  // namespace cteno
