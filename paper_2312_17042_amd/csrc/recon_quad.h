// Reconstruction of degree 2 and 3, a quad of lanes per cell: the device body
// shared by the single-mesh, the fused-stage and the batched serving kernels.
//
// A stage streams a cell's pseudo-inverses (186 entries at degree 3) once and
// does little arithmetic with them, so it is bound by memory as long as
// enough of that stream is in flight and the vector units are not busy
// otherwise.  The products run on the matrix cores, one small matrix product
// per cell: rows are coefficients, columns the variables, the inner index the
// slots.  Their operands lie where the loads put them (a lane holds one row's
// entries, or one variable's differences), and the result has one lane per
// variable with all its coefficients, where selection and face values run: a
// dozen accumulators instead of sixty, so the whole stream of a cell is
// requested before the first product.  The 4 x 4 instructions add their terms
// with one rounding each, slot after slot, like a chain of fused operations.
#pragma once
#include "kernels_common.h"

namespace cteno {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename real> struct StreamVec;
template <> struct StreamVec<float> { using T = f32x4; };
template <> struct StreamVec<double> { using T = f64x2; };

// value of x in lane u of each group of four lanes (a quad), by a DPP move
template <int u>
__device__ __forceinline__ float quad_bcast(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), u * 0x55, 0xF, 0xF, false));
}
template <int u>
__device__ __forceinline__ double quad_bcast(double x) {
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xFFFFFFFFll), u * 0x55, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), u * 0x55, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
// quad_bcast of an integer; u must be a constant after unrolling
__device__ __forceinline__ int quad_bcast_dyn(int u, int x) {
    switch (u) {
        case 0: return __builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, false);
        case 1: return __builtin_amdgcn_mov_dpp(x, 0x55, 0xF, 0xF, false);
        case 2: return __builtin_amdgcn_mov_dpp(x, 0xAA, 0xF, 0xF, false);
        default: return __builtin_amdgcn_mov_dpp(x, 0xFF, 0xF, 0xF, false);
    }
}
// the value of the other lane of each pair (0 <-> 1, 2 <-> 3)
__device__ __forceinline__ float pair_swap(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ double pair_swap(double x) {
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xFFFFFFFFll), 0xB1, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
// the value that lane `owner` of the quad holds in x[v] for the calling lane's v
template <int owner, typename real>
__device__ __forceinline__ real quad_take(const real (&x)[4], int v) {
    const real x0 = quad_bcast<owner>(x[0]), x1 = quad_bcast<owner>(x[1]);
    const real x2 = quad_bcast<owner>(x[2]), x3 = quad_bcast<owner>(x[3]);
    return v == 0 ? x0 : v == 1 ? x1 : v == 2 ? x2 : x3;
}
template <int owner, typename real>
__device__ __forceinline__ real quad_take(const real (&x)[1], int) { return quad_bcast<owner>(x[0]); }

// the state of the quad's cell in every lane
template <int NV>
__device__ __forceinline__ void quad_state(double un, double (&u)[NV]) {
    u[0] = quad_bcast<0>(un);
    if constexpr (NV == 4) {
        u[1] = quad_bcast<1>(un);
        u[2] = quad_bcast<2>(un);
        u[3] = quad_bcast<3>(un);
    }
}

// Transposes x[s] over the register index s and the lane's row of sixteen
// lanes i: afterwards x[i] holds, in row s, what x[s] held in row i.
__device__ __forceinline__ void rows_to_lanes(double (&x)[4]) {
    uint32_t h[2][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, x[s]);
        h[0][s] = (uint32_t)b;
        h[1][s] = (uint32_t)(b >> 32);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const auto y = __builtin_amdgcn_permlane32_swap(h[p][s], h[p][s + 2], false, false);
            h[p][s] = y[0];
            h[p][s + 2] = y[1];
        }
#pragma unroll
        for (int s = 0; s < 4; s += 2) {
            const auto y = __builtin_amdgcn_permlane16_swap(h[p][s], h[p][s + 1], false, false);
            h[p][s] = y[0];
            h[p][s + 1] = y[1];
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
        x[s] = __builtin_bit_cast(double, ((unsigned long long)h[1][s] << 32) | (unsigned long long)h[0][s]);
}

// a + b with both rounded: not contracted with the product that one of them is
template <typename real>
__device__ __forceinline__ real rounded_sum(real a, real b) {
#pragma clang fp contract(off)
    return a + b;
}

// constants of one reconstruction
template <typename real>
struct ReconArgs {
    const real *tab;        // device table: Gram matrix [K][K], face basis [3][2][K]
    real lam1, ct, eps;
    real lams[5];           // lambda_s for s_t = 2, 3, 4 (index s_t)
    real gamma;             // ratio of specific heats (positivity check)
    real lam_ratio[5];      // lambda_1 / lambda_s (index s_t)
    int positivity;         // 1: cell-average fallback for non-physical face states
    // entry k of the table, through the constant address space: a scalar load
    // also behind stores and barriers (as a vector load it would wait for the
    // stream that is in flight)
    __device__ __forceinline__ real entry(int k) const {
        return ((const __attribute__((address_space(4))) real *)tab)[k];
    }
};

// arrays of one mesh and state
template <typename real>
struct ReconPtrs {
    const double *U;        // AoS [Np][NV]
    const uint16_t *lslot;  // stencil entries as rows of the group (lslot_index)
    const int2 *desc;       // per group: first place in hlist, length
    const int32_t *hlist;   // the cells outside a group that its stencils reach
    const uint8_t *flags;   // [Np]
    const real *P;          // pseudo-inverse stream (quad_index)
    uint8_t *delta;         // AoS [Np][NV] (characteristic variables: [Np][3][NV])
    const real *fr;         // face records (characteristic variables only)
    unsigned long long *fb; // cells that took the positivity fallback (may be null)
    const int *done;        // the march's end (may be null)
};

// The lane's field (a conserved variable, or a characteristic field on one
// face): selection or CWENO weights, and the final coefficients in place in
// c1[K] (p_1 on entry); cd[3][2] the degree-1 directional coefficients.  VARS
// only decides which product of a directional indicator is rounded in FP32 (a
// march repeats its results only if that stays).
template <typename real, int K, int SCHEME, int GFORM, int DMODE, int VARS>
__device__ __forceinline__ int finish_field(const ReconArgs<real> a, real (&c1)[K], const real (&cd)[3][2], int fl,
                                            int adm, int st, real lams, real lratio, int forced) {
    int bits;
    if (DMODE == 2 && SCHEME != CTENO_SCHEME_CWENO) {
        bits = forced & adm;
    } else if (st == 1) {
        bits = 1;
    } else {
        // smoothness indicators: SI_1 = a1^T G a1, SI_s over the degree-1 block
        // of G.  FP64 sums the full quadratic form; FP32 its upper triangle,
        // whose off-diagonal entries the FP32 table holds doubled, at about
        // half the products.
        constexpr bool SYM = std::is_same<real, float>::value;
        real si[4];
        si[0] = 0;
#pragma unroll
        for (int p = 0; p < K; ++p) {
            real rp = 0;
#pragma unroll
            for (int q = SYM ? p : 0; q < K; ++q) rp += a.entry(p * K + q) * c1[q];
            si[0] += c1[p] * rp;
        }
        const real g00 = a.entry(0), g01 = a.entry(1), g10 = a.entry(K), g11 = a.entry(K + 1);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const real x0 = cd[q][0], x1 = cd[q][1];
            if constexpr (SYM && VARS) si[q + 1] = __builtin_fmaf(g11, x1 * x1, x0 * (g00 * x0 + g01 * x1));
            else if constexpr (SYM) si[q + 1] = x0 * (g00 * x0 + g01 * x1) + g11 * (x1 * x1);
            else si[q + 1] = x0 * (g00 * x0 + g01 * x1) + x1 * (g10 * x0 + g11 * x1);
        }
        if constexpr (SCHEME == CTENO_SCHEME_CWENO) {
            // every admissible stencil contributes: sum_s omega_s p_s, in place
            bits = adm;
            real w[4];
            cweno_weights<real>(si, adm, lams, a.lam1, lratio, a.eps, w);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                real x = w[0] * c1[k];
                if (k < 2) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if ((fl >> q) & 1) x += w[q + 1] * cd[q][k];
                }
                c1[k] = x;
            }
        } else {
            constexpr int SEL = SCHEME == CTENO_SCHEME_TENO ? CTENO_SCHEME_CTENO : SCHEME;
            constexpr int SGF = SCHEME == CTENO_SCHEME_TENO ? CTENO_GAMMA_PAPER : GFORM;
            bits = teno_bits<real, SEL, SGF>(si, adm, st, a.lam1, lams, lratio, a.ct, a.eps);
        }
    }
    // final coefficients: p_1, or the mean of the selected directional polynomials
    if (SCHEME != CTENO_SCHEME_CWENO && !(bits & 1)) {
        real s0 = 0, s1 = 0;
        int cnt = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if ((bits >> (q + 1)) & 1) { s0 += cd[q][0]; s1 += cd[q][1]; ++cnt; }
        c1[0] = cnt == 1 ? s0 : cnt == 2 ? (real)0.5 * s0 : fdiv(s0, (real)3);
        c1[1] = cnt == 1 ? s1 : cnt == 2 ? (real)0.5 * s1 : fdiv(s1, (real)3);
#pragma unroll
        for (int k = 2; k < K; ++k) c1[k] = 0;
    }
    return bits;
}

// The averages that the stencils of a group of 64 cells reach -- its own
// cells, then its listed neighbours -- go to LDS, one row of NV per cell.  A
// stencil entry is a row number: gathers of single averages from global
// memory took two of three slots of the address unit.
template <int NV>
struct GroupRows {
    static constexpr int RL = 256 / NV;   // rows that the group's threads write at once
    // the list's first HS shares are requested at once (NV = 4: 192 cells; the
    // usual list at degree 3 has 100, at most 135 in Morton order)
    static constexpr int HS = NV == 4 ? 3 : 1;
    int hid[HS];
    double hu[HS];
    // the threads' places in the list, t of the group's 256 (a place past the
    // list reads its first entry, or the pad)
    __device__ __forceinline__ static int place(int t) { return NV == 4 ? t >> 2 : t; }
    __device__ __forceinline__ void list(const int32_t *hlist, int2 desc, int t) {
        const int r = place(t);
#pragma unroll
        for (int k = 0; k < HS; ++k) hid[k] = hlist[desc.x + (r + k * RL < desc.y ? r + k * RL : 0)];
    }
    __device__ __forceinline__ void averages(const double *U, int v) {
#pragma unroll
        for (int k = 0; k < HS; ++k) hu[k] = U[(int64_t)hid[k] * NV + v];
    }
    __device__ __forceinline__ void store(double *rows, const double *U, const int32_t *hlist, int2 desc, int t, int v,
                                          double own) const {
        const int r0 = place(t);
        if (NV == 4 || (t & 3) == 0) rows[(t >> 2) * NV + v] = own;
#pragma unroll
        for (int k = 0; k < HS; ++k)
            if (r0 + k * RL < desc.y) rows[(64 + r0 + k * RL) * NV + v] = hu[k];
        for (int r = r0 + HS * RL; r < desc.y; r += RL)
            rows[(64 + r) * NV + v] = U[(int64_t)hlist[desc.x + r] * NV + v];
    }
};

struct RowIds3 { uint32_t w[3]; };
struct RowIds2 { uint32_t w[2]; };
template <int R> struct RowIds;
template <> struct RowIds<3> { using T = RowIds3; };
template <> struct RowIds<2> { using T = RowIds2; };

// a vector of the stream: nontemporal, or kept by the caches (stream_nontemporal)
template <bool NT, typename V>
__device__ __forceinline__ V stream_load(const V *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// A lane's share of its tile's row numbers and stream (16 cells, one wave).
// Lanes without an entry read another one's: no more bytes, and what they hold
// meets unused rows of the result or zero differences.
template <typename real, int R, bool NT> struct QuadStream;

template <int R, bool NT>
struct QuadStream<float, R, NT> {
    using D = QuadDims<R>;
    static constexpr int S = D::S, MA = D::MA, NAV = S * MA / 4;
    typename RowIds<R>::T ids;            // of slots q, q + 4, ... of the lane's cell
    f32x4 bA[NAV], bB[4];
    f32x2 tl;
    __device__ __forceinline__ void request_ids(const uint16_t *lslot, int64_t tile, int lane) {
        ids = reinterpret_cast<const typename RowIds<R>::T *>(lslot)[tile * 64 + lane];
    }
    __device__ __forceinline__ void request(const float *P, int64_t tile, int lane) {
        const float *__restrict__ Pt = P + (size_t)tile * (D::E * 16);
        auto ldv = [&](int off) { return stream_load<NT>(reinterpret_cast<const f32x4 *>(Pt + off)); };
        const int q = lane & 3, c16 = lane >> 2, o2 = q < 2 ? q : 2;
        constexpr int B0 = S * MA * 64;
        // in the order of their use, so that the products start with the first
#pragma unroll
        for (int g = 0; g < (S + 3) / 4; ++g) {
#pragma unroll
            for (int m = 0; m < MA; ++m)
                if (g * MA + m < NAV) bA[g * MA + m] = ldv(((g * MA + m) * 64 + lane) * 4);
            if (g < 3) bB[g] = ldv(B0 + ((g * 16 + c16) * 3 + o2) * 4);
            if (g == 3) bB[3] = ldv(B0 + 576 + c16 * 4);
            if (g == 4) tl = stream_load<NT>(reinterpret_cast<const f32x2 *>(Pt + B0 + 640 + c16 * 2));
        }
    }
    template <int NV>
    __device__ __forceinline__ void products(const float *, int64_t, const double *rows, int, int v, double U0,
                                             float (&ao)[D::K], float (&ad)[3][2]) {
        const char *rv = reinterpret_cast<const char *>(rows) + v * 8;
        f32x4 a[MA], x = {0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < MA; ++m) a[m] = f32x4{0, 0, 0, 0};
        // averages come from LDS three slots ahead of their products (six would
        // spill at five waves per SIMD)
        constexpr int LB = 3;
        static_assert(S % LB == 0, "slots in batches");
        double u[2][LB];
        auto fetch = [&](int b) {
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                const int j = b * LB + k;
                const uint32_t w = (uint32_t)quad_bcast_dyn(j & 3, (int)ids.w[j / 8]);
                u[b & 1][k] = *reinterpret_cast<const double *>(rv + ((j >> 2) & 1 ? w >> 16 : w & 0xFFFFu) * (NV * 8));
            }
        };
        fetch(0);
#pragma unroll
        for (int b = 0; b < S / LB; ++b) {
            if (b + 1 < S / LB) fetch(b + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                const int j = b * LB + k;
                const float d = (float)(u[b & 1][k] - U0);
#pragma unroll
                for (int m = 0; m < MA; ++m) {
                    const int p = j * MA + m;
                    a[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(bA[p / 4][p % 4], d, a[m], 0, 0, 0);
                }
                const float pb = j < 16 ? bB[j / 4 < 4 ? j / 4 : 0][j % 4] : tl[j & 1];
                x = __builtin_amdgcn_mfma_f32_4x4x1f32(pb, d, x, 0, 0, 0);
                if (j < 12 && j % 4 == 3) {   // directional group j / 4 is complete
                    ad[j / 4][0] = x[1];
                    ad[j / 4][1] = x[2];
                    x = f32x4{x[0], 0, 0, 0};
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int c = 0; c < 4; ++c) ao[4 * m + c] = a[m][c];
        ao[4 * MA] = x[0];
    }
};

template <int R, bool NT>
struct QuadStream<double, R, NT> {
    using D = QuadDims<R>;
    static constexpr int MA = D::MA, G = D::G;
    // the four quarters of the tile's cells; two of them are requested at once,
    // the others when a quarter's products have freed its registers.  At four
    // waves per SIMD this streams faster than all four quarters at three (k_stage,
    // 2M cells: 654 against 679 us; three quarters at three waves 690).
    static constexpr int NPRE = 2;
    typename RowIds<R>::T ids[4];         // of slots k, k + 4, ... (k = lane / 16) of cells 4 s + b (b = lane / 4 % 4)
    f64x2 dA[4][5], dB[4];
    double dA2[4], dB2[4], dB3[4], dB4[4];
    __device__ __forceinline__ void request_ids(const uint16_t *lslot, int64_t tile, int lane) {
        const auto *Sv = reinterpret_cast<const typename RowIds<R>::T *>(lslot) + tile * 64;
#pragma unroll
        for (int s = 0; s < 4; ++s) ids[s] = Sv[(4 * s + ((lane >> 2) & 3)) * 4 + (lane >> 4)];
    }
    __device__ __forceinline__ void quarter(const double *P, int64_t tile, int lane, int s) {
        const double *__restrict__ Pt = P + (size_t)tile * (D::E * 16) + s * (D::E * 4);
        auto ldv = [&](int off) { return stream_load<NT>(reinterpret_cast<const f64x2 *>(Pt + off)); };
        auto ld1 = [&](int off) { return stream_load<NT>(Pt + off); };
        const int q = lane & 3, kb = lane >> 2, o2 = q < 2 ? q : 2;
        constexpr int B0 = R == 3 ? 576 : 192;
        if constexpr (R == 3) {
#pragma unroll
            for (int g = 0; g < 4; ++g) dA[s][g] = ldv(g * 128 + lane * 2);
            dA[s][4] = ldv(512 + (lane & 31) * 2);
        } else {
            dA[s][0] = ldv(lane * 2);
            dA2[s] = ld1(128 + lane);
        }
        dB[s] = ldv(B0 + (kb * 3 + o2) * 2);
        dB2[s] = ld1(B0 + 96 + kb * 3 + o2);
        if constexpr (R == 3) {
            dB3[s] = ld1(B0 + 144 + kb);
            dB4[s] = ld1(B0 + 160 + (kb & 7));
        }
    }
    __device__ __forceinline__ void request(const double *P, int64_t tile, int lane) {
#pragma unroll
        for (int s = 0; s < NPRE; ++s) quarter(P, tile, lane, s);
    }
    template <int NV>
    __device__ __forceinline__ void products(const double *P, int64_t tile, const double *rows, int lane, int v, double,
                                             double (&ao)[D::K], double (&ad)[3][2]) {
        const char *rv = reinterpret_cast<const char *>(rows) + v * 8;
        // per s: full groups a[m], last group x[g] (row 0 runs on over g, rows
        // 1 and 2 are group g's directional coefficients)
        double a[MA][4], x[4][4];
        const bool row0lane = lane < 16;  // the lanes that hold row 0 of a result
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double u0 = rows[((int)(tile & 3) * 16 + 4 * s + ((lane >> 2) & 3)) * NV + v];
            double ug[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint32_t w = ids[s].w[g / 2];
                ug[g] = *reinterpret_cast<const double *>(rv + (g & 1 ? w >> 16 : w & 0xFFFFu) * (NV * 8));
            }
            double am[MA], xg = 0.0;
#pragma unroll
            for (int m = 0; m < MA; ++m) am[m] = 0.0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const double d = ug[g] - u0;
#pragma unroll
                for (int m = 0; m < MA; ++m) {
                    const double p = R == 3 ? dA[s][g < 5 ? g : 0][m] : (g < 2 ? dA[s][0][g & 1] : dA2[s]);
                    am[m] = __builtin_amdgcn_mfma_f64_4x4x4f64(p, d, am[m], 0, 0, 0);
                }
                const double pb = g < 2 ? dB[s][g & 1] : g == 2 ? dB2[s] : g == 3 ? dB3[s] : dB4[s];
                xg = __builtin_amdgcn_mfma_f64_4x4x4f64(pb, d, xg, 0, 0, 0);
                if (g < 3) {
                    x[g][s] = xg;
                    if (g < 2 || G > 3) xg = row0lane ? xg : 0.0;
                }
            }
            x[3][s] = xg;
#pragma unroll
            for (int m = 0; m < MA; ++m) a[m][s] = am[m];
            if (s + NPRE < 4) {
                __builtin_amdgcn_sched_barrier(0);
                quarter(P, tile, lane, s + NPRE);
            }
        }
        // results have lane 16 i + 4 b + v for row i of cell 4 s + b: swap s and
        // i, so that the lanes of cell 4 s + b hold its rows
#pragma unroll
        for (int m = 0; m < MA; ++m) {
            rows_to_lanes(a[m]);
#pragma unroll
            for (int c = 0; c < 4; ++c) ao[4 * m + c] = a[m][c];
        }
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            rows_to_lanes(x[g]);
            ad[g][0] = x[g][1];
            ad[g][1] = x[g][2];
        }
        rows_to_lanes(x[3]);
        ao[4 * MA] = x[3][0];
    }
};

// Central and directional coefficients of the lane's variable v, ao = P_c d
// and ad = P_s d.  il: the cell (below Np), t: the thread in its group's 256;
// U0: the cell's own average of variable v.  False (the same for the whole
// grid) when *done is set: the march is over; the flag is waited for together
// with the descriptor, before anything else is requested.  Holds a block
// barrier.
// Everything that is not the neighbours' averages is requested before the
// first wait; what the group's descriptor leads to (list, then averages) is
// the only chain.
template <typename real, int R, int NV, bool NT>
__device__ __forceinline__ bool quad_contract(const ReconPtrs<real> ptr, double *rows, int64_t il, int t, double &U0,
                                              int &fl, real (&ao)[QuadDims<R>::K], real (&ad)[3][2]) {
    const int lane = t & 63, v = NV == 4 ? t & 3 : 0;
    const int2 desc = ptr.desc[__builtin_amdgcn_readfirstlane((int)(il >> 6))];
    // (one wait for both: without a march the flag's place is the descriptors')
    const int stop = *(ptr.done ? ptr.done : &ptr.desc->x);
    if (ptr.done && stop) return false;
    const int64_t tile = __builtin_amdgcn_readfirstlane((int)(il >> 4));
    GroupRows<NV> gr;
    QuadStream<real, R, NT> qs;
    gr.list(ptr.hlist, desc, t);
    U0 = ptr.U[il * NV + v];
    fl = ptr.flags[il] & 7;
    qs.request_ids(ptr.lslot, tile, lane);
    qs.request(ptr.P, tile, lane);
    __builtin_amdgcn_sched_barrier(0);
    gr.averages(ptr.U, v);
    gr.store(rows, ptr.U, ptr.hlist, desc, t, v, U0);
    __syncthreads();
    qs.template products<NV>(ptr.P, tile, rows, lane, v, U0, ao, ad);
    return true;
}

// From the coefficients to the face Gauss-point values of the lane's variable v
// in out (NV = 1: of the one variable, in every lane), and the cell's selection
// bytes (DMODE 1).  live: the cell exists (padding cells of the last wave compute
// on padding data and report nothing).
template <typename real, int R, int NV, int SCHEME, int GFORM, int DMODE, int VARS>
__device__ __forceinline__ void recon_finish(const ReconArgs<real> a, const ReconPtrs<real> ptr, int64_t il, int q,
                                             bool live, double U0, int fl, real (&ao)[QuadDims<R>::K],
                                             real (&ad)[3][2], real (&out)[3][2]) {
    constexpr int K = QuadDims<R>::K;
    const int v = NV == 4 ? q : 0;
    const int adm = 1 | (fl << 1);
    const int st = 1 + __popc(fl);
    // static indices only: a dynamic index into the argument struct would
    // force it into scratch memory
    const real lams = st == 2 ? a.lams[2] : (st == 3 ? a.lams[3] : a.lams[4]);
    const real lratio = st == 2 ? a.lam_ratio[2] : (st == 3 ? a.lam_ratio[3] : a.lam_ratio[4]);
    // p_1 = (p_opt - sum_s lambda_s p_s) / lambda_1, in place of a_opt, with
    // one reciprocal of lambda_1; TENO keeps the central stencil's own polynomial
    const real ilam1 = frcp(a.lam1);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        real sm = ao[k];
        if (k < 2 && st > 1) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
                if ((fl >> s) & 1) sm -= lams * ad[s][k];
        }
        if (SCHEME != CTENO_SCHEME_TENO) ao[k] = st > 1 ? sm * ilam1 : sm;
    }
    constexpr int NB = VARS ? 3 : 1;      // selection bytes of this lane
    int dbyte[NB];
    if constexpr (VARS == 0) {
        dbyte[0] = finish_field<real, K, SCHEME, GFORM, DMODE, VARS>(a, ao, ad, fl, adm, st, lams, lratio,
                                                               DMODE == 2 ? ptr.delta[il * NV + v] : 0);
        // face Gauss-point values
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                real val = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) val += a.entry(K * K + (f * 2 + g) * K + k) * ao[k];
                out[f][g] = (real)(U0 + (double)val);
            }
    } else {
        // characteristic fields per face, lane v reconstructs field v: the
        // least-squares coefficients are linear in the data, so projecting
        // them with L_f equals reconstructing the projected averages W = L_f
        // U; the face values are U_0 + R_f (W(x_q) - W_0)
        static_assert(NV == 4, "characteristic variables need the Euler equations");
        const double Ud[4] = {quad_bcast<0>(U0), quad_bcast<1>(U0), quad_bcast<2>(U0), quad_bcast<3>(U0)};
        const real rho = (real)Ud[0], uu = (real)(Ud[1] / Ud[0]), vv = (real)(Ud[2] / Ud[0]);
        const real q2 = (real)0.5 * (uu * uu + vv * vv);
        const real pr = (a.gamma - 1) * ((real)Ud[3] - rho * q2);
        const real cs = fsqrt(fdiv(a.gamma * pr, rho)), H = fdiv(rounded_sum((real)Ud[3], pr), rho);
        const real b1 = fdiv(a.gamma - 1, cs * cs), b2 = b1 * q2, ic = frcp(cs);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            real nx, ny, len;
            uint32_t code;
            face_record<real>(ptr.fr, il, f, nx, ny, len, code);
            const real un = uu * nx + vv * ny, ut = -uu * ny + vv * nx;
            real Lr[4], Rr[4];      // row v of L_f and of R_f
            if (v == 0) {
                Lr[0] = (real)0.5 * (b2 + un * ic); Lr[1] = (real)-0.5 * (b1 * uu + nx * ic);
                Lr[2] = (real)-0.5 * (b1 * vv + ny * ic); Lr[3] = (real)0.5 * b1;
                Rr[0] = 1; Rr[1] = 1; Rr[2] = 0; Rr[3] = 1;
            } else if (v == 1) {
                Lr[0] = 1 - b2; Lr[1] = b1 * uu; Lr[2] = b1 * vv; Lr[3] = -b1;
                Rr[0] = uu - cs * nx; Rr[1] = uu; Rr[2] = -ny; Rr[3] = uu + cs * nx;
            } else if (v == 2) {
                Lr[0] = -ut; Lr[1] = -ny; Lr[2] = nx; Lr[3] = 0;
                Rr[0] = vv - cs * ny; Rr[1] = vv; Rr[2] = nx; Rr[3] = vv + cs * ny;
            } else {
                Lr[0] = (real)0.5 * (b2 - un * ic); Lr[1] = (real)-0.5 * (b1 * uu - nx * ic);
                Lr[2] = (real)-0.5 * (b1 * vv - ny * ic); Lr[3] = (real)0.5 * b1;
                Rr[0] = H - un * cs; Rr[1] = q2; Rr[2] = ut; Rr[3] = H + un * cs;
            }
            auto project = [&](real x) -> real {
                real y = 0;
                y += Lr[0] * quad_bcast<0>(x);
                y += Lr[1] * quad_bcast<1>(x);
                y += Lr[2] * quad_bcast<2>(x);
                y += Lr[3] * quad_bcast<3>(x);
                return y;
            };
            real c1[K], cd[3][2];
#pragma unroll
            for (int k = 0; k < K; ++k) c1[k] = project(ao[k]);
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int k = 0; k < 2; ++k) cd[s][k] = project(ad[s][k]);
            dbyte[f] = finish_field<real, K, SCHEME, GFORM, DMODE, VARS>(
                a, c1, cd, fl, adm, st, lams, lratio, DMODE == 2 ? ptr.delta[(il * 3 + f) * NV + v] : 0);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                real w = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) w += a.entry(K * K + (f * 2 + g) * K + k) * c1[k];
                real x = 0;
                x += Rr[0] * quad_bcast<0>(w);
                x += Rr[1] * quad_bcast<1>(w);
                x += Rr[2] * quad_bcast<2>(w);
                x += Rr[3] * quad_bcast<3>(w);
                out[f][g] = (real)(U0 + (double)x);
            }
        }
    }
    if constexpr (NV == 4) if (a.positivity) {
        // optional positivity fallback (not in the paper): a cell with a
        // non-physical state (density or pressure <= 0) at any of its Gauss
        // points uses its cell average at all of them; reported with bit 7
        // of its selection bytes and counted.  Without it the flux reports
        // the state.
        bool bad = false;
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const real r0 = quad_bcast<0>(out[f][g]), r1 = quad_bcast<1>(out[f][g]);
                const real r2 = quad_bcast<2>(out[f][g]), r3 = quad_bcast<3>(out[f][g]);
                const real pr = euler_pressure(a.gamma, r0, r1, r2, r3);
                bad |= !(r0 > 0) || !(pr > 0);
            }
        if (bad && live) {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int g = 0; g < 2; ++g) out[f][g] = (real)U0;
#pragma unroll
            for (int k = 0; k < NB; ++k) dbyte[k] |= 0x80;
            if (v == 0 && ptr.fb) atomicAdd(ptr.fb, 1ull);
        }
    }
    if (DMODE == 1 && live && q < NV) {
        if constexpr (VARS == 0) ptr.delta[il * NV + v] = (uint8_t)dbyte[0];
        else {
#pragma unroll
            for (int f = 0; f < 3; ++f) ptr.delta[(il * 3 + f) * NV + v] = (uint8_t)dbyte[f];
        }
    }
}

// Reconstruction of cell il by its quad (thread t of its group's 256; rows:
// the group's LDS rows).  mid() runs after the products, when the stream's
// registers are free: the caller's loads for what follows, which the
// selection's arithmetic then covers.  False when the march is over (out is
// not set).
template <typename real, int R, int NV, int SCHEME, int GFORM, int DMODE, int VARS, bool NT, class Mid>
__device__ __forceinline__ bool recon_quad(const ReconArgs<real> a, const ReconPtrs<real> ptr, double *rows,
                                           int64_t il, int t, bool live, Mid &&mid, double &U0,
                                           real (&out)[3][2]) {
    real ao[QuadDims<R>::K], ad[3][2];
    int fl;
    if (!quad_contract<real, R, NV, NT>(ptr, rows, il, t, U0, fl, ao, ad)) return false;
    mid();
    recon_finish<real, R, NV, SCHEME, GFORM, DMODE, VARS>(a, ptr, il, t & 3, live, U0, fl, ao, ad, out);
    return true;
}

// scheme constants of the reconstruction (linear weights of eq. e18 for every
// admissible-stencil count); the tables are on the device
template <typename real>
inline void fill_recon_constants(const DeviceMesh &m, ReconArgs<real> &a) {
    if constexpr (std::is_same<real, double>::value) a.tab = m.htab64;
    else a.tab = m.htab32;
    const double lam1 = 1.0 - 1.0 / m.lam1p;
    a.lam1 = (real)lam1;
    a.gamma = (real)m.gamma;
    a.ct = (real)m.ct;
    a.eps = (real)m.eps;
    a.positivity = m.positivity;
    for (int s = 0; s < 5; ++s) {
        const double ls = s >= 2 ? (1.0 - lam1) / (s - 1) : 0.0;
        a.lams[s] = (real)ls;
        a.lam_ratio[s] = s >= 2 ? (real)(lam1 / ls) : (real)1;
    }
}

}  // namespace cteno
