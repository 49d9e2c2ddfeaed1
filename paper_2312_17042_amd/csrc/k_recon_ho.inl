// Reconstruction of degree 4 to 6 (orders 5 to 7) for one arithmetic type;
// instantiated per type by k_recon_ho_f32.hip and k_recon_ho_f64.hip.
//
// A cell streams 532 (degree 4) to 1944 (degree 6) pseudo-inverse entries, which
// bounds the kernel as long as enough of them are in flight.  For the Euler
// equations the products run on the matrix cores as at degree 3 (recon_quad.h):
// rows are coefficients, columns the variables, the inner index the slots, each
// sum taken slot after slot with one rounding a term.  Against vector sums of
// four variables a lane, with two slots in flight: FP32, 500k cells of degree 6
// 870 -> 726 us (3.9 GB, 5.4 TB/s), 7k cells 42 -> 23 us; FP64, 215k cells of
// degree 4 224 -> 176 us (1.0 GB, 5.7 TB/s), 9.5k cells of degree 5 42 -> 21 us.
// One variable keeps a lane per cell.
#pragma once
#include "recon_quad.h"

namespace cteno {

template <typename real>
struct ReconHoArgs {
    int64_t N;
    const double *U;
    const int32_t *slot;
    const uint8_t *flags;
    const real *P;
    real *FV;                // AoS [Np][3][N_q][nv]
    uint8_t *delta;
    const int *done;
    const real *tab;
    const real *fr;          // face records (characteristic variables)
    real lams[5], lam_ratio[5];
    real lam1, ct, eps, gamma;
    int positivity;          // 1: cell-average fallback for non-physical face states
    unsigned long long *fb_count;   // cells that took the fallback (may be null)
    // the p_1 step's factors: (p_opt - p1_ls sum_s lambda_s p_s) / p1_l1,
    // (1, lambda_1) for the CTENO family, (0, 1) for TENO, which keeps p_opt
    real p1_ls, p1_l1;
    __device__ __forceinline__ real entry(int k) const {
        return ((const __attribute__((address_space(4))) real *)tab)[k];
    }
};

// one lane's field (a conserved variable, or a characteristic field on one
// face): selection or CWENO weights and the final coefficients, in place in
// c1[K] (p_1 on entry); cd[3][K_d] the directional coefficients
template <typename real, int K, int KD, int SCHEME, int GFORM, int DMODE>
__device__ __forceinline__ int finish_field_ho(const ReconHoArgs<real> a, real (&c1)[K], const real (&cd)[3][KD],
                                               int fl, int adm, int st, real lams, real lratio, int forced) {
    int bits;
    if (DMODE == 2 && SCHEME != CTENO_SCHEME_CWENO) {
        bits = forced & adm;
    } else if (st == 1) {
        bits = 1;
    } else {
        real si[4];
        si[0] = 0;
#pragma unroll
        for (int p = 0; p < K; ++p) {
            real rp = 0;
#pragma unroll
            for (int q = 0; q < K; ++q) rp += a.entry(p * K + q) * c1[q];
            si[0] += c1[p] * rp;
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            real sv = 0;
#pragma unroll
            for (int p = 0; p < KD; ++p) {
                real rp = 0;
#pragma unroll
                for (int q = 0; q < KD; ++q) rp += a.entry(p * K + q) * cd[s][q];
                sv += cd[s][p] * rp;
            }
            si[s + 1] = sv;
        }
        if constexpr (SCHEME == CTENO_SCHEME_CWENO) {
            // every admissible stencil contributes: sum_s omega_s p_s, in place
            bits = adm;
            real w[4];
            cweno_weights<real>(si, adm, lams, a.lam1, lratio, a.eps, w);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                real x = w[0] * c1[k];
                if (k < KD) {
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
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) c1[k] = 0;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if ((bits >> (q + 1)) & 1) {
                ++cnt;
#pragma unroll
                for (int k = 0; k < KD; ++k) c1[k] += cd[q][k];
            }
#pragma unroll
        for (int k = 0; k < KD; ++k) c1[k] = fdiv(c1[k], (real)cnt);
    }
    return bits;
}

// Row groups of a slot: NC hold central coefficients, those from D0 on
// directional ones (degree 4 and 6: group NC - 1 = D0 holds both).
template <int R>
struct HoGroups {
    using D = HoRows<R>;
    static constexpr int M = D::NF + (D::REM > 0);        // all
    static constexpr int NC = (D::K + 3) / 4, D0 = D::K / 4, ND = M - D0;
    static constexpr bool MIXED = D0 < NC;
};

// With variable groups (degrees 4 and 5) each directional row keeps three sums:
// a slot's products enter the sum of the stencil that its entry names, and with
// zero differences the other two.  These are the slot's differences for the
// three (a difference that is not finite stays so in all of them).
template <typename real>
__device__ __forceinline__ void ho_split(real d, uint32_t group, real (&ds)[3]) {
    const real z = d * 0;
#pragma unroll
    for (int s = 0; s < 3; ++s) ds[s] = group == (uint32_t)s ? d : z;
}

// FP32: a_opt = P_c d and a_s = P_s d of the lane's cell and variable, 16 cells
// per wave.  The row groups' results have a lane per variable with four
// coefficients each.  Two groups of slots are in flight ahead of the products (18
// KB a wave at degree 6); 160 to 220 registers, two or three waves per SIMD:
// held to three, degree 6 spills (726 -> 784 us, to four 1206).
template <int R>
__device__ __forceinline__ void ho_contract(const ReconHoArgs<float> a, int64_t i, int lane, double U0,
                                            float (&ao)[HoDims<R>::K], float (&ad)[3][HoDims<R>::KD]) {
    using D = HoRows<R>;
    using H = HoGroups<R>;
    constexpr int K = D::K, KD = D::C - K, NF = D::NF, REM = D::REM, G = D::G, MD = HoDims<R>::MD;
    constexpr bool VARG = HoDims<R>::VARG;
    constexpr int L = 2, NB = L + 1;
    const int q = lane & 3, c16 = lane >> 2;
    const float *__restrict__ Pt = a.P + (size_t)(i >> 4) * (D::E * 16);
    const int32_t *__restrict__ Si = a.slot + (size_t)(i >> 6) * (HoDims<R>::SP / 4) * 256 + (i & 63) * 4 + q;
    const double *__restrict__ Uv = a.U + q;
    uint32_t ent[G];                      // slot 4 g + q's
#pragma unroll
    for (int g = 0; g < G; ++g) ent[g] = (uint32_t)Si[g * 256];
    f32x4 b[NB][H::M];
    double u[NB][4];
    auto request = [&](int g) {
        const float *__restrict__ Pg = Pt + g * (64 * D::C);
        const bool tail = D::TAIL && g == G - 1;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (!tail || k < D::TAIL)
                u[g % NB][k] = Uv[(int64_t)((uint32_t)quad_bcast_dyn(k, (int)ent[g]) & kSlotIndexMask) * 4];
#pragma unroll
        for (int m = 0; m < NF; ++m) {
            if (!tail) b[g % NB][m] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Pg) + m * 64 + lane);
            else {
                const f32x2 x = __builtin_nontemporal_load(reinterpret_cast<const f32x2 *>(Pg) + m * 64 + lane);
                b[g % NB][m] = f32x4{x[0], x[1], 0, 0};
            }
        }
        if constexpr (REM > 0)
            b[g % NB][NF] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Pg + NF * 256) + c16 * REM +
                                                       (q < REM ? q : REM - 1));
    };
    f32x4 C[H::NC], X[VARG ? 3 : 1][H::ND];
#pragma unroll
    for (int m = 0; m < H::NC; ++m) C[m] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < (VARG ? 3 : 1); ++s)
#pragma unroll
        for (int m = 0; m < H::ND; ++m) X[s][m] = f32x4{0, 0, 0, 0};
    auto mma = [](float p, float d, f32x4 &x) { x = __builtin_amdgcn_mfma_f32_4x4x1f32(p, d, x, 0, 0, 0); };
#pragma unroll
    for (int g = 0; g < L; ++g) request(g);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g + L < G) request(g + L);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = 4 * g + k;
            if (j >= D::S) break;
            const float d = (float)(u[g % NB][k] - U0);
#pragma unroll
            for (int m = 0; m < H::NC; ++m) mma(b[g % NB][m][k], d, C[m]);
            if constexpr (VARG) {
                float ds[3];
                ho_split<float>(d, (uint32_t)quad_bcast_dyn(k, (int)ent[g]) >> kSlotGroupShift, ds);
#pragma unroll
                for (int m = 0; m < H::ND; ++m)
#pragma unroll
                    for (int s = 0; s < 3; ++s) mma(b[g % NB][H::D0 + m][k], ds[s], X[s][m]);
            } else {
#pragma unroll
                for (int m = 0; m < H::ND; ++m) mma(b[g % NB][H::D0 + m][k], d, X[0][m]);
                if (j % MD == MD - 1) {   // directional group j / MD is complete
#pragma unroll
                    for (int e = 0; e < KD; ++e) ad[j / MD][e] = X[0][(K + e) / 4 - H::D0][(K + e) % 4];
#pragma unroll
                    for (int m = 0; m < H::ND; ++m) X[0][m] = f32x4{0, 0, 0, 0};
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < K; ++e) ao[e] = C[e / 4][e % 4];
    if constexpr (VARG)
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int e = 0; e < KD; ++e) ad[s][e] = X[s][(K + e) / 4 - H::D0][(K + e) % 4];
}

// FP64: the four waves of a block take four of its 16 cells each (an instruction
// takes four slots of four cells; a wave with all 16 would hold 36 to 64 results
// beside the stream) and leave the coefficients in LDS, where one wave finds
// those of its lane's cell and variable: row r of lane l at ho_place(r, l).
// Results have lane 16 i + 4 b + v for row i: the swizzle spreads the rows of a
// store over the banks.  With characteristic variables three waves find them, one
// per face: each face has its own fields to select (122k cells of degree 6: 357
// us a stage; 935 with one wave for the three faces, 825 with vector sums).
__device__ __forceinline__ int ho_place(int row, int l) { return row * 64 + (l ^ ((row & 3) * 16)); }

template <int R>
__device__ __forceinline__ bool ho_contract_share(const ReconHoArgs<double> a, int64_t i0, int s, int lane,
                                                  double *coef) {
    using D = HoRows<R>;
    using H = HoGroups<R>;
    constexpr int K = D::K, KD = D::C - K, NF = D::NF, REM = D::REM, G = D::G, MD = HoDims<R>::MD;
    constexpr bool VARG = HoDims<R>::VARG;
    constexpr int NP = NF / 2;            // row groups in pairs
    // groups of four slots in flight ahead of the products (4, 3, 2: 3.6 to 5 KB
    // each; one more or less measures the same)
    constexpr int L = 8 - R, NB = L + 1;
    const int k = lane >> 4, b = (lane >> 2) & 3, v = lane & 3;
    const int64_t i = i0 + 4 * s + b;
    const double *__restrict__ Pt = a.P + (size_t)(i0 >> 4) * (D::E * 16) + s * (D::E * 4);
    const int32_t *__restrict__ Si = a.slot + (size_t)(i >> 6) * (HoDims<R>::SP / 4) * 256 + (i & 63) * 4 + k;
    const double *__restrict__ Uv = a.U + v;
    const int stop = *(a.done ? a.done : a.slot);
    uint32_t ent[G];
#pragma unroll
    for (int g = 0; g < G; ++g) ent[g] = (uint32_t)Si[g * 256];
    const double u0 = Uv[i * 4];
    f64x2 p2[NB][NP];
    double p1[NB][NF % 2 + 1], pr[NB];
    auto request = [&](int g) {
        const bool tail = D::TAIL && g == G - 1;          // (lanes without a slot: another one's, zero differences)
        const int n = tail ? 4 * D::TAIL : 16, l = tail ? lane & (4 * n - 1) : lane;
        const double *__restrict__ Pg = Pt + g * (16 * D::C);
#pragma unroll
        for (int p = 0; p < NP; ++p)
            p2[g % NB][p] = __builtin_nontemporal_load(reinterpret_cast<const f64x2 *>(Pg) + p * 4 * n + l);
        if constexpr (NF % 2 != 0) p1[g % NB][0] = __builtin_nontemporal_load(Pg + (NF - 1) * 4 * n + l);
        if constexpr (REM > 0)
            pr[g % NB] = __builtin_nontemporal_load(Pg + NF * 4 * n + (lane >> 2) * REM + (v < REM ? v : REM - 1));
    };
#pragma unroll
    for (int g = 0; g < L; ++g) request(g);
    __builtin_amdgcn_sched_barrier(0);
    if (a.done && stop) return false;
    double u[G];
#pragma unroll
    for (int g = 0; g < G; ++g) u[g] = Uv[(int64_t)(ent[g] & kSlotIndexMask) * 4];
    __builtin_amdgcn_sched_barrier(0);
    double C[H::NC], X[VARG ? 3 : 1][H::ND];
#pragma unroll
    for (int m = 0; m < H::NC; ++m) C[m] = 0;
#pragma unroll
    for (int t = 0; t < (VARG ? 3 : 1); ++t)
#pragma unroll
        for (int m = 0; m < H::ND; ++m) X[t][m] = 0;
    auto mma = [](double p, double d, double &x) { x = __builtin_amdgcn_mfma_f64_4x4x4f64(p, d, x, 0, 0, 0); };
    auto put = [&](int row, double x) { coef[ho_place(row + k, 16 * s + (lane & 15))] = x; };
    auto put_dir = [&](int t, const double (&x)[H::ND]) { // rows of stencil t
#pragma unroll
        for (int m = 0; m < H::ND; ++m) {
            const int e = 4 * (H::D0 + m) + k - K;
            if (e >= 0 && e < KD) coef[ho_place(K + t * KD + e, 16 * s + (lane & 15))] = x[m];
        }
    };
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g + L < G) request(g + L);
        __builtin_amdgcn_sched_barrier(0);
        const double d = u[g] - u0;
        double p[H::M];
#pragma unroll
        for (int m = 0; m < NF; ++m) p[m] = m < 2 * NP ? p2[g % NB][m / 2][m % 2] : p1[g % NB][0];
        if constexpr (REM > 0) p[NF] = pr[g % NB];
#pragma unroll
        for (int m = 0; m < H::NC; ++m) mma(p[m], d, C[m]);
        if constexpr (VARG) {
            double ds[3];
            ho_split<double>(d, ent[g] >> kSlotGroupShift, ds);
#pragma unroll
            for (int m = 0; m < H::ND; ++m)
#pragma unroll
                for (int t = 0; t < 3; ++t) mma(p[H::D0 + m], ds[t], X[t][m]);
        } else {
            // a directional group may end inside these four slots
            const int t = 4 * g / MD, e = (t + 1) * MD - 4 * g;   // its slots here: k < e
            if (e < 4) {
                const double d0 = k < e ? d : 0.0, d1 = k < e ? 0.0 : d;
#pragma unroll
                for (int m = 0; m < H::ND; ++m) mma(p[H::D0 + m], d0, X[0][m]);
                put_dir(t, X[0]);
#pragma unroll
                for (int m = 0; m < H::ND; ++m) {
                    X[0][m] = 0;
                    if (t < 2) mma(p[H::D0 + m], d1, X[0][m]);
                }
            } else {
#pragma unroll
                for (int m = 0; m < H::ND; ++m) mma(p[H::D0 + m], d, X[0][m]);
                if (e == 4) {
                    put_dir(t, X[0]);
#pragma unroll
                    for (int m = 0; m < H::ND; ++m) X[0][m] = 0;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (VARG)
#pragma unroll
        for (int t = 0; t < 3; ++t) put_dir(t, X[t]);
#pragma unroll
    for (int m = 0; m < H::NC; ++m)
        if (4 * m + k < K) put(4 * m, C[m]);
    return true;
}

// cells of a block: 256 lanes, a quad each (FP32 Euler), four waves for 16
// (FP64 Euler), or one lane each
template <typename real, int NV>
constexpr int ho_block_cells() { return NV == 1 ? 256 : std::is_same<real, float>::value ? 64 : 16; }

template <typename real, int R, int NV, int SCHEME, int GFORM, int DMODE, int VARS>
__global__ __launch_bounds__(256, (VARS && std::is_same<real, float>::value) || NV == 1 ? 1 : 2) void k_reconstruct_ho(const ReconHoArgs<real> a) {
    using D = HoDims<R>;
    constexpr int K = D::K, KD = D::KD, NQ = D::NQ;
    constexpr int BC = ho_block_cells<real, NV>();
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int v = threadIdx.x % NV;
    const int64_t i = blk * BC + (BC == 16 ? (threadIdx.x & 63) : threadIdx.x) / NV;
    const bool live = i < a.N;            // (padding cells compute on padding data and store nothing)
    if (NV == 1 && !live) return;
    const double U0 = a.U[i * NV + v];
    const int fl = a.flags[i] & 7;

    constexpr bool FACES = VARS && BC == 16;      // a wave per face
    int face = 0;
    real ao[K], ad[3][KD];
    if constexpr (NV == 4 && std::is_same<real, float>::value) {
        if (a.done && *a.done) return;
        ho_contract<R>(a, i, threadIdx.x & 63, U0, ao, ad);
    } else if constexpr (NV == 4) {
        __shared__ double coef[(K + 3 * KD) * 64];
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        if (!ho_contract_share<R>(a, blk * 16, wave, lane, coef)) return;
        __syncthreads();
        // characteristic variables: three of the waves take a face each
        if constexpr (FACES) face = wave;
        if (VARS ? wave == 3 : wave != (int)(blk & 3)) {
            if (VARS && a.positivity) __syncthreads();    // (the cells' flags, below)
            return;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) ao[k] = coef[ho_place(k, lane)];
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int k = 0; k < KD; ++k) ad[s][k] = coef[ho_place(K + s * KD + k, lane)];
    } else {
    constexpr int MD = D::MD, S = D::S, SP = D::SP, EPS = D::EPS, E = D::E, CT = 64;
    using V = typename Vec<real>::T;
    constexpr int VW = Vec<real>::W;
    constexpr int SV = EPS / VW;          // stream vectors per slot
    if (a.done && *a.done) return;
    const V *__restrict__ Pv = reinterpret_cast<const V *>(a.P) + (size_t)(i / CT) * (E / VW) * CT + (i % CT);
    const int32_t *__restrict__ Si = a.slot + (size_t)(i >> 6) * (SP / 4) * 256 + (i & 63) * 4;
    // a_opt = P_c d and a_s = P_s d, slot by slot (one lane per cell); the
    // next slot's stream vectors and entry are requested before the current
    // slot is used.  Variable groups: a slot's directional entries go to the
    // sums of the stencil its entry names
    real adt[KD];
#pragma unroll
    for (int k = 0; k < K; ++k) ao[k] = 0;
#pragma unroll
    for (int k = 0; k < KD; ++k) { adt[k] = 0; ad[0][k] = 0; ad[1][k] = 0; ad[2][k] = 0; }
    V cur[SV];
#pragma unroll
    for (int g = 0; g < SV; ++g) cur[g] = Pv[g * CT];
    uint32_t scur = (uint32_t)Si[0];
#pragma unroll 1
    for (int j = 0; j < S; ++j) {
        const int jn = j + 1 < S ? j + 1 : j;
        V nxt[SV];
#pragma unroll
        for (int g = 0; g < SV; ++g) nxt[g] = Pv[(jn * SV + g) * CT];
        const uint32_t sn = (uint32_t)Si[(jn >> 2) * 256 + (jn & 3)];
        const real d = (real)(a.U[(int64_t)(scur & kSlotIndexMask) * NV + v] - U0);
#pragma unroll
        for (int k = 0; k < K; ++k) ao[k] += comp(cur[k / VW], k % VW) * d;
        if constexpr (D::VARG) {
            const int gs = (int)(scur >> kSlotGroupShift);
            const real d0 = gs == 0 ? d : (real)0, d1 = gs == 1 ? d : (real)0, d2 = gs == 2 ? d : (real)0;
#pragma unroll
            for (int k = 0; k < KD; ++k) {
                const real p = comp(cur[(K + k) / VW], (K + k) % VW);
                ad[0][k] += p * d0;
                ad[1][k] += p * d1;
                ad[2][k] += p * d2;
            }
        } else {
#pragma unroll
            for (int k = 0; k < KD; ++k) adt[k] += comp(cur[(K + k) / VW], (K + k) % VW) * d;
            if (j % MD == MD - 1) {       // uniform: group j / MD is complete
                const int s = j / MD;
#pragma unroll
                for (int s2 = 0; s2 < 3; ++s2)
                    if (s2 == s)
#pragma unroll
                        for (int k = 0; k < KD; ++k) ad[s2][k] = adt[k];
#pragma unroll
                for (int k = 0; k < KD; ++k) adt[k] = 0;
            }
        }
#pragma unroll
        for (int g = 0; g < SV; ++g) cur[g] = nxt[g];
        scur = sn;
    }
    }

    const int adm = 1 | (fl << 1);
    const int st = 1 + __popc(fl);
    const real lams = st == 2 ? a.lams[2] : (st == 3 ? a.lams[3] : a.lams[4]);
    const real lratio = st == 2 ? a.lam_ratio[2] : (st == 3 ? a.lam_ratio[3] : a.lam_ratio[4]);
    // p_1 = (p_opt - sum_s lambda_s p_s) / lambda_1 (eq. e17), in place.
    // TENO keeps the central stencil's own polynomial: it runs the same step
    // with factors 0 and 1 from the arguments (exact: x - 0 y = x, x / 1 = x),
    // because without the step the compiler's schedule needs a third more
    // registers (110 instead of 81 VGPRs at r = 4, 187 instead of 145 at r = 6)
    {
        const real ls = lams * a.p1_ls, il1 = frcp(a.p1_l1);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            real sm = ao[k];
            if (k < KD && st > 1) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if ((fl >> q) & 1) sm -= ls * ad[q][k];
            }
            ao[k] = st > 1 ? sm * il1 : sm;
        }
    }
    real out[3][NQ];
    constexpr int NB = VARS ? 3 : 1;              // selection bytes of this lane
    int dbyte[NB];
    if constexpr (VARS == 0) {
        dbyte[0] = finish_field_ho<real, K, KD, SCHEME, GFORM, DMODE>(a, ao, ad, fl, adm, st, lams, lratio,
                                                                      DMODE == 2 ? a.delta[i * NV + v] : 0);
        // face Gauss-point values
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                real val = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) val += a.entry(K * K + (f * NQ + q) * K + k) * ao[k];
                out[f][q] = (real)(U0 + (double)val);
            }
    } else {
        // characteristic fields per face, lane v reconstructs field v: the
        // coefficients are projected with row v of L_f using the cell's
        // other lanes, the face values come back through row v of R_f
        static_assert(NV == 4, "characteristic variables need the Euler equations");
        const double Ud[4] = {quad_bcast<0>(U0), quad_bcast<1>(U0), quad_bcast<2>(U0), quad_bcast<3>(U0)};
        const real rho = (real)Ud[0], uu = (real)(Ud[1] / Ud[0]), vv = (real)(Ud[2] / Ud[0]);
        const real q2 = (real)0.5 * (uu * uu + vv * vv);
        const real pr = (a.gamma - 1) * ((real)Ud[3] - rho * q2);
        const real cs = fsqrt(fdiv(a.gamma * pr, rho)), H = fdiv((real)Ud[3] + pr, rho);
        const real b1 = fdiv(a.gamma - 1, cs * cs), b2 = b1 * q2, ic = frcp(cs);
#pragma unroll
        for (int w = 0; w < (FACES ? 1 : 3); ++w) {
            const int f = FACES ? face : w;
            real nx, ny, len;
            uint32_t code;
            face_record<real>(a.fr, i, f, nx, ny, len, code);
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
            auto project = [](const real (&row)[4], real x) -> real {
                real y = 0;
                y += row[0] * quad_bcast<0>(x);
                y += row[1] * quad_bcast<1>(x);
                y += row[2] * quad_bcast<2>(x);
                y += row[3] * quad_bcast<3>(x);
                return y;
            };
            real c1[K], cd[3][KD];
#pragma unroll
            for (int k = 0; k < K; ++k) c1[k] = project(Lr, ao[k]);
#pragma unroll
            for (int s2 = 0; s2 < 3; ++s2)
#pragma unroll
                for (int k = 0; k < KD; ++k) cd[s2][k] = project(Lr, ad[s2][k]);
            dbyte[w] = finish_field_ho<real, K, KD, SCHEME, GFORM, DMODE>(
                a, c1, cd, fl, adm, st, lams, lratio, DMODE == 2 ? a.delta[(i * 3 + f) * NV + v] : 0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                real x = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) x += a.entry(K * K + (f * NQ + q) * K + k) * c1[k];
                out[w][q] = (real)(U0 + (double)project(Rr, x));
            }
        }
    }
    if constexpr (NV == 4) if (a.positivity) {
        // optional positivity fallback (not in the paper; density or
        // pressure <= 0 at a Gauss point): the four lanes of the cell
        // exchange their values
        bool bad = false;
#pragma unroll
        for (int f = 0; f < (FACES ? 1 : 3); ++f)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const real r0 = quad_bcast<0>(out[f][q]), r1 = quad_bcast<1>(out[f][q]);
                const real r2 = quad_bcast<2>(out[f][q]), r3 = quad_bcast<3>(out[f][q]);
                const real pr = euler_pressure(a.gamma, r0, r1, r2, r3);
                bad |= !(r0 > 0) || !(pr > 0);
            }
        if constexpr (FACES) {
            __shared__ int badf[3][64];           // of the faces' waves
            badf[face][threadIdx.x & 63] = bad;
            __syncthreads();
            bad = badf[0][threadIdx.x & 63] | badf[1][threadIdx.x & 63] | badf[2][threadIdx.x & 63];
        }
        if (bad && live) {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int q = 0; q < NQ; ++q) out[f][q] = (real)U0;
#pragma unroll
            for (int k = 0; k < NB; ++k) dbyte[k] |= 0x80;
            if (v == 0 && face == 0 && a.fb_count) atomicAdd(a.fb_count, 1ull);
        }
    }
    if (!live) return;
    if (DMODE == 1) {
        if constexpr (VARS == 0) a.delta[i * NV + v] = (uint8_t)dbyte[0];
        else if constexpr (FACES) a.delta[(i * 3 + face) * NV + v] = (uint8_t)dbyte[0];
        else {
#pragma unroll
            for (int f = 0; f < 3; ++f) a.delta[(i * 3 + f) * NV + v] = (uint8_t)dbyte[f];
        }
    }
    if constexpr (FACES) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) a.FV[((i * 3 + face) * NQ + q) * NV + v] = out[0][q];
    } else {
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int q = 0; q < NQ; ++q) a.FV[((i * 3 + f) * NQ + q) * NV + v] = out[f][q];
    }
}

template <typename real, int R, int NV>
static hipError_t reconstruct_ho_t(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode,
                                   const int *done, hipStream_t st, unsigned long long *fb_count) {
    using D = HoDims<R>;
    ReconHoArgs<real> a;
    a.N = m.N;
    a.U = U;
    a.slot = m.slot;
    a.flags = m.flags;
    if constexpr (std::is_same<real, double>::value) { a.P = m.P64; a.tab = m.htab64; }
    else { a.P = m.P32; a.tab = m.htab32; }
    if (!a.P || !a.tab || m.E != (NV == 1 ? D::E : HoRows<R>::E)) return hipErrorInvalidValue;
    if constexpr (std::is_same<real, double>::value) a.fr = m.fr64;
    else a.fr = m.fr32;
    if (m.vars == CTENO_VARS_CHARACTERISTIC && (NV != 4 || !a.fr)) return hipErrorInvalidValue;
    a.FV = (real *)FV;
    a.delta = delta;
    a.done = done;
    const double lam1 = 1.0 - 1.0 / m.lam1p;
    a.lam1 = (real)lam1;
    a.gamma = (real)m.gamma;
    a.ct = (real)m.ct;
    a.eps = (real)m.eps;
    a.positivity = m.positivity;
    a.fb_count = fb_count;
    for (int s = 0; s < 5; ++s) {
        const double ls = s >= 2 ? (1.0 - lam1) / (s - 1) : 0.0;
        a.lams[s] = (real)ls;
        a.lam_ratio[s] = s >= 2 ? (real)(lam1 / ls) : (real)1;
    }
    a.p1_ls = m.scheme == CTENO_SCHEME_TENO ? (real)0 : (real)1;
    a.p1_l1 = m.scheme == CTENO_SCHEME_TENO ? (real)1 : a.lam1;
    constexpr int BC = ho_block_cells<real, NV>();
    const unsigned grid = (unsigned)((m.N + BC - 1) / BC);
#define HO_LAUNCH(SCH, GF, DM)                                                                               \
    do {                                                                                                     \
        if constexpr (NV == 4)                                                                               \
            if (m.vars == CTENO_VARS_CHARACTERISTIC) {                                                       \
                hipLaunchKernelGGL((k_reconstruct_ho<real, R, NV, SCH, GF, DM, 1>), dim3(grid), dim3(256), 0, st, \
                                   a);                                                                       \
                break;                                                                                       \
            }                                                                                                \
        hipLaunchKernelGGL((k_reconstruct_ho<real, R, NV, SCH, GF, DM, 0>), dim3(grid), dim3(256), 0, st, a);   \
    } while (0)
#define HO_DM(SCH, GF)                        \
    switch (dmode) {                          \
        case 0: HO_LAUNCH(SCH, GF, 0); break; \
        case 1: HO_LAUNCH(SCH, GF, 1); break; \
        default: HO_LAUNCH(SCH, GF, 2); break; \
    }
    if (m.scheme == CTENO_SCHEME_CTENOZ && m.gamma_form == CTENO_GAMMA_SCALED) { HO_DM(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_SCALED); }
    else if (m.scheme == CTENO_SCHEME_CTENOZ) { HO_DM(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_PAPER); }
    else if (m.scheme == CTENO_SCHEME_CWENO) { HO_DM(CTENO_SCHEME_CWENO, CTENO_GAMMA_PAPER); }
    else if (m.scheme == CTENO_SCHEME_TENO) { HO_DM(CTENO_SCHEME_TENO, CTENO_GAMMA_PAPER); }
    else if (m.gamma_form == CTENO_GAMMA_LAMBDA) { HO_DM(CTENO_SCHEME_CTENO, CTENO_GAMMA_LAMBDA); }
    else { HO_DM(CTENO_SCHEME_CTENO, CTENO_GAMMA_PAPER); }
#undef HO_DM
#undef HO_LAUNCH
    return hipGetLastError();
}

template <typename real>
hipError_t reconstruct_hi(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode,
                          const int *done, hipStream_t st, unsigned long long *fb_count) {
    if (m.nv == 4) {
        switch (m.r) {
            case 4: return reconstruct_ho_t<real, 4, 4>(m, U, FV, delta, dmode, done, st, fb_count);
            case 5: return reconstruct_ho_t<real, 5, 4>(m, U, FV, delta, dmode, done, st, fb_count);
            case 6: return reconstruct_ho_t<real, 6, 4>(m, U, FV, delta, dmode, done, st, fb_count);
        }
    } else {
        switch (m.r) {
            case 4: return reconstruct_ho_t<real, 4, 1>(m, U, FV, delta, dmode, done, st, fb_count);
            case 5: return reconstruct_ho_t<real, 5, 1>(m, U, FV, delta, dmode, done, st, fb_count);
            case 6: return reconstruct_ho_t<real, 6, 1>(m, U, FV, delta, dmode, done, st, fb_count);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace cteno
