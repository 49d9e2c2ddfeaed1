// Reconstruction of degree 2 and 3 (a quad of lanes per cell): the kernel and
// its launch, for one arithmetic type; instantiated per type by
// k_recon_f32.hip and k_recon_f64.hip.
#pragma once
#include "recon_quad.h"

namespace cteno {

template <typename real, int R, int NV, int SCHEME, int GFORM, int DMODE, int VARS, bool NT>
__global__ __launch_bounds__(256) void k_reconstruct(const ReconArgs<real> a, const ReconPtrs<real> ptr, int64_t N,
                                                     real *FV) {
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * 64 + (threadIdx.x >> 2);
    const int q = threadIdx.x & 3, v = NV == 4 ? q : 0;
    const bool live = i < N;
    extern __shared__ __align__(16) double rows[];
    double U0;
    real out[3][2];
    if (!recon_quad<real, R, NV, SCHEME, GFORM, DMODE, VARS, NT>(a, ptr, rows, i, threadIdx.x, live, [] {}, U0, out))
        return;
    if (!live || q >= NV) return;
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g) FV[((i * 3 + f) * 2 + g) * NV + v] = out[f][g];
}

template <typename real, int R, int NV, int VARS>
static void reconstruct_launch(const DeviceMesh &m, const ReconArgs<real> &a, const ReconPtrs<real> &p, real *FV,
                               int dmode, bool plain, unsigned grid, hipStream_t st) {
#define CT_LAUNCH(SCH, GF, DM)                                                                                    \
    do {                                                                                                          \
        if constexpr (DM == 0)                                                                                    \
            if (plain) {                                                                                          \
                hipLaunchKernelGGL((k_reconstruct<real, R, NV, SCH, GF, DM, VARS, false>), dim3(grid), dim3(256), \
                                   m.row_bytes(), st, a, p, m.N, FV);                                             \
                break;                                                                                            \
            }                                                                                                     \
        hipLaunchKernelGGL((k_reconstruct<real, R, NV, SCH, GF, DM, VARS, true>), dim3(grid), dim3(256),          \
                           m.row_bytes(), st, a, p, m.N, FV);                                                     \
    } while (0)
#define CT_DM(SCH, GF)                        \
    switch (dmode) {                          \
        case 0: CT_LAUNCH(SCH, GF, 0); break; \
        case 1: CT_LAUNCH(SCH, GF, 1); break; \
        default: CT_LAUNCH(SCH, GF, 2); break; \
    }
    if (m.scheme == CTENO_SCHEME_CTENOZ && m.gamma_form == CTENO_GAMMA_SCALED) { CT_DM(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_SCALED); }
    else if (m.scheme == CTENO_SCHEME_CTENOZ) { CT_DM(CTENO_SCHEME_CTENOZ, CTENO_GAMMA_PAPER); }
    else if (m.scheme == CTENO_SCHEME_CWENO) { CT_DM(CTENO_SCHEME_CWENO, CTENO_GAMMA_PAPER); }
    else if (m.scheme == CTENO_SCHEME_TENO) { CT_DM(CTENO_SCHEME_TENO, CTENO_GAMMA_PAPER); }
    else if (m.gamma_form == CTENO_GAMMA_LAMBDA) { CT_DM(CTENO_SCHEME_CTENO, CTENO_GAMMA_LAMBDA); }
    else { CT_DM(CTENO_SCHEME_CTENO, CTENO_GAMMA_PAPER); }
#undef CT_DM
#undef CT_LAUNCH
}

template <typename real, int R, int NV>
static hipError_t reconstruct_t(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode,
                                const int *done, hipStream_t st, unsigned long long *fb_count, bool stage) {
    if (m.E != QuadDims<R>::E || m.SP != QuadDims<R>::SP) return hipErrorInvalidValue;
    ReconArgs<real> a;
    fill_recon_constants<real>(m, a);
    ReconPtrs<real> p{};
    p.U = U;
    p.lslot = m.lslot;
    p.desc = m.desc;
    p.hlist = m.hlist;
    p.flags = m.flags;
    if constexpr (std::is_same<real, double>::value) { p.P = m.P64; p.fr = m.fr64; }
    else { p.P = m.P32; p.fr = m.fr32; }
    p.delta = delta;
    p.fb = fb_count;
    p.done = done;
    if (!p.P || !a.tab || !p.lslot || !p.desc || !p.hlist) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)(m.Np / 64);
    const bool plain = stage && !m.stream_nontemporal(std::is_same<real, float>::value);
    if (m.vars == CTENO_VARS_CHARACTERISTIC) {
        if constexpr (NV == 4) {
            if (!p.fr) return hipErrorInvalidValue;
            reconstruct_launch<real, R, NV, 1>(m, a, p, (real *)FV, dmode, plain, grid, st);
        } else {
            return hipErrorInvalidValue;
        }
    } else {
        reconstruct_launch<real, R, NV, 0>(m, a, p, (real *)FV, dmode, plain, grid, st);
    }
    return hipGetLastError();
}

template <typename real>
hipError_t reconstruct_lo(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode,
                          const int *done, hipStream_t st, unsigned long long *fb_count, bool stage) {
    if (m.nv == 4) {
        switch (m.r) {
            case 2: return reconstruct_t<real, 2, 4>(m, U, FV, delta, dmode, done, st, fb_count, stage);
            case 3: return reconstruct_t<real, 3, 4>(m, U, FV, delta, dmode, done, st, fb_count, stage);
        }
    } else {
        switch (m.r) {
            case 2: return reconstruct_t<real, 2, 1>(m, U, FV, delta, dmode, done, st, fb_count, stage);
            case 3: return reconstruct_t<real, 3, 1>(m, U, FV, delta, dmode, done, st, fb_count, stage);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace cteno
