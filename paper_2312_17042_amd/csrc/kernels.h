// Kernel launchers of the CTENO/CTENOZ library, implemented in k_precompute.hip
// (pseudo-inverses), k_recon_*.hip (reconstruction, per degree range and
// arithmetic type), k_stage_*.hip (fused stage of degree 2 and 3) and k_flux.hip
// (fluxes, RK stages, step control, serving batches, mesh lists, utilities);
// kernels_common.h and recon_quad.h hold the shared device code.
//
// HIP kernels (gfx950) of the CTENO/CTENOZ finite-volume hot path.
//
//   k_precompute   once per mesh, FP64: reference-space moments of every
//                  stencil cell (sec. 2.1), Householder QR of the M x K
//                  least-squares matrix and the pseudo-inverse
//                  P = R^-1 Q^T diag(|V'_m|), for the central stencil and
//                  the three directional stencils; FP32 copies on request.
//   k_reconstruct  per cell and stage, a quad of lanes per cell: neighbour
//                  averages, central and directional products P d on the
//                  matrix cores, p_1 (eq. e17), smoothness indicators, CTENO
//                  (Algorithm 1) / CTENOZ (Algorithm 2) selection, final
//                  polynomial at the face Gauss points.
//   k_flux         per cell and stage, a lane per face: HLLC (sec. 2.6) or
//                  upwind flux at the Gauss points, the residual of the
//                  semi-discrete form after eq. e1, and the SSP-RK3 stage;
//                  each interior face flux is evaluated identically by both
//                  of its cells (same operands, same order) so the update is
//                  conservative to FP64 round-off without atomics.
//   k_stage, k_stage_wide, k_stage_cross   degree 2 and 3: both in one kernel,
//                  face values in LDS, and the faces between its blocks.
//   k_control      per RK step, one block: time step from the reduced CFL
//                  bound, clipping to t_final, termination.
//
// Memory layout: the pseudo-inverse streams in tiles of 16 cells in the order
// that the matrix instructions read them (quad_index, ho_index), other static
// per-cell data in 64-cell tiles; the state and the face-point values are
// cell-major (array of structures) so a gather of one neighbour touches one
// cache line.
#pragma once

#include <algorithm>

#include "cteno_internal.h"

namespace cteno {

// Lists of the fused stage in one precision.  A block is bc cells: the faces
// that it evaluates alone (its boundary faces and the faces between two of its
// cells, once, from their owner), and the cells with a face to another block
// ("cross cells") with one record per such face ("side")
struct StageLists {
    bool fused = false;            // marches and stages run the fused kernels
    int bc = 64;
    int2 *fdesc = nullptr;         // per block its first listed face and their number
    void *frec = nullptr;          // [faces][4] normal, length, block face code (kBf*), of the precision type
    uint32_t *xid = nullptr;       // [Np] the cell's first side | its faces to other blocks << 28 (0: none)
    int2 *xcells = nullptr;        // [n_cross] cross cells, ascending, and their xid
    double *xarea = nullptr;       // [n_cross] their areas
    void *xrec = nullptr;          // [n_sides][4] normal, length, the other side | kNbOwner | kSideFar
    int64_t n_cross = 0, n_sides = 0;
    int64_t cross_blocks() const { return (n_cross + 63) / 64; }
};
// FP32 meshes from this many cells on take blocks of 256 cells (k_stage_wide):
// fewer faces lead to other blocks, but the four groups of a block run one
// after the other.  Both kernels of a stage together, blocks of 64 against 256
// cells, degree 3: 96 / 102 us at 500k cells, 186 / 189 at 1M, 288 / 283 at
// 1.4M, 402 / 392 at 2M, 1728 / 1545 at 8M.  Only where two groups' averages leave
// room for three blocks per CU (the usual lists take 13 KB; scattered numberings up
// to 90), and not for characteristic variables, whose selection per face leaves
// room for two waves per SIMD only (448 / 545 us at 1.6M).
constexpr int64_t kWideCells = 1200000;
// The fused stage runs where at most half of the cells' faces lead to other
// blocks: what it saves are the values of the others.  Morton order has 0.5 such
// faces a cell, a mesh numbered row by row 1.0, a random numbering 3.0.  20 steps
// at degree 3, fused / separate kernels, at 1.0, 1.4, 1.6, 2.4 and 3.0: 2M cells
// FP64 47.8 / 53.3, 53.4 / 54.4, 55.7 / 54.9, 62.5 / 58.4, 98.4 / 79.5 ms; mixed
// 26.9 / 27.1, 29.3 / 28.7, 30.4 / 29.2, 39.6 / 33.6, 70.3 / 59.0; 500k FP64 11.5 /
// 13.0, 13.0 / 13.2, 13.3 / 13.3, 15.2 / 13.9, 24.3 / 18.6.  FP64 with
// characteristic variables spends more on the selection and the line lies higher:
// 2M cells at 1.6, 2.4 and 3.0 65.5 / 67.2, 71.0 / 75.1, 112.1 / 104.1.
constexpr double kFusedFaces = 1.5, kFusedFacesChar64 = 2.75;
// Degree 2 and 3: what an RK stage reads and writes, of which the 256 MB
// memory-side cache keeps a stream that fits for the next stage, but not one that
// is loaded nontemporally.  20 steps, nontemporal / plain loads: one variable,
// degree 2, mixed 2677 / 2502 us at 400k cells (200 MB), 3100 / 2924 at 500k (250
// MB), 4191 / 4710 at 700k (350 MB); degree 3 mixed 2967 / 2787 at 200k (204 MB),
// 4523 / 5048 at 353k (360 MB); FP64 3845 / 3621 at 150k (264 MB), 4888 / 5270 at
// 200k.  Below, nontemporal streams stay in it too and leave the L2s to the
// averages: one variable, degree 2, mixed 1117 / 1183 at 100k (50 MB), 1395 / 1434
// at 150k (75 MB).  A single reconstruction finds its stream in memory, where
// nontemporal loads are the better ones (residual of 81k cells in FP64 74 / 78 us).
constexpr double kCachedStream[2] = {128e6, 268e6};
constexpr size_t kWideRowBytes = 28 * 1024;

struct DeviceMesh {
    int64_t N = 0, Np = 0;
    int r = 0, K = 0, S = 0, SP = 0, nv = 0, physics = 0;
    int scheme = 0, gamma_form = 0, precision = 0;
    int positivity = 0;            // 1: cell-average fallback for non-physical face states
    int vars = 0;                  // CTENO_VARS_CONSERVED | CTENO_VARS_CHARACTERISTIC
    int E = 0;                     // pseudo-inverse entries per cell
    int Kd = 0, Md = 0, Nq = 2;    // directional basis size and members, Gauss points per face
    double gamma = 1.4, ax = 0, ay = 0, lam1p = 1e4, ct = 1e-6, eps = 1e-12;
    double Lx = 0, Ly = 0;
    int32_t *slot = nullptr;       // vector-tiled [SP], VW 4 (r <= 3: while the mesh is uploaded)
    // r <= 3: the stencil entries as rows of the cell's group of 64 cells
    // (lslot_index): row < 64 a cell of the group, row - 64 a place in the
    // group's list of cells outside it
    uint16_t *lslot = nullptr;     // [Np][row_entries(r)]
    int2 *desc = nullptr;          // [groups()] first place in hlist (negative before its middle), its length
    int32_t *hlist = nullptr;
    int max_halo = 0;              // the longest list
    uint8_t *flags = nullptr;      // [Np]
    double *fr64 = nullptr;        // face records, vector-tiled [12], VW 2
    float *fr32 = nullptr;         // face records, vector-tiled [12], VW 4
    double *area = nullptr;        // [Np]
    double *P64 = nullptr;         // pseudo-inverse stream [Np][E] (r <= 3 quad_index, else ho_index, one variable avix; VW 2)
    float *P32 = nullptr;          // pseudo-inverse stream [Np][E] (VW 4)
    int32_t *perm = nullptr;       // internal -> user [N]
    double *bface = nullptr;       // [n_inflow][4]: first vertex and edge vector of each inflow face
    int64_t n_inflow = 0;
    double bst[2][4] = {};         // inflow states behind / ahead of the moving line
    double bline[3] = {};          // x = bline[0] + bline[1] y + bline[2] t
    double *htab64 = nullptr;      // Gram matrix [K][K] and face basis [3][Nq][K], FP64
    float *htab32 = nullptr;       // the same in FP32 (r <= 3: off-diagonal Gram entries above the diagonal doubled)
    RefTables tab;
    StageLists lists[2];           // fused stage (degree <= 3): FP64, FP32
    int64_t n_cross256 = 0;        // cells with a face to another 256-cell block
    int64_t blocks() const { return (N + 255) / 256; }
    int64_t groups() const { return Np / 64; }
    // LDS rows of one group
    size_t row_bytes() const { return (size_t)(64 + max_halo) * nv * sizeof(double); }
    bool stream_nontemporal(bool f32) const {
        const double cell = (double)E * (f32 ? 4 : 8) + 2.0 * row_entries(r) + 32.0 * nv + 100.0;
        return (double)N * cell < kCachedStream[0] || (double)N * cell > kCachedStream[1];
    }
    int64_t stage_blocks(bool f32) const { return (N + lists[f32].bc - 1) / lists[f32].bc; }
    // Per-block CFL minima of one march step that the control reduces: the
    // fused stage's second kernel's (which fold in the first kernel's, stored
    // behind them), or the only kernel's
    int64_t dt_parts(bool fused_run, bool f32) const {
        return !fused_run ? groups() : lists[f32].n_cross ? lists[f32].cross_blocks() : stage_blocks(f32);
    }
    int64_t dt_storage() const {
        return std::max({groups(), stage_blocks(false) + lists[0].cross_blocks(),
                         stage_blocks(true) + lists[1].cross_blocks()});
    }
    // selection bytes per cell: per variable, or per face and characteristic field
    int delta_bytes() const { return vars == CTENO_VARS_CHARACTERISTIC ? 3 * nv : nv; }
};

struct PrecomputeInputs {
    const double *verts;          // tiled [6]
    const uint8_t *slot_flag;     // tiled [S]
    const int8_t *slot_shift;     // tiled [2S]
    uint8_t *flags;               // [Np] in/out: inadmissible-by-rank bits cleared
    int *rank_fail;               // device counter of rank-deficient central systems
};

hipError_t launch_precompute(const DeviceMesh &m, const PrecomputeInputs &in, hipStream_t st);

// reconstruction of degree 2-3 (reconstruct_lo) and 4-6 (reconstruct_hi) in
// arithmetic `real` (float: mixed precision; double: FP64); instantiated in
// k_recon_f32/f64.hip and k_recon_ho_f32/f64.hip
template <typename real>
hipError_t reconstruct_lo(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode, const int *done,
                          hipStream_t st, unsigned long long *fb_count, bool stage);
template <typename real>
hipError_t reconstruct_hi(const DeviceMesh &m, const double *U, void *FV, uint8_t *delta, int dmode, const int *done,
                          hipStream_t st, unsigned long long *fb_count);

// reconstruction; dmode: 0 none, 1 write delta, 2 forced delta
// fb_count (may be null) counts the cells that take the positivity fallback;
// stage: of an RK stage, one of several on this mesh in a row (dmode 0)
hipError_t launch_reconstruct(const DeviceMesh &m, bool fp32, const double *U, void *FV, uint8_t *delta, int dmode,
                              const int *done, hipStream_t st, unsigned long long *fb_count = nullptr,
                              bool stage = false);

// flux / residual / RK stage.  mode: 0 outward face fluxes, 1 residual, 2 RK stage
struct FluxLaunch {
    int mode = 2;
    const void *FV = nullptr;
    const double *Un = nullptr, *Us = nullptr;
    double *Uout = nullptr;
    int stage = 0;
    const double *dt_ptr = nullptr;
    double dt_value = 0.0;
    void *flux_out = nullptr;    // AoS [Np][3][nv] of the precision type
    double *resid = nullptr;     // AoS [Np][nv]
    Ctrl *ctrl = nullptr;        // done / nonphysical (may be null); with dt_ptr also the march time
    int *nonphys = nullptr;      // non-physical flag when ctrl is null (may be null)
    double *dt_part = nullptr;   // per-block minima of the CFL bound (stage 2 of a march), or null
    double t_base = 0.0;         // time of the stage input when the march time is not on the device
    void *xterm = nullptr;       // FP32 fused stage: [2 n_sides][nv] floats, the cross cells' other terms
};
hipError_t launch_flux(const DeviceMesh &m, bool fp32, const FluxLaunch &f, hipStream_t st);

// Lists of the fused stage in one precision from the face records on the device,
// in two steps: the counts per group of 64 cells (listed faces, cross cells,
// sides) and the number of cells with a face to another 256-cell block; then,
// with the groups' offsets (exclusive sums of the counts), the lists.
struct BlockCounts {
    int32_t *faces, *cross, *sides;    // [groups()]
    int32_t *cross256;                 // one counter
};
hipError_t launch_block_counts(const DeviceMesh &m, bool f32, const BlockCounts &c, hipStream_t st);
hipError_t launch_block_lists(const DeviceMesh &m, bool f32, const BlockCounts &base, hipStream_t st);

// Fused SSP-RK3 stage of degree <= 3 (f.mode 2): part 0 reconstructs each
// block of cells into LDS, evaluates the faces inside the block and updates
// the cells whose faces all lie inside it; part 1 evaluates the faces between
// blocks, whose values part 0 leaves in f.FV ([n_sides][2][nv]), and updates
// their cells with the other faces' terms (f.xterm).  The two parts are launched in
// order, 0 then 1.
hipError_t launch_stage(const DeviceMesh &m, bool fp32, const FluxLaunch &f, const int *done, int part,
                        hipStream_t st, unsigned long long *fb_count);
template <typename real>
hipError_t stage_fused(const DeviceMesh &m, const FluxLaunch &f, const int *done, int part, hipStream_t st,
                       unsigned long long *fb_count);     // k_stage_f32.hip, k_stage_f64.hip

// minima of the CFL bound of state U over n_part shares of the cells into
// dt_part[n_part], from the face records of the stage kernels' precision (fp32) so a march's first step
// uses the same geometry as its later steps
hipError_t launch_dt_partials(const DeviceMesh &m, bool fp32, const double *U, double *dt_part, int64_t n_part,
                              hipStream_t st);
// step control; reduces dt_part[n_part] unless commit_only
hipError_t launch_control(Ctrl *ctrl, const double *dt_part, int64_t n_part, int commit_only, hipStream_t st);

// device descriptor of one active serving slot (one independent solve)
struct BatchSlot {
    int64_t N, block0, nblocks;     // cells; first global block; blocks of 256 cells
    const uint16_t *lslot;
    const int2 *desc;
    const int32_t *hlist;
    const uint8_t *flags;
    const float *P;                 // FP32 pseudo-inverse stream
    const float *fr;                // FP32 face records
    const double *area;
    double *U[3];                   // U^n, U^(1), U^(2)
    float *FV;
    double *dt_part;                // [4 nblocks]
    Ctrl *ctrl;
};
// one SSP-RK3 step (control + 3 x (reconstruction, flux/RK)) of every slot in
// tab[0 .. *n_slots); grids of max_slots and max_blocks blocks (blocks past the
// active range exit at once).  FP32 reconstruction/flux, Euler, r = 2 or 3.
// proto.max_halo: the longest neighbour list of a group that a slot may have.
hipError_t launch_batch_step(const DeviceMesh &proto, const BatchSlot *tab, const int *n_slots, int max_slots,
                             int64_t max_blocks, hipStream_t st);

// neighbour lists of the 64-cell groups: their lengths into len[groups()], then
// (their places set in m.desc) the lists and the stencil entries as rows
hipError_t launch_halo_counts(const DeviceMesh &m, int32_t *len, hipStream_t st);
hipError_t launch_halo_lists(const DeviceMesh &m, hipStream_t st);

// layout conversions between caller order/layout and internal order/layout
hipError_t launch_user_to_state(const DeviceMesh &m, const double *user, double *state, hipStream_t st);
hipError_t launch_state_to_user(const DeviceMesh &m, const double *state, double *user, hipStream_t st);
hipError_t launch_fv_to_user(const DeviceMesh &m, bool fp32, const void *fv, void *user, hipStream_t st);
hipError_t launch_fv_from_user(const DeviceMesh &m, bool fp32, const void *user, void *fv, hipStream_t st);
hipError_t launch_flux_to_user(const DeviceMesh &m, bool fp32, const void *fo, void *user, hipStream_t st);
hipError_t launch_delta_to_user(const DeviceMesh &m, const uint8_t *d, uint8_t *user, hipStream_t st);
hipError_t launch_delta_from_user(const DeviceMesh &m, const uint8_t *user, uint8_t *d, hipStream_t st);
hipError_t launch_count_diff(const DeviceMesh &m, const uint8_t *a, const uint8_t *b, unsigned long long *count,
                             hipStream_t st);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t st);
hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, size_t n, hipStream_t st);

// Fixed device scratch of the allocation-free entry point (one array per
// device, held until the process ends).  scratch_init records its device
// address for `device`, which must be the current device; it is called
// once per device by cteno_ctx_create.  scratch_device_ptr returns the
// recorded address, or null before scratch_init succeeded on that device.
constexpr size_t kScratchBytes = size_t(32) << 20;
constexpr int kMaxDevices = 64;
hipError_t scratch_init(int device);
void *scratch_device_ptr(int device);
hipError_t launch_copy16(void *dst, const void *src, size_t n16, hipStream_t st);
// dst[a][e] = entry e of cell idx[a] of the pseudo-inverse stream (exactly one of
// src64 / src32; entries in pinv_offset's order at r <= 3), or of the slot
// table (srci, E = SP)
hipError_t launch_gather_entries(const DeviceMesh &m, int n, const int32_t *idx, int E, const double *src64,
                                 const float *src32, const int32_t *srci, double *dst, hipStream_t st);

}  // namespace cteno
