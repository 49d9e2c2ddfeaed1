// Internal declarations of the CTENO/CTENOZ MI355X library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <utility>
#include <string>
#include <vector>

#include "../../include/cteno.h"

namespace cteno {

// ---------------------------------------------------------------------------
// sizes
// ---------------------------------------------------------------------------
constexpr int kTile = 64;          // cells per tile of the tiled per-cell arrays (one wave)
constexpr int kNq = 2;             // Gauss points per face for degree <= 3
constexpr int kMaxR = 6;
constexpr int kMaxK = 27;          // K at degree 6
constexpr int kMaxS = 54;          // slots at degree 6
constexpr int kMaxNq = 4;          // Gauss points per face at degree 6
constexpr int kDirSlots = 4;       // M_d = 2 K_d with K_d = 2 (degree-1 directional, r <= 3)

inline int dims_K(int r) { return (r + 1) * (r + 2) / 2 - 1; }
inline int dims_M(int r) { return 2 * dims_K(r); }
// directional degree: 1 up to cubic, ceil(r/2) above (third-order directional
// stencils for the fifth-order scheme)
inline int dims_rd(int r) { return r <= 3 ? 1 : (r + 1) / 2; }
inline int dims_Kd(int r) { return dims_K(dims_rd(r)); }
inline int dims_Md(int r) { return 2 * dims_Kd(r); }
// Slots of a cell's stream.  Up to cubic (and at degree 6, where
// 3 M_d = M): the three directional groups of M_d slots first (a group's
// members, then other central cells or pads), then the rest of the central
// stencil.  At degrees 4 and 5 (M < 3 M_d; the directional stencils, subsets
// of the central one, hold at most M cells together): exactly the M central
// cells, the members of the three directional stencils first, one stencil
// after the other, then the central cells of no directional stencil.
inline bool ho_var_groups(int r) { return r >= 4 && dims_M(r) < 3 * dims_Md(r); }
inline int dims_S(int r) {
    if (ho_var_groups(r)) return dims_M(r);
    return dims_M(r) > 3 * dims_Md(r) ? dims_M(r) : 3 * dims_Md(r);
}
inline int dims_Nq(int r) { return (r + 2) / 2; }
// r >= 4: every slot carries K central and K_d directional entries; scalar
// physics pads them to a multiple of 4, so that a lane per cell reads each slot
// as a whole number of 16-byte vectors
inline int ho_slot_entries(int r, int nv) {
    const int n = dims_K(r) + dims_Kd(r);
    return nv == 1 ? (n + 3) / 4 * 4 : n;
}

// tiled index: per-cell array with E entries, 64-cell tiles, entry-major inside a tile
__host__ __device__ inline size_t tix(int64_t i, int e, int E) {
    return ((size_t)(i >> 6) * E + e) * kTile + (i & 63);
}
// vector-tiled index (array of structures of arrays): entries are grouped in
// vectors of VW consecutive entries per cell, vectors tiled like tix; a lane
// reads VW entries with one 16-byte load and a wave reads 1 KiB contiguously.
// E must be a multiple of VW.  Returns the scalar index of entry e.
__host__ __device__ inline size_t avix(int64_t i, int e, int E, int VW) {
    return ((((size_t)(i >> 6) * (E / VW) + e / VW) * kTile + (i & 63)) * VW) + (e % VW);
}
inline int64_t pad64(int64_t n) { return (n + kTile - 1) / kTile * kTile; }
inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

// Entries of a cell's pseudo-inverse stream, slot by slot.  r <= 3: for slot j
// the K central entries P_c[k][j], then (j < 12) the two directional entries
// P_d[j/4][c][j%4]; pinv_offset is slot j's first entry in that order (the
// order of the stream in memory is quad_index's).
__host__ __device__ constexpr int pinv_offset(int j, int K) {
    return j <= 12 ? j * (K + 2) : 12 * (K + 2) + (j - 12) * K;
}
inline int pinv_entries(int r, int nv) {
    return r <= 3 ? pinv_offset(dims_S(r), dims_K(r)) : dims_S(r) * ho_slot_entries(r, nv);
}
// r <= 3: the stream feeds 4 x 4 matrix instructions, four coefficients (rows)
// by the variables (columns).  The K + 2 coefficients of a slot form MA full row
// groups of central ones (0..3, and 4..7 at degree 3) and one last group: the
// last central coefficient (row 0) and the two directional ones of slots 0..11
// (rows 1 and 2).
template <int R>
struct QuadDims {
    static constexpr int K = (R + 1) * (R + 2) / 2 - 1;
    static constexpr int M = 2 * K;
    static constexpr int S = M > 12 ? M : 12;
    static constexpr int SP = (S + 3) / 4 * 4;
    static constexpr int MA = R == 3 ? 2 : 1;
    static constexpr int G = (S + 3) / 4;          // groups of four slots
    static constexpr int SK = (G + 1) / 2 * 2;     // row numbers per cell and slot % 4
    static constexpr int E = pinv_offset(S, K);
    static_assert(K == 4 * MA + 1, "row groups of degree 2 and 3");
};
// Scalar index of coefficient e (0..K-1 central, K, K + 1 directional) of slot j
// of cell i, in tiles of 16 cells (one wave).
//   FP32 (VW 4): an instruction takes one slot of 16 cells, lane 4 c + o row o
//   of cell c.  A lane's entries in slot order, in vectors of four (rows of 64
//   lanes): the full groups; then the last group's of slots 0..11 for rows 0..2;
//   then its row 0 of slots 12..15 (a vector) and 16, 17 (a pair).
//   FP64 (VW 2): an instruction takes four slots of four cells, lane 16 k + 4 b
//   + o slot 4 g + k, row o of cell 4 s + b.  Per s: the full groups in pairs
//   (degree 3: both groups of a g; degree 2: g = 0, 1, then g = 2 alone; the
//   last g of degree 3 has k < 2 only); the last group's g = 0, 1 in pairs and
//   g = 2 alone for rows 0..2, then row 0 of g = 3 and (k < 2) g = 4.
template <int R>
__host__ __device__ inline size_t quad_index(int64_t i, int j, int e, int VW) {
    using D = QuadDims<R>;
    constexpr int MA = D::MA, NA = D::S * MA;
    const int c16 = (int)(i & 15);
    const size_t base = (size_t)(i >> 4) * (D::E * 16);
    const int m = e / 4, o = e % 4;                 // last group: m = MA, o = 0..2
    if (VW == 4) {
        if (m < MA) {
            const int p = j * MA + m;
            return base + (size_t)((p / 4 * 16 + c16) * 4 + o) * 4 + p % 4;
        }
        const size_t b = base + NA * 64;
        if (j < 12) return b + (size_t)((j / 4 * 16 + c16) * 3 + o) * 4 + j % 4;
        if (j < 16) return b + 576 + c16 * 4 + (j - 12);
        return b + 640 + c16 * 2 + (j - 16);
    }
    const int k = j & 3, g = j >> 2, kb = 4 * k + (c16 & 3), lane = 4 * kb + o;
    const size_t sb = base + (size_t)(c16 >> 2) * (D::E * 4);
    if (m < MA) {
        if (R == 3) return sb + (size_t)g * 128 + lane * 2 + m;
        return g < 2 ? sb + lane * 2 + g : sb + 128 + lane;
    }
    const size_t b = sb + (R == 3 ? 576 : 192);
    if (g < 2) return b + (kb * 3 + o) * 2 + g;
    if (g == 2) return b + 96 + kb * 3 + o;
    return b + 144 + (g - 3) * 16 + kb;
}
// index of slot j's entry in a mesh's row-number table: per cell the slots 0, 4,
// 8, ..., then 1, 5, 9, ... (padded to SK each)
template <int R>
__host__ __device__ inline size_t lslot_index(int64_t i, int j) {
    constexpr int SK = QuadDims<R>::SK;
    return (size_t)i * (4 * SK) + (j & 3) * SK + (j >> 2);
}
inline int row_entries(int r) { return 4 * (r == 2 ? QuadDims<2>::SK : QuadDims<3>::SK); }
// entry e in pinv_offset's order
template <int R>
__host__ __device__ inline size_t quad_index_entry(int64_t i, int e, int VW) {
    constexpr int K = QuadDims<R>::K;
    const int j = e < 12 * (K + 2) ? e / (K + 2) : 12 + (e - 12 * (K + 2)) / K;
    return quad_index<R>(i, j, e - pinv_offset(j, K), VW);
}
// Degree 4 to 6, Euler: the K + K_d coefficients of a slot as NF full row groups
// of four and REM rows more, in tiles of 16 cells.  Coefficient e of slot j:
//   FP32 (VW 4): by groups of four slots (two in degree 6's last).  Lane 4 c + o
//   has row o of cell c: per row group a vector of its entries in slot order;
//   the REM rows likewise without gaps.
//   FP64 (VW 2): by cells 4 s + b, then groups of four slots.  Lane 16 k + 4 b +
//   o has slot 4 g + k, row o: row groups in pairs (a vector), then a single one,
//   then the REM rows without gaps.
template <int R>
struct HoRows {
    static constexpr int K = (R + 1) * (R + 2) / 2 - 1;
    static constexpr int RD = (R + 1) / 2;
    static constexpr int C = K + (RD + 1) * (RD + 2) / 2 - 1;
    static constexpr int S = R == 6 ? 54 : 2 * K;
    static constexpr int NF = C / 4, REM = C % 4;
    static constexpr int G = (S + 3) / 4, TAIL = S % 4;    // slots of an incomplete last group
    static constexpr int E = S * C;
    static_assert(REM == 0 || TAIL == 0, "an incomplete group of slots has full row groups only");
};
template <int R>
__host__ __device__ inline size_t ho_index(int64_t i, int j, int e, int VW) {
    using D = HoRows<R>;
    const int c16 = (int)(i & 15), g = j >> 2, k = j & 3, m = e / 4, o = e % 4;
    const size_t base = (size_t)(i >> 4) * (D::E * 16);
    if (VW == 4) {
        const size_t b = base + (size_t)g * (64 * D::C);
        if (D::TAIL && g == D::G - 1) return b + (size_t)(m * 64 + 4 * c16 + o) * D::TAIL + k;
        if (m < D::NF) return b + (size_t)(m * 64 + 4 * c16 + o) * 4 + k;
        return b + D::NF * 256 + (size_t)(c16 * D::REM + o) * 4 + k;
    }
    const int n = D::TAIL && g == D::G - 1 ? 4 * D::TAIL : 16;     // (slot, cell) pairs of the group
    const int kb = 4 * k + (c16 & 3), lane = 4 * kb + o;
    const size_t b = base + (size_t)(c16 >> 2) * (D::E * 4) + (size_t)g * (16 * D::C);
    if (m < (D::NF & ~1)) return b + (size_t)((m / 2) * 4 * n + lane) * 2 + m % 2;
    if (m < D::NF) return b + (size_t)m * 4 * n + lane;
    return b + (size_t)D::NF * 4 * n + kb * D::REM + o;
}

// neighbour code per cell face: bit 31 set = boundary (bits 0..1 = kind),
// else bits 0..27 neighbour (internal index), 28..29 neighbour's local
// face, bit 30 = this cell owns the face
constexpr uint32_t kNbBoundary = 0x80000000u;
constexpr uint32_t kNbOwner = 0x40000000u;
constexpr uint32_t kNbIndexMask = 0x0FFFFFFFu;
// boundary faces: kind in bits 0-1; an inflow face's row in the inflow table in bits 2-29
constexpr uint32_t kNbInflowMask = 0x0FFFFFFFu;
// listed faces of a fused-stage block (at most 256 cells): bits 0..7 the
// evaluating cell in the block, 8..9 its local face; bits 10..17 the other cell
// and 18..19 its local face, or bit 31 and the boundary kind in bits 10..11
constexpr uint32_t kBfBoundary = 0x80000000u;
// side records: the other side's number in bits 0..27, kNbOwner, and whether the
// other cell lies in another 256-cell block
constexpr uint32_t kSideFar = 0x80000000u;
// slot entries at degree >= 4: bits 0..27 the cell (internal index), bits
// 28..29 the directional stencil (face 0..2) that holds it, 3 for none
constexpr uint32_t kSlotIndexMask = 0x0FFFFFFFu;
constexpr int kSlotGroupShift = 28;
constexpr uint32_t kSlotNoGroup = 3u;

// allocator whose new elements are left uninitialised (default-initialised):
// for arrays that the parallel mesh layout writes in full, so that no serial
// zero fill runs first
template <typename T>
struct NoInitAlloc : std::allocator<T> {
    template <typename U> struct rebind { using other = NoInitAlloc<U>; };
    NoInitAlloc() = default;
    template <typename U> NoInitAlloc(const NoInitAlloc<U> &) noexcept {}
    template <typename U> void construct(U *p) noexcept { ::new (static_cast<void *>(p)) U; }
    template <typename U, typename... A> void construct(U *p, A &&...a) {
        ::new (static_cast<void *>(p)) U(std::forward<A>(a)...);
    }
};
template <typename T> using raw_vector = std::vector<T, NoInitAlloc<T>>;

// ---------------------------------------------------------------------------
// host mesh builder output (all in internal order unless noted)
// ---------------------------------------------------------------------------
struct HostMesh {
    int N = 0, r = 0, K = 0, M = 0, S = 0, nv = 0, Kd = 0, Md = 0, Nq = 0;
    int per_x = 0, per_y = 0;
    double Lx = 0, Ly = 0;
    int64_t n_faces = 0, n_boundary = 0;
    int n_inadmissible = 0;
    std::vector<int32_t> perm;     // internal -> user
    std::vector<int32_t> iperm;    // user -> internal
    // user-order stencils (for inspection)
    std::vector<int32_t> cen_user;     // [N][M] ascending user ids
    std::vector<int32_t> dir_user;     // [N][3][Md] user ids, -1 padded
    std::vector<int32_t> dirn_user;    // [N][3]
    // internal-order device inputs
    int SP = 0;                        // slots padded to a multiple of 4
    raw_vector<int32_t> slot;          // vector-tiled [SP] (VW 4): internal cell index (self for pads)
    raw_vector<uint8_t> slot_flag;     // tiled [S]: bit0 central member, bit1 directional member
    raw_vector<int8_t> slot_shift;     // tiled [2*S]: periodic image shift (x then y)
    raw_vector<uint8_t> flags;         // [Npad]: bit s = directional stencil of face s admissible
    raw_vector<double> verts;          // tiled [6]: CCW vertex coordinates x0,y0,x1,y1,x2,y2
    // face records: per local face (nx, ny, |A|, neighbour code), vector-tiled
    raw_vector<double> fr64;           // [12] entries, VW 2; code stored in the low bits of the double
    raw_vector<float> fr32;            // [12] entries, VW 4; code stored as the float's bits
    raw_vector<double> area;           // [Npad]
    // inflow faces: first vertex (x, y) and edge vector, rows in internal cell order
    std::vector<double> bface;         // [n_inflow][4]
    double bst[2][4] = {};             // prescribed states behind / ahead of the moving line
    double bline[3] = {};              // x = bline[0] + bline[1] y + bline[2] t
};

// host threads the calling thread's mesh builds may use (default 16)
void set_builder_threads(int n);
// returns CTENO_OK or an error (message in err)
cteno_status build_host_mesh(const cteno_mesh_desc &d, const cteno_scheme &s, HostMesh &hm, std::string &err);

// ---------------------------------------------------------------------------
// constant tables of the reference triangle (host-computed, FP64)
// ---------------------------------------------------------------------------
struct RefTables {
    int K = 0, Nq = 0;
    int ex[kMaxK][2];               // exponents of psi_k
    double mean[kMaxK];             // mean of psi_k over the reference triangle
    double gram[kMaxK][kMaxK];      // smoothness-indicator Gram matrix
    double basis[3][kMaxNq][kMaxK]; // phi_k at the face Gauss points
    double gq[kMaxNq], gw[kMaxNq];  // Gauss points and weights on [0, 1]
};
void make_ref_tables(int r, RefTables &t);

// ---------------------------------------------------------------------------
// device-side control block of a time march
// ---------------------------------------------------------------------------
struct Ctrl {
    double t, t_next, t_final, dt, cfl;
    unsigned long long dt_cand_bits;   // min over cells of the dt bound (bits of a positive double)
    long long step, max_steps;
    int done, pending, nonphysical, pad;
    unsigned long long fallbacks;      // cells x stages that took the positivity fallback
};

}  // namespace cteno
