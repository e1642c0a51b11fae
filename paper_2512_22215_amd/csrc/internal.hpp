// Internal declarations of the LDU pressure-solve library (gfx950).
//
// Data layout in HBM, per multigrid level:
//  - face form (owner, neighbour, upper, lower: the lduMatrix arrays of
//    paper Sec. 2.1) plus ownStart[i], the first face owned by cell i;
//  - a sliced-ELLPACK copy for the product kernels: rows in slices of 64
//    (one wavefront), slice s holding width_s = max row length in the slice;
//    entry k of row r = 64 s + lane sits at sptr[s] + 64 k + lane, so a
//    wavefront streams 64 consecutive int32 columns and 64 consecutive values
//    per step.  Row entries are column-sorted: the "lower" faces (columns
//    below the row) first, then the "upper" ones.  Padding entries point at
//    their own row with value 0.  val holds A, valT holds A^T at the same
//    positions, so the transposed product runs the same kernel.
//  - levels whose row lengths vary (the Galerkin coarse levels: 3 to ~27
//    entries, which pads max-width slices by 40-50%) use compressed slices:
//    inside each slice of 64 rows the rows are ordered by length (longest
//    first; perm maps a slice position to its row, iperm back), and entry k
//    of lane l is stored at sptr[s] + otab[tptr[s] + k] + l, where
//    otab[tptr[s] + k] counts the entries of the slice's first k columns.
//    Nothing is padded, and a row's loads and stores stay inside the slice's
//    own cache lines.
//  - 16-bit columns: for each stored column k of a slice (a "slot": the k-th
//    entries of the slice's rows), cbase holds the smallest column of the
//    slot and c16 each entry's column minus that base.  Slots that span at
//    most 65535 columns use them in the product kernels (2 bytes per entry
//    instead of 4, and a shorter stream between the reuses of x); wider
//    slots have base -1 and read the 32-bit columns.  A level without any
//    narrow slot keeps c16 = NULL.  The slot of (s, k) is (sptr[s] / 64) + k
//    in plain slices and tptr[s] + k in compressed ones (which keep 32-bit
//    columns).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <stdexcept>
#include <string>
#include <vector>

#include "arena.hpp"
#include "ldu.h"

namespace ldu {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxGrid = 2048;     // streaming kernels: at most this many blocks
// FP64 products on plain slices: at most this many blocks walk slices (the
// rest only contribute zero partials).  Four waves per SIMD instead of eight
// keep fewer of the streamed matrix lines in flight, so more of x survives
// in L2 between its reuses one mesh plane apart.
#ifndef LDU_PLAIN_F64_BLOCKS
#define LDU_PLAIN_F64_BLOCKS 1024
#endif
constexpr int kPlainF64ProductBlocks = LDU_PLAIN_F64_BLOCKS;
#ifndef LDU_CMP_BATCH
#define LDU_CMP_BATCH 24
#endif
constexpr int kCmpBatch = LDU_CMP_BATCH;  // compressed-slice row products: entries per batch
// level-0 vector kernels stream their vectors with nontemporal loads and
// stores above this many cells: four FP64 vectors then exceed the 256 MB
// Infinity Cache, which below it keeps them between kernels
#ifndef LDU_STREAM_NT_CELLS
#define LDU_STREAM_NT_CELLS 12000000
#endif
constexpr int64_t kStreamNtCells = LDU_STREAM_NT_CELLS;
// diagonal CG and PBiCG run an iteration as two kernels up to this many cells
// (the product forms the new direction in its gathers), as three above.  CG,
// two against three kernels: 32^3 2.87 and 3.50 ms, 48^3 4.79 and 5.73, 64^3
// 9.03 and 8.72, 100^3 50.6 and 26.3; PBiCG: 32^3 1.33 and 1.37 ms, 64^3 2.68
// and 2.39
#ifndef LDU_FUSED_CG_CELLS
#define LDU_FUSED_CG_CELLS 160000
#endif
constexpr int64_t kFusedCgCells = LDU_FUSED_CG_CELLS;
constexpr int64_t kFusedBicgCells = 1 << 16;
// blocks of the CG forms' vector updates, whose partials every block of the
// next kernel reads (512, 1024 and 2048: 28.0, 26.3 and 27.5 ms for diagonal
// CG at 100^3, 117.0, 108.9 and 109.4 ms at 150^3)
#ifndef LDU_CG_BLOCKS
#define LDU_CG_BLOCKS 1024
#endif
constexpr int kCgBlocks = LDU_CG_BLOCKS;
// above this many cells they run on kMaxGrid blocks: with four waves a SIMD the
// streams of one kernel leave HBM bandwidth unused, and reading twice the partials
// costs less.  1024 and 2048 blocks, us an iteration of diagonal CG in FP64 and
// mixed: 128^3 61.9 and 62.0, 41.5 and 42.9; 160^3 119.2 and 120.2, 72.2 and
// 72.8; 200^3 240.0 and 236.3, 130.8 and 131.0; 256^3 502 and 492, 293 and 278
// (with reductions of their own: 496, 283)
constexpr int64_t kCgWideCells = 6000000;
// Meshes of at least this many cells are checked for a scattered numbering
// when a hierarchy is built; levels above kRenumberRows are renumbered.
// Shuffled boxes, levels as they are and renumbered, default GAMG to 1e-8: 48^3
// 9.9 and 10.7 ms, 64^3 17.0 and 13.3, 80^3 20.2 and 14.9, 100^3 45.1 and 26.3;
// CG + V-cycle, merged: 4.1 and 4.1, 7.3 and 5.8, 11.5 and 7.8, 26.2 and 13.2;
// set-up 17.2 and 19.1, 21.2 and 22.7, 24.8 and 26.1, 31.0 and 34.4.  From
// 500,000 cells one solve pays for the copies; below, the break-even lies near
// 64^3 and a caller of one loose solve would lose.  Renumbering levels of more
// than 4000, 20,000 and 100,000 rows: set-up and GAMG at 128^3 46.2 + 34.3, 45.4
// + 34.4 and 44.4 + 34.8 ms, CG + V-cycle at 100^3 13.3, 13.4 and 13.9 ms.
#ifndef LDU_RENUMBER_CELLS
#define LDU_RENUMBER_CELLS 500000
#endif
constexpr int64_t kRenumberCells = LDU_RENUMBER_CELLS;
constexpr int32_t kRenumberRows = 20000;
// A matrix is read with the default cache policy (SellView::stream false) when
// it and the vectors used between two passes over it fit the 256 MB Infinity
// Cache, else nontemporally, so that it leaves the vectors there.  Diagonal CG,
// streaming against keeping the matrix: 100^3 (100 MB) 26.3 and 24.9 ms, 125^3
// (211 MB) 57.9 and 52.2, 150^3 (364 MB) 109.0 and 118.3; PBiCG 100^3 (188 MB)
// 7.49 and 6.80 ms, 125^3 (367 MB) 12.8 and 13.3; standalone GAMG, whose
// cycles sweep a level several times in a row, 128^3 33.6 and 31.9 ms; CG +
// V-cycle passes over each level's operators once in turn and streams them
// (100^3 15.5 and 16.3 ms, 200^3 125.0 and 132.8).
constexpr int64_t kCacheBytes = int64_t(240) << 20;
constexpr int kMaxLevels = 64;
constexpr int kMaxCoarseRow = 128; // widest coarse-level row the setup supports
constexpr double kCoarsestTol = 1e-10;
// residual history entries kept on the device per solve (the first ones)
constexpr int64_t kMaxHistory = int64_t(1) << 20;
// largest coarsest level (with off-diagonal entries) the single-workgroup CG
// accepts: its iteration cap max(2n, 100) keeps that kernel to a fraction of
// a second; a hierarchy cut off above it (max_levels, stalled coarsening) is
// refused at setup
constexpr int kMaxCoarsest = 8192;

// ---------------------------------------------------------------- errors
void hip_fail(hipError_t e, const char *what, const char *file, int line);
#define HIP_CHECK(x)                                                        \
    do {                                                                    \
        hipError_t e_ = (x);                                                \
        if (e_ != hipSuccess) ::ldu::hip_fail(e_, #x, __FILE__, __LINE__); \
    } while (0)

// ---------------------------------------------------------------- views
template <typename T>
struct SellView {
    int32_t n;
    int64_t nslices;
    const int64_t *sptr;
    const int32_t *col;
    const T *val;
    const T *diag;
    const int32_t *perm;   // row stored at slice position p (NULL: identity)
    const int32_t *iperm;  // slice position of row i (NULL: identity)
    const int32_t *pdeg;   // compressed slices: entries of the row at position p
    const int32_t *tptr;   // compressed slices: start of slice s in otab
    const int32_t *otab;   // compressed slices: offset of entry k within slice s
    const uint16_t *c16;   // column minus its slot base (NULL: use col)
    const int32_t *cbase;  // smallest column of each slot (-1: slot uses col)
    bool stream = true;    // columns and values are read past the caches
};

// scalars shared between the kernels of one solve; device resident
struct DevScalars {
    double rr, bb, rz, rho, pq, alpha, beta, res, bnorm, tol;
    double maxabs, scale;       // mixed: ||r||_inf of the outer residual
    double r0, inner_tol;       // mixed inner CG
    double inner_now;           // mixed: current inner tolerance
    double mean;                // coarsest: rhs mean
    int iters, max_iter, done, status;
    int inner_iters, inner_max, inner_done;
    int x_pending;              // CG: the iteration's x += alpha p is formed but not yet applied
    unsigned int ticket;        // grid reduction arrival counter (always 0 between kernels)
    unsigned int pad2_;
};

// done codes
enum { kRunning = 0, kConverged = 1, kMaxIter = 2, kFailed = 3 };

// ---------------------------------------------------------------- storage
struct DeviceBuffer {
    void *p = nullptr;
    size_t bytes = 0;
};

struct Sell {
    int32_t n = 0;
    int64_t nslices = 0, nnz = 0;
    int64_t *sptr = nullptr;
    int32_t *col = nullptr;
    double *val = nullptr, *valT = nullptr;
    float *val32 = nullptr, *valT32 = nullptr;
    double *diag = nullptr;
    float *diag32 = nullptr;
    // compressed slices (levels with uneven rows): lanes sorted by row length
    int32_t *perm = nullptr, *iperm = nullptr, *pdeg = nullptr, *tptr = nullptr, *otab = nullptr;
    // 16-bit column offsets and slot bases (c16 NULL when some slot is too wide)
    uint16_t *c16 = nullptr;
    int32_t *cbase = nullptr;

    // bytes of one pass over columns and values of this size each
    int64_t bytes(size_t value) const {
        return nnz * (int64_t)((c16 ? sizeof(uint16_t) : sizeof(int32_t)) + value);
    }
    __host__ __device__ SellView<double> view(bool transpose) const {
        return {n,    nslices, sptr, col,  transpose ? valT : val, diag, perm, iperm, pdeg,
                tptr, otab,    c16,  cbase};
    }
    __host__ __device__ SellView<float> view32(bool transpose) const {
        return {n,    nslices, sptr, col,  transpose ? valT32 : val32, diag32, perm, iperm, pdeg,
                tptr, otab,    c16,  cbase};
    }
};

// rows stored one after another, each row's entries contiguous and in
// column order (the restriction operators R)
template <typename T>
struct CsrView {
    int32_t n;
    const int64_t *rptr;
    const int32_t *col;
    const T *val;
    int group;  // lanes that share a row in the product kernel
    int64_t nnz;
};

struct Csr {
    int32_t n = 0;
    int64_t nnz = 0;
    int64_t *rptr = nullptr;  // [n + 1]
    int32_t *col = nullptr;
    double *val = nullptr, *valT = nullptr;
    float *val32 = nullptr, *valT32 = nullptr;
    int group = 1;
    __host__ __device__ CsrView<double> view(bool transpose) const {
        return {n, rptr, col, transpose ? valT : val, group, nnz};
    }
    __host__ __device__ CsrView<float> view32(bool transpose) const {
        return {n, rptr, col, transpose ? valT32 : val32, group, nnz};
    }
};

// lanes per row of a CSR product: the power of two nearest the mean row
// length over this many entries per lane, from 1 to 16 (every lane then
// loads its few entries at once, so a long row costs one round trip instead
// of a chain of batches)
#ifndef LDU_CSR_ENTRIES_PER_LANE
#define LDU_CSR_ENTRIES_PER_LANE 2
#endif
constexpr int kCsrEntriesPerLane = LDU_CSR_ENTRIES_PER_LANE;
constexpr int kCsrBatch = 8;  // entries a lane loads before its gathers
// a CSR operator of at most this many bytes (columns and values) is read with
// the default cache policy, so that it stays in the Infinity Cache from one
// V-cycle to the next; a larger one streams past it.  CG + V-cycle, streaming
// every operator against keeping the small ones: 100^3 17.0 -> 16.6 ms, mixed
// 128^3 31.7 -> 30.1 ms; keeping an operator of 83 MB as well (151x143x139
// step): 13.8 -> 14.1 ms
constexpr int64_t kCsrCachedBytes = int64_t(64) << 20;
// restriction operators with at most this many rows are stored in CSR: there
// a row's lanes load its entries in one round trip.  Above it compressed
// slices win: a lane per row keeps the matrix stream coalesced, and there
// are enough rows to hide the chain of batches
#ifndef LDU_R_CSR_MAX_ROWS
#define LDU_R_CSR_MAX_ROWS 300000
#endif
constexpr int64_t kCsrMaxRows = LDU_R_CSR_MAX_ROWS;

struct Level {
    int32_t n = 0;
    int64_t nf = 0;
    int32_t *own = nullptr, *nb = nullptr;
    double *upper = nullptr, *lower = nullptr, *diag = nullptr;
    int64_t *ownStart = nullptr;          // [n+1]
    int64_t *slotU = nullptr, *slotL = nullptr;  // [nf] positions in the SELL arrays
    Sell A;
    int32_t *src = nullptr;  // renumbered levels: source of each entry of A (-1: padding)
    int32_t *order = nullptr;  // and the cell of each position
    // aggregation to the next level (absent on the coarsest level)
    int32_t nc = 0;
    int32_t *agg = nullptr, *aggStart = nullptr, *aggCells = nullptr;
    // the fine faces each Galerkin sum visits, in its order: per coarse face
    // (cfStart[ncf+1], cfFace: f if the fine owner lies in the coarse owner,
    // else ~f), and per coarse cell its internal fine faces (ciStart, ciFace)
    int64_t *cfStart = nullptr, *ciStart = nullptr;
    int32_t *cfFace = nullptr, *ciFace = nullptr;
    // the down leg of a cycle with one Jacobi pre-sweep from zero as one
    // operator: R = P^T (I - omega A D^-1), a row per coarse cell over this
    // level's columns (valT: the same for A^T), in compressed slices (R) when
    // it has more than kCsrMaxRows rows, else in CSR (Rc)
    Sell R;
    Csr Rc;
    // on a plain-slice level whose R would need compressed slices, the down
    // leg runs over this level's own slices instead: t = (I - omega A D^-1) r
    // with the values -omega a_ij / D_j stored at A's positions (ah; ahT the
    // same for A^T; padding 0), then the member sums of t
    double *ah = nullptr, *ahT = nullptr;
    // scaled slices: A's columns mapped to aggregates, for the up leg's
    // A P e_c (ac32 only when some slot is too wide for 16 bits)
    uint16_t *ac16 = nullptr;
    int32_t *acbase = nullptr, *ac32 = nullptr;
    float *ah32 = nullptr, *ahT32 = nullptr;
    // on small levels (kUpRows) the up leg of the same cycles as one operator
    // over the stacked vector (r, e_c): e = U (r, e_c), a row per cell
    Csr Uc;
    // small levels of the other Jacobi cycles (several pre-sweeps, or scaled
    // corrections): rows of A with their Q entries behind (V; qptr: where they
    // start), and the restriction of the residual over (r, e) (W)
    Csr V, W;
    int64_t *qptr = nullptr;
    int64_t *w_src = nullptr, *w_src0 = nullptr;  // sources of W's entries, as R's
    int32_t *w_srcn = nullptr;                    // (count 0: a member, value 1)
    double g_omega = 0.0;
    bool g_ready = false;                 // V's and W's values match the coefficients
    bool g_wide = false;                  // a row is too wide for V or W
    int64_t *r_src = nullptr;             // sources of R's entries, by entry in runs:
    int64_t *r_src0 = nullptr;            //   first source of each entry of R
    int32_t *r_srcn = nullptr;            //   and their count (source -1: a diagonal)
    double r_omega = 0.0;                 // omega the values of R were made for
    bool r_ready = false;                 // R's values match the coefficients
    int singular = 0;                     // coarsest level: A 1 = 0
    int max_row = 0;                      // longest row (off-diagonal entries)
    // V-cycle work vectors
    double *r = nullptr, *e = nullptr, *e2 = nullptr, *t = nullptr;
    float *r32 = nullptr, *e32 = nullptr, *e232 = nullptr, *t32 = nullptr;
    // second ping-pong buffer of the two-stage Gauss-Seidel inner steps
    // (allocated when a cycle asks for three or more of them)
    double *w = nullptr;
    float *w32 = nullptr;
};

}  // namespace ldu

// the opaque handle of the C ABI
struct ldu_t {
    int device = 0;
    bool poisoned = false;
    ldu::ChunkPool pool;         // chunks of the temporary arenas of one call
    ldu::Arena arena;            // level-0 and solver buffers
    ldu::Arena gamg_arena;       // hierarchy buffers (rebuilt by gamg_setup)
    ldu::Level L0;
    std::vector<ldu::Level> levels;  // levels[0] aliases L0's arrays when built
    // the same levels renumbered for the solves, on a large mesh whose own
    // numbering scatters its neighbours (gamg.hip, NumberingScope; empty on
    // other meshes).  Small levels share their arrays with `levels`.
    ldu::Level inner_L0;
    std::vector<ldu::Level> inner;
    int32_t *inner_order = nullptr;          // cell of each inner position, level 0
    double *inner_b = nullptr, *inner_x = nullptr;
    bool inner_stale = false;        // the renumbered levels wait for the last coefficients
    bool gamg_ready = false;
    ldu_gamg_opts gamg_opts{};
    bool f32_ready = false;          // FP32 copies of level values exist
    // solver buffers
    double *r = nullptr, *p = nullptr, *q = nullptr;
    double *z = nullptr, *p2 = nullptr;  // z = M^-1 r, and p's second buffer (two-kernel CG)
    double *rt = nullptr, *pt = nullptr, *qt = nullptr;  // PBiCG shadow vectors
    double *zt = nullptr, *pt2 = nullptr;
    float *r32 = nullptr, *p32 = nullptr, *q32 = nullptr, *d32 = nullptr;
    double *partials = nullptr;      // [4 * kMaxGrid]
    ldu::DevScalars *dev = nullptr;  // [2]: the second for kernels that pass scalars on
    ldu::DevScalars *host = nullptr; // pinned mirror
    double *hist = nullptr;          // device residual history
    int hist_cap = 0;
    int *flag = nullptr;             // device error flag (validation)
    int *hflag = nullptr;            // pinned
    double *coarse_work = nullptr;   // coarsest-level CG scratch (5 n doubles)
    double *dic_dt = nullptr;        // coarsest-level DIC pivots
    bool dic_ready = false;          // dic_dt matches the current coarsest values
    bool dic_ok = false;             // every pivot usable (else diagonal fallback)
};

namespace ldu {

// ---------------------------------------------------------------- launch helpers
inline int stream_grid_slices(int64_t nslices) {
    int64_t g = (nslices + kWavesPerBlock - 1) / kWavesPerBlock;
    if (g > kMaxGrid) g = kMaxGrid;
    if (g >= 64) g &= ~int64_t(7);
    if (g < 1) g = 1;
    return (int)g;
}
// blocks of a CG form's vector updates over n cells, at most G
inline int cg_blocks(int64_t n, int G) {
    const int most = n > kCgWideCells ? kMaxGrid : kCgBlocks;
    return G < most ? G : most;
}
inline int64_t slices_of(int64_t n) { return (n + kWave - 1) / kWave; }

// relayout.hip
void build_level_sell(ldu_t *h, Arena &ar, Level &L, bool validate, hipStream_t st);
void set_level_values(Level &L, hipStream_t st);   // face values -> SELL values
// slices for n rows of the given lengths (device array), plain or compressed;
// returns the number of slots
int64_t layout_rows(Sell &A, int32_t n, const int32_t *deg, int64_t nnz, Arena &ar, Arena &tmp,
                    hipStream_t st);
// the columns of a level's plain slices mapped through its aggregate map
void aggregate_columns(Level &L, Arena &ar, Arena &tmp, hipStream_t st);
// A with its rows in the order `order` (cell of each position; place: position
// of each cell) and its columns renumbered, each row in ascending column order
void build_renumbered(const Sell &A, int64_t nf, const int32_t *order, const int32_t *place,
                      Level &out, Arena &ar, hipStream_t st);
void renumbered_values(const Sell &A, Level &L, hipStream_t st);
bool scattered_numbering(ldu_t *h, hipStream_t st);
void gather_cells(const double *a, const int32_t *order, double *out, int64_t n, hipStream_t st);
void scatter_cells(const double *a, const int32_t *order, double *out, int64_t n, hipStream_t st);
void build_sliced_rows(Sell &A, int32_t n, const int32_t *deg, Arena &ar,
                       hipStream_t st);  // compressed slices for given row lengths
void assemble_pressure(ldu_t *h, const double *gamma, const double *w, const double *mag_sf,
                       const double *delta, const double *diag_bc, const double *phi,
                       const double *b_bc, double *b, hipStream_t st);
void ensure_f32(Level &L, Arena &ar, bool own, hipStream_t st);
void refresh_f32(Level &L, hipStream_t st);
void exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, Arena &tmp,
                        hipStream_t st);  // out has n+1 entries
void scan_counts_i32(const int32_t *cnt, int32_t *out, int64_t n, Arena &tmp,
                     hipStream_t st);     // out has n+1 entries, int32
void check_finite(ldu_t *h, const double *a, int64_t n, hipStream_t st);

// spmv_pcg.hip
void launch_amul(const SellView<double> &A, const double *x, double *y, hipStream_t st);
void launch_amul32(const SellView<float> &A, const float *x, float *y, hipStream_t st);
void read_scalars(ldu_t *h, hipStream_t st);
int next_batch(double res0, double res, int steps, double tol, int first, int most);
void set_scalars_for_solve(ldu_t *h, double tol, int max_iter, hipStream_t st);
double residual_norm(ldu_t *h, const Level &L, bool tr, const double *b,
                     const double *x, double *r_out, hipStream_t st);
int pcg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o,
             bool tr, ldu_stats *stats, hipStream_t st, bool own_hist = true);
int pbicg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
               ldu_stats *stats, hipStream_t st);
int pcg_mixed(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o,
              bool tr, ldu_stats *stats, hipStream_t st);
void ensure_hist(ldu_t *h, int64_t entries);
// noalloc.hip: the allocation-free diagonal-PCG entry point's static scratch
constexpr int64_t kNoAllocMaxCells = int64_t(1) << 20;
constexpr int kNoAllocHistory = 4096;
void noalloc_init(int device);
int pcg_fp64_noalloc(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o,
                     ldu_stats *stats, hipStream_t st);
void copy_history(ldu_t *h, ldu_stats *stats, int count, hipStream_t st);
void launch_coeff_grad(const Level &L, const double *lam, const double *x,
                       double *gd, double *gu, double *gl, hipStream_t st);
void launch_residual_cycle(ldu_t *h, const SellView<double> &A, const double *b,
                           const double *x, double *r, bool maxabs, int grid,
                           hipStream_t st);
void zero_vector(double *a, int64_t n, hipStream_t st);
void launch_residual_plain(ldu_t *h, const SellView<double> &A, const double *b,
                           const double *x, double *r, bool write_hist, int grid,
                           hipStream_t st);
// q = A p and the partials of p.q, unless the scalars in ds say done
void launch_product_dot(ldu_t *h, const SellView<double> &A, const double *p, double *q, int grid,
                        const DevScalars *ds, hipStream_t st);
void set_done(ldu_t *h, int done, hipStream_t st);
// convergence step after an r update whose partials hold ||r||^2
void launch_converge(ldu_t *h, const double *partials, int grid, hipStream_t st);
// x += alpha p if a stopped CG still owes it
void launch_x_pending(ldu_t *h, double *x, const double *p, int32_t n, int64_t S, int grid,
                      hipStream_t st);

// gamg.hip
void gamg_build(ldu_t *h, const ldu_gamg_opts &o, hipStream_t st);
void gamg_refresh_values(ldu_t *h, hipStream_t st);
int gamg_fp64(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o,
              bool tr, ldu_stats *stats, hipStream_t st);
int gamg_mixed(ldu_t *h, const double *b, double *x, const ldu_gamg_opts &o,
               bool tr, ldu_stats *stats, hipStream_t st);
void gamg_vcycle64(ldu_t *h, const double *r, double *e, const ldu_gamg_opts &o,
                   bool tr, hipStream_t st);
int pcg_gamg_fp64(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                  ldu_stats *stats, hipStream_t st);
int pcg_gamg_mixed(ldu_t *h, const double *b, double *x, const ldu_pcg_opts &o, bool tr,
                   ldu_stats *stats, hipStream_t st);
void launch_mx_q(ldu_t *h, const SellView<float> &A32, int G, hipStream_t st);
void launch_mx_update_plain(ldu_t *h, int32_t n, int64_t S, int G, int Gq, hipStream_t st);
void set_inner(ldu_t *h, double inner_tol, int inner_max, hipStream_t st);
void launch_mx_refine(ldu_t *h, double *x, int32_t n, int64_t S, int G, hipStream_t st);

}  // namespace ldu
