// Internal declarations shared by the library's HIP translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <functional>
#include <string>
#include <vector>

#include "lsqr_mi355x.h"

namespace lsqr {

constexpr int kBlock = 256;          // threads per workgroup (4 wave64)
constexpr int kStateWords = 32;      // doubles per per-iteration state row

// Per-iteration state row S[k] (doubles), written by the update kernel of
// iteration k (k = 0 is the start) and read by the next iteration.
enum StateField {
    S_ALPHA = 0,    // alpha_{k+1}
    S_BETA = 1,     // beta_{k+1}
    S_RHOBAR = 2,   // rhobar_{k+1}
    S_PHIBAR = 3,   // phibar_{k+1} = |rbar_k| estimate
    S_RHO = 4,
    S_C = 5,
    S_S = 6,
    S_THETA = 7,
    S_PHI = 8,
    S_PSI = 9,      // |A_D^T rbar_k| estimate
    S_ETA = 10,     // psi_k |D^-1 v_{k+1}| / |Abar^T bbar|
    S_VNORM = 11,   // |D^-1 v_{k+1}|
    S_ARNORM0 = 12, // |Abar^T bbar| (row 0 only; LSMR: alpha_1 beta_1)
    // LSMR (Fong & Saunders): the second rotation chain and the |r| chain;
    // S_PHIBAR holds |r_k|, S_PSI |A_D^T r_k| = |zetabar_{k+1}|
    S_ALPHABAR = 13,
    S_ZETABAR = 14,
    S_CBAR = 15,
    S_SBAR = 16,
    S_ZETA = 17,
    S_BETADD = 18,
    S_BETAD = 19,
    S_RHODOLD = 20,
    S_TAUTILDE = 21,
    S_THETATILDE = 22,
    S_METHOD = 23,  // row 0: 0 LSQR, 1 LSMR (written by the start step)
};

// Control words (int32) on the device.
enum CtlField {
    C_STOP = 0,     // 1 once the solve has stopped
    C_ISTOP = 1,    // stop reason
    C_ITERS = 2,    // iterations completed
    C_ERR = 3,      // 1 if a scalar became non-finite
    C_CNT0 = 4,     // iteration counter read by iterations of parity 0
    C_CNT1 = 5,     // ... parity 1
    C_KMAX = 6,     // iteration limit of the current solve
    C_REQ = 7,      // fused iterations: a stop the forward kernel asked for
    C_WORDS = 8,
};

enum { MODE_ITER = 0, MODE_INIT = 1, MODE_OPERATOR = 2 };

// Element types of stored matrix values and of vectors.
enum ValType { VT_F64 = 0, VT_F32 = 1, VT_BF16 = 2, VT_F16 = 3 };
size_t vt_size(int vt);

struct Problem {
    int64_t m = 0, n = 0, nnz = 0;
    int32_t nx = 0, ny = 0, nz = 0;
    double w = 0.0, damp = 0.0;
};

// Data rows of the forward product.
// Most columns a row group may hold (its part of D v is staged in LDS: 56 KB
// at FP64, within the 64 KB a workgroup may take on any CDNA part).
constexpr int kLcolMaxCap = 7168;

struct RowFmt {
    int vt = VT_F64;
    const int64_t *rp = nullptr;       // [m+1] value offsets
    const int32_t *ci = nullptr;       // [nnz] columns (plain CSR)
    const void *val = nullptr;
    const float *sigma = nullptr;      // [m] row scales (quantised values) or nullptr
    int lpr = 64;                      // lanes per row (plain CSR)
    // plain CSR with 64 lanes per row: a launch of wgrid workgroups takes
    // contiguous row ranges balanced in entries, wrow[p] .. wrow[p+1]-1, one
    // per workgroup (its waves interleaved) or per wave (fwd_pipe_parts);
    // other launch sizes take rows w, w + waves, ...
    const int32_t *wrow = nullptr;     // [fwd_pipe_parts(wgrid) + 1]
    int wgrid = 0;
    // row groups with local columns (used instead of ci when slot is set):
    // group g = rows gp[g] .. gp[g+1]-1, its sorted columns gcol[gcp[g] ..
    // gcp[g+1]-1] (at most gcap), slot[p] = position of entry p's column
    // in its group's list.  With slot set, wrow holds the launch's group
    // ranges (wrow[b] .. wrow[b+1]-1 for workgroup b of wgrid).
    const int32_t *gp = nullptr;       // [ngroups + 1]
    const int64_t *gcp = nullptr;      // [ngroups + 1]
    const int32_t *gcol = nullptr;
    const uint16_t *slot = nullptr;    // [nnz]
    int ngroups = 0;
    int gcap = 0;                      // columns per group at most (<= kLcolMaxCap)
    int padded = 0;                    // zero elements val and slot hold past the last entry
};

// The row-group kernel with entries in pairs reads two values and two slots
// at a time from even positions, and one element past the last entry
// (RowFmt::padded).
static inline bool lcol_pairs_ok(const RowFmt &R)
{
    const uintptr_t w = 2 * (uintptr_t)vt_size(R.vt);
    return R.padded >= 1 && ((uintptr_t)R.val & (w - 1)) == 0 && ((uintptr_t)R.slot & 3u) == 0;
}

// Entries in quads (4- and 2-byte values): four values and four slots from
// positions that are multiples of four, and up to three elements past the
// last entry.  Measured on the paper-shaped system against pairs: FP32
// 699 -> 655 us, FP16 569 -> 527 us, BF16 585 -> 566 us.
#ifndef LSQR_FWD_QUADS
#define LSQR_FWD_QUADS 1
#endif
static inline bool lcol_quads_ok(const RowFmt &R)
{
    const uintptr_t w = 4 * (uintptr_t)vt_size(R.vt);
    return LSQR_FWD_QUADS && vt_size(R.vt) <= 4 && R.padded >= 3 && ((uintptr_t)R.val & (w - 1)) == 0 &&
           ((uintptr_t)R.slot & 7u) == 0;
}

// Entries in octets (16-bit codes): eight codes and eight slots, one 16-byte
// load each, from positions that are multiples of eight, and up to seven
// elements past the last entry.  Measured on the config-1 system against
// quads: BF16 532 -> 507 us, FP16 506 -> 467 us.
#ifndef LSQR_FWD_OCTS
#define LSQR_FWD_OCTS 1
#endif
static inline bool lcol_octs_ok(const RowFmt &R)
{
    return LSQR_FWD_OCTS && vt_size(R.vt) == 2 && R.padded >= 7 && ((uintptr_t)R.val & 15u) == 0 &&
           ((uintptr_t)R.slot & 15u) == 0;
}

// Parts of a node's runs with a stored value offset: a kernel whose 4 or 16
// waves share a node starts them there.
constexpr int kNodeParts = 16;
// Waves that share a node's runs in the transposed product (depth-pair
// layouts): 16 on grids of up to kWideNodes nodes, where a workgroup of 4 waves
// per node leaves most of the device idle, if a node has runs for them: at least
// 400, and twice as many as there are nodes (the more nodes, the more waves of
// the 4-wave workgroups are in flight already); else 4.  Transposed product, 4 ->
// 16 waves (us, FP64 / BF16): 64 nodes, 573 runs each 8.1 -> 6.6 / 7.2 -> 6.9; 256
// nodes, 274 runs 8.3 -> 7.6 / 6.8 -> 7.3, 561 runs 11 -> 8.4 / 8.7 -> 8.2, 3,825
// runs 50 -> 24 / 40 -> 16; 484 nodes, 375 runs 14.1 -> 14.4 / 9.2 -> 12.4, 1,366
// runs 38 -> 22 / 24 -> 16; 625 nodes, 752 runs 18.9 -> 18.9 / 15 -> 19, 1,254 runs
// 27 -> 22 / 20 -> 21; 729 nodes, 317 runs 9.7 -> 17 / 8.2 -> 18, 1,149 runs 24 -> 23
// / 19 -> 21, 2,095 runs 45 -> 31 / 33 -> 25; 784 nodes, 1,082 runs 31 -> 32 / 19 ->
// 25, 2,119 runs 59 -> 44 / 35 -> 30, 127 M entries 310 -> 208 / 171 -> 91; 1,024
// nodes 60 -> 60 / 34 -> 40; 3,136 nodes 152 -> 179 / 69 -> 106.
constexpr int64_t kWideNodes = 800;
static inline int adj_node_waves(int64_t nodes, int64_t runs)
{
    const int64_t each = nodes <= 200 ? 400 : 2 * nodes;
    return nodes <= kWideNodes && runs > each * nodes ? 16 : 4;
}

// Unknowns of the fused small step (k_fwd_small): D v sits in LDS (48 KB in
// FP64) and every workgroup forms all of it, 6 elements per thread.
constexpr int kSmallCols = 6144;
// Lanes per row of the fused small step, four entries each (eight 16-bit codes):
// the fewest whose reach holds 1.25 average rows; a longer row is loaded in
// further turns.  Lanes past a row's end are lost: FP64 rows of 44 entries on 64
// lanes 515 us an iteration (2,304 unknowns, 50 M entries; separate launches 414),
// on 16 lanes 328; FP32 rows of 92 on 64 lanes 294 (262), on 32 lanes 221; BF16
// rows of 20 on 16 lanes 441 (344), on 4 lanes 237.
static inline int small_reach(int vt) { return vt_size(vt) == 2 ? 8 : 4; }
static inline int small_lanes(int vt, double avg_row)
{
    const int E = small_reach(vt);
    const double lanes = 1.25 * avg_row / E;
    return lanes <= 4 ? 4 : lanes <= 16 ? 16 : lanes <= 32 || E == 8 ? 32 : 64;
}
// Where the fused step pays.  Up to 1,536 unknowns (6 for each of 256 threads)
// always: separate launches over fused, 192 to 1,440 unknowns, 30 k to 50 M
// entries, 1.0 to 1.3.  Past that every workgroup's pass over all unknowns has to
// be worth the launch it saves, so the entries decide: 6,144 unknowns in FP64 0.95
// with 100 k entries, 1.04 with 1 M, 1.2 with 50 M; FP32 0.90, 0.99, 1.2 (1.07 with
// 3 M); BF16 0.84, 0.95, 1.3 (1.07 with 3 M); 2,304 unknowns 0.98, 1.07, 1.2; 0.98,
// 1.05, 1.2; 0.93, 1.0, 1.3.  FP32 rows that fill less than 0.6 of their lanes'
// reach stay separate past 16 M entries (50 M: 0.86 to 0.95).
static inline bool small_pays(int vt, int64_t n, int64_t m, int64_t nnz)
{
    if (m < 1 || n > kSmallCols) return false;
    if (n > 1536 && nnz < (vt == VT_F64 ? 100 : vt == VT_F32 ? 200 : 300) * n) return false;
    const double avg = (double)nnz / (double)m;
    return vt != VT_F32 || nnz <= ((int64_t)1 << 24) || avg >= 0.6 * small_reach(vt) * small_lanes(vt, avg);
}

// Stored transpose (CSC) for the transposed product.
struct ColFmt {
    int vt = VT_F64;
    const int64_t *cp = nullptr;       // [n+1]
    const int32_t *ri = nullptr;       // [nnz] rows, ascending within a column
    const void *val = nullptr;
    int lpc = 64;
    // Node runs (used instead of the CSC when nrp is set; val then holds the
    // values in node-major run order).  Node k = columns [k nz, (k+1) nz).
    const int64_t *nrp = nullptr;      // [nnodes+1] runs of node k: [nrp[k], nrp[k+1])
    const int64_t *nvq = nullptr;      // [kNodeParts nnodes+1] value offset of each part of a node's
                                       // runs (part w from run r0 + c w / kNodeParts on)
    const uint32_t *nrow = nullptr;    // [nruns] data row of the run
    const uint16_t *ndesc = nullptr;   // [nruns] (iz0 << 8) | len
    const int32_t *norder = nullptr;   // [nnodes] nodes by decreasing work
    int waves = 4;                     // per node (adj_node_waves)
    int pairs = 0;                     // W = 2, 4 or 8: val / nvq in the layout of W
                                       // depths to a word (k_adj_npair<W>)
};

// Type-dispatched launchers (kernels_f64.hip, kernels_f32.hip).
void launch_init(hipStream_t st, const Problem &P, int grid, int vec, const double *rhs, int full,
                 void *T0, const float *sigma, void *Ts0, double *y, void *vzero, double *part,
                 int *ctl, int kmax);
// Workgroups of the pipelined CSR forward product that the device holds at
// once (0 when R does not use it), and its balanced wave partition.
int fwd_pipe_grid(int vec, const RowFmt &R);
int fwd_pipe_parts(int grid);          // row ranges of the balanced partition for a grid
// Workgroups of the node-run transposed product the device holds at once (0
// when C does not use it).
int adj_nruns_grid(int vec, const ColFmt &C);
void launch_wave_rows(hipStream_t st, const int64_t *rp, int64_t m, int waves, int32_t *wrow);
// Row groups (RowFmt::slot): workgroups of k_fwd_lcol the device holds at once
// (0 without groups) and the balanced group ranges of a launch of `parts`.
int fwd_lcol_grid(int vec, const RowFmt &R);
void launch_group_parts(hipStream_t st, const int64_t *rp, const int32_t *gp, int ng, int parts,
                        int32_t *wgrp);
void launch_fwd(hipStream_t st, const Problem &P, int grid, int vec, const RowFmt &R,
                const void *z, const void *Tprev, void *Tcur, void *Ts, double *part_out,
                const double *part_v, int np_v, double *S, int *ctl, int parity, double tol,
                int mode);
void launch_adj(hipStream_t st, const Problem &P, int grid, int vec, const ColFmt &C,
                const double *d, const void *T, const void *Tg, const void *v, void *q,
                double *part_out, const double *part_t, int np_t, double *S, int *ctl,
                int parity, int mode, int data_only, double *cur = nullptr);
// hbar != nullptr selects the LSMR step (w then holds LSMR's h).
void launch_update(hipStream_t st, const Problem &P, int grid, int vec, const double *d,
                   const void *q, void *v, double *w, double *y, void *z, double *part_out,
                   const double *part_q, int np_q, double *S, int *ctl, int parity, int mode,
                   double *hbar, double *cur = nullptr);
// The fused step of small systems (k_fwd_small): iteration k's forward product
// after the update of iteration k - 1.
struct SmallStep {
    const RowFmt *R = nullptr;         // CSR rows (value type, lanes per row)
    const uint16_t *col16 = nullptr;   // [nnz + 8] columns
    const int32_t *wrow = nullptr;     // [grid+1] balanced row ranges
    int grid = 1, threads = 1024, lanes = 64;
    const double *d = nullptr;
    const void *z = nullptr, *q = nullptr;
    void *v = nullptr;
    double *w = nullptr, *y = nullptr, *hbar = nullptr;
    const void *Tprev = nullptr;
    void *Tcur = nullptr, *Ts = nullptr;
    double *part_t = nullptr;          // out
    const double *part_q = nullptr, *part_v = nullptr;
    int np_q = 0, np_v = 0;
    double *S = nullptr, *cur = nullptr;
    int *ctl = nullptr;
    int parity = 0;
    double tol = 0.0;
};
void launch_small(hipStream_t st, const Problem &P, int vec, const SmallStep &q);
void launch_col16(hipStream_t st, int64_t nnz, const int32_t *ci, uint16_t *col16);

// Helpers (kernels_common.hip).
void launch_finalize(hipStream_t st, const Problem &P, int grid, const double *d,
                     const double *y, double *dm, const double *part_v, int np_v, double *S,
                     int *ctl, double tol, int accumulate);
void launch_scale_vec(hipStream_t st, int64_t n, const double *d, const double *x, double *z);
void launch_fill(hipStream_t st, int64_t n, double value, double *x);
void launch_jacobi(hipStream_t st, const Problem &P, const ColFmt &C, double *d);
void launch_check_vec(hipStream_t st, int64_t n, const double *x, int positive, int *flag);
// The values of the node runs in the layout of W depths to a word (W = 1:
// plain), run r from start[r] on: iz0 mod W zeros, its len values in[src[r]
// ..], zeros up to a multiple of W (elements of elem_bytes = 2, 4 or 8).
void launch_gather_runs(hipStream_t st, int64_t nr, const uint32_t *src, const uint32_t *start,
                        const uint16_t *desc, int W, const void *in, void *out, int elem_bytes);
void launch_convert_f32(hipStream_t st, int64_t nnz, const double *src, float *dst);
void launch_row_scales(hipStream_t st, int64_t m, const int64_t *rp, const double *val, int vt,
                       float *sigma);
void launch_quantise_rows(hipStream_t st, int64_t m, const int64_t *rp, const double *val,
                          const float *sigma, int vt, uint16_t *q);
void launch_quantise_cols(hipStream_t st, int64_t nnz, const int32_t *ri, const double *cv,
                          const float *sigma, int vt, uint16_t *q);
// rbar = bbar - y in FP64 (y = NULL: rbar = bbar); partials of |rbar|^2
void launch_residual(hipStream_t st, const Problem &P, int grid, const double *dt,
                     const double *y, double *rbar, double *part);
void launch_sum_partials(hipStream_t st, const double *part, int np, double *out);

// Transpose (transpose.hip).
struct Allocator {
    lsqr_alloc_fn alloc = nullptr;
    lsqr_free_fn dealloc = nullptr;
    void *user = nullptr;
    void *get(size_t bytes);
    void put(void *p, size_t bytes);
};
hipError_t build_transpose(hipStream_t st, Allocator &al, int64_t m, int64_t n, int64_t nnz,
                           const int64_t *rp, const int32_t *ci, const double *val,
                           int64_t *col_ptr, int32_t *row_idx, double *cval, std::string &err);

// ptr[c] = first position whose key is >= c, c = 0 .. n (keys ascending).
void launch_key_ptr(hipStream_t st, int64_t count, int64_t n, const uint32_t *keys, int64_t *ptr);

// Planning of the stored formats on the device (plan.hip).  The runs of a
// CSR structure (maximal stretches of consecutive columns inside one lateral
// node), in row order and in node-major order (rows ascending); nz <= 64,
// nnz < 2^32.
struct RunPlan {
    int64_t nr = 0;
    int64_t *rrp = nullptr;                        // [m+1] runs of row i: rrp[i] .. rrp[i+1]-1
    uint32_t *src = nullptr, *row = nullptr;       // [nr] position of the first value, row
    uint32_t *col0 = nullptr;                      // [nr] first column
    uint8_t *len = nullptr;                        // [nr]
    int64_t *nrp = nullptr;                        // [nnodes+1]
    uint32_t *nsrc = nullptr, *nrow = nullptr;     // [nr] node-major: src, row
    uint16_t *ndesc = nullptr;                     // [nr] (iz0 << 8) | len
    uint32_t *rrid = nullptr;                      // [nr] node-major index of the row order's runs, or nullptr
    int32_t *norder = nullptr;                     // [nnodes] by decreasing run count, stable
};
// Columns a device-planned row group can index (its column set sits in LDS as
// bits, 32 KB, with a rank per word, 16 KB); larger grids group on the host.
constexpr int64_t kPlanMaxCols = (int64_t)1 << 18;
bool plan_groups_fit(int64_t n, int nz);
// cnt[i] = runs of row i; info[0] = validation flags of the CSR (when check
// holds its values: 1 row_ptr, 2 column range, 4 column order, 8 non-finite),
// info[1] = longest row.
hipError_t plan_scan_rows(hipStream_t st, int64_t m, int64_t n, int64_t nnz, int nz, const int64_t *rp,
                          const int32_t *ci, const double *check, uint32_t *cnt, int *info);
hipError_t plan_row_runs(hipStream_t st, Allocator &al, int64_t m, const uint32_t *cnt, int64_t *rrp, int64_t *nr);
// Fills R's row order and key / idx (node and position of every run).
hipError_t plan_emit_runs(hipStream_t st, int64_t m, int nz, const int64_t *rp, const int32_t *ci,
                          const RunPlan &R, uint32_t *key, uint32_t *idx);
// Fills R's node-major order; padded[0..2] = value positions of the layouts of
// 2, 4 and 8 depths to a word.  key and idx are overwritten.
hipError_t plan_node_runs(hipStream_t st, Allocator &al, int64_t nn, int nz, RunPlan &R, uint32_t *key,
                          uint32_t *idx, uint64_t *padded);
// Value position of every run (start) and of every node's parts (nvq) in
// the layout of W depths to a word, `total` positions in all.
hipError_t plan_layout(hipStream_t st, Allocator &al, int64_t nn, const RunPlan &R, int W, int64_t total,
                       uint32_t *start, int64_t *nvq);
hipError_t plan_csc(hipStream_t st, Allocator &al, int64_t n, int nz, int64_t nnz, const RunPlan &R,
                    const int64_t *nvq, const double *nval, int64_t *cp, int32_t *ri, double *cv);
hipError_t plan_group_bounds(hipStream_t st, Allocator &al, int64_t m, int64_t n, int cap, const RunPlan &R,
                             std::vector<int32_t> &gp);
hipError_t plan_group_sizes(hipStream_t st, Allocator &al, int64_t n, int ng, const int32_t *gp, const RunPlan &R,
                            int64_t *gcp, int64_t *total);
hipError_t plan_group_lists(hipStream_t st, int64_t n, int ng, const int32_t *gp, const RunPlan &R,
                            const int64_t *rp, const int32_t *ci, const int64_t *gcp, int32_t *gcol, uint16_t *slot);

// Row blocks of the batched products (nz <= 32): consecutive data rows that cross
// the same lateral nodes, at most 20 to a block.  A pair is a (block, node) with
// an entry, nodes ascending in a block.  Its FP32 values are a tile per quad of
// rows, [depths d0 .. d0+nd_q-1][4 rows] with zeros where a row has no entry, one
// quad after the other: periods reach down to different depths, so one window
// for all rows of a block would store about two values per entry.
constexpr int kBlockRows = 20, kQuads = kBlockRows / 4;
constexpr int64_t kPlanMaxNodes = (int64_t)1 << 17;    // a block's node set sits in LDS
struct RowBlocks {
    int nb = 0;
    int rows_max = 0;                  // most rows of a block
    int64_t np = 0;
    int32_t *row0 = nullptr;           // [nb+1] first row
    uint32_t *pptr = nullptr;          // [nb+1] pairs of block b: pptr[b] .. pptr[b+1]-1
    uint4 *pair = nullptr;             // [np] node | d0 << 20 | largest nd_q << 26, position of
                                       // the tiles / 4 floats, nd_q << 6 q (30 bits), units of 4
    float *val = nullptr;              // the tiles
    int64_t *nptr = nullptr;           // [nnodes+1] node-major pairs (blocks ascending)
    uint4 *nlist = nullptr;            // [np] position, first row, rows | d0 << 8 | units << 16, nd_q
    int32_t *norder = nullptr;         // [nnodes] by decreasing number of pairs
};
// Builds B (buffers from keep, which returns nullptr when out of memory); sets
// B.nb = 0, keeping nothing, when the rows share too few nodes for blocks to
// pay or the structure is past a limit.
hipError_t plan_row_blocks(hipStream_t st, Allocator &al, int64_t m, int64_t n, int nz, const int64_t *rp,
                           const int32_t *ci, const double *va, RowBlocks &B,
                           const std::function<void *(size_t)> &keep);

}  // namespace lsqr
