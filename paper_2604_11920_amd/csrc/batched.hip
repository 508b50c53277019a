// Batched multi right-hand-side LSQR: host runtime of lsqr_solve_batched,
// the block operator entry points and the schedule autotuner.
//
// All systems' iterations are captured into one hipGraph (a block of up to 32
// iterations x every system x three kernel stages) and replayed; each
// system's right-hand sides carry their own FP64 scalars on the device.
#include <math.h>

#include <algorithm>
#include <vector>

#include "ctx.h"
#include "lsqr_batched.cuh"

using namespace lsqr;

namespace {

int pow2_at_least(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Row blocks, but for one right-hand side where a node has fewer than 2.5 pairs:
// a workgroup per node has little to do (both products of 3,185 nodes and 66
// paths of 13 periods: 23.5 us, over runs and entries 19.3; of two right-hand
// sides 23.7 and 23.9; of one with 253 paths 27.3 and 29.0).
bool use_row_blocks(const lsqr_ctx *c, int R)
{
    return c->rb.nb && (R > 1 || 2 * c->rb.np >= 5 * (c->P.n / c->P.nz));
}

BArgs base_args(lsqr_ctx *c, BatchEngine &B)
{
    BArgs a{};
    a.rp = c->rp; a.ci = c->ci; a.va = c->va32;
    a.cp = c->cp; a.ri = c->ri; a.cv = c->cv32;
    if (c->nval32 && c->P.nz <= kMaxNzBatched) {   // transposed product over node runs
        a.nrp = c->nrp; a.nvq = c->nvq; a.nrow = c->nrow; a.ndesc = c->ndesc;
        a.norder = c->norder; a.nval = c->nval32;
        if (B.Pr) { a.rrp = c->rrp; a.rrid = c->rrid; a.Pr = B.Pr; a.g_pr = B.g_adj; }
    }
    if (use_row_blocks(c, B.R)) a.rb = c->rb;
    a.va64 = c->va; a.cv64 = c->cv;
    a.d = c->d;
    a.m = c->P.m; a.n = (int)c->P.n; a.nx = c->P.nx; a.ny = c->P.ny; a.nz = c->P.nz;
    a.w = c->P.w; a.damp = c->P.damp;
    a.R = B.R;
    a.act = B.act; a.why = B.why; a.ctl = B.ctl; a.S = B.S;
    return a;
}

// Forward: 8 waves share a block's pairs up to this many blocks (a workgroup
// each), where 4 waves each leave compute units idle.  4 -> 8 waves, us of a
// batched iteration (nodes, depths): 32 right-hand sides, 177 blocks 32.8 -> 30.5
// (256, 9) and 140 -> 134 (3,136, 12); 494 blocks 43.5 -> 42.3 and 68 -> 66 (528, 20);
// 658 blocks 50.0 -> 48.8, 82.5 -> 84.9 (528, 20), 90.3 -> 91.7 (1,122, 16); 968 blocks
// 60.1 -> 61.6 and 88 -> 94.  Of 128,000 unknowns (6,400, 20), where the smoothing and
// damping rows are most of the launch, 177 blocks 282 -> 290, 968 blocks 351 -> 358.
// 8 right-hand sides: 177 blocks 25.4 -> 24.7 and 105 -> 92 (6,400, 20); 767 blocks
// 38.9 -> 39.1, 55.4 -> 54.6 (900, 20), 130 -> 124 (6,400, 20); 968 blocks 44.1 ->
// 45.3, 56 -> 59 (528, 20), 144 -> 142.
template <int RT>
bool few_blocks(const BArgs &a)
{
    return a.rb.nb <= (RT > 16 ? 576 : 768) && (RT <= 16 || a.n <= 65536);
}

// Transposed: 8 waves share a node's pairs where the nodes are at most the
// workgroups of 4 waves that the device holds at once (768 for 32 right-hand
// sides and more than 16 depths, else 1,024; of 8 waves it holds 256 and 512) and
// a node has pairs for them.  4 -> 8 waves, us of a batched iteration (nodes,
// pairs a node): 32 right-hand sides of 20 depths 65.8 -> 69.7 (528, 33), 84.9 ->
// 76.3 (528, 41), 154 -> 131 (528, 141), 92 -> 102 (900, 31), 150 -> 167 (900, 101);
// of 9 depths 30.5 -> 27.0 (256, 18), 48.8 -> 39.9 (256, 69), 60.9 -> 61.0 (1,024,
// 25), 75.6 -> 72.1 (1,024, 33).  8 of them: 24.7 -> 22.9 (256, 18), 29.8 -> 27.3 (528,
// 11), 33.6 -> 35.8 (900, 10), 42.0 -> 42.2 (900, 25), 48.8 -> 44.9 (900, 31), 35.3 ->
// 36.3 (1,024, 25), 47.1 -> 41.2 (1,024, 33), 110.5 -> 115.4 (3,136, 53); the product
// alone of 16 on 256 nodes of 9 pairs 7.1 -> 6.6, on 756 of 8 8.8 -> 8.1.
template <int RT, int MT>
bool few_nodes(const BArgs &a)
{
    const bool big = RT > 16 && MT == 2;
    const int64_t nn = a.n / a.nz, pairs = nn > 768 ? 28 : big ? 40 : 6;
    return nn <= (big ? 768 : 1024) && a.rb.np >= pairs * nn;
}

template <int RT, int KS, int MT>
void launch_fwd_rb(hipStream_t st, int grid, const BArgs &a)
{
    if (few_blocks<RT>(a))
        hipLaunchKernelGGL((k_bfwd_rb<RT, KS, MT, 8>), dim3(grid), dim3(512), 0, st, a);
    else
        hipLaunchKernelGGL((k_bfwd_rb<RT, KS, MT, 4>), dim3(grid), dim3(256), 0, st, a);
}

template <int RT, int MT, int QM>
void launch_adj_rb(hipStream_t st, int grid, const BArgs &a)
{
    if (few_nodes<RT, MT>(a))
        hipLaunchKernelGGL((k_badj_rb<RT, MT, QM, 8>), dim3(grid), dim3(512), 0, st, a);
    else
        hipLaunchKernelGGL((k_badj_rb<RT, MT, QM, 4>), dim3(grid), dim3(256), 0, st, a);
}

template <int RT>
void launch_tile(hipStream_t st, int kind, int grid, const BArgs &a)
{
    switch (kind) {
    case 0: hipLaunchKernelGGL((k_binit<RT>), dim3(grid), dim3(kBlock), 0, st, a); break;
    case 1:
        if (a.rb.nb) {                // row blocks
            const bool two = a.rb.rows_max > 16;
            if (a.nz <= 12) two ? launch_fwd_rb<RT, 3, 2>(st, grid, a) : launch_fwd_rb<RT, 3, 1>(st, grid, a);
            else if (a.nz <= 20) two ? launch_fwd_rb<RT, 5, 2>(st, grid, a) : launch_fwd_rb<RT, 5, 1>(st, grid, a);
            else two ? launch_fwd_rb<RT, 8, 2>(st, grid, a) : launch_fwd_rb<RT, 8, 1>(st, grid, a);
        } else if (a.Pr && RT == 32) {       // two-phase product over the node runs
            hipLaunchKernelGGL(k_bfwd_pr32, dim3(a.g_pr), dim3(kBlock), 0, st, a);
            hipLaunchKernelGGL((k_bfwd<RT>), dim3(grid), dim3(kBlock), 0, st, a);
        } else {                      // entry-wise over the CSR rows
            BArgs b = a;
            b.Pr = nullptr;
            hipLaunchKernelGGL((k_bfwd<RT>), dim3(grid), dim3(kBlock), 0, st, b);
        }
        break;
    default:
        if (a.rb.nb) {
            const bool two = a.rb.rows_max > 16;
            if (a.nz <= 16) two ? launch_adj_rb<RT, 1, 5>(st, grid, a) : launch_adj_rb<RT, 1, 4>(st, grid, a);
            else two ? launch_adj_rb<RT, 2, 5>(st, grid, a) : launch_adj_rb<RT, 2, 4>(st, grid, a);
        } else if (a.nrp && RT == 32) hipLaunchKernelGGL(k_badj_mfma32, dim3(grid), dim3(kBlock), 0, st, a);
        else if (a.nrp) hipLaunchKernelGGL((k_badj_nruns<RT>), dim3(grid), dim3(kBlock), 0, st, a);
        else hipLaunchKernelGGL((k_badj<RT>), dim3(grid), dim3(kBlock), 0, st, a);
        break;
    }
}

void launch_tiled(hipStream_t st, int kind, int grid, BArgs a, int R, int rt)
{
    for (int r0 = 0; r0 < R; r0 += rt) {
        a.r0 = r0;
        switch (rt) {
        case 1: launch_tile<1>(st, kind, grid, a); break;
        case 2: launch_tile<2>(st, kind, grid, a); break;
        case 4: launch_tile<4>(st, kind, grid, a); break;
        case 8: launch_tile<8>(st, kind, grid, a); break;
        case 16: launch_tile<16>(st, kind, grid, a); break;
        default: launch_tile<32>(st, kind, grid, a); break;
        }
    }
}

// FP32 copies of the values (the batched kernels read FP32): in row blocks where
// the rows share their nodes, else row-major, column-major and node-major.
lsqr_status ensure_fp32(lsqr_ctx *c, hipStream_t st, int R)
{
    const int64_t nnz = c->P.nnz;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (!c->rb_tried) HIP_TRY(c, hipStreamIsCapturing(st, &cap));
    if (!c->rb_tried && cap == hipStreamCaptureStatusNone) {      // the planning waits for the stream
        std::vector<void *> kept;
        if (nnz > 0 && nnz < ((int64_t)1 << 32) && c->P.m < ((int64_t)1 << 31)) {
            const hipError_t e = plan_row_blocks(st, c->al, c->P.m, c->P.n, c->P.nz, c->rp, c->ci, c->va, c->rb,
                                                 [&](size_t b) {
                                                     void *p = ctx_alloc_bytes(c, b);
                                                     if (p) kept.push_back(p);
                                                     return p;
                                                 });
            if (e != hipSuccess) {
                for (void *p : kept) ctx_release(c, p);
                c->rb = RowBlocks{};
                if (e != hipErrorOutOfMemory)              // out of memory: the other layouts
                    return fail(c, LSQR_E_DEVICE, std::string("row blocks: ") + hipGetErrorString(e));
            }
        }
        c->rb_tried = true;
    }
    if (use_row_blocks(c, R)) return LSQR_OK;
    const lsqr_status s = ensure_values32(c, st, true);       // nval32: the transposed block product
    if (s != LSQR_OK) return s;
    HIP_TRY(c, hipGetLastError());
    return LSQR_OK;
}

int cap(int64_t work, int per, int lim)
{
    int64_t b = (work + per - 1) / per;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, lim));
}

// Gives back the batch buffers.
void release_batch(lsqr_ctx *c)
{
    BatchEngine &B = c->beng;
    for (void *p : {(void *)B.T[0], (void *)B.T[1], (void *)B.V, (void *)B.Q, (void *)B.Z,
                    (void *)B.W, (void *)B.Y, (void *)B.rhs, (void *)B.dm, (void *)B.P1,
                    (void *)B.P2, (void *)B.P3, (void *)B.S, (void *)B.act, (void *)B.why, (void *)B.ctl,
                    (void *)B.Pr, (void *)B.X, (void *)B.F, (void *)B.rsum})
        if (p) ctx_release(c, p);
    B = BatchEngine{};
}

// Workgroups at most, where no schedule is set: 2,048 over row blocks, over the
// entries of up to this many rows, and for the transposed product over node runs;
// else 1,024.  1,024 -> 2,048 workgroups (us): entries of 13,366 rows and 8
// right-hand sides 73 -> 62, of 20,920 rows 249 -> 204, of 44,891 rows 442 -> 415, but
// of 53,464 rows 631 -> 666 and of 73,306 rows 606 -> 645; node runs with 32 531 ->
// 418 and 269 -> 202, with 8 156 -> 160 and 450 -> 444; columns (more than 32
// depths) 2,026 -> 2,274, 436 -> 479 and 58 -> 62.
constexpr int64_t kMoreRows = 49152;

// Buffers for R right-hand sides and `iters` iterations; all or none.
lsqr_status ensure_batch(lsqr_ctx *c, hipStream_t st, int R, int iters)
{
    BatchEngine &B = c->beng;
    const int64_t m = c->P.m, n = c->P.n, mb = m + 2 * n;
    lsqr_status s = ensure_fp32(c, st, R);
    if (s != LSQR_OK) return s;
    const int keep_rt = B.tuned || B.R == R ? B.rt : 0, keep_grid = B.tuned || B.R == R ? B.grid : 0;
    auto refuse = [&]() {             // nothing half made; the schedule stays for the next call
        release_batch(c);
        if (keep_rt) { B.rt = keep_rt; B.grid = keep_grid; B.tuned = 1; }
        return fail(c, LSQR_E_OOM, "device allocation failed");
    };
    if (B.R != R) {
        release_batch(c);
        B.R = R;
        B.rt = keep_rt && keep_rt <= R ? keep_rt : std::min(R, 32);
        B.grid = keep_grid;
        B.T[0] = ctx_alloc<float>(c, mb * R);
        B.T[1] = ctx_alloc<float>(c, mb * R);
        B.V = ctx_alloc<float>(c, n * R);
        B.Q = ctx_alloc<float>(c, n * R);
        B.Z = ctx_alloc<float>(c, n * R);
        B.W = ctx_alloc<double>(c, n * R);
        B.Y = ctx_alloc<double>(c, n * R);
        B.rhs = ctx_alloc<double>(c, std::max<int64_t>(m, 1) * R);
        B.dm = ctx_alloc<double>(c, n * R);
        B.P1 = ctx_alloc<double>(c, (size_t)2048 * R);
        B.P2 = ctx_alloc<double>(c, (size_t)2048 * R);
        B.P3 = ctx_alloc<double>(c, (size_t)2048 * R);
        B.act = ctx_alloc<int>(c, R);
        B.why = ctx_alloc<int>(c, R);
        B.ctl = ctx_alloc<int>(c, C_WORDS);
        if (!B.T[0] || !B.T[1] || !B.V || !B.Q || !B.Z || !B.W || !B.Y || !B.rhs || !B.dm ||
            !B.P1 || !B.P2 || !B.P3 || !B.act || !B.why || !B.ctl)
            return refuse();
        // per-run partial rows of the two-phase forward product (node runs)
        if (!use_row_blocks(c, R) && c->rrid && c->nval32 && c->P.nz <= kMaxNzBatched) {
            B.Pr = ctx_alloc<float>(c, std::max<int64_t>(c->nnruns, 1) * R);
            if (!B.Pr) return refuse();
        }
    }
    const int64_t need = (int64_t)iters + 2;
    if (B.s_rows < need) {
        if (B.S) ctx_release(c, B.S);
        B.s_rows = 0;
        const int64_t rows = std::max<int64_t>(need, 512);
        B.S = ctx_alloc<double>(c, (size_t)rows * R * kStateWords);
        if (!B.S) return refuse();
        B.s_rows = rows;
    }
    const bool rb = use_row_blocks(c, R), runs = c->nval32 && c->P.nz <= kMaxNzBatched;
    const int gf = B.grid ? B.grid : rb || m <= kMoreRows ? 2048 : 1024;
    const int ga = B.grid ? B.grid : rb || runs ? 2048 : 1024;
    // a workgroup per row block, and enough of them for the smoothing and damping
    // rows (4 a thread: 60 blocks, 18,000 unknowns and 32 right-hand sides took
    // 86 us for both products, now 37)
    if (rb) B.g_fwd = cap(std::max<int64_t>(c->rb.nb, (2 * n * R + 1023) / 1024), 1, gf);
    else B.g_fwd = cap(m * 64, kBlock, gf);
    if (rb || runs) B.g_adj = (int)std::max<int64_t>(1, std::min<int64_t>(n / c->P.nz, ga));   // a workgroup per lateral node
    else B.g_adj = cap(n * 64, kBlock, ga);
    B.g_upd = cap(n * R, kBlock, 512);
    return LSQR_OK;
}

void batch_init(lsqr_ctx *c, hipStream_t st, double tol, bool full = false)
{
    BatchEngine &B = c->beng;
    BArgs a = base_args(c, B);
    a.rhs = full ? B.F : B.rhs; a.rhs_full = full ? 1 : 0;
    a.Tcur = B.T[0]; a.V = B.V; a.Y = B.Y; a.W = B.W; a.Zout = B.Z; a.Q = B.Q;
    a.tol = tol;
    a.part_out = B.P1;
    launch_tiled(st, 0, B.g_fwd, a, B.R, B.rt);
    a.mode = MODE_INIT;
    a.part_in = B.P1; a.np_in = B.g_fwd; a.part_out = B.P2;
    launch_tiled(st, 2, B.g_adj, a, B.R, B.rt);
    a.part_in = B.P2; a.np_in = B.g_adj; a.part_out = B.P3;
    hipLaunchKernelGGL(k_bupdate, dim3(B.g_upd), dim3(kBlock), 0, st, a);
}

void batch_iter(lsqr_ctx *c, hipStream_t st, int p, double tol)
{
    BatchEngine &B = c->beng;
    BArgs a = base_args(c, B);
    a.parity = p; a.mode = MODE_ITER; a.tol = tol;
    a.V = B.V; a.Q = B.Q; a.W = B.W; a.Y = B.Y;
    // forward: T[1-p] = A_D Z - alpha U
    a.Z = B.Z; a.Tprev = B.T[p]; a.Tcur = B.T[1 - p];
    a.part_in = B.P3; a.np_in = B.g_upd; a.part_out = B.P1;
    launch_tiled(st, 1, B.g_fwd, a, B.R, B.rt);
    // transposed: Q = D A^T T / beta - beta V
    a.part_in = B.P1; a.np_in = B.g_fwd; a.part_out = B.P2;
    launch_tiled(st, 2, B.g_adj, a, B.R, B.rt);
    // update
    a.part_in = B.P2; a.np_in = B.g_adj; a.part_out = B.P3; a.Zout = B.Z;
    hipLaunchKernelGGL(k_bupdate, dim3(B.g_upd), dim3(kBlock), 0, st, a);
}

__global__ void k_set_kmax(int *ctl, int kmax) { ctl[C_KMAX] = kmax; }

// dst += src.
__global__ void k_blk_add(int64_t count, const double *src, double *dst)
{
#pragma clang fp contract(off)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = dst[i] + src[i];
}

int grid_for(int64_t work) { return cap(work, 256, 4096); }

// Checks shared by the batched entry points.
lsqr_status batch_args(lsqr_ctx *const *ctxs, int nsys, int nrhs, const double *const *dt,
                       lsqr_mem vec_mem, int iters, double tol, double *const *dm)
{
    if (!ctxs || nsys < 1) return fail(nullptr, LSQR_E_INVALID_ARG, "need at least one context");
    for (int s = 0; s < nsys; ++s)
        if (!ctxs[s]) return fail(nullptr, LSQR_E_INVALID_ARG, "context is NULL");
    lsqr_ctx *c0 = ctxs[0];
    if (nrhs < 1 || nrhs > kMaxRhs) return fail(c0, LSQR_E_INVALID_ARG, "nrhs must be in 1..32");
    if (!dt || !dm) return fail(c0, LSQR_E_INVALID_ARG, "dt and dm must not be NULL");
    if (iters < 0) return fail(c0, LSQR_E_INVALID_ARG, "iters must be >= 0");
    if (!(tol >= 0.0) || !isfinite(tol)) return fail(c0, LSQR_E_INVALID_ARG, "tol must be finite and >= 0");
    if (vec_mem != LSQR_MEM_HOST && vec_mem != LSQR_MEM_DEVICE)
        return fail(c0, LSQR_E_INVALID_ARG, "unknown memory kind");
    for (int s = 0; s < nsys; ++s) {
        if (!dt[s] || !dm[s]) return fail(c0, LSQR_E_INVALID_ARG, "dt[s] and dm[s] must not be NULL");
        if (ctxs[s]->device != c0->device) return fail(c0, LSQR_E_INVALID_ARG, "contexts on different devices");
        if (vec_mem == LSQR_MEM_HOST)
            for (int64_t i = 0; i < ctxs[s]->P.m * (int64_t)nrhs; ++i)
                if (!isfinite(dt[s][i])) return fail(c0, LSQR_E_NONFINITE, "non-finite value in dt");
    }
    return LSQR_OK;
}

// Copies every system's [m][nrhs] right-hand sides into its padded [m][R]
// block B.rhs (buffers for `iters` iterations made ready first).
lsqr_status batch_load_rhs(lsqr_ctx *const *ctxs, int nsys, int nrhs, int R, const double *const *dt,
                           lsqr_mem vec_mem, int iters)
{
    lsqr_ctx *c0 = ctxs[0];
    hipStream_t st = c0->st;
    const hipMemcpyKind kin = vec_mem == LSQR_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        lsqr_status e = ensure_batch(c, st, R, iters);
        if (e != LSQR_OK) return fail(c0, e, c->err);
        BatchEngine &B = c->beng;
        if (R != nrhs) launch_fill(st, std::max<int64_t>(c->P.m, 1) * R, 0.0, B.rhs);
        if (c->P.m > 0)
            HIP_TRY(c0, hipMemcpy2DAsync(B.rhs, R * sizeof(double), dt[s], nrhs * sizeof(double),
                                         nrhs * sizeof(double), c->P.m, kin, st));
    }
    HIP_TRY(c0, hipGetLastError());
    return LSQR_OK;
}

// Runs every system's batch from its start (B.rhs, or B.F when full) for up
// to `iters` iterations: a captured graph of a block of iterations of all
// systems, replayed while any right-hand side is active, then single
// iterations; leaves dm = D y of every system in its B.dm.
lsqr_status batch_run(lsqr_ctx *const *ctxs, int nsys, int nrhs, int R, int iters, double tol,
                      bool full)
{
    lsqr_ctx *c0 = ctxs[0];
    hipStream_t st = c0->st;
    for (int s = 0; s < nsys; ++s) {
        batch_init(ctxs[s], st, tol, full);
        hipLaunchKernelGGL(k_set_kmax, dim3(1), dim3(1), 0, st, ctxs[s]->beng.ctl, iters);
    }
    HIP_TRY(c0, hipGetLastError());
    int done = 0;
    bool stopped = false;
    std::vector<int> hact((size_t)R);
    auto poll = [&]() -> lsqr_status {
        int live = 0;
        for (int s = 0; s < nsys; ++s) {
            HIP_TRY(c0, hipMemcpyAsync(hact.data(), ctxs[s]->beng.act, R * sizeof(int),
                                       hipMemcpyDeviceToHost, st));
            HIP_TRY(c0, hipStreamSynchronize(st));
            for (int r = 0; r < nrhs; ++r) live += hact[r];
        }
        stopped = live == 0;
        return LSQR_OK;
    };
    const int gb = std::min(iters, tol > 0.0 ? c0->check_every : 32) & ~1;
    lsqr_status e;
    if (gb >= 2 && !(c0->flags & LSQR_FLAG_NO_GRAPH)) {
        if (!c0->cap_st) HIP_TRY(c0, hipStreamCreateWithFlags(&c0->cap_st, hipStreamNonBlocking));
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        HIP_TRY(c0, hipStreamBeginCapture(c0->cap_st, hipStreamCaptureModeThreadLocal));
        for (int i = 0; i < gb; ++i)
            for (int s = 0; s < nsys; ++s) batch_iter(ctxs[s], c0->cap_st, i & 1, tol);
        HIP_TRY(c0, hipStreamEndCapture(c0->cap_st, &graph));
        hipError_t ge = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ge != hipSuccess) return fail(c0, LSQR_E_DEVICE, std::string("hipGraphInstantiate: ") + hipGetErrorString(ge));
        while (!stopped && iters - done >= gb) {
            hipError_t le = hipGraphLaunch(exec, st);
            if (le != hipSuccess) {
                (void)hipGraphExecDestroy(exec);
                return fail(c0, LSQR_E_DEVICE, std::string("hipGraphLaunch: ") + hipGetErrorString(le));
            }
            done += gb;
            if (tol > 0.0 && done < iters && (e = poll()) != LSQR_OK) { (void)hipGraphExecDestroy(exec); return e; }
        }
        (void)hipStreamSynchronize(st);
        (void)hipGraphExecDestroy(exec);
    }
    while (!stopped && done < iters) {
        for (int s = 0; s < nsys; ++s) batch_iter(ctxs[s], st, done & 1, tol);
        ++done;
        if (tol > 0.0 && done % c0->check_every == 0 && done < iters && (e = poll()) != LSQR_OK) return e;
    }
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        BatchEngine &B = c->beng;
        BArgs a = base_args(c, B);
        a.Y = B.Y; a.tol = tol; a.part_in = B.P3; a.np_in = B.g_upd;
        hipLaunchKernelGGL(k_bfinal, dim3(cap(c->P.n * R, kBlock, 1024)), dim3(kBlock), 0, st, a, B.dm);
    }
    HIP_TRY(c0, hipGetLastError());
    return LSQR_OK;
}

// The state rows of system c's last batch run: per right-hand side r <
// nrhs its stop reason, the last iteration it advanced (klast) and the rows
// hs [(kdone + 1)][R][kStateWords]; err |= the device error flag.
lsqr_status batch_state(lsqr_ctx *c0, lsqr_ctx *c, int nrhs, int &err, std::vector<int> &why,
                        std::vector<int> &klast, std::vector<double> &hs, int &kdone)
{
    BatchEngine &B = c->beng;
    const int R = B.R;
    int ctl[C_WORDS];
    why.assign((size_t)R, 0);
    klast.assign((size_t)nrhs, 0);
    HIP_TRY(c0, hipStreamSynchronize(c0->st));     // the copies below are not on it
    HIP_TRY(c0, hipMemcpy(ctl, B.ctl, sizeof(ctl), hipMemcpyDeviceToHost));
    HIP_TRY(c0, hipMemcpy(why.data(), B.why, R * sizeof(int), hipMemcpyDeviceToHost));
    kdone = ctl[C_ITERS];
    err |= ctl[C_ERR];
    hs.assign((size_t)(kdone + 1) * R * kStateWords, 0.0);
    HIP_TRY(c0, hipMemcpy(hs.data(), B.S, hs.size() * sizeof(double), hipMemcpyDeviceToHost));
    for (int r = 0; r < nrhs; ++r) {
        int kl = 0;
        for (int k = 1; k <= kdone; ++k) {
            const double *Sk = hs.data() + ((size_t)k * R + r) * kStateWords;
            const double *Sp = hs.data() + ((size_t)(k - 1) * R + r) * kStateWords;
            if (Sk[S_PHIBAR] != Sp[S_PHIBAR] || Sk[S_PSI] != Sp[S_PSI]) kl = k;
        }
        if (why[r] == 0) kl = 0;
        if (why[r] == 2) kl = kdone;
        klast[(size_t)r] = kl;
    }
    return LSQR_OK;
}

// FP64 refinement scratch of a context (allocated on first use).
lsqr_status ensure_refine_buffers(lsqr_ctx *c)
{
    const int64_t n = c->P.n, mb = c->P.m + 2 * n;
    BatchEngine &B = c->beng;
    if (!B.X) B.X = ctx_alloc<double>(c, n * B.R);
    if (!B.F) B.F = ctx_alloc<double>(c, mb * B.R);
    if (!B.rsum) B.rsum = ctx_alloc<double>(c, (size_t)4 * B.R);
    if (!B.X || !B.F || !B.rsum)
        return fail(c, LSQR_E_OOM, "device allocation failed");
    return LSQR_OK;
}

}  // namespace

extern "C" {

lsqr_status lsqr_solve_batched(lsqr_ctx *const *ctxs, int nsys, int nrhs, const double *const *dt,
                               lsqr_mem vec_mem, int iters, double tol, double *const *dm,
                               double *const *res_hist, lsqr_info *info)
{
    lsqr_status e = batch_args(ctxs, nsys, nrhs, dt, vec_mem, iters, tol, dm);
    if (e != LSQR_OK) return e;
    lsqr_ctx *c0 = ctxs[0];
    DeviceGuard dg(c0->device);
    hipStream_t st = c0->st;
    const int R = pow2_at_least(nrhs);
    const hipMemcpyKind kout = vec_mem == LSQR_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    // the batch runs on the first context's stream, after each context's own work
    for (int s = 1; s < nsys; ++s)
        if (ctxs[s]->st != st) HIP_TRY(c0, hipStreamSynchronize(ctxs[s]->st));
    if ((e = batch_load_rhs(ctxs, nsys, nrhs, R, dt, vec_mem, iters)) != LSQR_OK) return e;
    if ((e = batch_run(ctxs, nsys, nrhs, R, iters, tol, false)) != LSQR_OK) return e;
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        HIP_TRY(c0, hipMemcpy2DAsync(dm[s], nrhs * sizeof(double), c->beng.dm, R * sizeof(double),
                                     nrhs * sizeof(double), c->P.n, kout, st));
    }
    HIP_TRY(c0, hipGetLastError());
    HIP_TRY(c0, hipStreamSynchronize(st));
    int err = 0;
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        std::vector<int> why, klast;
        std::vector<double> hs;
        int kdone = 0;
        if ((e = batch_state(c0, c, nrhs, err, why, klast, hs, kdone)) != LSQR_OK) return e;
        for (int r = 0; r < nrhs; ++r) {
            const int kl = klast[(size_t)r];
            if (res_hist && res_hist[s]) {
                double *h = res_hist[s];
                for (int k = 0; k <= iters; ++k)
                    for (int f = 0; f < 3; ++f) h[((size_t)k * nrhs + r) * 3 + f] = NAN;
                for (int k = 0; k <= kl; ++k) {
                    const double *Sk = hs.data() + ((size_t)k * R + r) * kStateWords;
                    double *o = h + ((size_t)k * nrhs + r) * 3;
                    if (why[r] == 0) { o[0] = Sk[S_BETA]; o[1] = 0.0; o[2] = 0.0; break; }
                    o[0] = Sk[S_PHIBAR]; o[1] = Sk[S_PSI]; o[2] = Sk[S_ETA];
                }
            }
            if (info) {
                lsqr_info &I = info[(size_t)s * nrhs + r];
                const double *Sk = hs.data() + ((size_t)kl * R + r) * kStateWords;
                I.istop = why[r];
                I.iters = kl;
                I.sweeps = 0;
                I.fallback_used = c->fallback_used;
                I.inner_fp32 = 0;
                I.eta = why[r] == 0 ? 0.0 : Sk[S_ETA];
                I.phibar = why[r] == 0 ? Sk[S_BETA] : Sk[S_PHIBAR];
                I.eta_final_fp64 = NAN;
            }
        }
    }
    if (err) return fail(c0, LSQR_E_NONFINITE, "a solver scalar became non-finite");
    return LSQR_OK;
}

lsqr_status lsqr_solve_batched_refined(lsqr_ctx *const *ctxs, int nsys, int nrhs,
                                       const double *const *dt, lsqr_mem vec_mem, int iters,
                                       double tol, double inner_tol, int sweeps,
                                       double *const *dm, lsqr_info *info)
{
    lsqr_status e = batch_args(ctxs, nsys, nrhs, dt, vec_mem, iters, tol, dm);
    if (e != LSQR_OK) return e;
    lsqr_ctx *c0 = ctxs[0];
    if (!(tol > 0.0)) return fail(c0, LSQR_E_INVALID_ARG, "the refined batch needs tol > 0");
    if (!(inner_tol >= 0.0 && inner_tol < 1.0))
        return fail(c0, LSQR_E_INVALID_ARG, "inner_tol must be in [0, 1)");
    if (sweeps < 1) return fail(c0, LSQR_E_INVALID_ARG, "sweeps must be >= 1");
    for (int s = 0; s < nsys; ++s)
        if (!(ctxs[s]->P.damp > 0.0))
            return fail(c0, LSQR_E_UNSUPPORTED, "the refinement needs damp > 0 (its correction goes into the damping block)");
    DeviceGuard dg(c0->device);
    hipStream_t st = c0->st;
    const int R = pow2_at_least(nrhs);
    const hipMemcpyKind kout = vec_mem == LSQR_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    for (int s = 1; s < nsys; ++s)
        if (ctxs[s]->st != st) HIP_TRY(c0, hipStreamSynchronize(ctxs[s]->st));
    if ((e = batch_load_rhs(ctxs, nsys, nrhs, R, dt, vec_mem, iters)) != LSQR_OK) return e;
    // per system and right-hand side: |Abar^T bbar|, eta, stop reason, work
    const size_t NR = (size_t)nsys * nrhs;
    std::vector<double> arnorm(NR, 0.0), eta(NR, INFINITY), eta_prev(NR, INFINITY), rn(NR, 0.0);
    std::vector<int> istop(NR, 2), total(NR, 0), nsw(NR, 0), live(NR, 1);
    std::vector<double> hsum((size_t)4 * R);
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        if ((e = ensure_refine_buffers(c)) != LSQR_OK) return fail(c0, e, c->err);
        launch_fill(st, c->P.n * R, 0.0, c->beng.X);
    }
    for (int sw = 0;; ++sw) {
        // FP64 residual rbar of every right-hand side (in F) and Abar^T rbar (in dm)
        for (int s = 0; s < nsys; ++s) {
            lsqr_ctx *c = ctxs[s];
            BatchEngine &B = c->beng;
            const Problem &P = c->P;
            RefArgs a{c->rp, c->ci, c->va, P.m, (int)P.n, P.nx, P.ny, P.nz, R, P.w, P.damp,
                      B.rhs, sw > 0 ? B.X : nullptr, B.F, B.dm, B.P1};
            const int gf = cap(P.m + 2 * P.n, 4, 2048), ga = cap(P.n, 4, 2048);
            hipLaunchKernelGGL(k_ref_fwd, dim3(gf), dim3(kBlock), 0, st, a);
            hipLaunchKernelGGL(k_ref_sum, dim3(1), dim3(kBlock), 0, st, gf, R, (const double *)B.P1, B.rsum);
            a.ptr = c->cp; a.idx = c->ri; a.val = c->cv; a.part = B.P2;
            hipLaunchKernelGGL(k_ref_adj, dim3(ga), dim3(kBlock), 0, st, a);
            hipLaunchKernelGGL(k_ref_sum, dim3(1), dim3(kBlock), 0, st, ga, R, (const double *)B.P2, B.rsum + 1);
        }
        HIP_TRY(c0, hipGetLastError());
        for (int s = 0; s < nsys; ++s) {
            lsqr_ctx *c = ctxs[s];
            BatchEngine &B = c->beng;
            HIP_TRY(c0, hipMemcpyAsync(hsum.data(), B.rsum, 4 * R * sizeof(double), hipMemcpyDeviceToHost, st));
            HIP_TRY(c0, hipStreamSynchronize(st));
            uint32_t mask = 0;
            for (int r = 0; r < nrhs; ++r) {
                const size_t k = (size_t)s * nrhs + r;
                if (!live[k]) continue;
                const double an = sqrt(hsum[4 * (size_t)r + 1]);
                if (sw == 0) {                     // rbar = bbar: |Abar^T bbar|
                    arnorm[k] = an;
                    if (!(an > 0.0)) { istop[k] = 0; live[k] = 0; eta[k] = 0.0; continue; }
                }
                rn[k] = sqrt(hsum[4 * (size_t)r]);
                eta[k] = an / arnorm[k];
                if (!isfinite(eta[k])) return fail(c0, LSQR_E_NONFINITE, "refinement residual became non-finite");
                if (eta[k] <= tol) { istop[k] = 1; live[k] = 0; }
                else if (sw >= sweeps) { istop[k] = 2; live[k] = 0; }
                else if (sw > 0 && eta[k] > 0.5 * eta_prev[k]) { istop[k] = 4; live[k] = 0; }
                if (live[k]) mask |= 1u << r;
                eta_prev[k] = eta[k];
            }
            // the next inner right-hand side f = [0; 0; (Abar^T rbar) / damp] (refine.hip)
            hipLaunchKernelGGL(k_ref_rhs, dim3(grid_for((c->P.m + 2 * c->P.n) * R)), dim3(256), 0, st,
                               (c->P.m + c->P.n) * R, c->P.n * (int64_t)R, R, c->P.damp, mask, (const double *)B.dm, B.F);
        }
        int any = 0;
        for (size_t k = 0; k < NR; ++k) any |= live[k];
        if (!any) break;
        // inner batched LSQR on (Ahat D, f) for every right-hand side; x += D y
        if ((e = batch_run(ctxs, nsys, nrhs, R, iters, inner_tol, true)) != LSQR_OK) return e;
        int err = 0;
        for (int s = 0; s < nsys; ++s) {
            lsqr_ctx *c = ctxs[s];
            BatchEngine &B = c->beng;
            hipLaunchKernelGGL(k_blk_add, dim3(grid_for(c->P.n * R)), dim3(256), 0, st,
                               c->P.n * (int64_t)R, (const double *)B.dm, B.X);
            std::vector<int> why, klast;
            std::vector<double> hs;
            int kdone = 0;
            if ((e = batch_state(c0, c, nrhs, err, why, klast, hs, kdone)) != LSQR_OK) return e;
            for (int r = 0; r < nrhs; ++r) {
                const size_t k = (size_t)s * nrhs + r;
                if (!live[k]) continue;
                total[k] += klast[(size_t)r];
                nsw[k] += 1;
            }
        }
        if (err) return fail(c0, LSQR_E_NONFINITE, "a solver scalar became non-finite");
    }
    for (int s = 0; s < nsys; ++s) {
        lsqr_ctx *c = ctxs[s];
        HIP_TRY(c0, hipMemcpy2DAsync(dm[s], nrhs * sizeof(double), c->beng.X, R * sizeof(double),
                                     nrhs * sizeof(double), c->P.n, kout, st));
    }
    HIP_TRY(c0, hipGetLastError());
    HIP_TRY(c0, hipStreamSynchronize(st));
    if (info)
        for (size_t k = 0; k < NR; ++k) {
            lsqr_info &I = info[k];
            I.istop = istop[k];
            I.iters = total[k];
            I.sweeps = nsw[k];
            I.fallback_used = ctxs[k / nrhs]->fallback_used;
            I.inner_fp32 = 0;
            I.eta = eta[k];
            I.phibar = rn[k];
            I.eta_final_fp64 = eta[k];
        }
    return LSQR_OK;
}

lsqr_status lsqr_apply_block(lsqr_ctx *c, int nrhs, const float *x, float *y)
{
    if (!c) return fail(nullptr, LSQR_E_INVALID_ARG, "ctx is NULL");
    if (!x || !y) return fail(c, LSQR_E_INVALID_ARG, "x and y must not be NULL");
    if (nrhs < 1 || nrhs > kMaxRhs || (nrhs & (nrhs - 1)))
        return fail(c, LSQR_E_INVALID_ARG, "nrhs must be a power of two <= 32");
    DeviceGuard dg(c->device);
    lsqr_status e = ensure_batch(c, c->st, nrhs, 1);
    if (e != LSQR_OK) return e;
    BatchEngine &B = c->beng;
    BArgs a = base_args(c, B);
    a.mode = MODE_OPERATOR; a.Z = x; a.Tcur = y; a.part_out = B.P1;
    launch_tiled(c->st, 1, B.g_fwd, a, B.R, B.rt);
    HIP_TRY(c, hipGetLastError());
    return LSQR_OK;
}

lsqr_status lsqr_apply_t_block(lsqr_ctx *c, int nrhs, const float *y, float *x)
{
    if (!c) return fail(nullptr, LSQR_E_INVALID_ARG, "ctx is NULL");
    if (!x || !y) return fail(c, LSQR_E_INVALID_ARG, "x and y must not be NULL");
    if (nrhs < 1 || nrhs > kMaxRhs || (nrhs & (nrhs - 1)))
        return fail(c, LSQR_E_INVALID_ARG, "nrhs must be a power of two <= 32");
    if (nrhs >= 4 && ((uintptr_t)y & 15u))                // rows of y are read as 16-byte vectors
        return fail(c, LSQR_E_INVALID_ARG, "y must be 16-byte aligned when nrhs >= 4");
    DeviceGuard dg(c->device);
    lsqr_status e = ensure_batch(c, c->st, nrhs, 1);
    if (e != LSQR_OK) return e;
    BatchEngine &B = c->beng;
    BArgs a = base_args(c, B);
    a.mode = MODE_OPERATOR; a.Tcur = const_cast<float *>(y); a.Q = x; a.part_out = B.P2;
    launch_tiled(c->st, 2, B.g_adj, a, B.R, B.rt);
    HIP_TRY(c, hipGetLastError());
    return LSQR_OK;
}

lsqr_status lsqr_set_batch_config(lsqr_ctx *c, const lsqr_batch_cfg *cfg)
{
    if (!c || !cfg) return fail(c, LSQR_E_INVALID_ARG, "ctx and cfg must not be NULL");
    const int rt = cfg->rhs_tile, g = cfg->grid;
    if (rt < 1 || rt > kMaxRhs || (rt & (rt - 1)) || g < 1 || g > 2048)
        return fail(c, LSQR_E_INVALID_ARG, "rhs_tile must be a power of two <= 32, grid in 1..2048");
    c->beng.rt = rt;
    c->beng.grid = g;
    c->beng.tuned = 1;
    return LSQR_OK;
}

lsqr_status lsqr_autotune_batched(lsqr_ctx *c, int nrhs, int probe_iters, lsqr_batch_cfg *best)
{
    if (!c || !best) return fail(c, LSQR_E_INVALID_ARG, "ctx and best must not be NULL");
    if (nrhs < 1 || nrhs > kMaxRhs) return fail(c, LSQR_E_INVALID_ARG, "nrhs must be in 1..32");
    if (probe_iters < 2) probe_iters = 2;
    DeviceGuard dg(c->device);
    const int R = pow2_at_least(nrhs);
    hipStream_t st = c->st;
    hipEvent_t e0, e1;
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    lsqr_batch_cfg top{0, 0, INFINITY};
    const int tiles[] = {8, 16, 32};
    const int grids[] = {256, 512, 1024, 2048};
    for (int rt : tiles) {
        if (rt > R) continue;
        for (int g : grids) {
            BatchEngine &B = c->beng;
            B.rt = rt;
            B.grid = g;
            B.tuned = 1;
            lsqr_status e = ensure_batch(c, st, R, probe_iters);
            if (e != LSQR_OK) { (void)hipEventDestroy(e0); (void)hipEventDestroy(e1); return e; }
            launch_fill(st, std::max<int64_t>(c->P.m, 1) * R, 1.0, B.rhs);
            std::vector<float> ms;
            for (int rep = 0; rep < 5; ++rep) {
                batch_init(c, st, 0.0);
                hipLaunchKernelGGL(k_set_kmax, dim3(1), dim3(1), 0, st, B.ctl, probe_iters);
                (void)hipEventRecord(e0, st);
                for (int i = 0; i < probe_iters; ++i) batch_iter(c, st, i & 1, 0.0);
                (void)hipEventRecord(e1, st);
                HIP_TRY(c, hipEventSynchronize(e1));
                float t = 0.f;
                HIP_TRY(c, hipEventElapsedTime(&t, e0, e1));
                ms.push_back(t / (float)probe_iters);
            }
            std::sort(ms.begin(), ms.end());
            const double med = ms[ms.size() / 2];
            if (med < top.ms_per_iter) top = lsqr_batch_cfg{rt, g, med};
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    c->beng.rt = top.rhs_tile;
    c->beng.grid = top.grid;
    c->beng.tuned = 1;
    lsqr_status e = ensure_batch(c, st, R, 1);
    if (e != LSQR_OK) return e;
    *best = top;
    return LSQR_OK;
}

}  // extern "C"
