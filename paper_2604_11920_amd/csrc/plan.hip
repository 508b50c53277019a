// Device-side planning of the stored formats from the CSR structure: the row
// scan (validation, runs per row, longest row), the node runs in row and in
// node-major order with their value positions, the CSC derived from them, and
// the row groups with their column lists and slots.  Every result equals the
// host builders' in runs_host.h.
//
// The host builders walked every entry on at most 16 threads after a copy of
// the structure over PCIe; here the structure stays in HBM and is read a
// handful of times, so the planning is bound by the value copies it writes.
// A system of 100 M entries (7,140 paths x 14 periods on an 80 x 80 x 20 grid),
// from ray polylines to a ready FP64 solver: 418 -> 13 ms.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include <algorithm>
#include <vector>

#include "lsqr_kernels.cuh"

namespace lsqr {

namespace {

int blocks(int64_t work, int per, int cap)
{
    const int64_t b = (work + per - 1) / per;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

int bits_for(int64_t n)               // bits of 0 .. n-1
{
    int b = 1;
    while (b < 32 && ((int64_t)1 << b) < n) ++b;
    return b;
}

// ------------------------------------------------------------- row scan --
// A wave per row: the number of runs that start in it (maximal stretches of
// consecutive columns inside one lateral node) and, over all rows, the longest
// row (info[1]).  CHECK: info[0] |= 1 row_ptr decreasing or out of range, 2
// column out of range, 4 columns not strictly increasing, 8 non-finite value;
// a row whose bounds are bad is not read.  A wave per row in place of a thread
// per row (whose lanes read 64 rows at a stride): 5.1 -> 0.50 ms at 100 M
// entries.
template <bool CHECK>
__global__ __launch_bounds__(kBlock) void k_scan_rows(int64_t m, int64_t n, int64_t nnz, FastDiv nz,
                                                      const int64_t *rp, const int32_t *ci,
                                                      const double *va, uint32_t *cnt, int *info)
{
    __shared__ int sh[2];
    if (threadIdx.x < 2) sh[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    int f = 0, longest = 0;
    for (int64_t row = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); row < m; row += waves) {
        const int64_t s = rp[row], e = rp[row + 1];
        if (CHECK && (s < 0 || e < s || e > nnz)) {
            f |= 1;
            if (lane == 0) cnt[row] = 0u;
            continue;
        }
        int runs = 0;
        for (int64_t p0 = s; p0 < e; p0 += 64) {
            const int64_t p = p0 + lane;
            bool start = false;
            if (p < e) {
                const int c = ci[p], prev = p > s ? ci[p - 1] : -2;
                start = p == s || c != prev + 1 || nz.mod((uint32_t)c) == 0;
                if (CHECK) {
                    if (c < 0 || c >= n) f |= 2;
                    if (p > s && c <= prev) f |= 4;
                    if (!isfinite(va[p])) f |= 8;
                }
            }
            runs += __popcll(__ballot(start));
        }
        longest = max(longest, (int)min(e - s, (int64_t)0x7fffffff));
        if (lane == 0) cnt[row] = (uint32_t)runs;
    }
    if (f) atomicOr(&sh[0], f);
    if (lane == 0) atomicMax(&sh[1], longest);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (sh[0]) atomicOr(&info[0], sh[0]);
        atomicMax(&info[1], sh[1]);
    }
}

// The runs in row order (a wave per row): position of the first value, row,
// first column, node; idx = 0, 1, ...
__global__ __launch_bounds__(kBlock) void k_emit_runs(int64_t m, FastDiv nz, const int64_t *rp,
                                                      const int32_t *ci, const int64_t *rrp,
                                                      uint32_t *src, uint32_t *row_of, uint32_t *col0,
                                                      uint32_t *key, uint32_t *idx)
{
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t row = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); row < m; row += waves) {
        const int64_t s = rp[row], e = rp[row + 1];
        int64_t base = rrp[row];
        for (int64_t p0 = s; p0 < e; p0 += 64) {
            const int64_t p = p0 + lane;
            bool start = false;
            int c = 0;
            if (p < e) {
                c = ci[p];
                start = p == s || c != ci[p - 1] + 1 || nz.mod((uint32_t)c) == 0;
            }
            const uint64_t mask = __ballot(start);
            if (start) {
                const int64_t q = base + __popcll(mask & (((uint64_t)1 << lane) - 1));
                src[q] = (uint32_t)p;
                row_of[q] = (uint32_t)row;
                col0[q] = (uint32_t)c;
                key[q] = nz.div((uint32_t)c);
                idx[q] = (uint32_t)q;
            }
            base += __popcll(mask);
        }
    }
}

// Length of run q: to the next run of its row, else to the row's end.
__global__ void k_run_len(int64_t nr, const int64_t *rp, const uint32_t *src, const uint32_t *row_of,
                          uint8_t *len)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nr;
         q += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t row = row_of[q];
        const int64_t end = q + 1 < nr && row_of[q + 1] == row ? (int64_t)src[q + 1] : rp[row + 1];
        len[q] = (uint8_t)(end - (int64_t)src[q]);
    }
}

// Elements of a run in the layout of W depths to a word (W = 1: its length).
template <int W>
struct PaddedLen {
    __host__ __device__ uint32_t operator()(uint16_t d) const
    {
        const uint32_t len = d & 255u, pre = (uint32_t)(d >> 8) & (W - 1);
        return (len + pre + W - 1) & ~(uint32_t)(W - 1);
    }
};

// The runs in node-major order: run r is run perm[r] of the row order.  The
// totals of the padded lengths (W = 2, 4, 8) go to tot.
__global__ __launch_bounds__(kBlock) void k_node_runs(int64_t nr, FastDiv nz, const uint32_t *perm,
                                                      const uint32_t *src, const uint32_t *row_of,
                                                      const uint32_t *col0, const uint8_t *len,
                                                      uint32_t *nsrc, uint32_t *nrow, uint16_t *ndesc,
                                                      uint32_t *rrid, unsigned long long *tot)
{
    __shared__ unsigned long long sh[3];
    if (threadIdx.x < 3) sh[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long t2 = 0, t4 = 0, t8 = 0;
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < nr; r += (int64_t)gridDim.x * kBlock) {
        const uint32_t q = perm[r];
        const uint16_t d = (uint16_t)(nz.mod(col0[q]) << 8 | len[q]);
        nsrc[r] = src[q];
        nrow[r] = row_of[q];
        ndesc[r] = d;
        if (rrid) rrid[q] = (uint32_t)r;
        t2 += PaddedLen<2>{}(d);
        t4 += PaddedLen<4>{}(d);
        t8 += PaddedLen<8>{}(d);
    }
    atomicAdd(&sh[0], t2);
    atomicAdd(&sh[1], t4);
    atomicAdd(&sh[2], t8);
    __syncthreads();
    if (threadIdx.x < 3) atomicAdd(&tot[threadIdx.x], sh[threadIdx.x]);
}

// Value offset of each part of every node's runs (part w starts at run r0 + c
// w / kNodeParts, as in the kernels); start[r] = value position of run r.
__global__ void k_parts(int64_t nn, int64_t nr, const int64_t *nrp, const uint32_t *start,
                           int64_t total, int64_t *nvq)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= kNodeParts * nn;
         i += (int64_t)gridDim.x * blockDim.x) {
        int64_t q = nr;
        if (i < kNodeParts * nn) {
            const int64_t r0 = nrp[i / kNodeParts], c = nrp[i / kNodeParts + 1] - r0;
            q = r0 + c * (i % kNodeParts) / kNodeParts;
        }
        nvq[i] = q < nr ? (int64_t)start[q] : total;
    }
}

__global__ void k_order_keys(int64_t nn, const int64_t *nrp, uint32_t *key, uint32_t *node)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nn;
         k += (int64_t)gridDim.x * blockDim.x) {
        key[k] = ~(uint32_t)(nrp[k + 1] - nrp[k]);           // ascending = decreasing run count
        node[k] = (uint32_t)k;
    }
}

// ------------------------------------------------------------------- CSC --
// A workgroup per node; its kCscParts waves take fixed parts of the node's
// runs.  Lane d < nz counts the runs of the part that cover depth d
// (FILL = false: cnt[(node nz + d) kCscParts + part]); with the counts scanned
// in that order, cnt holds where each (column, part) starts, and the fill pass
// writes rows and values: per chunk of 64 runs and depth, the runs covering it
// go to consecutive positions, rows ascending.  Rows and values leave in
// coalesced stores and the values come in through the runs' own lines, in
// place of a radix sort of every entry's column and two gathers per entry:
// 7.0 -> 1.6 ms at 100 M entries, and 1.2 ms with the values read in node order.
constexpr int kCscParts = 8;

template <bool FILL>
__global__ __launch_bounds__(64 * kCscParts) void k_csc(int64_t nn, int nz, const int64_t *nrp,
                                                        const uint16_t *ndesc, const uint32_t *nrow,
                                                        const int64_t *nvq, const double *nval,
                                                        uint32_t *cnt, int32_t *ri, double *cv)
{
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    for (int64_t k = blockIdx.x; k < nn; k += gridDim.x) {
        const int64_t r0 = nrp[k], c = nrp[k + 1] - r0;
        const int64_t rs = r0 + c * part / kCscParts, re = r0 + c * (part + 1) / kCscParts;
        uint32_t *mine = cnt + (k * nz + lane) * kCscParts + part;
        uint32_t at = FILL && lane < nz ? *mine : 0u;        // depth `lane`: next position, or count
        const double *v = FILL ? nval + nvq[kNodeParts * k + kNodeParts / kCscParts * part] : nullptr;
        for (int64_t b = rs; b < re; b += 64) {
            const int64_t r = b + lane;
            const uint32_t d = r < re ? ndesc[r] : 0u;
            const int iz0 = (int)(d >> 8), len = (int)(d & 255u);
            uint32_t row = 0;
            int src = 0;                                     // value of depth 0 of the run, from v on
            if (FILL) {
                if (r < re) row = nrow[r];
                const int incl = wave_incl_scan(len);
                src = incl - len - iz0;
            }
            for (int z = 0; z < nz; ++z) {
                const bool in = (unsigned)(z - iz0) < (unsigned)len;
                const uint64_t mask = __ballot(in);
                if (FILL) {
                    const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)at, z);
                    if (in) {
                        const uint32_t p = base + (uint32_t)__popcll(mask & (((uint64_t)1 << lane) - 1));
                        ri[p] = (int32_t)row;
                        cv[p] = v[src + z];
                    }
                }
                if (lane == z) at += (uint32_t)__popcll(mask);
            }
            if (FILL) v += __builtin_amdgcn_readlane(src + iz0 + len, 63);
        }
        if (!FILL && lane < nz) *mine = at;
    }
}

__global__ void k_csc_ptr(int64_t n, int64_t nnz, const uint32_t *cnt, int64_t *cp)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j <= n;
         j += (int64_t)gridDim.x * blockDim.x)
        cp[j] = j < n ? (int64_t)cnt[j * kCscParts] : nnz;
}

// ------------------------------------------------------------ row groups --
// A set of columns as bits in LDS: adds the run [c, c + len), len <= 64, and
// returns how many of its columns were new (f: the new bits of its words).
struct Fresh { uint32_t f[3]; };
__device__ __forceinline__ void run_words(uint32_t c, uint32_t len, uint32_t (&w)[3])
{
    const uint64_t ones = len >= 64 ? ~(uint64_t)0 : ((uint64_t)1 << len) - 1;
    const uint32_t sh = c & 31u;
    const uint64_t lo = ones << sh;
    w[0] = (uint32_t)lo;
    w[1] = (uint32_t)(lo >> 32);
    w[2] = sh ? (uint32_t)(ones >> (64 - sh)) : 0u;
}
__device__ __forceinline__ int add_run(uint32_t *bits, uint32_t c, uint32_t len, Fresh &F)
{
    uint32_t w[3];
    run_words(c, len, w);
    int n = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        F.f[i] = w[i] ? w[i] & ~atomicOr(&bits[(c >> 5) + i], w[i]) : 0u;
        n += __popc(F.f[i]);
    }
    return n;
}

// One wave adds the runs from q on to a set of `cnt` columns, 64 at a time while
// the set stays within cap (rows play no part in the size of a union); the 64
// that overflow it are taken out again and added row by row.  The row that no
// longer fits, m past the last run, or -1 when qend comes first (cnt is then the
// size of the set).
__device__ __forceinline__ int32_t wave_extent(uint32_t *bits, int64_t q, int64_t qend, int64_t nr, int cap, int &cnt,
                                               int64_t m, const uint32_t *col0, const uint8_t *len,
                                               const uint32_t *row_of)
{
    const int lane = threadIdx.x & 63;
    uint32_t c = 0, l = 0;
    if (q + lane < nr) { c = col0[q + lane]; l = len[q + lane]; }
    while (q < qend) {
        uint32_t cn = 0, ln = 0;
        if (q + 64 + lane < nr) { cn = col0[q + 64 + lane]; ln = len[q + 64 + lane]; }
        Fresh F;
        const int tot = group_sum<64>(add_run(bits, c, l, F));
        if (cnt + tot > cap) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (F.f[i]) atomicAnd(&bits[(c >> 5) + i], ~F.f[i]);
            const uint32_t row = q + lane < nr ? row_of[q + lane] : 0u;
            uint64_t todo = __ballot(q + lane < nr);
            while (todo) {
                const uint32_t ri = (uint32_t)__builtin_amdgcn_readlane((int)row, __ffsll((unsigned long long)todo) - 1);
                const bool mine = q + lane < nr && row == ri;
                cnt += group_sum<64>(mine ? add_run(bits, c, l, F) : 0);
                todo &= ~__ballot(mine);
                if (cnt > cap) return (int32_t)ri;
            }
        }
        else cnt += tot;
        q += 64;
        c = cn;
        l = ln;
    }
    return q < nr ? -1 : (int32_t)m;
}

// ext[s] = first row that no longer fits the group that starts at row s (the
// union of the columns of rows s .. ext[s] - 1 holds at most cap, with row
// ext[s] more): the greedy boundaries are then the chain 0, ext[0], ext[ext[0]],
// ...  One wave per start, its column set as bits in LDS.  Every start is tried
// because the chain itself is serial: at 100 M entries, 1.4 ms for all of them.
// A start whose group is longer than `most` runs gets -1: without that limit
// the work grows with the square of the rows where few columns are met (one
// group of all rows on a grid of cap + 1 unknowns).
__global__ __launch_bounds__(64) void k_group_extent(int64_t m, int words, int cap, int64_t most, const int64_t *rrp,
                                                     const uint32_t *col0, const uint8_t *len,
                                                     const uint32_t *row_of, int32_t *ext)
{
    extern __shared__ uint32_t bits[];
    const int lane = threadIdx.x;
    const int64_t nr = rrp[m];
    for (int64_t s = blockIdx.x; s < m; s += gridDim.x) {
        for (int w = lane; w < words; w += 64) bits[w] = 0u;
        __syncthreads();
        int cnt = 0;
        const int64_t q = rrp[s];
        const int32_t e = wave_extent(bits, q, min(nr, q + most), nr, cap, cnt, m, col0, len, row_of);
        if (lane == 0) ext[s] = e;
        __syncthreads();
    }
}

// The chain from row s on, for starts without an extent: one workgroup adds a
// group's runs 1,024 at a time, and its first wave finds the row in the 1,024
// that overflow.  Ends at the first start that has one (or m); *count ends of
// groups in `ends`.  Linear in the runs, since the groups do not overlap.
__global__ __launch_bounds__(1024) void k_group_walk(int64_t m, int words, int cap, int64_t s, const int64_t *rrp,
                                                     const uint32_t *col0, const uint8_t *len,
                                                     const uint32_t *row_of, const int32_t *ext, int32_t *ends,
                                                     int32_t *count)
{
    extern __shared__ uint32_t bits[];
    __shared__ int sums[16];
    __shared__ int32_t end;
    const int tid = threadIdx.x;
    const int64_t nr = rrp[m];
    int groups = 0;
    do {
        for (int w = tid; w < words; w += 1024) bits[w] = 0u;
        __syncthreads();
        int cnt = 0;
        int64_t q = rrp[s];
        uint32_t c = 0, l = 0;
        if (q + tid < nr) { c = col0[q + tid]; l = len[q + tid]; }
        bool over = false;
        while (q < nr) {
            uint32_t cn = 0, ln = 0;
            if (q + 1024 + tid < nr) { cn = col0[q + 1024 + tid]; ln = len[q + 1024 + tid]; }
            Fresh F;
            const int t = group_sum<64>(add_run(bits, c, l, F));
            if ((tid & 63) == 0) sums[tid >> 6] = t;
            __syncthreads();
            int tot = 0;
#pragma unroll
            for (int w = 0; w < 16; ++w) tot += sums[w];
            __syncthreads();
            if (cnt + tot > cap) {                        // uniform
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (F.f[i]) atomicAnd(&bits[(c >> 5) + i], ~F.f[i]);
                over = true;
                break;
            }
            cnt += tot;
            q += 1024;
            c = cn;
            l = ln;
        }
        __syncthreads();
        if (tid < 64) {
            const int32_t e = over ? wave_extent(bits, q, nr, nr, cap, cnt, m, col0, len, row_of) : (int32_t)m;
            if (tid == 0) {
                end = e;
                ends[groups] = e;
            }
        }
        ++groups;
        __syncthreads();
        s = end;
        __syncthreads();
    } while (s < m && ext[s] < 0);
    if (tid == 0) *count = groups;
}

// A workgroup per group: its columns as bits in LDS.  EMIT = false: their
// number to gcnt.  EMIT = true: the sorted list at gcol[gcp[g]] and, for every
// entry of the group's rows, the rank of its column (bits below it in its word
// plus the rank of the word); gridDim.y workgroups share the entries of a group.
template <bool EMIT>
__global__ __launch_bounds__(kBlock) void k_group_cols(int ng, int words, const int32_t *gp,
                                                       const int64_t *rrp, const uint32_t *col0,
                                                       const uint8_t *len, const int64_t *rp,
                                                       const int32_t *ci, uint32_t *gcnt,
                                                       const int64_t *gcp, int32_t *gcol, uint16_t *slot)
{
    extern __shared__ uint32_t bits[];
    uint16_t *rank = (uint16_t *)(bits + words);
    __shared__ int ws[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int per = (words + kBlock - 1) / kBlock;
    for (int g = blockIdx.x; g < ng; g += gridDim.x) {
        for (int w = threadIdx.x; w < words; w += kBlock) bits[w] = 0u;
        __syncthreads();
        const int64_t r0 = gp[g], r1 = gp[g + 1];
        for (int64_t q = rrp[r0] + threadIdx.x; q < rrp[r1]; q += kBlock) {
            uint32_t w[3];
            const uint32_t c = col0[q];
            run_words(c, len[q], w);
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (w[i]) atomicOr(&bits[(c >> 5) + i], w[i]);
        }
        __syncthreads();
        const int w0 = min(words, (int)threadIdx.x * per), w1 = min(words, w0 + per);
        int mine = 0;
        for (int w = w0; w < w1; ++w) mine += __popc(bits[w]);
        const int incl = wave_incl_scan(mine);
        if (lane == 63) ws[wid] = incl;
        __syncthreads();
        if (!EMIT) {
            if (threadIdx.x == 0) gcnt[g] = (uint32_t)(ws[0] + ws[1] + ws[2] + ws[3]);
        } else {
            int at = incl - mine;
            for (int w = 0; w < wid; ++w) at += ws[w];
            const int64_t base = gcp[g];
            for (int w = w0; w < w1; ++w) {
                rank[w] = (uint16_t)at;
                for (uint32_t b = bits[w]; b; b &= b - 1, ++at)
                    if (blockIdx.y == 0) gcol[base + at] = 32 * w + __ffs((int)b) - 1;
            }
            __syncthreads();
            const int64_t p0 = rp[r0], np = rp[r1] - p0, pe = p0 + np * (blockIdx.y + 1) / gridDim.y;
            for (int64_t p = p0 + np * blockIdx.y / gridDim.y + threadIdx.x; p < pe; p += kBlock) {
                const int c = ci[p];
                slot[p] = (uint16_t)(rank[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u)));
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ row blocks --
// Segments of row i: its entries at one lateral node.  cnt[i] (EMIT = false),
// else node, row, position of the first entry at srp[i] on.
template <bool EMIT>
__global__ __launch_bounds__(kBlock) void k_segments(int64_t m, FastDiv nz, const int64_t *rp, const int32_t *ci,
                                                     uint32_t *cnt, const int64_t *srp, uint32_t *node,
                                                     uint32_t *row_of, uint32_t *pos)
{
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t row = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); row < m; row += waves) {
        const int64_t s = rp[row], e = rp[row + 1];
        int64_t base = EMIT ? srp[row] : 0;
        for (int64_t p0 = s; p0 < e; p0 += 64) {
            const int64_t p = p0 + lane;
            bool start = false;
            int k = 0;
            if (p < e) {
                k = (int)nz.div((uint32_t)ci[p]);
                start = p == s || (int)nz.div((uint32_t)ci[p - 1]) != k;
            }
            const uint64_t mask = __ballot(start);
            if (EMIT && start) {
                const int64_t q = base + __popcll(mask & (((uint64_t)1 << lane) - 1));
                node[q] = (uint32_t)k;
                row_of[q] = (uint32_t)row;
                pos[q] = (uint32_t)p;
            }
            base += __popcll(mask);
        }
        if (!EMIT && lane == 0) cnt[row] = (uint32_t)base;
    }
}

// cut[i] = 1 when rows i - 1 and i share fewer than half of the larger one's
// nodes (a wave per row; both lists ascend).
__global__ __launch_bounds__(kBlock) void k_row_cuts(int64_t m, const int64_t *srp, const uint32_t *node,
                                                     uint8_t *cut)
{
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t row = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); row < m; row += waves) {
        if (row == 0) {
            if (lane == 0) cut[0] = 1;
            continue;
        }
        const int64_t a0 = srp[row - 1], a1 = srp[row], b1 = srp[row + 1];
        int common = 0;
        for (int64_t q = a1 + lane; q < b1; q += 64) {
            const uint32_t k = node[q];
            int64_t lo = a0, hi = a1;
            while (lo < hi) {
                const int64_t mid = (lo + hi) / 2;
                if (node[mid] < k) lo = mid + 1;
                else hi = mid;
            }
            common += lo < a1 && node[lo] == k;
        }
        common = group_sum<64>(common);
        if (lane == 0) cut[row] = 2 * (int64_t)common < max(a1 - a0, b1 - a1);
    }
}

// A workgroup per block.  FILL = false: its pairs (ucnt).  FILL = true: its
// pairs' nodes and blocks, and the pair of every segment (slot).
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_blocks(int nb, int nwords, const int32_t *row0, const int64_t *srp,
                                                   const uint32_t *node, uint32_t *ucnt, const uint32_t *pptr,
                                                   uint32_t *pnode, uint32_t *pblk, uint32_t *slot)
{
    extern __shared__ uint32_t bits[];
    uint32_t *rank = bits + nwords;
    __shared__ int ws[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int per = (nwords + kBlock - 1) / kBlock;
    for (int b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t q0 = srp[row0[b]], q1 = srp[row0[b + 1]];
        for (int w = threadIdx.x; w < nwords; w += kBlock) bits[w] = 0u;
        __syncthreads();
        for (int64_t q = q0 + threadIdx.x; q < q1; q += kBlock) atomicOr(&bits[node[q] >> 5], 1u << (node[q] & 31u));
        __syncthreads();
        const int w0 = min(nwords, (int)threadIdx.x * per), w1 = min(nwords, w0 + per);
        int set = 0;
        for (int w = w0; w < w1; ++w) set += __popc(bits[w]);
        const int incl = wave_incl_scan(set);
        if (lane == 63) ws[wid] = incl;
        __syncthreads();
        if (!FILL) {
            if (threadIdx.x == 0) ucnt[b] = (uint32_t)(ws[0] + ws[1] + ws[2] + ws[3]);
        } else {
            const uint32_t p0 = pptr[b];
            int at = incl - set;
            for (int w = 0; w < wid; ++w) at += ws[w];
            for (int w = w0; w < w1; ++w) {
                rank[w] = (uint32_t)at;
                for (uint32_t v = bits[w]; v; v &= v - 1, ++at) {
                    pnode[p0 + at] = (uint32_t)(32 * w + __ffs((int)v) - 1);
                    pblk[p0 + at] = (uint32_t)b;
                }
            }
            __syncthreads();
            for (int64_t q = q0 + threadIdx.x; q < q1; q += kBlock) {
                const uint32_t k = node[q];
                slot[q] = p0 + rank[k >> 5] + (uint32_t)__popc(bits[k >> 5] & ((1u << (k & 31u)) - 1u));
            }
        }
        __syncthreads();
    }
}

// First depth of every pair (lo, from 32 on) and end of the depths of each of
// its row quads (hi, from 0 on).
__global__ void k_windows(int64_t ns, FastDiv nz, const int64_t *rp, const int32_t *ci, const uint32_t *row_of,
                          const uint32_t *pos, const uint32_t *slot, const uint32_t *pblk, const int32_t *row0,
                          uint32_t *lo, uint32_t *hi)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < ns;
         q += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t row = row_of[q], p = slot[q];
        const int64_t end = q + 1 < ns && row_of[q + 1] == row ? (int64_t)pos[q + 1] : rp[row + 1];
        atomicMin(&lo[p], nz.mod((uint32_t)ci[pos[q]]));
        atomicMax(&hi[(int64_t)p * kQuads + ((int)row - row0[pblk[p]]) / 4], nz.mod((uint32_t)ci[end - 1]) + 1u);
    }
}

// 16-byte units of every pair: the depths of its quads.
__global__ void k_tile_size(int64_t np, const uint32_t *lo, const uint32_t *hi, uint32_t *size)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (int64_t)gridDim.x * blockDim.x) {
        uint32_t u = 0;
        for (int q = 0; q < kQuads; ++q) u += max(hi[p * kQuads + q], lo[p]) - lo[p];
        size[p] = u;
    }
}

__global__ void k_pairs(int64_t np, const uint32_t *pnode, const uint32_t *lo, const uint32_t *hi,
                        const uint32_t *size, const int64_t *off, uint4 *pair, uint32_t *key, uint32_t *idx)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += (int64_t)gridDim.x * blockDim.x) {
        uint32_t nds = 0, most = 0;
        for (int q = 0; q < kQuads; ++q) {
            const uint32_t nd = max(hi[p * kQuads + q], lo[p]) - lo[p];
            nds |= nd << (6 * q);
            most = max(most, nd);
        }
        pair[p] = make_uint4(pnode[p] | lo[p] << 20 | most << 26, (uint32_t)off[p], nds, size[p]);
        key[p] = pnode[p];
        idx[p] = (uint32_t)p;
    }
}

// Values of the segments (16 lanes each) into the tiles, zeroed before.
__global__ __launch_bounds__(256) void k_tile_values(int64_t ns, FastDiv nz, const int64_t *rp, const int32_t *ci,
                                                     const double *va, const uint32_t *row_of,
                                                     const uint32_t *pos, const uint32_t *slot,
                                                     const uint32_t *pblk, const int32_t *row0,
                                                     const uint4 *pair, float *val)
{
    const int l = threadIdx.x & 15;
    for (int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4; q < ns; q += (int64_t)gridDim.x * 16) {
        const uint32_t row = row_of[q], p = slot[q];
        const uint4 t = pair[p];
        const int r = (int)row - row0[pblk[p]], d0 = (int)((t.x >> 20) & 31u);
        int64_t u = t.y;
        for (int c = 0; c < r / 4; ++c) u += (t.z >> (6 * c)) & 63u;
        const int64_t end = q + 1 < ns && row_of[q + 1] == row ? (int64_t)pos[q + 1] : rp[row + 1];
        float *o = val + 4 * u + (r & 3);
        for (int64_t k = pos[q] + l; k < end; k += 16) o[4 * ((int)nz.mod((uint32_t)ci[k]) - d0)] = (float)va[k];
    }
}

__global__ void k_node_pairs(int64_t np, const uint32_t *perm, const uint32_t *pblk, const uint4 *pair,
                             const int32_t *row0, uint4 *nlist)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < np; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = perm[i], b = pblk[p];
        const uint4 t = pair[p];
        const int r0 = row0[b];
        nlist[i] = make_uint4(t.y, (uint32_t)r0,
                              (uint32_t)(row0[b + 1] - r0) | ((t.x >> 20) & 31u) << 8 | t.w << 16, t.z);
    }
}

// Temporary device memory of one planning call, given back when it ends (after
// the stream has finished with it).
struct Temps {
    hipStream_t st;
    Allocator &al;
    std::vector<std::pair<void *, size_t>> held;
    bool ok = true;
    Temps(hipStream_t s, Allocator &a) : st(s), al(a) {}
    ~Temps()
    {
        if (held.empty()) return;
        (void)hipStreamSynchronize(st);
        for (auto &h : held) al.put(h.first, h.second);
    }
    void *bytes(size_t b)
    {
        void *p = al.get(b);
        if (p) held.push_back({p, b});
        else ok = false;
        return p;
    }
    template <class T> T *get(int64_t count) { return (T *)bytes((size_t)std::max<int64_t>(count, 1) * sizeof(T)); }
};

template <class In, class Out, class Init>
hipError_t scan_exclusive(Temps &tm, In in, Out out, Init init, int64_t count)
{
    size_t b = 0;
    hipError_t e = rocprim::exclusive_scan(nullptr, b, in, out, init, (size_t)count, rocprim::plus<Init>(), tm.st);
    if (e != hipSuccess) return e;
    void *t = tm.bytes(b);
    if (!t) return hipErrorOutOfMemory;
    return rocprim::exclusive_scan(t, b, in, out, init, (size_t)count, rocprim::plus<Init>(), tm.st);
}

hipError_t sort_pairs(Temps &tm, rocprim::double_buffer<uint32_t> &keys,
                      rocprim::double_buffer<uint32_t> &vals, int64_t count, int bits)
{
    size_t b = 0;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, b, keys, vals, (size_t)count, 0, bits, tm.st);
    if (e != hipSuccess) return e;
    void *t = tm.bytes(b);
    if (!t) return hipErrorOutOfMemory;
    return rocprim::radix_sort_pairs(t, b, keys, vals, (size_t)count, 0, bits, tm.st);
}

template <int W>
hipError_t starts(Temps &tm, const RunPlan &R, uint32_t *start)
{
    return scan_exclusive(tm, rocprim::make_transform_iterator(R.ndesc, PaddedLen<W>{}), start, (uint32_t)0, R.nr);
}

#define PL_TRY(expr)                          \
    do {                                      \
        const hipError_t _e = (expr);         \
        if (_e != hipSuccess) return _e;      \
    } while (0)
#define PL_OK(tm) PL_TRY((tm).ok ? hipSuccess : hipErrorOutOfMemory)

}  // namespace

hipError_t plan_scan_rows(hipStream_t st, int64_t m, int64_t n, int64_t nnz, int nz, const int64_t *rp,
                          const int32_t *ci, const double *check, uint32_t *cnt, int *info)
{
    PL_TRY(hipMemsetAsync(info, 0, 2 * sizeof(int), st));
    const int g = blocks(m, kBlock / 64, 8192);
    if (check) hipLaunchKernelGGL((k_scan_rows<true>), dim3(g), dim3(kBlock), 0, st, m, n, nnz, FastDiv((uint32_t)nz), rp, ci, check, cnt, info);
    else hipLaunchKernelGGL((k_scan_rows<false>), dim3(g), dim3(kBlock), 0, st, m, n, nnz, FastDiv((uint32_t)nz), rp, ci, check, cnt, info);
    return hipGetLastError();
}

hipError_t plan_row_runs(hipStream_t st, Allocator &al, int64_t m, const uint32_t *cnt, int64_t *rrp,
                         int64_t *nr)
{
    Temps tm(st, al);
    PL_TRY(scan_exclusive(tm, cnt, rrp, (int64_t)0, m + 1));
    PL_TRY(hipMemcpyAsync(nr, rrp + m, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    return hipStreamSynchronize(st);
}

hipError_t plan_emit_runs(hipStream_t st, int64_t m, int nz, const int64_t *rp, const int32_t *ci,
                          const RunPlan &R, uint32_t *key, uint32_t *idx)
{
    hipLaunchKernelGGL(k_emit_runs, dim3(blocks(m, kBlock / 64, 16384)), dim3(kBlock), 0, st, m, FastDiv((uint32_t)nz), rp, ci,
                       R.rrp, R.src, R.row, R.col0, key, idx);
    hipLaunchKernelGGL(k_run_len, dim3(blocks(R.nr, 256, 16384)), dim3(256), 0, st, R.nr, rp, R.src, R.row, R.len);
    return hipGetLastError();
}

hipError_t plan_node_runs(hipStream_t st, Allocator &al, int64_t nn, int nz, RunPlan &R, uint32_t *key,
                          uint32_t *idx, uint64_t *padded)
{
    Temps tm(st, al);
    uint32_t *k1 = tm.get<uint32_t>(R.nr), *i1 = tm.get<uint32_t>(R.nr);
    unsigned long long *tot = tm.get<unsigned long long>(3);
    uint32_t *ok0 = tm.get<uint32_t>(nn), *ok1 = tm.get<uint32_t>(nn), *on0 = tm.get<uint32_t>(nn);
    PL_OK(tm);
    rocprim::double_buffer<uint32_t> keys(key, k1), vals(idx, i1);
    PL_TRY(sort_pairs(tm, keys, vals, R.nr, bits_for(nn)));
    launch_key_ptr(st, R.nr, nn, keys.current(), R.nrp);
    PL_TRY(hipMemsetAsync(tot, 0, 3 * sizeof(unsigned long long), st));
    hipLaunchKernelGGL(k_node_runs, dim3(blocks(R.nr, kBlock, 8192)), dim3(kBlock), 0, st, R.nr, FastDiv((uint32_t)nz),
                       vals.current(), R.src, R.row, R.col0, R.len, R.nsrc, R.nrow, R.ndesc, R.rrid, tot);
    hipLaunchKernelGGL(k_order_keys, dim3(blocks(nn, 256, 1024)), dim3(256), 0, st, nn, R.nrp, ok0, on0);
    rocprim::double_buffer<uint32_t> okey(ok0, ok1), onode(on0, (uint32_t *)R.norder);
    PL_TRY(sort_pairs(tm, okey, onode, nn, 32));
    if (onode.current() != (uint32_t *)R.norder)
        PL_TRY(hipMemcpyAsync(R.norder, onode.current(), nn * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
    PL_TRY(hipMemcpyAsync(padded, tot, 3 * sizeof(uint64_t), hipMemcpyDeviceToHost, st));
    return hipStreamSynchronize(st);
}

hipError_t plan_layout(hipStream_t st, Allocator &al, int64_t nn, const RunPlan &R, int W, int64_t total,
                       uint32_t *start, int64_t *nvq)
{
    Temps tm(st, al);
    switch (W) {
    case 1: PL_TRY((starts<1>(tm, R, start))); break;
    case 2: PL_TRY((starts<2>(tm, R, start))); break;
    case 4: PL_TRY((starts<4>(tm, R, start))); break;
    default: PL_TRY((starts<8>(tm, R, start))); break;
    }
    hipLaunchKernelGGL(k_parts, dim3(blocks(kNodeParts * nn + 1, 256, 4096)), dim3(256), 0, st, nn, R.nr, R.nrp,
                       start, total, nvq);
    return hipGetLastError();
}

hipError_t plan_csc(hipStream_t st, Allocator &al, int64_t n, int nz, int64_t nnz, const RunPlan &R,
                    const int64_t *nvq, const double *nval, int64_t *cp, int32_t *ri, double *cv)
{
    Temps tm(st, al);
    uint32_t *cnt = tm.get<uint32_t>(n * kCscParts), *at = tm.get<uint32_t>(n * kCscParts);
    PL_OK(tm);
    const int64_t nn = n / nz;
    const int g = (int)std::min<int64_t>(nn, 16384);
    hipLaunchKernelGGL((k_csc<false>), dim3(g), dim3(64 * kCscParts), 0, st, nn, nz, R.nrp, R.ndesc, R.nrow,
                       nvq, nval, cnt, ri, cv);
    PL_TRY(scan_exclusive(tm, cnt, at, (uint32_t)0, n * kCscParts));
    hipLaunchKernelGGL(k_csc_ptr, dim3(blocks(n + 1, 256, 4096)), dim3(256), 0, st, n, nnz, at, cp);
    hipLaunchKernelGGL((k_csc<true>), dim3(g), dim3(64 * kCscParts), 0, st, nn, nz, R.nrp, R.ndesc, R.nrow,
                       nvq, nval, at, ri, cv);
    return hipGetLastError();
}

bool plan_groups_fit(int64_t n, int nz) { return n <= kPlanMaxCols && nz <= 64; }

// Runs that all starts of k_group_extent may look at together: 64 times the runs
// there are, or this many where that is more (about 25 ms).
constexpr int64_t kExtentRuns = (int64_t)1 << 31;

hipError_t plan_group_bounds(hipStream_t st, Allocator &al, int64_t m, int64_t n, int cap, const RunPlan &R,
                             std::vector<int32_t> &gp)
{
    gp.assign(1, 0);
    if (n <= cap) {                                        // every set of rows fits
        gp.push_back((int32_t)m);
        return hipSuccess;
    }
    Temps tm(st, al);
    int32_t *ext = tm.get<int32_t>(m);
    PL_OK(tm);
    const int words = (int)((n + 31) / 32);
    const int64_t most = std::max(64 * ((R.nr + m - 1) / m), kExtentRuns / m);
    hipLaunchKernelGGL(k_group_extent, dim3(blocks(m, 1, 1 << 20)), dim3(64), words * 4, st, m, words, cap, most,
                       R.rrp, R.col0, R.len, R.row, ext);
    PL_TRY(hipGetLastError());
    std::vector<int32_t> h((size_t)m);
    PL_TRY(hipMemcpyAsync(h.data(), ext, m * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    PL_TRY(hipStreamSynchronize(st));
    int32_t *ends = nullptr;                               // [1 + m]: their number, then the ends
    std::vector<int32_t> walked;
    for (int64_t s = 0; s < m; s = gp.back()) {
        if (h[(size_t)s] >= 0) {
            if (h[(size_t)s] <= s || h[(size_t)s] > m) return hipErrorUnknown;
            gp.push_back(h[(size_t)s]);
            continue;
        }
        if (!ends) ends = tm.get<int32_t>(1 + m);
        PL_OK(tm);
        hipLaunchKernelGGL(k_group_walk, dim3(1), dim3(1024), words * 4, st, m, words, cap, s, R.rrp, R.col0, R.len,
                           R.row, ext, ends + 1, ends);
        PL_TRY(hipGetLastError());
        int32_t count = 0;
        PL_TRY(hipMemcpyAsync(&count, ends, sizeof(count), hipMemcpyDeviceToHost, st));
        PL_TRY(hipStreamSynchronize(st));
        if (count < 1 || count > m - s) return hipErrorUnknown;
        walked.resize((size_t)count);
        PL_TRY(hipMemcpyAsync(walked.data(), ends + 1, count * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        PL_TRY(hipStreamSynchronize(st));
        for (int32_t e : walked) {
            if (e <= gp.back() || e > m) return hipErrorUnknown;
            gp.push_back(e);
        }
    }
    return hipSuccess;
}

hipError_t plan_group_sizes(hipStream_t st, Allocator &al, int64_t n, int ng, const int32_t *gp, const RunPlan &R,
                            int64_t *gcp, int64_t *total)
{
    Temps tm(st, al);
    uint32_t *cnt = tm.get<uint32_t>(ng + 1);
    PL_OK(tm);
    const int words = (int)((n + 31) / 32);
    PL_TRY(hipMemsetAsync(cnt + ng, 0, sizeof(uint32_t), st));
    hipLaunchKernelGGL((k_group_cols<false>), dim3(blocks(ng, 1, 1 << 20)), dim3(kBlock), words * 4, st, ng, words,
                       gp, R.rrp, R.col0, R.len, (const int64_t *)nullptr, (const int32_t *)nullptr, cnt,
                       (const int64_t *)nullptr, (int32_t *)nullptr, (uint16_t *)nullptr);
    PL_TRY(scan_exclusive(tm, cnt, gcp, (int64_t)0, (int64_t)ng + 1));
    PL_TRY(hipMemcpyAsync(total, gcp + ng, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    return hipStreamSynchronize(st);
}

hipError_t plan_group_lists(hipStream_t st, int64_t n, int ng, const int32_t *gp, const RunPlan &R,
                            const int64_t *rp, const int32_t *ci, const int64_t *gcp, int32_t *gcol, uint16_t *slot)
{
    const int words = (int)((n + 31) / 32);
    // long groups: their entries (not their runs) are shared by up to 256 workgroups
    const int parts = blocks(R.nr / std::max(ng, 1), 1 << 15, 256);
    hipLaunchKernelGGL((k_group_cols<true>), dim3(blocks(ng, 1, 1 << 20), parts), dim3(kBlock), words * 6 + 4, st, ng, words,
                       gp, R.rrp, R.col0, R.len, rp, ci, (uint32_t *)nullptr, gcp, gcol, slot);
    return hipGetLastError();
}

// Blocks pay where a pair serves at least 4.5 (row, node) segments: a pair costs
// its nodes' rows and its products whatever its rows hold.  Both products of 32
// right-hand sides at 3 and 5 periods a path: 1,690 and 1,870 us, over runs and
// entries 1,290 and 2,000; of 8: 332 and 351 us against 349 and 526.  And where the
// tiles hold at most two values per entry: past that they are more to read than
// the entries with their columns.
constexpr int64_t kMinSegmentsPer2Pairs = 9, kMaxTileFill = 2;

hipError_t plan_row_blocks(hipStream_t st, Allocator &al, int64_t m, int64_t n, int nz, const int64_t *rp,
                           const int32_t *ci, const double *va, RowBlocks &B,
                           const std::function<void *(size_t)> &keep)
{
    B = RowBlocks{};
    const int64_t nn = n / nz;
    if (m < 1 || nz > 32 || nn > kPlanMaxNodes) return hipSuccess;
    Temps tm(st, al);
    uint32_t *cnt = tm.get<uint32_t>(m + 1);
    int64_t *srp = tm.get<int64_t>(m + 1);
    uint8_t *cut = tm.get<uint8_t>(m);
    PL_OK(tm);
    const int gr = blocks(m, kBlock / 64, 16384);
    hipLaunchKernelGGL((k_segments<false>), dim3(gr), dim3(kBlock), 0, st, m, FastDiv((uint32_t)nz), rp, ci, cnt,
                       (const int64_t *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr);
    PL_TRY(scan_exclusive(tm, cnt, srp, (int64_t)0, m + 1));
    int64_t ends[2] = {0, 0};                              // segments, entries
    PL_TRY(hipMemcpyAsync(&ends[0], srp + m, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    PL_TRY(hipMemcpyAsync(&ends[1], rp + m, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    PL_TRY(hipStreamSynchronize(st));
    const int64_t ns = ends[0];
    if (ns == 0) return hipSuccess;
    uint32_t *node = tm.get<uint32_t>(ns), *row_of = tm.get<uint32_t>(ns), *pos = tm.get<uint32_t>(ns);
    uint32_t *slot = tm.get<uint32_t>(ns);
    PL_OK(tm);
    hipLaunchKernelGGL((k_segments<true>), dim3(gr), dim3(kBlock), 0, st, m, FastDiv((uint32_t)nz), rp, ci, (uint32_t *)nullptr, srp,
                       node, row_of, pos);
    hipLaunchKernelGGL(k_row_cuts, dim3(gr), dim3(kBlock), 0, st, m, srp, node, cut);
    // blocks: the rows between two cuts in equal parts, of at most 20 where most
    // rows lie in runs of 17 to 20 (one block instead of two), else of at most 16
    // (the kernels of one row tile).  32 right-hand sides, 19 rows a path, both
    // products: 2.95 ms with 20, 3.62 with 16; 8, 13 rows a path: 494 and 471 us.
    std::vector<uint8_t> hc((size_t)m);
    PL_TRY(hipMemcpyAsync(hc.data(), cut, (size_t)m, hipMemcpyDeviceToHost, st));
    PL_TRY(hipStreamSynchronize(st));
    std::vector<int32_t> r0;
    int rows_max = 0;
    int64_t between = 0;
    for (int64_t i = 0, e = 0; i < m; i = e) {
        for (e = i + 1; e < m && !hc[(size_t)e];) ++e;
        if (e - i > 16 && e - i <= kBlockRows) between += e - i;
    }
    const int64_t limit = 2 * between > m ? kBlockRows : 16;
    for (int64_t i = 0; i < m;) {
        int64_t e = i + 1;
        while (e < m && !hc[(size_t)e]) ++e;
        const int64_t parts = (e - i + limit - 1) / limit;
        for (int64_t k = 0; k < parts; ++k) r0.push_back((int32_t)(i + (e - i) * k / parts));
        rows_max = std::max(rows_max, (int)((e - i + parts - 1) / parts));
        i = e;
    }
    const int nb = (int)r0.size();
    r0.push_back((int32_t)m);
    int32_t *row0 = tm.get<int32_t>(nb + 1);
    uint32_t *ucnt = tm.get<uint32_t>(nb + 1);
    uint32_t *pptr = tm.get<uint32_t>(nb + 1);
    PL_OK(tm);
    PL_TRY(hipMemcpyAsync(row0, r0.data(), (nb + 1) * sizeof(int32_t), hipMemcpyHostToDevice, st));
    const int nw = (int)((nn + 31) / 32);
    const int gb = blocks(nb, 1, 1 << 20);
    hipLaunchKernelGGL((k_blocks<false>), dim3(gb), dim3(kBlock), nw * 8, st, nb, nw, row0, srp, node, ucnt,
                       (const uint32_t *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr);
    PL_TRY(scan_exclusive(tm, ucnt, pptr, (uint32_t)0, (int64_t)nb + 1));
    uint32_t hp = 0;
    PL_TRY(hipMemcpyAsync(&hp, pptr + nb, sizeof(hp), hipMemcpyDeviceToHost, st));
    PL_TRY(hipStreamSynchronize(st));
    const int64_t np = hp;
    if (2 * ns < kMinSegmentsPer2Pairs * np) return hipSuccess;
    uint32_t *pnode = tm.get<uint32_t>(np), *pblk = tm.get<uint32_t>(np), *lo = tm.get<uint32_t>(np);
    uint32_t *hi = tm.get<uint32_t>(np * kQuads), *size = tm.get<uint32_t>(np + 1);
    int64_t *off = tm.get<int64_t>(np + 1);
    PL_OK(tm);
    PL_TRY(hipMemsetAsync(lo, 0x7f, np * sizeof(uint32_t), st));
    PL_TRY(hipMemsetAsync(hi, 0, np * kQuads * sizeof(uint32_t), st));
    hipLaunchKernelGGL((k_blocks<true>), dim3(gb), dim3(kBlock), nw * 8, st, nb, nw, row0, srp, node,
                       (uint32_t *)nullptr, pptr, pnode, pblk, slot);
    const int gp = blocks(np, 256, 16384);
    hipLaunchKernelGGL(k_windows, dim3(blocks(ns, 256, 16384)), dim3(256), 0, st, ns, FastDiv((uint32_t)nz), rp, ci, row_of, pos, slot, pblk,
                       row0, lo, hi);
    hipLaunchKernelGGL(k_tile_size, dim3(gp), dim3(256), 0, st, np, lo, hi, size);
    PL_TRY(scan_exclusive(tm, size, off, (int64_t)0, np + 1));
    int64_t units = 0;
    PL_TRY(hipMemcpyAsync(&units, off + np, sizeof(units), hipMemcpyDeviceToHost, st));
    PL_TRY(hipStreamSynchronize(st));
    if (units >= ((int64_t)1 << 32) || 4 * units > kMaxTileFill * ends[1] + 4 * np) return hipSuccess;
    const size_t vbytes = (size_t)units * 16;
    B.row0 = (int32_t *)keep((nb + 1) * sizeof(int32_t));
    B.pptr = (uint32_t *)keep((nb + 1) * sizeof(uint32_t));
    B.pair = (uint4 *)keep(np * sizeof(uint4));
    B.val = (float *)keep(vbytes);
    B.nptr = (int64_t *)keep((nn + 1) * sizeof(int64_t));
    B.nlist = (uint4 *)keep(np * sizeof(uint4));
    B.norder = (int32_t *)keep(nn * sizeof(int32_t));
    uint32_t *k0 = tm.get<uint32_t>(np), *k1 = tm.get<uint32_t>(np);
    uint32_t *i0 = tm.get<uint32_t>(np), *i1 = tm.get<uint32_t>(np);
    uint32_t *ok0 = tm.get<uint32_t>(nn), *ok1 = tm.get<uint32_t>(nn), *on0 = tm.get<uint32_t>(nn);
    PL_OK(tm);
    if (!B.row0 || !B.pptr || !B.pair || !B.val || !B.nptr || !B.nlist || !B.norder) return hipErrorOutOfMemory;
    PL_TRY(hipMemcpyAsync(B.row0, row0, (nb + 1) * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
    PL_TRY(hipMemcpyAsync(B.pptr, pptr, (nb + 1) * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
    PL_TRY(hipMemsetAsync(B.val, 0, vbytes, st));
    hipLaunchKernelGGL(k_pairs, dim3(gp), dim3(256), 0, st, np, pnode, lo, hi, size, off, B.pair, k0, i0);
    hipLaunchKernelGGL(k_tile_values, dim3(blocks(ns, 16, 65536)), dim3(256), 0, st, ns, FastDiv((uint32_t)nz), rp, ci, va, row_of, pos,
                       slot, pblk, row0, B.pair, B.val);
    rocprim::double_buffer<uint32_t> keys(k0, k1), idx(i0, i1);
    PL_TRY(sort_pairs(tm, keys, idx, np, bits_for(nn)));
    launch_key_ptr(st, np, nn, keys.current(), B.nptr);
    hipLaunchKernelGGL(k_node_pairs, dim3(gp), dim3(256), 0, st, np, idx.current(), pblk, B.pair, row0, B.nlist);
    hipLaunchKernelGGL(k_order_keys, dim3(blocks(nn, 256, 1024)), dim3(256), 0, st, nn, B.nptr, ok0, on0);
    rocprim::double_buffer<uint32_t> okey(ok0, ok1), onode(on0, (uint32_t *)B.norder);
    PL_TRY(sort_pairs(tm, okey, onode, nn, 32));
    if (onode.current() != (uint32_t *)B.norder)
        PL_TRY(hipMemcpyAsync(B.norder, onode.current(), nn * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
    PL_TRY(hipGetLastError());
    PL_TRY(hipStreamSynchronize(st));
    B.nb = nb;
    B.rows_max = rows_max;
    B.np = np;
    return hipSuccess;
}

}  // namespace lsqr
