// Learned column scaling: per-column features, the MLP 6 -> 64 -> 64 -> 1
// (GELU, softplus output) for inference in BF16 (weights and activations
// rounded to nearest-even, FP32 accumulation), and FP32 training kernels
// (forward/backward per sample, per-parameter gradient sums in a fixed order,
// Adam).  The multiplier softplus(z) scales the Jacobi column scale.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "ctx.h"
#include "lsqr_kernels.cuh"

using namespace lsqr;

namespace {

constexpr int H = 64;
constexpr int NF = 6;
// flat parameter layout: W1 [H][NF], b1 [H], W2 [H][H], b2 [H], W3 [H], b3 [1]
constexpr int OW1 = 0, OB1 = OW1 + H * NF, OW2 = OB1 + H, OB2 = OW2 + H * H, OW3 = OB2 + H,
              OB3 = OW3 + H, NP = OB3 + 1;
static_assert(NP == LSQR_MLP_NPARAMS, "parameter count");

__device__ __forceinline__ float gelu(float x)
{
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad(float x)
{
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) +
           x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

__device__ __forceinline__ float softplus(float z)
{
    return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));
}

__device__ __forceinline__ float sigmoid(float z) { return 0.5f * (1.0f + tanhf(0.5f * z)); }

// FP32 -> BF16 -> FP32, round to nearest even (finite inputs)
__device__ __forceinline__ float bf16r(float x)
{
    uint32_t u = __float_as_uint(x);
    const uint32_t lsb = (u >> 16) & 1u;
    u += 0x7FFFu + lsb;
    return __uint_as_float(u & 0xFFFF0000u);
}

// ----------------------------------------------------------------- features --
// Both kernels stream the matrix once (12 bytes an entry: 160 us on 95 M entries at
// the rate of a streaming read), a wave per row or column with four loads a lane
// in flight, sums in the order of the entries: 276 -> 268 and 450 -> 443 us, so
// they are not bound by latency but by the FP64 and address arithmetic of each
// entry, the columns also by the gather of the rows' centroids.
constexpr int kFeatUnroll = 4;

__global__ __launch_bounds__(256) void k_row_centroid(int64_t m, FastDiv fz, const int64_t *rp, const int32_t *ci,
                                                      const double *va, double *cen)
{
    const int lane = threadIdx.x & 63;
    const double zden = fz.d > 1 ? (double)(fz.d - 1) : 1.0;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; i < m;
         i += ((int64_t)gridDim.x * blockDim.x) >> 6) {
        double sa = 0.0, sz = 0.0;
        const int64_t end = rp[i + 1];
        for (int64_t e = rp[i] + lane; e < end; e += 64 * kFeatUnroll) {
            double v[kFeatUnroll];
            int c[kFeatUnroll];
#pragma unroll
            for (int u = 0; u < kFeatUnroll; ++u) {
                const int64_t q = min(e + 64 * u, end - 1);
                v[u] = __builtin_nontemporal_load(va + q);
                c[u] = __builtin_nontemporal_load(ci + q);
            }
#pragma unroll
            for (int u = 0; u < kFeatUnroll; ++u)
                if (e + 64 * u < end) {
                    const double a = fabs(v[u]);
                    sa += a;
                    sz += a * (double)fz.mod((uint32_t)c[u]);
                }
        }
        sa = group_sum<64>(sa);
        sz = group_sum<64>(sz);
        if (lane == 0) cen[i] = sa > 0.0 ? sz / sa / zden : 0.0;
    }
}

__global__ __launch_bounds__(256) void k_col_features(int n, int nx, int ny, int nz, double w, double damp,
                                                      const int64_t *cp, const int32_t *ri, const double *cv,
                                                      const double *cen, float *feat)
{
    const int lane = threadIdx.x & 63;
    const double zden = nz > 1 ? (double)(nz - 1) : 1.0;
    for (int j = (int)((((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6)); j < n;
         j += (int)(((int64_t)gridDim.x * blockDim.x) >> 6)) {
        double g2 = 0.0, ca = 0.0, c1 = 0.0, c2 = 0.0;
        const int64_t end = cp[j + 1];
        for (int64_t p = cp[j] + lane; p < end; p += 64 * kFeatUnroll) {
            double v[kFeatUnroll], ce[kFeatUnroll];
            int r[kFeatUnroll];
#pragma unroll
            for (int u = 0; u < kFeatUnroll; ++u) {
                const int64_t q = min(p + 64 * u, end - 1);
                r[u] = __builtin_nontemporal_load(ri + q);
                v[u] = __builtin_nontemporal_load(cv + q);
            }
#pragma unroll
            for (int u = 0; u < kFeatUnroll; ++u) ce[u] = cen[r[u]];
#pragma unroll
            for (int u = 0; u < kFeatUnroll; ++u)
                if (p + 64 * u < end) {
                    const double g = v[u], a = fabs(g), c = ce[u];
                    g2 += g * g;
                    ca += a;
                    c1 += a * c;
                    c2 += a * c * c;
                }
        }
        g2 = group_sum<64>(g2);
        ca = group_sum<64>(ca);
        c1 = group_sum<64>(c1);
        c2 = group_sum<64>(c2);
        if (lane == 0) {
            const int iz = j % nz, ixy = j / nz, ix = ixy % nx, iy = ixy / nx;
            const int sxy = nx * nz;
            int deg = 0;
            double nb = 0.0;
            auto hit = [&](int q) { return (double)(cp[q + 1] - cp[q]); };
            if (ix > 0) { nb += hit(j - nz); ++deg; }
            if (ix < nx - 1) { nb += hit(j + nz); ++deg; }
            if (iy > 0) { nb += hit(j - sxy); ++deg; }
            if (iy < ny - 1) { nb += hit(j + sxy); ++deg; }
            if (iz > 0) { nb += hit(j - 1); ++deg; }
            if (iz < nz - 1) { nb += hit(j + 1); ++deg; }
            const double colnorm2 = g2 + w * w * (double)(deg * deg + deg) + damp * damp;
            const double mean = ca > 0.0 ? c1 / ca : 0.0;
            const double var = ca > 0.0 ? c2 / ca - mean * mean : 0.0;
            float *f = feat + (int64_t)j * NF;
            f[0] = (float)(0.5 * log10(colnorm2));
            f[1] = (float)log1p(hit(j));
            f[2] = (float)((double)iz / zden);
            f[3] = (float)mean;
            f[4] = (float)sqrt(var > 0.0 ? var : 0.0);
            f[5] = (float)log1p(deg > 0 ? nb / (double)deg : 0.0);
        }
    }
}

// ---------------------------------------------------------------- inference --
struct Norm {
    float mean[NF], inv_std[NF];
};

// Sums over the system's columns of the features flagged in `mask` (FP64, fixed
// order): workgroup b adds its columns' to part[b][NF].  One workgroup for all
// took 335 us on 128,000 columns, now 5 us.
constexpr int kMeanParts = 64;

__global__ __launch_bounds__(256) void k_feature_sums(int n, const float *feat, unsigned mask,
                                                      double *part)
{
    __shared__ double acc[4];
    const int per = (n + kMeanParts - 1) / kMeanParts, j0 = blockIdx.x * per, j1 = min(n, j0 + per);
    for (int f = 0; f < NF; ++f) {
        double sum = 0.0;
        if ((mask >> f) & 1u)
            for (int j = j0 + threadIdx.x; j < j1; j += 256) sum += (double)feat[(int64_t)j * NF + f];
        sum = group_sum<64>(sum);
        if ((threadIdx.x & 63) == 0) acc[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) part[blockIdx.x * NF + f] = ((acc[0] + acc[1]) + acc[2]) + acc[3];
        __syncthreads();
    }
}

// d_j = djac_j * softplus(z_j), BF16 weights and activations, FP32 sums.
// Features flagged in `mask` are centred on the system's own means (part:
// k_feature_sums).
__global__ __launch_bounds__(256) void k_mlp_infer(int n, const float *params, Norm nrm,
                                                   unsigned mask, const double *part,
                                                   const float *feat, const double *djac,
                                                   double *d)
{
    __shared__ float W[NP];
    __shared__ float mu[NF];
    for (int i = threadIdx.x; i < NP; i += blockDim.x) W[i] = bf16r(params[i]);
    static_assert(kMeanParts == 64, "a lane per partial sum");
    for (int f = threadIdx.x >> 6; f < NF; f += 4) {
        const double sum = group_sum<64>(part[(threadIdx.x & 63) * NF + f]);
        if ((threadIdx.x & 63) == 0) mu[f] = ((mask >> f) & 1u) ? (float)(sum / (double)n) : nrm.mean[f];
    }
    __syncthreads();
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        float x[NF];
        for (int f = 0; f < NF; ++f)
            x[f] = bf16r((feat[(int64_t)j * NF + f] - mu[f]) * nrm.inv_std[f]);
        float h1[H];
        for (int k = 0; k < H; ++k) {
            float a = W[OB1 + k];
            for (int f = 0; f < NF; ++f) a = fmaf(W[OW1 + k * NF + f], x[f], a);
            h1[k] = bf16r(gelu(a));
        }
        float z = W[OB3];
        for (int k = 0; k < H; ++k) {
            float a = W[OB2 + k];
            for (int l = 0; l < H; ++l) a = fmaf(W[OW2 + k * H + l], h1[l], a);
            z = fmaf(W[OW3 + k], bf16r(gelu(a)), z);
        }
        d[j] = djac[j] * (double)softplus(z);
    }
}

// ----------------------------------------------------------------- training --
// Forward and backward of a minibatch and its weight gradient in one kernel:
// a workgroup takes tiles of kTile samples, 8 to a wave, lane k of a wave
// owning neuron k of both hidden layers (the 8 samples' activations are read
// from LDS as broadcasts, W2 by row and by column with a padded row, both
// without bank conflicts; per neuron the sums run over the inputs in order).
// The tile's activations and deltas stay in LDS, and every thread then adds
// its 16 entries of d2 h1^T (and the smaller blocks) over the tile's samples
// in FP64; k_mlp_reduce adds the workgroups' partial gradients in order.
// What bounds it is latency, a chain of ~20 LDS phases per tile: at the
// default minibatch of 4,096, 99 us (one thread per sample on 16 workgroups)
// plus 1,043 us for the weight gradient (one thread per parameter walking
// the whole batch) became 24.5 us plus 4.8 us for k_mlp_reduce.  Tiles of 16
// samples measured 22.0 + 7.3 us: the same.
constexpr int kTile = 32;                 // samples per workgroup and tile
constexpr int kTW = kTile / 4;            // samples per wave
constexpr int kW2S = H + 1;               // padded row of W2 in LDS
constexpr int kTS = kTW + 4;              // padded row of the per-neuron sample arrays
constexpr int kMaxTileGroups = 512;       // workgroups (partial gradients) at most

// the kTW samples of one neuron (or feature) of a wave
__device__ __forceinline__ void ld_samples(const float *p, float (&v)[kTW])
{
#pragma unroll
    for (int q = 0; q < kTW / 4; ++q) {
        const float4 a = *(const float4 *)(p + 4 * q);
        v[4 * q] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
    }
}
__device__ __forceinline__ void st_samples(float *p, const float (&v)[kTW])
{
#pragma unroll
    for (int q = 0; q < kTW / 4; ++q)
        *(float4 *)(p + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

// Partial gradient of workgroup b in gpart[b][NP] (FP64), its part of the
// squared residuals in part[b].
__global__ __launch_bounds__(256) void k_mlp_grad(int B, const float *params, const float *x,
                                                  const float *target, double *gpart, double *part)
{
    static_assert(kTW % 4 == 0, "whole float4s of samples");
    __shared__ float w2[H * kW2S];
    __shared__ __align__(16) float h1s[4][H * kTS], h2s[4][H * kTS], d1s[4][H * kTS], d2s[4][H * kTS];
    // per wave and sample: the features, then dz and 1, as rows of kTS like the
    // neurons', so that a product of two rows covers every small parameter
    __shared__ __align__(16) float xs[4][(NF + 2) * kTS];
    __shared__ double lds[4];
    const int k = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < H * H; i += 256) w2[(i / H) * kW2S + i % H] = params[OW2 + i];
    float w1[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) w1[f] = params[OW1 + k * NF + f];
    const float b1 = params[OB1 + k], b2 = params[OB2 + k], w3 = params[OW3 + k], b3 = params[OB3];
    // the thread's entries of W2: rows tk + 16 i, columns tl + 16 j
    const int tk = threadIdx.x >> 4, tl = threadIdx.x & 15;
    double g2[4][4] = {}, gs[3] = {0.0, 0.0, 0.0};
    // the thread's parameters outside W2 (W1 and b1, the first OW2, then b2, W3,
    // b3): each the sum over the samples of one row times another
    constexpr int NS = NP - H * H;
    const float *ra[3], *rb[3];
    int sa[3], sb[3];                     // strides from wave to wave
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int q = threadIdx.x + 256 * u, p = q < OW2 ? q : q + H * H;
        ra[u] = rb[u] = &xs[0][(NF + 1) * kTS];
        sa[u] = sb[u] = (NF + 2) * kTS;
        if (p < OB1) { ra[u] = &d1s[0][p / NF * kTS]; sa[u] = H * kTS; rb[u] = &xs[0][p % NF * kTS]; }
        else if (p < OW2) { ra[u] = &d1s[0][(p - OB1) * kTS]; sa[u] = H * kTS; }
        else if (p < OW3) { ra[u] = &d2s[0][(p - OB2) * kTS]; sa[u] = H * kTS; }
        else if (p < OB3) { ra[u] = &h2s[0][(p - OW3) * kTS]; sa[u] = H * kTS; rb[u] = &xs[0][NF * kTS]; }
        else if (p < NP) rb[u] = &xs[0][NF * kTS];
    }
    double sq = 0.0;
    const int tiles = (B + kTile - 1) / kTile;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        __syncthreads();                  // w2 is in place, the previous tile's reads are done
        if (threadIdx.x < kTile * NF) {
            const int i = threadIdx.x / NF, f = threadIdx.x % NF, b = t * kTile + i;
            xs[i / kTW][f * kTS + i % kTW] = b < B ? x[(int64_t)b * NF + f] : 0.0f;
        }
        if (threadIdx.x < kTile) xs[threadIdx.x / kTW][(NF + 1) * kTS + threadIdx.x % kTW] = 1.0f;
        __syncthreads();
        const int s0 = wid * kTW;
        float a1[kTW], a2[kTW], h[kTW];
#pragma unroll
        for (int s = 0; s < kTW; ++s) {
            float a = b1;
#pragma unroll
            for (int f = 0; f < NF; ++f) a = fmaf(w1[f], xs[wid][f * kTS + s], a);
            a1[s] = a;
            h[s] = gelu(a);
            a2[s] = b2;
        }
        st_samples(&h1s[wid][k * kTS], h);
        __syncthreads();
#pragma unroll 8
        for (int l = 0; l < H; ++l) {
            ld_samples(&h1s[wid][l * kTS], h);
            const float w = w2[k * kW2S + l];
#pragma unroll
            for (int s = 0; s < kTW; ++s) a2[s] = fmaf(w, h[s], a2[s]);
        }
        float d[kTW];
#pragma unroll
        for (int s = 0; s < kTW; ++s) {
            h[s] = gelu(a2[s]);
            const float z = b3 + group_sum<64>(w3 * h[s]);
            const int b = t * kTile + s0 + s;
            const float sp = softplus(z);
            const float r = b < B ? logf(sp) - target[b] : 0.0f;
            const float dz = b < B ? 2.0f * r / (float)B * sigmoid(z) / sp : 0.0f;
            if (k == 0) {
                sq += (double)r * (double)r;
                xs[wid][NF * kTS + s] = dz;
            }
            d[s] = dz * w3 * gelu_grad(a2[s]);
        }
        st_samples(&h2s[wid][k * kTS], h);
        st_samples(&d2s[wid][k * kTS], d);
        __syncthreads();
        float e[kTW] = {};
#pragma unroll 8
        for (int q = 0; q < H; ++q) {
            ld_samples(&d2s[wid][q * kTS], h);
            const float w = w2[q * kW2S + k];
#pragma unroll
            for (int s = 0; s < kTW; ++s) e[s] = fmaf(w, h[s], e[s]);
        }
#pragma unroll
        for (int s = 0; s < kTW; ++s) e[s] *= gelu_grad(a1[s]);
        st_samples(&d1s[wid][k * kTS], e);
        __syncthreads();
        // the tile's weight gradient, samples in order
        for (int w = 0; w < 4; ++w) {
            float dv[4][kTW], hv[4][kTW];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ld_samples(&d2s[w][(tk + 16 * i) * kTS], dv[i]);
                ld_samples(&h1s[w][(tl + 16 * i) * kTS], hv[i]);
            }
#pragma unroll
            for (int s = 0; s < kTW; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) g2[i][j] = fma((double)dv[i][s], (double)hv[j][s], g2[i][j]);
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                if (threadIdx.x + 256 * u >= NS) continue;
                float av[kTW], bv[kTW];
                ld_samples(ra[u] + w * sa[u], av);
                ld_samples(rb[u] + w * sb[u], bv);
#pragma unroll
                for (int s = 0; s < kTW; ++s) gs[u] += (double)av[s] * (double)bv[s];
            }
        }
    }
    double *g = gpart + (int64_t)blockIdx.x * NP;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) g[OW2 + (tk + 16 * i) * H + tl + 16 * j] = g2[i][j];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int q = threadIdx.x + 256 * u;
        if (q < NS) g[q < OW2 ? q : q + H * H] = gs[u];
    }
    const double tot = block_sum(sq, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Gradient = sum of the np partial gradients (16 runs of workgroups in order,
// then the runs in order: fixed), rounded to FP32; with lr > 0 also the Adam
// step.  16 parameters to a workgroup, so 293 workgroups share the read.
__global__ __launch_bounds__(256) void k_mlp_reduce(int np, const double *gpart, float *grad,
                                                    float *params, float *m, float *v, float lr,
                                                    float b1c, float b2c)
{
    __shared__ double acc[16][16];
    const int c = threadIdx.x & 15, q = threadIdx.x >> 4, p = blockIdx.x * 16 + c;
    double s = 0.0;
    if (p < NP)
        for (int b = np * q / 16; b < np * (q + 1) / 16; ++b) s += gpart[(int64_t)b * NP + p];
    acc[q][c] = s;
    __syncthreads();
    if (q != 0 || p >= NP) return;
    for (int r = 1; r < 16; ++r) s += acc[r][c];
    const float gi = (float)s;
    grad[p] = gi;
    if (!(lr > 0.0f)) return;
    const float mi = 0.9f * m[p] + 0.1f * gi;
    const float vi = 0.999f * v[p] + 0.001f * gi * gi;
    m[p] = mi;
    v[p] = vi;
    params[p] -= lr * (mi / b1c) / (sqrtf(vi / b2c) + 1e-8f);
}

}  // namespace

struct lsqr_trainer {
    hipStream_t st = nullptr;
    lsqr::Allocator al;
    int max_batch = 0;
    int t = 0;
    float *params = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
    double *gpart = nullptr, *part = nullptr, *sum = nullptr;
    double *hsum = nullptr;
    std::string err;
};

// Device buffers of a trainer and their sizes (bytes), in one place so that
// creation and release agree.
constexpr int kTrainerBuffers = 7;

static int tile_groups(int batch) { return std::min(kMaxTileGroups, (batch + kTile - 1) / kTile); }

static void trainer_buffers(lsqr_trainer *t, void **(&ptrs)[kTrainerBuffers],
                            size_t (&bytes)[kTrainerBuffers])
{
    const size_t G = (size_t)tile_groups(t->max_batch);
    void **p[kTrainerBuffers] = {(void **)&t->params, (void **)&t->m, (void **)&t->v,
                                 (void **)&t->grad, (void **)&t->gpart, (void **)&t->part,
                                 (void **)&t->sum};
    const size_t b[kTrainerBuffers] = {NP * 4, NP * 4, NP * 4, NP * 4, G * NP * 8, G * 8, 8};
    for (int i = 0; i < kTrainerBuffers; ++i) { ptrs[i] = p[i]; bytes[i] = b[i]; }
}

static void trainer_free(lsqr_trainer *t)
{
    void **ptrs[kTrainerBuffers];
    size_t bytes[kTrainerBuffers];
    trainer_buffers(t, ptrs, bytes);
    for (int i = 0; i < kTrainerBuffers; ++i)
        if (*ptrs[i]) t->al.put(*ptrs[i], bytes[i]);
    if (t->hsum) (void)hipHostFree(t->hsum);
    delete t;
}

// Scratch of lsqr_mlp_scale_noalloc: the Jacobi scale of up to
// LSQR_NOALLOC_MAX_COLS columns followed by the features' partial sums.  Host code
// never passes this name to a kernel or a copy: it reads the array's device
// address once per device (hipGetSymbolAddress) and uses that address.
static __device__ __align__(256) double scratch[LSQR_NOALLOC_MAX_COLS + NF * kMeanParts];

static std::mutex g_scratch_mu;
static std::vector<double *> g_scratch_ptr;      // per device; null until looked up

static lsqr_status scratch_address(lsqr_ctx *c, double **out)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    const int dev = c->device;
    if (dev < 0) return fail(c, LSQR_E_DEVICE, "invalid device of the context");
    if ((size_t)dev >= g_scratch_ptr.size()) g_scratch_ptr.resize(dev + 1, nullptr);
    if (!g_scratch_ptr[dev]) {
        double *p = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(c, LSQR_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") +
                                              hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LSQR_OK;
}

extern "C" {

lsqr_status lsqr_column_features(lsqr_ctx *c, float *feat)
{
    if (!c || !feat) return fail(c, LSQR_E_INVALID_ARG, "ctx and feat must not be NULL");
    DeviceGuard dg(c->device);
    const Problem &P = c->P;
    double *cen = ctx_alloc<double>(c, std::max<int64_t>(P.m, 1));
    if (!cen) return fail(c, LSQR_E_OOM, "device allocation failed");
    const int gr = (int)std::min<int64_t>(std::max<int64_t>((P.m * 64 + 255) / 256, 1), 65536);
    hipLaunchKernelGGL(k_row_centroid, dim3(gr), dim3(256), 0, c->st, P.m, FastDiv((uint32_t)P.nz),
                       c->rp, c->ci, c->va, cen);
    const int gc = (int)std::min<int64_t>(std::max<int64_t>((P.n * 64 + 255) / 256, 1), 65536);
    hipLaunchKernelGGL(k_col_features, dim3(gc), dim3(256), 0, c->st, (int)P.n, P.nx, P.ny, P.nz,
                       P.w, P.damp, c->cp, c->ri, c->cv, cen, feat);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->st));
    ctx_release(c, cen);
    return LSQR_OK;
}

// Inference with the Jacobi scale and the features' partial sums in
// djac [n + NF kMeanParts].
static lsqr_status mlp_scale_into(lsqr_ctx *c, const float *params, const Norm &nrm,
                                  unsigned centre, const float *feat, double *d, double *djac)
{
    const Problem &P = c->P;
    double *part = djac + P.n;
    launch_jacobi(c->st, P, c->C64, djac);
    hipLaunchKernelGGL(k_feature_sums, dim3(kMeanParts), dim3(256), 0, c->st, (int)P.n, feat, centre,
                       part);
    const int g = (int)std::min<int64_t>((P.n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_mlp_infer, dim3(std::max(g, 1)), dim3(256), 0, c->st, (int)P.n, params,
                       nrm, centre, (const double *)part, feat, (const double *)djac, d);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->st));
    return LSQR_OK;
}

static lsqr_status mlp_scale_args(lsqr_ctx *c, const float *params, const float *mean,
                                  const float *std, unsigned centre, const float *feat, double *d,
                                  Norm &nrm)
{
    if (!c || !params || !mean || !std || !feat || !d)
        return fail(c, LSQR_E_INVALID_ARG, "arguments must not be NULL");
    if (centre >> NF) return fail(c, LSQR_E_INVALID_ARG, "centre flags only features 0..5");
    for (int f = 0; f < NF; ++f) {
        if (!(std[f] > 0.0f) || !isfinite(std[f]) || !isfinite(mean[f]))
            return fail(c, LSQR_E_INVALID_ARG, "standardisation must be finite with std > 0");
        nrm.mean[f] = mean[f];
        nrm.inv_std[f] = 1.0f / std[f];
    }
    return LSQR_OK;
}

lsqr_status lsqr_mlp_scale(lsqr_ctx *c, const float *params, const float *mean, const float *std,
                           unsigned centre, const float *feat, double *d)
{
    Norm nrm;
    lsqr_status s = mlp_scale_args(c, params, mean, std, centre, feat, d, nrm);
    if (s != LSQR_OK) return s;
    DeviceGuard dg(c->device);
    double *djac = ctx_alloc<double>(c, c->P.n + NF * kMeanParts);
    if (!djac) return fail(c, LSQR_E_OOM, "device allocation failed");
    s = mlp_scale_into(c, params, nrm, centre, feat, d, djac);
    ctx_release(c, djac);
    return s;
}

lsqr_status lsqr_mlp_scale_noalloc(lsqr_ctx *c, const float *params, const float *mean,
                                   const float *std, unsigned centre, const float *feat, double *d)
{
    Norm nrm;
    lsqr_status s = mlp_scale_args(c, params, mean, std, centre, feat, d, nrm);
    if (s != LSQR_OK) return s;
    if (c->P.n > LSQR_NOALLOC_MAX_COLS)
        return fail(c, LSQR_E_INVALID_ARG,
                    "lsqr_mlp_scale_noalloc: n = " + std::to_string(c->P.n) +
                        " columns exceeds the static scratch of " +
                        std::to_string((long long)LSQR_NOALLOC_MAX_COLS) +
                        " (use lsqr_mlp_scale)");
    DeviceGuard dg(c->device);
    double *djac = nullptr;
    s = scratch_address(c, &djac);
    if (s != LSQR_OK) return s;
    // every element the kernels read is written first in the same call (the
    // Jacobi scale of all n columns, then the partial sums): nothing to clear
    return mlp_scale_into(c, params, nrm, centre, feat, d, djac);
}

static thread_local std::string t_err;

lsqr_status lsqr_trainer_create(int max_batch, const float *params, void *stream,
                                lsqr_alloc_fn alloc, lsqr_free_fn dealloc, void *alloc_user,
                                lsqr_trainer **out)
{
    if (!out || !params || max_batch < 1) {
        t_err = "invalid arguments";
        return LSQR_E_INVALID_ARG;
    }
    *out = nullptr;
    lsqr_trainer *t = new lsqr_trainer();
    t->st = (hipStream_t)stream;
    t->al.alloc = alloc;
    t->al.dealloc = dealloc;
    t->al.user = alloc_user;
    t->max_batch = max_batch;
    void **ptrs[kTrainerBuffers];
    size_t bytes[kTrainerBuffers];
    trainer_buffers(t, ptrs, bytes);
    bool ok = true;
    for (int i = 0; i < kTrainerBuffers && ok; ++i) ok = (*ptrs[i] = t->al.get(bytes[i])) != nullptr;
    ok = ok && hipHostMalloc((void **)&t->hsum, 8, hipHostMallocDefault) == hipSuccess;
    if (!ok) {
        trainer_free(t);
        t_err = "device allocation failed";
        return LSQR_E_OOM;
    }
    if (hipMemcpy(t->params, params, NP * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(t->m, 0, NP * 4) != hipSuccess || hipMemset(t->v, 0, NP * 4) != hipSuccess) {
        trainer_free(t);
        t_err = "device copy failed";
        return LSQR_E_DEVICE;
    }
    *out = t;
    return LSQR_OK;
}

// The gradient of a minibatch into t->grad; with lr > 0 the Adam step too.
static lsqr_status trainer_grad(lsqr_trainer *t, int batch, const float *x, const float *target,
                                double *loss, float lr, float b1c, float b2c)
{
    const int groups = tile_groups(batch);
    hipLaunchKernelGGL(k_mlp_grad, dim3(groups), dim3(256), 0, t->st, batch, t->params, x, target,
                       t->gpart, t->part);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NP + 15) / 16), dim3(256), 0, t->st, groups, t->gpart,
                       t->grad, t->params, t->m, t->v, lr, b1c, b2c);
    if (loss) {
        launch_sum_partials(t->st, t->part, groups, t->sum);
        if (hipMemcpyAsync(t->hsum, t->sum, 8, hipMemcpyDeviceToHost, t->st) != hipSuccess ||
            hipStreamSynchronize(t->st) != hipSuccess) {
            t->err = "device copy failed";
            return LSQR_E_DEVICE;
        }
        *loss = t->hsum[0] / (double)batch;
    }
    if (hipGetLastError() != hipSuccess) {
        t->err = "kernel launch failed";
        return LSQR_E_DEVICE;
    }
    return LSQR_OK;
}

lsqr_status lsqr_trainer_grad(lsqr_trainer *t, int batch, const float *x, const float *target,
                              float *grad, double *loss)
{
    if (!t || !x || !target || batch < 1 || batch > t->max_batch) return LSQR_E_INVALID_ARG;
    lsqr_status s = trainer_grad(t, batch, x, target, loss, 0.0f, 1.0f, 1.0f);
    if (s != LSQR_OK) return s;
    if (grad && hipMemcpyAsync(grad, t->grad, NP * 4, hipMemcpyDeviceToDevice, t->st) != hipSuccess)
        return LSQR_E_DEVICE;
    return hipStreamSynchronize(t->st) == hipSuccess ? LSQR_OK : LSQR_E_DEVICE;
}

lsqr_status lsqr_trainer_step(lsqr_trainer *t, int batch, const float *x, const float *target,
                              float lr, double *loss)
{
    if (!t || !x || !target || batch < 1 || batch > t->max_batch || !(lr > 0.0f)) return LSQR_E_INVALID_ARG;
    const int n = t->t + 1;
    const float b1c = 1.0f - powf(0.9f, (float)n), b2c = 1.0f - powf(0.999f, (float)n);
    lsqr_status s = trainer_grad(t, batch, x, target, loss, lr, b1c, b2c);
    if (s == LSQR_OK) t->t = n;
    return s;
}

lsqr_status lsqr_trainer_params(const lsqr_trainer *t, float *params, float *params_device)
{
    if (!t || (!params && !params_device)) return LSQR_E_INVALID_ARG;
    if (params && hipMemcpyAsync(params, t->params, NP * 4, hipMemcpyDeviceToHost, t->st) != hipSuccess)
        return LSQR_E_DEVICE;
    if (params_device &&
        hipMemcpyAsync(params_device, t->params, NP * 4, hipMemcpyDeviceToDevice, t->st) != hipSuccess)
        return LSQR_E_DEVICE;
    return hipStreamSynchronize(t->st) == hipSuccess ? LSQR_OK : LSQR_E_DEVICE;
}

void lsqr_trainer_destroy(lsqr_trainer *t)
{
    if (!t) return;
    if (t->st) (void)hipStreamSynchronize(t->st);
    trainer_free(t);
}

}  // extern "C"
