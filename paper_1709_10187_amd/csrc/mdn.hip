// Mixture-density network of the learned escape surrogate: forward, likelihood, backward
// and Adam on BF16 matrix cores (v_mfma_f32_32x32x16_bf16, FP32 accumulation).
//
// Network: x (16) -> 256 -> 256 -> 256 -> 128, exact (erf) GELU on the hidden layers; the
// 128 outputs parameterise a 16-component mixture over (exit face, y1, y2) (component k:
// logit o[k], face logits o[16+2k+f], mean / log-sigma of y1 at o[48+k] / o[64+k], of y2
// at o[80+k] / o[96+k], correlation 0.95 tanh(o[112+k]); log-sigmas clamped to [-6, 4]).
// The loss is the mean negative log-likelihood of the targets.
//
// The products are small (4096 rows x 170 k weights in training), so what bounds them is the
// number of launches and passes over memory, not the matrix cores:
//   mdn_rows   everything that is local to a row, one block per 32 rows: the four layers, and for
//              training the likelihood and the three backward products.  Eight waves own 32
//              output columns each; activations stay in LDS, the GELU derivatives of the three
//              hidden layers in the registers of the lanes that will need them.  Weights are
//              read from L2 in the order of the MFMA operand (refresh_bf16 lays them out), 1 KiB
//              contiguous per load.  The same kernel computes the surrogate's inputs and sampling
//              records when a cloud's window is evaluated.
//   mdn_wgrad  all four weight gradients and the bias gradients, contracted over the batch from
//              operands that mdn_rows left in MFMA order ([feature][32 rows] per row tile, so no
//              transposition and no LDS), split over the batch into FP32 partials;
//   mdn_reduce adds the partials in a fixed order (the result does not depend on timing).
// One training step of 4096 rows takes 4 launches and 53 us (268 us and 30 launches with one launch
// per product, operands staged and transposed through LDS); the 40 000 records of sixteen clouds
// 66 us on the device (10 batches of 7 launches, 750 us).  What is left: the row kernel's 128
// blocks for 4096 rows fill half of the compute units, and its time is the serial chain of seven
// products with ~50 instructions of erfc per activation.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "rddmc_internal.h"
#include "surrogate_dev.h"

namespace rddmc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t f2bf(float f)
{   // round to nearest even
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ---- parameter layout ---------------------------------------------------------------
constexpr int kIn = 16, kHid = 256, kOut = 128, kComp = 16;
constexpr int kMaxSplits = 16;     // K splits of a weight-gradient product
constexpr int64_t kW1 = 0, kB1 = kW1 + kIn * kHid, kW2 = kB1 + kHid, kB2 = kW2 + kHid * kHid, kW3 = kB2 + kHid,
                  kB3 = kW3 + kHid * kHid, kW4 = kB3 + kHid, kB4 = kW4 + kHid * kOut, kNParams = kB4 + kOut;
constexpr int64_t kLayerW[4] = {kW1, kW2, kW3, kW4};
constexpr int64_t kLayerB[4] = {kB1, kB2, kB3, kB4};
constexpr int kLayerIn[4] = {kIn, kHid, kHid, kHid};
constexpr int kLayerOut[4] = {kHid, kHid, kHid, kOut};

// Parameter buffer: f32 theta, Adam m, Adam v, grad (kNParams each), then two bf16 copies of
// every W in MFMA operand order: wt for the forward product (contraction over the inputs), w for
// the backward one (contraction over the outputs).
struct ParamView {
    float *theta, *m, *v, *grad;
    uint16_t *w, *wt;     // bf16, kNParams entries each (bias slots unused)
};

// Place of element (k, n) of a [K, N] right operand in MFMA order: 32-column tiles, 16-deep
// steps, 64 lanes (column n % 32, half (k % 16) / 8) of 8 consecutive k.
__host__ __device__ inline int64_t frag_of(int k, int n, int K)
{
    return ((((int64_t)(n >> 5) * (K >> 4) + (k >> 4)) << 6) + (n & 31) + (((k >> 3) & 1) << 5)) * 8 + (k & 7);
}

__host__ __device__ inline ParamView param_view(void *base)
{
    ParamView p;
    float *f = static_cast<float *>(base);
    p.theta = f;
    p.m = f + kNParams;
    p.v = f + 2 * kNParams;
    p.grad = f + 3 * kNParams;
    p.w = reinterpret_cast<uint16_t *>(f + 4 * kNParams);
    p.wt = p.w + kNParams;
    return p;
}
constexpr uint64_t kParamBytes = 4ull * 4 * kNParams + 2ull * 2 * kNParams;

// Work buffer for a batch of up to `cap` samples (cap a multiple of 32).  Activations and
// gradients are kept per 32-row tile as [feature][32 rows], the operand order of mdn_wgrad.
struct WorkView {
    uint16_t *act[4];              // the inputs of layer l: [tile][16 or 256][32]
    uint16_t *d[4];                // d loss / d (pre-activation of layer l): [tile][256 or 128][32]
    float *part;                   // [kMaxSplits, kNParams] partial gradients
    float *lossp;                  // [cap / 32] loss of each row tile
};

__host__ __device__ inline WorkView work_view(void *base, int64_t cap)
{
    WorkView w;
    uint8_t *p = static_cast<uint8_t *>(base);
    auto take = [&](uint64_t bytes) {
        uint8_t *q = p;
        p += (bytes + 255) & ~255ull;
        return q;
    };
    for (int l = 0; l < 4; ++l) w.act[l] = reinterpret_cast<uint16_t *>(take(2ull * cap * kLayerIn[l]));
    for (int l = 0; l < 4; ++l) w.d[l] = reinterpret_cast<uint16_t *>(take(2ull * cap * kLayerOut[l]));
    w.part = reinterpret_cast<float *>(take(4ull * kMaxSplits * kNParams));
    w.lossp = reinterpret_cast<float *>(take(4ull * (cap / 32)));
    return w;
}

__host__ inline uint64_t work_bytes_for(int64_t cap)
{
    WorkView w = work_view(nullptr, cap);
    return reinterpret_cast<uint64_t>(w.lossp) + ((4ull * (cap / 32) + 255) & ~255ull);
}

// ---- small kernels --------------------------------------------------------------------
// bf16 copies of one weight (parameter i), in both operand orders
__device__ __forceinline__ void refresh_weight(const ParamView &p, int64_t i, float theta)
{
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int64_t w0 = kLayerW[l];
        const int K = kLayerIn[l], N = kLayerOut[l];
        if (i >= w0 && i < w0 + (int64_t)K * N) {
            const int k = (int)(i - w0) / N, n = (int)(i - w0) % N;
            const uint16_t b = f2bf(theta);
            p.wt[w0 + frag_of(k, n, K)] = b;
            if (l > 0) p.w[w0 + frag_of(n, k, N)] = b;   // the inputs need no gradient
        }
    }
}

__global__ void refresh_bf16(ParamView p)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kNParams) refresh_weight(p, i, p.theta[i]);
}

// Glorot-uniform weights and zero biases from a Philox-free hash of (seed, index): the
// initial point only needs to be reproducible.
__global__ void init_params(ParamView p, uint64_t seed)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    float val = 0.0f;
    for (int l = 0; l < 4; ++l) {
        const int64_t w0 = kLayerW[l], n = (int64_t)kLayerIn[l] * kLayerOut[l];
        if (i >= w0 && i < w0 + n) {
            uint64_t z = seed * 0x9E3779B97F4A7C15ull + (uint64_t)i * 0xD1B54A32D192ED03ull + 0x632BE59BD9B4E019ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            const float u = ((float)(z >> 40) + 0.5f) * 5.9604644775390625e-8f;
            const float lim = sqrtf(6.0f / (float)(kLayerIn[l] + kLayerOut[l]));
            val = (2.0f * u - 1.0f) * lim;
        }
    }
    p.theta[i] = val;
    p.m[i] = 0.0f;
    p.v[i] = 0.0f;
    p.grad[i] = 0.0f;
}

// ---- everything local to a row -------------------------------------------------------------
constexpr int kRows = 32, kLd = kHid + 8, kLdO = kOut + 4;   // rows per block, padded LDS rows

// What a block of mdn_rows reads and writes besides the parameters.
struct RowArgs {
    const float *x;        // f32 [n, 16] inputs (kForward, kTrain)
    const float *y;        // f32 [n, 3] targets (kTrain)
    float *out;            // kForward: f32 [n, 128] raw outputs; kRecords: records of rows 0 .. n-1
    int64_t n;
    WorkView w;            // kTrain
    const uint8_t *tb, *surr;   // kRecords: tables and surrogate header
};
enum RowMode : int { kForward = 0, kTrain = 1, kRecords = 2 };

// The wave's 32 x 32 tile of H [32, K] B [K, .] for output columns 32 tile ..: H in LDS, B in MFMA
// order in global memory.  Lane l supplies row l % 32 of H and column l % 32 of B, k-slice
// [(l / 32) * 8, +8) of each 16-deep step; accumulator r holds row 8 (r / 4) + 4 (l / 32) + (r % 4),
// column l % 32.
template <int K>
__device__ __forceinline__ f32x16 product(const uint16_t *__restrict__ H, const uint16_t *__restrict__ B, int tile,
                                          int lane)
{
    constexpr int S = K / 16;
    const bf16x8 *bp = reinterpret_cast<const bf16x8 *>(B) + (int64_t)tile * S * 64 + lane;
    const uint16_t *ap = H + (lane & 31) * kLd + ((lane >> 5) << 3);
    bf16x8 b[S];
#pragma unroll
    for (int s = 0; s < S; ++s) b[s] = bp[s * 64];
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(ap + 16 * s), b[s], acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ int acc_row(int r, int lane) { return ((r >> 2) << 3) + ((lane >> 5) << 2) + (r & 3); }

// The lane's 16 values (one column) into LDS H[row][col] and, if T, the tile's [feature][32 rows]
__device__ __forceinline__ void put_rows(uint16_t *__restrict__ H, uint16_t *__restrict__ T, int col, int lane,
                                         const uint16_t *v)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) H[acc_row(r, lane) * kLd + col] = v[r];
    if (T) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<uint2 *>(T + col * 32 + 8 * q + ((lane >> 5) << 2)) =
                make_uint2(v[4 * q] | ((uint32_t)v[4 * q + 1] << 16), v[4 * q + 2] | ((uint32_t)v[4 * q + 3] << 16));
    }
}

// One hidden layer of the forward pass: H <- bf16 gelu(H W + b); `gd` receives gelu' of the
// lane's pre-activations.
template <int K, bool TRAIN>
__device__ __forceinline__ void hidden(uint16_t *__restrict__ Hin, uint16_t *__restrict__ Hout, const ParamView &p, int l,
                                       uint16_t *T, int wave, int lane, float *gd)
{
    const f32x16 acc = product<K>(Hin, p.wt + kLayerW[l], wave, lane);
    const int col = 32 * wave + (lane & 31);
    const float bias = p.theta[kLayerB[l] + col];
    uint16_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float z = acc[r] + bias;
        const float e = erfcf(-z * 0.70710678118654752f);   // gelu and its derivative share it
        v[r] = f2bf(0.5f * z * e);
        if (TRAIN) gd[r] = 0.5f * e + z * 0.39894228040143268f * __expf(-0.5f * z * z);
    }
    put_rows(Hout, T, col, lane, v);
}

// One backward product: D <- bf16 (D W^T) * gelu'.
template <int K>
__device__ __forceinline__ void backward(const uint16_t *__restrict__ Din, uint16_t *__restrict__ Dout, const ParamView &p,
                                         int l, uint16_t *T, int wave, int lane, const float *gd)
{
    const f32x16 acc = product<K>(Din, p.w + kLayerW[l], wave, lane);
    uint16_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = f2bf(acc[r] * gd[r]);
    put_rows(Dout, T, 32 * wave + (lane & 31), lane, v);
}

// The likelihood of one row and d(mean NLL)/d(o), by its 16 lanes (lane k: component k); q: the
// row's 128 outputs in LDS, lcs: 16 floats of scratch of the row, g: the row's gradient (bf16).
// Sums over components run in order in every lane, so they do not depend on the layout.
__device__ __forceinline__ float row_nll(const float *__restrict__ q, const float *__restrict__ y, bool live, float inv_n,
                                         int k, float *__restrict__ lcs, uint16_t *__restrict__ g)
{
    const int f = live ? (int)y[0] : 0;
    const float y1 = live ? y[1] : 0.0f, y2 = live ? y[2] : 0.0f;
    float amax = -INFINITY;
    for (int c = 0; c < kComp; ++c) amax = fmaxf(amax, q[c]);
    float asum = 0.0f;
    for (int c = 0; c < kComp; ++c) asum += __expf(q[c] - amax);
    const float log_asum = amax + __logf(asum);
    const float f0 = q[16 + 2 * k], f1 = q[17 + 2 * k];
    const float fm = fmaxf(f0, f1);
    const float e0 = __expf(f0 - fm), e1 = __expf(f1 - fm);
    const float lse_f = fm + __logf(e0 + e1);
    const float s1r = q[64 + k], s2r = q[96 + k];
    const float s1 = fminf(fmaxf(s1r, -6.0f), 4.0f), s2 = fminf(fmaxf(s2r, -6.0f), 4.0f);
    const float rr = tanhf(q[112 + k]);
    const float rho = 0.95f * rr;
    const float e1s = __expf(-s1), e2s = __expf(-s2);
    const float z1 = (y1 - q[48 + k]) * e1s, z2 = (y2 - q[80 + k]) * e2s;
    const float om = 1.0f - rho * rho;
    const float qq = (z1 * z1 - 2.0f * rho * z1 * z2 + z2 * z2) / om;
    const float lc = (q[k] - log_asum) + ((f ? f1 : f0) - lse_f) +
                     (-1.8378770664093453f - s1 - s2 - 0.5f * __logf(om) - 0.5f * qq);
    lcs[k] = lc;
    __syncthreads();
    float lmax = -INFINITY;
    for (int c = 0; c < kComp; ++c) lmax = fmaxf(lmax, lcs[c]);
    float lsum = 0.0f;
    for (int c = 0; c < kComp; ++c) lsum += __expf(lcs[c] - lmax);
    const float ll = lmax + __logf(lsum);
    const float w = __expf(lc - ll);
    const float pi = __expf(q[k] - log_asum);
    const float p0 = e0 / (e0 + e1), p1 = e1 / (e0 + e1);
    const float dq1 = (2.0f * z1 - 2.0f * rho * z2) / om, dq2 = (2.0f * z2 - 2.0f * rho * z1) / om;
    const float dqr = (-2.0f * z1 * z2) / om + qq * (2.0f * rho) / om;
    const float in1 = (s1r > -6.0f && s1r < 4.0f) ? 1.0f : 0.0f;
    const float in2 = (s2r > -6.0f && s2r < 4.0f) ? 1.0f : 0.0f;
    // padding rows contribute nothing
    g[k] = live ? f2bf((pi - w) * inv_n) : (uint16_t)0;
    g[16 + 2 * k] = live ? f2bf(w * (p0 - (f == 0 ? 1.0f : 0.0f)) * inv_n) : (uint16_t)0;
    g[17 + 2 * k] = live ? f2bf(w * (p1 - (f == 1 ? 1.0f : 0.0f)) * inv_n) : (uint16_t)0;
    g[48 + k] = live ? f2bf(-w * 0.5f * dq1 * e1s * inv_n) : (uint16_t)0;
    g[64 + k] = live ? f2bf(-w * (-1.0f + 0.5f * dq1 * z1) * in1 * inv_n) : (uint16_t)0;
    g[80 + k] = live ? f2bf(-w * 0.5f * dq2 * e2s * inv_n) : (uint16_t)0;
    g[96 + k] = live ? f2bf(-w * (-1.0f + 0.5f * dq2 * z2) * in2 * inv_n) : (uint16_t)0;
    g[112 + k] = live ? f2bf(-w * (rho / om - 0.5f * dqr) * 0.95f * (1.0f - rr * rr) * inv_n) : (uint16_t)0;
    return ll;
}

// The sampling record of one window state from its outputs q (LDS), by its 16 lanes.
__device__ __forceinline__ void row_record(const float *__restrict__ q, float S, float wd, int k, float *__restrict__ r)
{
    float amax = -INFINITY;
    for (int c = 0; c < kComp; ++c) amax = fmaxf(amax, q[c]);
    float sum = 0.0f, cum = 0.0f;
    for (int c = 0; c < kComp; ++c) {
        sum += __expf(q[c] - amax);
        if (c == k) cum = sum;
    }
    r[kRecCdf + k] = k == 15 ? 1.0f : cum / sum;
    r[kRecPf0 + k] = 1.0f / (1.0f + __expf(q[17 + 2 * k] - q[16 + 2 * k]));
    r[kRecMu1 + k] = q[48 + k];
    r[kRecSg1 + k] = __expf(fminf(fmaxf(q[64 + k], -6.0f), 4.0f));
    r[kRecMu2 + k] = q[80 + k];
    r[kRecSg2 + k] = __expf(fminf(fmaxf(q[96 + k], -6.0f), 4.0f));
    r[kRecRho + k] = 0.95f * tanhf(q[112 + k]);
    r[kRecS + k] = k == 0 ? S : (k == kRecW - kRecS ? wd : 0.0f);
}

template <int MODE>
__global__ __launch_bounds__(512) void mdn_rows(ParamView p, RowArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t H[2][kRows * kLd];
    __shared__ float O[kRows * kLdO];
    __shared__ float scr[kRows * kComp];     // component log-likelihoods; states' scales
    __shared__ float rowloss[kRows];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t tile = blockIdx.x, row0 = tile * kRows;
    constexpr bool TRAIN = MODE == kTrain;
    // inputs (bf16; rows past n are zero)
    if (MODE == kRecords) {
        if (t < kRows) {
            float f[kSurrIn], S = 0.0f, wd = 0.0f;
            for (int k = 0; k < kSurrIn; ++k) f[k] = 0.0f;
            if (row0 + t < a.n) surr_state_features(a.tb, a.surr, (uint64_t)(row0 + t), f, S, wd);
            for (int k = 0; k < kIn; ++k) H[0][t * kLd + k] = f2bf(f[k]);
            scr[2 * t] = S;
            scr[2 * t + 1] = wd;
        }
    } else {
        const int r = t >> 4, k = t & 15;
        const uint16_t v = row0 + r < a.n ? f2bf(a.x[(row0 + r) * kIn + k]) : (uint16_t)0;
        H[0][r * kLd + k] = v;
        if (TRAIN) a.w.act[0][(tile * kIn + k) * 32 + r] = v;
    }
    __syncthreads();
    uint16_t *T1 = TRAIN ? a.w.act[1] + tile * kHid * 32 : nullptr;
    uint16_t *T2 = TRAIN ? a.w.act[2] + tile * kHid * 32 : nullptr;
    uint16_t *T3 = TRAIN ? a.w.act[3] + tile * kHid * 32 : nullptr;
    float gd1[16], gd2[16], gd3[16];
    hidden<kIn, TRAIN>(H[0], H[1], p, 0, T1, wave, lane, gd1);
    __syncthreads();
    hidden<kHid, TRAIN>(H[1], H[0], p, 1, T2, wave, lane, gd2);
    __syncthreads();
    hidden<kHid, TRAIN>(H[0], H[1], p, 2, T3, wave, lane, gd3);
    __syncthreads();
    if (wave < kOut / 32) {
        const f32x16 acc = product<kHid>(H[1], p.wt + kLayerW[3], wave, lane);
        const int col = 32 * wave + (lane & 31);
        const float bias = p.theta[kLayerB[3] + col];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = acc_row(r, lane);
            const float v = acc[r] + bias;
            if (MODE == kForward) {
                if (row0 + row < a.n) a.out[(row0 + row) * kOut + col] = v;
            } else {
                O[row * kLdO + col] = v;
            }
        }
    }
    if (MODE == kForward) return;
    __syncthreads();
    const int r = t >> 4, k = t & 15;
    const bool live = row0 + r < a.n;
    if (MODE == kRecords) {
        if (live) row_record(O + r * kLdO, scr[2 * r], scr[2 * r + 1], k, a.out + (row0 + r) * kSurrRec);
        return;
    }
    const float ll = row_nll(O + r * kLdO, a.y + 3 * (row0 + r), live, 1.0f / (float)a.n, k, scr + r * kComp, H[0] + r * kLd);
    if (k == 0) rowloss[r] = live ? -ll / (float)a.n : 0.0f;
    __syncthreads();
    if (t == 0) {   // the tile's share of the mean NLL
        float v = 0.0f;
        for (int q = 0; q < kRows; ++q) v += rowloss[q];
        a.w.lossp[tile] = v;
    }
    {
        const int c = t >> 2, q0 = (t & 3) << 3;
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = H[0][(q0 + e) * kLd + c];
        *reinterpret_cast<uint4 *>(a.w.d[3] + (tile * kOut + c) * 32 + q0) =
            make_uint4(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16), v[4] | ((uint32_t)v[5] << 16),
                       v[6] | ((uint32_t)v[7] << 16));
    }
    backward<kOut>(H[0], H[1], p, 3, a.w.d[2] + tile * kHid * 32, wave, lane, gd3);
    __syncthreads();
    backward<kHid>(H[1], H[0], p, 2, a.w.d[1] + tile * kHid * 32, wave, lane, gd2);
    __syncthreads();
    backward<kHid>(H[0], H[1], p, 1, a.w.d[0] + tile * kHid * 32, wave, lane, gd1);
}

// ---- weight and bias gradients ------------------------------------------------------------------
// Block: one 64 x 64 tile of one layer's dW = act^T d over one range of row tiles, 32 x 32 per
// wave; the waves of the first tile row also sum d's columns (the bias gradient).  Partials go
// to part[split][parameter].
constexpr int kWgTiles[4] = {4, 16, 16, 8};      // 64 x 64 tiles of each layer (16 inputs: one row)
constexpr int kWgAll = 44;

template <int L>
__device__ __forceinline__ void wgrad_tile(const WorkView &w, int tile, int lo, int hi, float *__restrict__ P, int wave,
                                           int lane)
{
    constexpr int K = kLayerIn[L], N = kLayerOut[L];
    const int m0 = (tile / (N / 64)) * 64 + ((wave >> 1) << 5), n0 = (tile % (N / 64)) * 64 + ((wave & 1) << 5);
    if (m0 >= K) return;
    const int m = m0 + (lane & 31), n = n0 + (lane & 31), kh = (lane >> 5) << 3;
    const bool in = m < K;
    const uint16_t *A = w.act[L] + (int64_t)(in ? m : 0) * 32 + kh;
    const uint16_t *B = w.d[L] + (int64_t)n * 32 + kh;
    const bool bias = m0 == 0;
    float db = 0.0f;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll 4
    for (int q = lo; q < hi; ++q) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint4 av = *reinterpret_cast<const uint4 *>(A + (int64_t)q * K * 32 + 16 * h);
            const uint4 bv = *reinterpret_cast<const uint4 *>(B + (int64_t)q * N * 32 + 16 * h);
            if (!in) av = make_uint4(0u, 0u, 0u, 0u);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                          acc, 0, 0, 0);
            if (bias) {
                const uint32_t u[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) db += bf2f((uint16_t)u[e]) + bf2f((uint16_t)(u[e] >> 16));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = m0 + acc_row(r, lane);
        if (row < K) P[kLayerW[L] + (int64_t)row * N + n] = acc[r];
    }
    if (bias) {
        db += __shfl_xor(db, 32);
        if (lane < 32) P[kLayerB[L] + n] = db;
    }
}

__global__ __launch_bounds__(256) void mdn_wgrad(WorkView w, int tiles, int splits)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int split = blockIdx.x / kWgAll;
    int b = blockIdx.x % kWgAll;
    const int per = (tiles + splits - 1) / splits;
    const int lo = split * per, hi = min(tiles, lo + per);
    float *P = w.part + (int64_t)split * kNParams;
    if (b < kWgTiles[0]) return wgrad_tile<0>(w, b, lo, hi, P, wave, lane);
    b -= kWgTiles[0];
    if (b < kWgTiles[1]) return wgrad_tile<1>(w, b, lo, hi, P, wave, lane);
    b -= kWgTiles[1];
    if (b < kWgTiles[2]) return wgrad_tile<2>(w, b, lo, hi, P, wave, lane);
    wgrad_tile<3>(w, b - kWgTiles[2], lo, hi, P, wave, lane);
}

// grad = the partials' sum, splits in order; the loss, row tiles in order (64 strided sums, then
// in lane order).
__global__ __launch_bounds__(256) void mdn_reduce(ParamView p, WorkView w, int splits, int tiles, float *__restrict__ loss)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kNParams) {
        float v = 0.0f;
        for (int q = 0; q < splits; ++q) v += w.part[(int64_t)q * kNParams + i];
        p.grad[i] = v;
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && loss) {
        float v = 0.0f;
        for (int q = threadIdx.x; q < tiles; q += 64) v += w.lossp[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (threadIdx.x == 0) *loss = v;
    }
}

__global__ void adam_kernel(ParamView p, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    const float g = p.grad[i];
    const float m = b1 * p.m[i] + (1.0f - b1) * g;
    const float v = b2 * p.v[i] + (1.0f - b2) * g * g;
    p.m[i] = m;
    p.v[i] = v;
    const float th = p.theta[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
    p.theta[i] = th;
    refresh_weight(p, i, th);
}

}  // namespace

uint64_t mdn_param_bytes() { return kParamBytes; }
uint64_t mdn_work_bytes(int64_t cap) { return work_bytes_for(cap); }
int64_t mdn_n_params() { return kNParams; }

hipError_t mdn_init(void *d_params, uint64_t seed, hipStream_t s)
{
    ParamView p = param_view(d_params);
    init_params<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(p, seed);
    refresh_bf16<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t mdn_refresh(void *d_params, hipStream_t s)
{
    ParamView p = param_view(d_params);
    refresh_bf16<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t mdn_forward(void *d_params, const float *d_x, int n, float *d_out, hipStream_t s)
{
    if (!d_out) return hipSuccess;
    RowArgs a{};
    a.x = d_x;
    a.out = d_out;
    a.n = n;
    mdn_rows<kForward><<<(unsigned)((n + kRows - 1) / kRows), 512, 0, s>>>(param_view(d_params), a);
    return hipGetLastError();
}

hipError_t mdn_records(void *d_params, const uint8_t *d_tables, const uint8_t *d_surr, uint64_t n, float *d_rec,
                       hipStream_t s)
{
    if (n == 0) return hipSuccess;
    RowArgs a{};
    a.tb = d_tables;
    a.surr = d_surr;
    a.out = d_rec;
    a.n = (int64_t)n;
    mdn_rows<kRecords><<<(unsigned)((n + kRows - 1) / kRows), 512, 0, s>>>(param_view(d_params), a);
    return hipGetLastError();
}

hipError_t mdn_loss_grad(void *d_params, void *d_work, int64_t cap, const float *d_x, const float *d_y, int n,
                         float *d_loss, hipStream_t s)
{
    const ParamView p = param_view(d_params);
    RowArgs a{};
    a.x = d_x;
    a.y = d_y;
    a.n = n;
    a.w = work_view(d_work, cap);
    const int tiles = (n + kRows - 1) / kRows;
    // ranges of the batch for the weight gradients: at least 256 rows each
    const int splits = std::max(1, std::min(kMaxSplits, tiles * kRows / 256));
    mdn_rows<kTrain><<<(unsigned)tiles, 512, 0, s>>>(p, a);
    mdn_wgrad<<<(unsigned)(kWgAll * splits), 256, 0, s>>>(a.w, tiles, splits);
    mdn_reduce<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(p, a.w, splits, tiles, d_loss);
    return hipGetLastError();
}

hipError_t mdn_adam(void *d_params, int64_t step, float lr, hipStream_t s)
{
    ParamView p = param_view(d_params);
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    adam_kernel<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(p, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace rddmc
