// Learned measurement-noise model: features, inference and training kernels.
//
// Training minimises the Gaussian negative log-likelihood 1/2 (s + r^2 e^-s)
// of residuals r = D - Z between a frame's measured depth D and the depth Z
// of the fused surface raycast from that frame's pose, with s = log sigma^2
// predicted from the pixel's features.  Forward, backward and the Adam update
// are hand-written: the two layer-2 products of the backward pass run on the
// matrix cores like the forward product.
#include "tsdf_internal.h"
#include "mlp_device.h"
#include "mlp_features.h"
#include "tsdf_mlp.h"

namespace tsdf {

// ---------------------------------------------------------------- features

__global__ __launch_bounds__(256) void features_kernel(const float *__restrict__ depth, int W, int H, double fx,
                                                       double fy, double cx, double cy, float4 *__restrict__ feat,
                                                       uint8_t *__restrict__ valid)
{
    __shared__ FeatLds L;
    const int i0 = blockIdx.x * kFeatTile, j0 = blockIdx.y * kFeatTile;
    float f[4];
    const bool ok = tile_features(L, depth, W, H, fx, fy, cx, cy, i0, j0, threadIdx.x, f);
    const int i = i0 + threadIdx.x % kFeatTile, j = j0 + threadIdx.x / kFeatTile;
    if (i < W && j < H) {
        feat[(size_t)j * W + i] = make_float4(f[0], f[1], f[2], f[3]);
        valid[(size_t)j * W + i] = ok ? 1 : 0;
    }
}

// ---------------------------------------------------------------- forward

__global__ __launch_bounds__(256) void forward_kernel(const uint16_t *__restrict__ params,
                                                      const float4 *__restrict__ x, int64_t n, float *__restrict__ s)
{
    __shared__ MlpParamsLds P;
    __shared__ MlpInferLds Wl[4];
    mlp_stage_params(P, params, threadIdx.x, 256);
    __syncthreads();
    const int64_t k = blockIdx.x * 256ll + threadIdx.x;
    float4 xv = k < n ? x[k] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float xa[4] = {xv.x, xv.y, xv.z, xv.w};
    // the same forward pass as the integration path
    const float out = mlp_infer_wave(P, params, Wl[threadIdx.x >> 6], xa, threadIdx.x & 63);
    if (k < n) s[k] = out;
}

// ---------------------------------------------------------------- training

// Sample index of position k in the epoch's visiting order: an affine
// permutation k -> (a k + b) mod n with a coprime to n (chosen by the host).
// (a < n and k < n <= 2^31 keep a k + b inside 64 bits).  `inv` is
// floor((2^64 - 1) / n): the quotient from its high product is at most two
// short, which replaces two 64-bit divisions per sample.
__device__ __forceinline__ uint64_t mod_n(uint64_t x, uint64_t n, uint64_t inv)
{
    uint64_t r = x - __umul64hi(x, inv) * n;
    if (r >= n) r -= n;
    if (r >= n) r -= n;
    return r;
}
__device__ __forceinline__ int64_t visit(int64_t k, int64_t n, uint64_t inv, uint64_t a, uint64_t b)
{
    return (int64_t)mod_n(a * mod_n((uint64_t)k, (uint64_t)n, inv) + b, (uint64_t)n, inv);
}

constexpr int kTrainSamples = 128;   // per workgroup
constexpr int kTrainWaves = 4;       // 32 samples (one matrix tile) each
constexpr int kTS = 40;              // row stride of the bf16 tiles: 16-byte rows of 8, spread over the banks

// Per-wavefront scratch.  The bf16 activations and errors are kept in both
// orders (sample rows, unit rows), so that every matrix operand is one 16-byte
// read per lane and K step.
struct TrainWaveLds {
    union {
        struct {
            alignas(16) uint16_t h1[32][kTS];    // [sample][unit]
            alignas(16) uint16_t h1t[32][kTS];   // [unit][sample]
            union {
                struct {
                    alignas(16) uint16_t e2[32][kTS];    // bf16(dL/da2), [sample][unit]
                    alignas(16) uint16_t e2t[32][kTS];   // [unit][sample]
                };
                float t3[32][kMlpHidden + 1];    // before them: output-layer terms per (sample, unit)
            };
        };
        float dw2[kMlpHidden * kMlpHidden];      // the wavefront's dW2, once the tiles are dead
    };
    alignas(16) float g1[32][36];                // silu'(a1), [unit][sample]
    alignas(16) float x0[32][4];
    alignas(16) float ds[32];
    float red[kMlpHidden * kMlpIn + 3 * kMlpHidden + 2];   // the wavefront's other gradients and loss
};
struct TrainLds {
    MlpParamsLds P;
    alignas(16) uint16_t w2[32][kTS];    // W2 as bf16 bits, [out][in]
    alignas(16) uint16_t w2t[32][kTS];   // [in][out]
    TrainWaveLds wave[kTrainWaves];
};
static_assert(sizeof(TrainLds) <= 80 * 1024, "two workgroups per CU");

__device__ __forceinline__ i16x8_t tile_operand(const uint16_t *row)
{
    return *(const i16x8_t *)row;
}

// One workgroup = 128 samples of the batch, 32 per wavefront; writes the
// workgroup's summed gradient (1249 values) and loss into partial[blockIdx.x].
//
// A batch of 65536 gives the chip 2048 wavefronts, two per SIMD, so the kernel
// is one wavefront's chain of instruction latencies: 32 samples a wavefront
// rather than 64 halve it, the sums over samples run down the accumulator rows
// a lane holds (layer 1 took 160 butterfly sums of six exchanges each), and no
// activation is computed twice.  In the accumulator layout a lane holds unit
// o = lane % 32 of the samples 8 (q / 4) + 4 (lane / 32) + q % 4.
__global__ __launch_bounds__(64 * kTrainWaves) __attribute__((amdgpu_waves_per_eu(2))) void train_kernel(const uint16_t *__restrict__ params,
                                                                 const float4 *__restrict__ x,
                                                                 const float *__restrict__ r, int64_t n_samples,
                                                                 uint64_t n_inv, int64_t first, int64_t batch,
                                                                 uint64_t pa, uint64_t pb, float *__restrict__ partial)
{
    __shared__ TrainLds S;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    constexpr int NT = 64 * kTrainWaves;
    TrainWaveLds &W = S.wave[wv];
    // this lane's sample, loaded ahead of the parameters (lanes m and m + 32 share it)
    const int m = lane & 31, hf = lane >> 5;
    const int64_t kb = blockIdx.x * (int64_t)kTrainSamples + 32 * wv + m;   // position inside the batch
    const bool live = kb < batch;
    float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
    float rr = 0.f;
    if (live) {
        const int64_t idx = visit(first + kb, n_samples, n_inv, pa, pb);
        xv = x[idx];
        rr = r[idx];
    }
    mlp_stage_params(S.P, params, tid, NT);
#pragma unroll
    for (int q = 0; q < kMlpHidden * kMlpHidden / NT; ++q) {
        const int e = tid + q * NT, o = e >> 5, i = e & 31;
        const uint16_t w = params[MLP_W2 + e];
        S.w2[o][i] = w;
        S.w2t[i][o] = w;
    }
    __syncthreads();

    // layer 1: this lane's sample, units 16 hf .. 16 hf + 15
    const float x0[4] = {bf16_round(xv.x), bf16_round(xv.y), bf16_round(xv.z), bf16_round(xv.w)};
    if (hf == 0) *(float4 *)W.x0[m] = make_float4(x0[0], x0[1], x0[2], x0[3]);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int o = 16 * hf + q;
        float a = S.P.p[MLP_B1 + o];
#pragma unroll
        for (int i = 0; i < kMlpIn; ++i) a += S.P.p[MLP_W1 + o * kMlpIn + i] * x0[i];
        const uint16_t h = bf16_bits(silu(a));
        W.h1[m][o] = h;
        W.h1t[o][m] = h;
        W.g1[o][m] = silu_grad(a);
    }
    __syncthreads();

    // layer 2: a2[m][o] = sum_i h1[m][i] W2[o][i] + b2[o]
    const int col = lane & 31, kh = 8 * hf;
    f32x16_t c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t a2 = c;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
        a2 = mfma_bf16_k16(tile_operand(&W.h1[col][16 * kk + kh]), tile_operand(&S.w2[col][16 * kk + kh]), a2);
    const float b2 = S.P.p[MLP_B2 + col], w3 = S.P.p[MLP_W3 + col];
    float h2[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        a2[q] += b2;
        h2[q] = bf16_round(silu(a2[q]));
        W.t3[8 * (q >> 2) + 4 * hf + (q & 3)][col] = w3 * h2[q];
    }
    __syncthreads();

    // output of this lane's sample: each half sums 16 units
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += W.t3[m][16 * hf + q];
    s += __shfl_xor(s, 32);
    s += S.P.p[MLP_B3];
    const float e = __expf(-s);
    const float loss = live ? 0.5f * (s + rr * rr * e) : 0.0f;
    const float ds = live ? 0.5f * (1.0f - rr * rr * e) : 0.0f;
    if (hf == 0) W.ds[m] = ds;
    __syncthreads();

    // output layer and dL/da2
    float gW3 = 0.f, gb2 = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 d4 = *(const float4 *)&W.ds[8 * g + 4 * hf];
        const float d[4] = {d4.x, d4.y, d4.z, d4.w};
        uint16_t eb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = 4 * g + k;
            const float da2 = d[k] * w3 * silu_grad(a2[q]);
            gW3 += d[k] * h2[q];
            gb2 += da2;
            eb[k] = bf16_bits(da2);
            W.e2[8 * g + 4 * hf + k][col] = eb[k];
        }
        *(uint2 *)&W.e2t[col][8 * g + 4 * hf] =
            make_uint2((uint32_t)eb[0] | ((uint32_t)eb[1] << 16), (uint32_t)eb[2] | ((uint32_t)eb[3] << 16));
    }
    __syncthreads();

    // dW2[o][i] = sum_m e2[m][o] h1[m][i] and dh1[m][i] = sum_o e2[m][o] W2[o][i]
    f32x16_t w2c = c, dh = c;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        w2c = mfma_bf16_k16(tile_operand(&W.e2t[col][16 * kk + kh]), tile_operand(&W.h1t[col][16 * kk + kh]), w2c);
        dh = mfma_bf16_k16(tile_operand(&W.e2[col][16 * kk + kh]), tile_operand(&S.w2t[col][16 * kk + kh]), dh);
    }
    // layer 1, unit col: da1 = dh1 silu'(a1); dW1 = sum_m da1 x0^T, db1 = sum_m da1
    float gw[kMlpIn] = {0.f, 0.f, 0.f, 0.f}, gb1 = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 s4 = *(const float4 *)&W.g1[col][8 * g + 4 * hf];
        const float sg[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float da1 = dh[4 * g + k] * sg[k];
            const float4 xq = *(const float4 *)W.x0[8 * g + 4 * hf + k];
            gb1 += da1;
            gw[0] += da1 * xq.x;
            gw[1] += da1 * xq.y;
            gw[2] += da1 * xq.z;
            gw[3] += da1 * xq.w;
        }
    }
    // the two row halves of a unit, then the samples' own sums over the 32 lanes of one half
    gb1 += __shfl_xor(gb1, 32);
    gb2 += __shfl_xor(gb2, 32);
    gW3 += __shfl_xor(gW3, 32);
#pragma unroll
    for (int i = 0; i < kMlpIn; ++i) gw[i] += __shfl_xor(gw[i], 32);
    float b3s = ds, ls = loss;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
        b3s += __shfl_xor(b3s, off);
        ls += __shfl_xor(ls, off);
    }
    __syncthreads();   // every wavefront has read its tiles: their space takes dW2
#pragma unroll
    for (int q = 0; q < 16; ++q) W.dw2[(8 * (q >> 2) + 4 * hf + (q & 3)) * kMlpHidden + col] = w2c[q];
    if (hf == 0) {
#pragma unroll
        for (int i = 0; i < kMlpIn; ++i) W.red[col * kMlpIn + i] = gw[i];
        W.red[kMlpHidden * kMlpIn + col] = gb1;
        W.red[kMlpHidden * kMlpIn + kMlpHidden + col] = gb2;
        W.red[kMlpHidden * kMlpIn + 2 * kMlpHidden + col] = gW3;
        if (lane == 0) {
            W.red[kMlpHidden * kMlpIn + 3 * kMlpHidden] = b3s;
            W.red[kMlpHidden * kMlpIn + 3 * kMlpHidden + 1] = ls;
        }
    }
    __syncthreads();
    float *out = partial + (size_t)blockIdx.x * kMlpParamsPadded;
    for (int k = tid; k < kMlpHidden * kMlpIn + 3 * kMlpHidden + 2; k += NT) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < kTrainWaves; ++w) v += S.wave[w].red[k];
        int dst;
        if (k < 128) dst = MLP_W1 + k;
        else if (k < 160) dst = MLP_B1 + (k - 128);
        else if (k < 192) dst = MLP_B2 + (k - 160);
        else if (k < 224) dst = MLP_W3 + (k - 192);
        else if (k == 224) dst = MLP_B3;
        else dst = kMlpParams;   // loss, stored in the padding
        out[dst] = v;
    }
#pragma unroll
    for (int q = 0; q < kMlpHidden * kMlpHidden / NT; ++q) {
        const int k = tid + q * NT;
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < kTrainWaves; ++w) v += S.wave[w].dw2[k];
        out[MLP_W2 + k] = v;
    }
}

// grad[p] = (sum over workgroups of partial[wg][p]) / batch in double; loss
// likewise.  One workgroup per 64 parameters: its 16 wavefronts take every
// 16th partial each (consecutive lanes read consecutive parameters), then add
// up through LDS.  One lane per parameter over all partials is a chain of 512
// loads: 122 us for a batch of 65536, against 5 us.
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(64 * kReduceWaves) void reduce_kernel(const float *__restrict__ partial, int n_wg,
                                                                   int64_t batch, float *__restrict__ grad,
                                                                   float *__restrict__ loss)
{
    __shared__ double sum[kReduceWaves][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    double acc = 0.0;
    if (p <= kMlpParams) {
        const float *src = partial + p;
#pragma unroll 8
        for (int w = wv; w < n_wg; w += kReduceWaves) acc += src[(size_t)w * kMlpParamsPadded];
    }
    sum[wv][lane] = acc;
    __syncthreads();
    if (wv != 0 || p > kMlpParams) return;
    acc = 0.0;
#pragma unroll
    for (int w = 0; w < kReduceWaves; ++w) acc += sum[w][lane];
    if (p < kMlpParams) grad[p] = (float)(acc / (double)batch);
    else if (loss) loss[0] = (float)(acc / (double)batch);
}

// Adam on float32 master weights; the bf16 parameters are their rounding.
__global__ void adam_kernel(float *__restrict__ master, float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ grad, uint16_t *__restrict__ params, int step, float lr,
                            float beta1, float beta2, float eps)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kMlpParams) return;
    const float g = grad[p];
    const float mn = beta1 * m[p] + (1.0f - beta1) * g;
    const float vn = beta2 * v[p] + (1.0f - beta2) * g * g;
    m[p] = mn;
    v[p] = vn;
    const float mh = mn / (1.0f - powf(beta1, (float)step));
    const float vh = vn / (1.0f - powf(beta2, (float)step));
    const float w = master[p] - lr * mh / (sqrtf(vh) + eps);
    master[p] = w;
    params[p] = bf16_bits(w);
}

// Training samples of one frame: pixels with a measurement, valid features
// and a raycast hit; residual r = D - (camera z of the hit).  Pass 1 counts
// per workgroup, pass 2 scans the counts, pass 3 writes in pixel order.
__device__ __forceinline__ bool sample_of(const float *depth, const float4 *feat, const uint8_t *valid,
                                          const float4 *vertex, const Camera &cam, size_t k, float &res)
{
    const float D = depth[k];
    if (!(D > 0.0f) || !isfinite(D) || !valid[k]) return false;
    const float4 vt = vertex[k];
    if (!(vt.w > 0.0f)) return false;
    const double z = cam.R[2] * ((double)vt.x - cam.t[0]) + cam.R[5] * ((double)vt.y - cam.t[1]) +
                     cam.R[8] * ((double)vt.z - cam.t[2]);
    res = (float)((double)D - z);
    return true;
}

__global__ __launch_bounds__(256) void sample_count_kernel(const float *depth, const float4 *feat,
                                                           const uint8_t *valid, const float4 *vertex, Camera cam,
                                                           int64_t n, uint32_t *counts)
{
    const size_t k = blockIdx.x * 256ull + threadIdx.x;
    float res;
    const bool ok = k < (size_t)n && sample_of(depth, feat, valid, vertex, cam, k, res);
    const int c = __syncthreads_count(ok);
    if (threadIdx.x == 0) counts[blockIdx.x] = (uint32_t)c;
}

// Exclusive scan of the workgroups' counts on top of the running total, by one
// workgroup: 1024 counts a round, four per lane (a single lane takes a round
// trip per count: 62 us for the 1200 of a 640x480 frame, against 4 us).
__global__ __launch_bounds__(256) void scan_kernel(const uint32_t *__restrict__ counts, int nblocks,
                                                   uint64_t *__restrict__ base, uint64_t *__restrict__ total)
{
    __shared__ uint32_t wave_sum[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint64_t carry = total[0];
    for (int b0 = 0; b0 < nblocks; b0 += 1024) {
        const int k0 = b0 + 4 * threadIdx.x;
        uint32_t c[4], s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = k0 + q < nblocks ? counts[k0 + q] : 0u;
            s += c[q];
        }
        uint32_t inc = s;   // (at most 1024 counts of 256: 32 bits)
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)inc, off);
            if (lane >= off) inc += y;
        }
        if (lane == 63) wave_sum[wv] = inc;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wv) before += wave_sum[w];
            all += wave_sum[w];
        }
        uint64_t run = carry + before + inc - s;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (k0 + q < nblocks) base[k0 + q] = run;
            run += c[q];
        }
        carry += all;
        __syncthreads();   // the next round rewrites the wavefronts' sums
    }
    if (threadIdx.x == 0) total[0] = carry;
}

__global__ __launch_bounds__(256) void sample_write_kernel(const float *depth, const float4 *feat,
                                                           const uint8_t *valid, const float4 *vertex, Camera cam,
                                                           int64_t n, const uint64_t *base, int64_t cap,
                                                           float4 *xout, float *rout)
{
    __shared__ uint32_t wave_counts[4];
    const size_t k = blockIdx.x * 256ull + threadIdx.x;
    float res = 0.0f;
    const bool ok = k < (size_t)n && sample_of(depth, feat, valid, vertex, cam, k, res);
    const unsigned long long m = __ballot(ok);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) wave_counts[wv] = (uint32_t)__popcll(m);
    __syncthreads();
    uint64_t off = base[blockIdx.x];
    for (int w = 0; w < wv; ++w) off += wave_counts[w];
    off += (uint64_t)__popcll(m & ((1ull << lane) - 1ull));
    if (ok && (int64_t)off < cap) {
        xout[off] = feat[k];
        rout[off] = res;
    }
}

}  // namespace tsdf

using namespace tsdf;

extern "C" {

tsdf_status tsdf_mlp_features(const float *depth_dev, const tsdf_intrinsics *K, float *feat_dev, uint8_t *valid_dev,
                              hipStream_t stream)
{
    if (!depth_dev || !K || !feat_dev || !valid_dev || !(K->fx > 0) || !(K->fy > 0) || K->width <= 0 ||
        K->height <= 0)
        return TSDF_EINVAL;
    dim3 grid((K->width + kFeatTile - 1) / kFeatTile, (K->height + kFeatTile - 1) / kFeatTile);
    hipLaunchKernelGGL(features_kernel, grid, dim3(256), 0, stream, depth_dev, K->width, K->height, K->fx, K->fy,
                       K->cx, K->cy, (float4 *)feat_dev, valid_dev);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

tsdf_status tsdf_mlp_forward(const void *params_dev, const float *x_dev, int64_t n, float *s_dev, hipStream_t stream)
{
    if (!params_dev || n < 0 || (n > 0 && (!x_dev || !s_dev))) return TSDF_EINVAL;
    if (n == 0) return TSDF_OK;
    dim3 grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(forward_kernel, grid, dim3(256), 0, stream, (const uint16_t *)params_dev,
                       (const float4 *)x_dev, n, s_dev);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

uint64_t tsdf_mlp_workspace_bytes(int64_t batch)
{
    if (batch <= 0) return 0;
    return (uint64_t)((batch + kTrainSamples - 1) / kTrainSamples) * kMlpParamsPadded * sizeof(float);
}

tsdf_status tsdf_mlp_loss_grad(const void *params_dev, const float *x_dev, const float *r_dev, int64_t n_samples,
                               int64_t first, int64_t batch, uint64_t perm_a, uint64_t perm_b, void *workspace_dev,
                               float *grad_dev, float *loss_dev, hipStream_t stream)
{
    if (!params_dev || !x_dev || !r_dev || !workspace_dev || !grad_dev || n_samples <= 0 || batch <= 0 || first < 0)
        return TSDF_EINVAL;
    if (perm_a == 0 || perm_a >= (uint64_t)n_samples || perm_b >= (uint64_t)n_samples || n_samples > (1ll << 31))
        return TSDF_EINVAL;
    const int n_wg = (int)((batch + kTrainSamples - 1) / kTrainSamples);
    const uint64_t n_inv = ~0ull / (uint64_t)n_samples;
    hipLaunchKernelGGL(train_kernel, dim3(n_wg), dim3(64 * kTrainWaves), 0, stream, (const uint16_t *)params_dev,
                       (const float4 *)x_dev, r_dev, n_samples, n_inv, first, batch, perm_a, perm_b,
                       (float *)workspace_dev);
    if (hipGetLastError() != hipSuccess) return TSDF_EHIP;
    hipLaunchKernelGGL(reduce_kernel, dim3((kMlpParams + 1 + 63) / 64), dim3(64 * kReduceWaves), 0, stream,
                       (const float *)workspace_dev, n_wg, batch, grad_dev, loss_dev);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

tsdf_status tsdf_mlp_adam_step(float *master_dev, float *m_dev, float *v_dev, const float *grad_dev, void *params_dev,
                               int32_t step, float lr, float beta1, float beta2, float eps, hipStream_t stream)
{
    if (!master_dev || !m_dev || !v_dev || !grad_dev || !params_dev || step < 1 || !(lr > 0) || !(beta1 >= 0) ||
        !(beta1 < 1) || !(beta2 >= 0) || !(beta2 < 1) || !(eps > 0))
        return TSDF_EINVAL;
    hipLaunchKernelGGL(adam_kernel, dim3((kMlpParams + 255) / 256), dim3(256), 0, stream, master_dev, m_dev, v_dev,
                       grad_dev, (uint16_t *)params_dev, step, lr, beta1, beta2, eps);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

uint64_t tsdf_mlp_samples_workspace_bytes(int32_t width, int32_t height)
{
    const uint64_t nb = ((uint64_t)width * height + 255) / 256;
    return nb * 4 + nb * 8 + 8;
}

tsdf_status tsdf_mlp_collect_samples(const float *depth_dev, const float *feat_dev, const uint8_t *valid_dev,
                                     const float *vertex_dev, const tsdf_intrinsics *K, const double pose_c2w[12],
                                     void *workspace_dev, uint64_t *count_dev, int64_t cap, float *x_out_dev,
                                     float *r_out_dev, hipStream_t stream)
{
    if (!depth_dev || !feat_dev || !valid_dev || !vertex_dev || !K || !pose_c2w || !workspace_dev || !count_dev ||
        cap < 0 || (cap > 0 && (!x_out_dev || !r_out_dev)) || K->width <= 0 || K->height <= 0)
        return TSDF_EINVAL;
    Camera cam;
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) cam.R[3 * r + c] = pose_c2w[4 * r + c];
        cam.t[r] = pose_c2w[4 * r + 3];
    }
    cam.fx = K->fx;
    cam.fy = K->fy;
    cam.cx = K->cx;
    cam.cy = K->cy;
    cam.width = K->width;
    cam.height = K->height;
    const int64_t n = (int64_t)K->width * K->height;
    const int nb = (int)((n + 255) / 256);
    uint32_t *counts = (uint32_t *)workspace_dev;
    uint64_t *base = (uint64_t *)((uint8_t *)workspace_dev + (((uint64_t)nb * 4 + 7) & ~7ull));
    hipLaunchKernelGGL(sample_count_kernel, dim3(nb), dim3(256), 0, stream, depth_dev, (const float4 *)feat_dev,
                       valid_dev, (const float4 *)vertex_dev, cam, n, counts);
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(256), 0, stream, (const uint32_t *)counts, nb, base, count_dev);
    hipLaunchKernelGGL(sample_write_kernel, dim3(nb), dim3(256), 0, stream, depth_dev, (const float4 *)feat_dev,
                       valid_dev, (const float4 *)vertex_dev, cam, n, (const uint64_t *)base, cap,
                       (float4 *)x_out_dev, r_out_dev);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

}  // extern "C"
