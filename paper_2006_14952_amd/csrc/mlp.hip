// Learned acceptance / order selector: training kernels (FP32 forward, softmax
// cross-entropy, backward, Adam), BF16 MFMA inference, model upload and loading, and
// the training-data entry point (candidate export + labels).
#include <stdio.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "mlp.h"
#include "state.h"

namespace hfmm {

int run_labels(fmm_tree *t, const fmm_params *P, const double *aref_sorted, double eps, float *feats, int *labels,
               float *errs, int cap, int *dcounter, hipStream_t st);
int upward(fmm_tree *t, const fmm_params *P, hipStream_t st);

// ---------------------------------------------------------------------------
// model state (one model per process, on the device current at upload)

static std::mutex g_model_mu;
static MacModel g_hmodel;
static MacModel *g_dmodel = nullptr;
static bool g_have_model = false;
static uint64_t g_model_serial = 0;  // changes with every model set or cleared

uint64_t model_serial()
{
    std::lock_guard<std::mutex> lk(g_model_mu);
    return g_model_serial;
}

const MacModel *current_model(MacModel *host_copy)
{
    std::lock_guard<std::mutex> lk(g_model_mu);
    if (!g_have_model) return nullptr;
    if (host_copy) *host_copy = g_hmodel;
    return g_dmodel;
}

static short host_bf16(float x)
{
    uint32_t u;
    memcpy(&u, &x, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

// MFMA B-operand fragments: lane l holds W[k = 16 kc + 4 (l / 16) + r][j = 16 u + l % 16].
static void build_model(const float *w, const float *mu, const float *isd, double theta_max, int safety, MacModel &M)
{
    memset(&M, 0, sizeof(M));
    for (int u = 0; u < 4; ++u)
        for (int l = 0; l < 64; ++l)
            for (int r = 0; r < 4; ++r) {
                int k = 4 * (l / 16) + r, j = 16 * u + l % 16;
                M.w.w1[u][l][r] = host_bf16(w[kOffW1 + k * kHid + j]);
            }
    // 16x16x32 steps: K slot r of lane l in step kc multiplies the hidden unit that the
    // previous layer's output fragments leave there, 16 (2 kc + r / 4) + 4 (l / 16) + r % 4
    for (int kc = 0; kc < 2; ++kc)
        for (int u = 0; u < 4; ++u)
            for (int l = 0; l < 64; ++l)
                for (int r = 0; r < 8; ++r) {
                    int k = 16 * (2 * kc + r / 4) + 4 * (l / 16) + r % 4, j = 16 * u + l % 16;
                    M.w.w2[kc][u][l][r] = host_bf16(w[kOffW2 + k * kHid + j]);
                }
    for (int kc = 0; kc < 2; ++kc)
        for (int l = 0; l < 64; ++l)
            for (int r = 0; r < 8; ++r) {
                int k = 16 * (2 * kc + r / 4) + 4 * (l / 16) + r % 4, j = l % 16;
                M.w.w3[kc][l][r] = j < kCls ? host_bf16(w[kOffW3 + k * kCls + j]) : 0;
            }
    for (int j = 0; j < kHid; ++j) {
        M.w.b1[j] = w[kOffB1 + j];
        M.w.b2[j] = w[kOffB2 + j];
    }
    for (int j = 0; j < 16; ++j) M.w.b3[j] = j < kCls ? w[kOffB3 + j] : 0.0f;
    for (int k = 0; k < kFeat; ++k) {
        M.w.mu[k] = mu[k];
        M.w.isd[k] = isd[k];
    }
    M.theta_max = theta_max;
    M.safety = safety;
}

// ---------------------------------------------------------------------------
// training kernels (FP32)

typedef float f4 __attribute__((ext_vector_type(4)));

// Forward pass, FP32 matrix cores (16x16x4), a wave per 16 samples.  The product is taken
// transposed (weights as the A operand): lane l holds sample l % 16, and the output register r
// of unit block u, unit 16 u + 4 (l / 16) + r, is the B operand of one K step of the next
// layer, whose weights are loaded in that order.  Activations and weights stay in registers
// (a wave loads the weights once and walks the samples); bound by the matrix cores, 96
// products of 1024 multiply-adds per 16 samples.  400,000 samples: a thread per sample with its
// activations in scratch memory 151 us (30 TFLOP/s), this form 46 us (98 TFLOP/s of 157).
__global__ __launch_bounds__(256) void k_mlp_fwd(const float *__restrict__ w, const float *__restrict__ mu,
                                                 const float *__restrict__ isd, const float *__restrict__ X, int B,
                                                 float *__restrict__ Z)
{
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    float w1[4][4], w2[4][4][4], w3[4][4];  // [unit block][K step]
    f4 b1[4], b2[4], b3, mul, sub;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w1[u][q] = w[kOffW1 + (4 * g + q) * kHid + 16 * u + n];
            w3[u][q] = n < kCls ? w[kOffW3 + (16 * u + 4 * g + q) * kCls + n] : 0.0f;
            b1[u][q] = w[kOffB1 + 16 * u + 4 * g + q];
            b2[u][q] = w[kOffB2 + 16 * u + 4 * g + q];
#pragma unroll
            for (int v = 0; v < 4; ++v) w2[u][v][q] = w[kOffW2 + (16 * v + 4 * g + q) * kHid + 16 * u + n];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        b3[q] = 4 * g + q < kCls ? w[kOffB3 + 4 * g + q] : 0.0f;
        sub[q] = mu[4 * g + q];
        mul[q] = isd[4 * g + q];
    }
    const int nwave = gridDim.x * (blockDim.x / 64), tiles = (B + 15) / 16;
    for (int t = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6); t < tiles; t += nwave) {
        const int s = 16 * t + n;
        f4 x = {0, 0, 0, 0};
        if (s < B)
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = (X[(size_t)s * kFeat + 4 * g + q] - sub[q]) * mul[q];
        f4 h1[4], h2[4], z = b3;
#pragma unroll
        for (int u = 0; u < 4; ++u) h1[u] = b1[u];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) h1[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[u][q], x[q], h1[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            h2[u] = b2[u];
#pragma unroll
            for (int q = 0; q < 4; ++q) h1[u][q] = fmaxf(h1[u][q], 0.0f);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    h2[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[u][v][q], h1[v][q], h2[u], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                z = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[v][q], fmaxf(h2[v][q], 0.0f), z, 0, 0, 0);
        if (s < B && g < 2)
#pragma unroll
            for (int q = 0; q < 4; ++q) Z[(size_t)s * kCls + 4 * g + q] = z[q];
    }
}

// Loss and gradient of the class-weighted softmax cross-entropy (mean over the batch by the
// weights' sum) in one pass: a workgroup takes tiles of 32 samples through the forward pass,
// the loss and the backward pass in LDS, and keeps its share of every parameter's gradient in
// registers (4x4 of the 64x64 weights per thread) until its last tile; part[blk] receives it,
// summed by k_mlp_gsum in a fixed order.  Each sample's sums run over the inputs in order.
// wsum_dev != nullptr: the weight sum is read from device memory (k_class_wsum), a label
// outside [0, kCls) has weight 0 and a zero weight sum gives zero loss and gradient.
// Bound by latency and LDS reads (276 Mflop at 8192 samples).  One thread per parameter
// summing over the whole batch took 2.1 ms of a 2.5 ms step at 8192 samples; this form 26 us and the
// sum 5 us of 0.10 ms (the rest is the host reading the labels for the weights' sum).
constexpr int kTrainTile = 32, kTrainBlocks = 256;  // 256 tiles of 32: one per CU at 8192 samples
constexpr int kW2Row = kHid + 4;                    // row stride in LDS: 16-byte reads of rows, fewer conflicts

__global__ __launch_bounds__(256) void k_mlp_train(const float *__restrict__ w, const float *__restrict__ mu,
                                                   const float *__restrict__ isd, const float *__restrict__ X,
                                                   const int *__restrict__ y, const float *__restrict__ cw, int B,
                                                   float wsum, const float *__restrict__ wsum_dev,
                                                   float *__restrict__ part, float *__restrict__ loss)
{
    __shared__ __align__(16) float w1[kFeat * kHid], w2[kHid * kW2Row], w3[kHid * kCls], bias[2 * kHid + kCls];
    __shared__ __align__(16) float xn[kTrainTile][kFeat], h1[kTrainTile][kHid], h2[kTrainTile][kHid],
        d1[kTrainTile][kHid], d2[kTrainTile][kHid], zs[kTrainTile][kCls], dz[kTrainTile][kCls];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16, s0 = 2 * ty, u0 = 4 * tx;
    for (int k = tid; k < kFeat * kHid; k += 256) w1[k] = w[kOffW1 + k];
    for (int k = tid; k < kHid * kHid; k += 256) w2[k / kHid * kW2Row + k % kHid] = w[kOffW2 + k];
    for (int k = tid; k < kHid * kCls; k += 256) w3[k] = w[kOffW3 + k];
    if (tid < kHid) bias[tid] = w[kOffB1 + tid];
    else if (tid < 2 * kHid) bias[tid] = w[kOffB2 + tid - kHid];
    else if (tid < 2 * kHid + kCls) bias[tid] = w[kOffB3 + tid - 2 * kHid];
    float g1[4] = {0, 0, 0, 0}, g2[4][4] = {}, g3[2] = {0, 0}, gb = 0.0f, total = 0.0f;
    const int tiles = (B + kTrainTile - 1) / kTrainTile;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        __syncthreads();
        for (int k = tid; k < kTrainTile * kFeat; k += 256) {
            const int s = t * kTrainTile + k / kFeat, f = k % kFeat;
            (&xn[0][0])[k] = s < B ? (X[(size_t)s * kFeat + f] - mu[f]) * isd[f] : 0.0f;
        }
        __syncthreads();
        // 2 samples x 4 units per thread
        auto layer = [&](const float *in, int nin, const float *wt, int row, const float *b, float (*out)[kHid])
            __attribute__((always_inline)) {
            float a0[4], a1[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) a0[q] = a1[q] = b[u0 + q];
#pragma unroll 8
            for (int k = 0; k < nin; ++k) {
                const float4 v = *reinterpret_cast<const float4 *>(wt + k * row + u0);
                const float p0 = in[s0 * nin + k], p1 = in[(s0 + 1) * nin + k];
                a0[0] = fmaf(p0, v.x, a0[0]); a0[1] = fmaf(p0, v.y, a0[1]);
                a0[2] = fmaf(p0, v.z, a0[2]); a0[3] = fmaf(p0, v.w, a0[3]);
                a1[0] = fmaf(p1, v.x, a1[0]); a1[1] = fmaf(p1, v.y, a1[1]);
                a1[2] = fmaf(p1, v.z, a1[2]); a1[3] = fmaf(p1, v.w, a1[3]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                out[s0][u0 + q] = fmaxf(a0[q], 0.0f);
                out[s0 + 1][u0 + q] = fmaxf(a1[q], 0.0f);
            }
        };
        layer(&xn[0][0], kFeat, w1, kHid, bias, h1);
        __syncthreads();
        layer(&h1[0][0], kHid, w2, kW2Row, bias + kHid, h2);
        __syncthreads();
        {  // one logit per thread
            const int s = tid / kCls, c = tid % kCls;
            float v = bias[2 * kHid + c];
#pragma unroll 8
            for (int k = 0; k < kHid; ++k) v = fmaf(h2[s][k], w3[k * kCls + c], v);
            zs[s][c] = v;
        }
        __syncthreads();
        if (tid < kTrainTile) {
            const int s = t * kTrainTile + tid;
            float z[kCls], m = -3.0e38f, se = 0.0f, wc = 0.0f;
            for (int k = 0; k < kCls; ++k) {
                z[k] = zs[tid][k];
                m = fmaxf(m, z[k]);
            }
            for (int k = 0; k < kCls; ++k) se += expf(z[k] - m);
            int c = s < B ? y[s] : 0;
            if (s >= B) {
                wc = 0.0f;
            } else if (wsum_dev) {
                const float ws = *wsum_dev;
                const bool ok = c >= 0 && c < kCls && ws > 0.0f;
                wc = ok ? cw[c] / ws : 0.0f;
                c = ok ? c : 0;
            } else {
                wc = cw[c] / wsum;
            }
            if (s < B) total += wc * (logf(se) + m - zs[tid][c]);
            for (int k = 0; k < kCls; ++k)
                dz[tid][k] = s < B ? wc * (expf(z[k] - m) / se - (k == c ? 1.0f : 0.0f)) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v = 0.0f;
#pragma unroll
                for (int c = 0; c < kCls; ++c) v = fmaf(dz[s0 + r][c], w3[(u0 + q) * kCls + c], v);
                d2[s0 + r][u0 + q] = h2[s0 + r][u0 + q] > 0.0f ? v : 0.0f;
            }
        __syncthreads();
        {
            float a[2][4] = {};
#pragma unroll 4
            for (int j = 0; j < kHid; j += 4) {
                const float4 p0 = *reinterpret_cast<const float4 *>(&d2[s0][j]),
                             p1 = *reinterpret_cast<const float4 *>(&d2[s0 + 1][j]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 v = *reinterpret_cast<const float4 *>(w2 + (u0 + q) * kW2Row + j);
                    a[0][q] = fmaf(p0.w, v.w, fmaf(p0.z, v.z, fmaf(p0.y, v.y, fmaf(p0.x, v.x, a[0][q]))));
                    a[1][q] = fmaf(p1.w, v.w, fmaf(p1.z, v.z, fmaf(p1.y, v.y, fmaf(p1.x, v.x, a[1][q]))));
                }
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) d1[s0 + r][u0 + q] = h1[s0 + r][u0 + q] > 0.0f ? a[r][q] : 0.0f;
        }
        __syncthreads();
        // gradients: rows 4 ty .. 4 ty + 3 of W2, row ty of W1, columns u0 .. u0 + 3; two of W3
        const int i3 = tid / 4, c3 = 2 * (tid % 4);
#pragma unroll 4
        for (int s = 0; s < kTrainTile; ++s) {
            const float4 v = *reinterpret_cast<const float4 *>(&d2[s][u0]), p = *reinterpret_cast<const float4 *>(&h1[s][4 * ty]),
                         e = *reinterpret_cast<const float4 *>(&d1[s][u0]);
            const float pv[4] = {p.x, p.y, p.z, p.w}, xi = xn[s][ty], hi = h2[s][i3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                g2[q][0] = fmaf(pv[q], v.x, g2[q][0]);
                g2[q][1] = fmaf(pv[q], v.y, g2[q][1]);
                g2[q][2] = fmaf(pv[q], v.z, g2[q][2]);
                g2[q][3] = fmaf(pv[q], v.w, g2[q][3]);
            }
            g1[0] = fmaf(xi, e.x, g1[0]);
            g1[1] = fmaf(xi, e.y, g1[1]);
            g1[2] = fmaf(xi, e.z, g1[2]);
            g1[3] = fmaf(xi, e.w, g1[3]);
            g3[0] = fmaf(hi, dz[s][c3], g3[0]);
            g3[1] = fmaf(hi, dz[s][c3 + 1], g3[1]);
            if (tid < kHid) gb += d1[s][tid];
            else if (tid < 2 * kHid) gb += d2[s][tid - kHid];
            else if (tid < 2 * kHid + kCls) gb += dz[s][tid - 2 * kHid];
        }
    }
    float *o = part + (size_t)blockIdx.x * kNParam;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        o[kOffW1 + ty * kHid + u0 + q] = g1[q];
#pragma unroll
        for (int r = 0; r < 4; ++r) o[kOffW2 + (4 * ty + r) * kHid + u0 + q] = g2[r][q];
    }
    o[kOffW3 + (tid / 4) * kCls + 2 * (tid % 4)] = g3[0];
    o[kOffW3 + (tid / 4) * kCls + 2 * (tid % 4) + 1] = g3[1];
    if (tid < kHid) o[kOffB1 + tid] = gb;
    else if (tid < 2 * kHid) o[kOffB2 + tid - kHid] = gb;
    else if (tid < 2 * kHid + kCls) o[kOffB3 + tid - 2 * kHid] = gb;
    if (tid < 64) {
        for (int k = 32; k > 0; k >>= 1) total += __shfl_xor(total, k, 64);
        if (tid == 0) atomicAdd(loss, total);
    }
}

// Sum of the workgroups' gradients, 64 parameters per workgroup: each of its four waves takes
// a quarter of the rows, in order.
__global__ __launch_bounds__(256) void k_mlp_gsum(const float *__restrict__ part, int nb, float *__restrict__ g)
{
    __shared__ float q[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    const int r0 = (int)((int64_t)nb * w / 4), r1 = (int)((int64_t)nb * (w + 1) / 4);
    float v = 0.0f;
    if (p < kNParam) {
#pragma unroll 8
        for (int r = r0; r < r1; ++r) v += part[(size_t)r * kNParam + p];
    }
    q[w][lane] = v;
    __syncthreads();
    if (w == 0 && p < kNParam) g[p] = (q[0][lane] + q[1][lane]) + (q[2][lane] + q[3][lane]);
}

static int train_blocks(int B)
{
    const int t = (B + kTrainTile - 1) / kTrainTile;
    return t < kTrainBlocks ? t : kTrainBlocks;
}

// Sum of the class weights of the batch's labels (labels outside [0, kCls) count 0),
// added into *wsum (which the caller cleared).
__global__ void k_class_wsum(const int *__restrict__ y, const float *__restrict__ cw, int B, float *__restrict__ wsum)
{
    float v = 0.0f;
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < B; s += gridDim.x * blockDim.x) {
        const int c = y[s];
        v += (c >= 0 && c < kCls) ? cw[c] : 0.0f;
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(wsum, v);
}

// Sets n floats to zero (a kernel, not a memset: also valid inside a recorded graph).
__global__ void k_fill_zero(float *__restrict__ p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       int n, float lr, float b1, float b2, float eps, float wd, float c1, float c2)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    float gp = g[p] + wd * w[p];
    float mp = b1 * m[p] + (1.0f - b1) * gp;
    float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    w[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

// inference with the loaded model: 64 samples per wave, BF16 MFMA (as in the traversal)
__global__ __launch_bounds__(64) void k_mlp_infer(const MacModel *__restrict__ M, const float *__restrict__ X, int B,
                                                  float *__restrict__ Z)
{
    __shared__ __align__(16) short act[64 * kActRow];
    int s = blockIdx.x * 64 + threadIdx.x;
    float f[kFeat], lg[kCls];
    for (int k = 0; k < kFeat; ++k) f[k] = s < B ? X[(size_t)s * kFeat + k] : 0.0f;
    mlp_logits_wave(M->w, f, act, lg);
    if (s < B)
        for (int k = 0; k < kCls; ++k) Z[(size_t)s * kCls + k] = lg[k];
}

static std::mutex g_train_mu;
static DevBuf g_part;  // the workgroups' gradients of fmm_mlp_grad

// Scratch of fmm_mlp_grad_noalloc: a fixed device array (one copy per GPU, held until the
// process ends) for the workgroups' gradients, plus the class-weight sum.  Host code never
// passes the array's name to a kernel or copy: it uses the device address hipGetSymbolAddress
// returns for the device that is current, taken once per device.
constexpr int kNoAllocMaxB = 8192;
constexpr size_t kNoAllocFloats = (size_t)kTrainBlocks * kNParam + 64;
static __device__ __align__(256) float scratch[kNoAllocFloats];
constexpr int kMaxDevices = 64;
static float *g_scratch_dev[kMaxDevices];
static std::mutex g_scratch_mu;

static int scratch_address(float **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return set_error(FMM_ERR_HIP, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return set_error(FMM_ERR_ARG, "device %d beyond the %d supported", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
            return set_error(FMM_ERR_HIP, "hipGetSymbolAddress of the training scratch");
        g_scratch_dev[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_dev[dev];
    return 0;
}

}  // namespace hfmm

using namespace hfmm;

extern "C" {

int fmm_set_mac_model(const float *params, const float *mu, const float *isd, double theta_max, int safety)
{
    if (!params || !mu || !isd) {
        std::lock_guard<std::mutex> lk(g_model_mu);
        g_have_model = false;
        ++g_model_serial;
        return 0;
    }
    if (!(theta_max > 0) || !(theta_max < 0.75)) return set_error(FMM_ERR_ARG, "theta_max must be in (0, 0.75)");
    if (safety < 0 || safety > 6) return set_error(FMM_ERR_ARG, "safety must be in [0, 6]");
    MacModel M;
    build_model(params, mu, isd, theta_max, safety, M);
    std::lock_guard<std::mutex> lk(g_model_mu);
    if (!g_dmodel && hipMalloc(&g_dmodel, sizeof(MacModel)) != hipSuccess) {
        g_dmodel = nullptr;
        return set_error(FMM_ERR_NOMEM, "model allocation");
    }
    if (hipMemcpy(g_dmodel, &M, sizeof(M), hipMemcpyHostToDevice) != hipSuccess)
        return set_error(FMM_ERR_HIP, "model upload");
    g_hmodel = M;
    g_have_model = true;
    ++g_model_serial;
    return 0;
}

// File layout (little endian): "HFMMMAC1", int32 version (1), nfeat (16), hidden (64),
// nclass (8); double theta_max, eps_label; int32 safety, reserved; float mu[16], isd[16],
// params[5768] (FP32 master), adam_m[5768], adam_v[5768]; int64 step; int32 len; JSON.
int fmm_load_mac_model(const char *path)
{
    if (!path) return fmm_set_mac_model(nullptr, nullptr, nullptr, 0.0, 0);
    FILE *f = fopen(path, "rb");
    if (!f) return set_error(FMM_ERR_ARG, "cannot open model file %s", path);
    char magic[8];
    int hdr[4];
    double th[2];
    int sf[2];
    std::vector<float> mu(kFeat), isd(kFeat), w(kNParam);
    bool ok = fread(magic, 1, 8, f) == 8 && memcmp(magic, "HFMMMAC1", 8) == 0 && fread(hdr, 4, 4, f) == 4 &&
              hdr[0] == 1 && hdr[1] == kFeat && hdr[2] == kHid && hdr[3] == kCls && fread(th, 8, 2, f) == 2 &&
              fread(sf, 4, 2, f) == 2 && fread(mu.data(), 4, kFeat, f) == (size_t)kFeat &&
              fread(isd.data(), 4, kFeat, f) == (size_t)kFeat && fread(w.data(), 4, kNParam, f) == (size_t)kNParam;
    fclose(f);
    if (!ok) return set_error(FMM_ERR_ARG, "%s is not a selector model file of this version", path);
    return fmm_set_mac_model(w.data(), mu.data(), isd.data(), th[0], sf[0]);
}

int fmm_mlp_forward(const float *params, const float *mu, const float *isd, const float *X, int B, float *logits,
                    void *stream)
{
    if (B < 0 || (B > 0 && (!params || !mu || !isd || !X || !logits))) return set_error(FMM_ERR_ARG, "bad arguments");
    if (B == 0) return 0;
    const int nb = (B + 63) / 64;  // a wave per 16 samples, four waves per workgroup
    k_mlp_fwd<<<nb < 512 ? nb : 512, 256, 0, (hipStream_t)stream>>>(params, mu, isd, X, B, logits);
    return hip_check(hipGetLastError(), "mlp forward");
}

int fmm_mlp_infer(const float *X, int B, float *logits, void *stream)
{
    if (B < 0 || (B > 0 && (!X || !logits))) return set_error(FMM_ERR_ARG, "bad arguments");
    const MacModel *M = current_model(nullptr);
    if (!M) return set_error(FMM_ERR_STATE, "no selector model loaded");
    if (B == 0) return 0;
    k_mlp_infer<<<(B + 63) / 64, 64, 0, (hipStream_t)stream>>>(M, X, B, logits);
    return hip_check(hipGetLastError(), "mlp infer");
}

int fmm_mlp_grad(const float *params, const float *mu, const float *isd, const float *X, const int *y,
                 const float *class_w, int B, float *grad, float *loss, void *stream)
{
    if (B <= 0 || !params || !mu || !isd || !X || !y || !class_w || !grad || !loss)
        return set_error(FMM_ERR_ARG, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    std::lock_guard<std::mutex> lk(g_train_mu);
    const size_t b = (size_t)B;
    const int nb = train_blocks(B);
    int rc = grow(g_part, (size_t)nb * kNParam * 4);
    if (rc) return rc;
    std::vector<float> cw(kCls);
    if (hipMemcpy(cw.data(), class_w, kCls * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return set_error(FMM_ERR_HIP, "class weights");
    std::vector<int> hy(B);
    if (hipMemcpy(hy.data(), y, b * 4, hipMemcpyDeviceToHost) != hipSuccess) return set_error(FMM_ERR_HIP, "labels");
    float wsum = 0.0f;
    for (int s = 0; s < B; ++s) wsum += cw[hy[s]];
    if (!(wsum > 0)) return set_error(FMM_ERR_ARG, "class weights sum to zero");
    if (int rc = hip_check(hipMemsetAsync(loss, 0, 4, st), "mlp loss")) return rc;
    k_mlp_train<<<nb, 256, 0, st>>>(params, mu, isd, X, y, class_w, B, wsum, nullptr, ptr<float>(g_part), loss);
    k_mlp_gsum<<<(kNParam + 63) / 64, 256, 0, st>>>(ptr<float>(g_part), nb, grad);
    rc = hip_check(hipGetLastError(), "mlp grad");
    if (!rc) rc = hip_check(hipStreamSynchronize(st), "mlp grad");  // scratch is shared between calls
    return rc;
}

int fmm_mlp_grad_noalloc(const float *params, const float *mu, const float *isd, const float *X, const int *y,
                         const float *class_w, int B, float *grad, float *loss, void *stream)
{
    if (B <= 0 || !params || !mu || !isd || !X || !y || !class_w || !grad || !loss)
        return set_error(FMM_ERR_ARG, "bad arguments");
    if (B > kNoAllocMaxB)
        return set_error(FMM_ERR_ARG, "batch of %d exceeds the %d samples of the fixed scratch", B, kNoAllocMaxB);
    float *sc = nullptr;
    if (int rc = scratch_address(&sc)) return rc;
    hipStream_t st = (hipStream_t)stream;
    float *wsum = sc + (size_t)kTrainBlocks * kNParam;  // past the gradients
    const int nb = train_blocks(B);
    k_fill_zero<<<1, 64, 0, st>>>(wsum, 1);
    k_fill_zero<<<1, 64, 0, st>>>(loss, 1);
    k_class_wsum<<<nb < 64 ? nb : 64, 128, 0, st>>>(y, class_w, B, wsum);
    k_mlp_train<<<nb, 256, 0, st>>>(params, mu, isd, X, y, class_w, B, 0.0f, wsum, sc, loss);
    k_mlp_gsum<<<(kNParam + 63) / 64, 256, 0, st>>>(sc, nb, grad);
    return hip_check(hipGetLastError(), "mlp grad (fixed scratch)");
}

int fmm_mlp_adam(float *params, const float *grad, float *m, float *v, int64_t step, float lr, float beta1, float beta2,
                 float eps, float weight_decay, void *stream)
{
    if (!params || !grad || !m || !v || step < 1) return set_error(FMM_ERR_ARG, "bad arguments");
    float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    k_adam<<<(kNParam + 255) / 256, 256, 0, (hipStream_t)stream>>>(params, grad, m, v, kNParam, lr, beta1, beta2, eps,
                                                                   weight_decay, c1, c2);
    return hip_check(hipGetLastError(), "adam");
}

}  // extern "C"
