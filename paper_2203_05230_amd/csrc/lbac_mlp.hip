// Training of the learned closure's network on the GPU: a 25 -> 64 -> 64 -> 2
// multilayer perceptron with tanh-GELU, mean-squared-error loss and Adam.
//
// FP32 throughout, on the FP32 matrix cores (16x16x4 MFMA, FP32 products and
// sums), every reduction in a fixed order so a training run is reproducible:
//   mlp_block_kernel   four wavefronts per 16 samples: the forward pass
//                      (Z1 = W1 X + b1, H1 = gelu(Z1), Z2 = W2 H1 + b2,
//                      H2 = gelu(Z2), out = W3 H2 + b3), and for training the
//                      backward pass (d3 = 2 (out - y) / B,
//                      d2 = (W3^T d3) * gelu'(Z2), d1 = (W2^T d2) * gelu'(Z1))
//                      and the block's share of the gradient
//                      (dW1 = d1 X^T, dW2 = d2 H1^T, dW3 = d3 H2^T, db = row
//                      sums of d) and of the loss, written to per-block rows
//   mlp_reduce_kernel  the gradient as the sum of the blocks' rows in a
//                      fixed order, then (training) the Adam update (Kingma
//                      & Ba, Algorithm 1); the loss as the sum of the blocks'
//                      shares in a fixed order
// MFMA operands: lane l of a 16x16x4 product supplies A[l % 16][k] and
// B[k][l % 16] with k the lane group l / 16 of the K-step, and receives
// D[4 (l / 16) + i][l % 16], i = 0..3.  The forward products keep features on
// the M side and samples on N, so the accumulator of a layer holds, in lane
// (g, n), features 16 mt + 4 g + i of sample n (mt: the wavefront), which is
// the next layer's B operand for the K-steps (mt, i), read back from LDS; the
// weight products take the 16 samples as K from LDS.
// Parameter layout: W1[64][25], b1[64], W2[64][64], b2[64], W3[2][64], b3[2].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "lbac.h"

namespace {

constexpr int kIn = 25, kH = 64, kOut = 2;
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH,
              ob3 = oW3 + kOut * kH, kNParam = ob3 + kOut;
static_assert(kNParam == LBAC_MLP_NPARAM, "parameter count");
constexpr float kGeluK = 0.7978845608028654f;  // sqrt(2/pi)
constexpr int kNS = 16;                        // samples a workgroup takes at a time
constexpr int kKin = 28;                       // inputs padded to whole K-steps of 4

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// gelu(x) and its derivative from one tanh
struct Gelu {
    float v, d;
};
__device__ __forceinline__ Gelu gelu(float x) {
    const float t = tanhf(kGeluK * (x + 0.044715f * x * x * x));
    return {0.5f * x * (1.0f + t),
            0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * kGeluK * (1.0f + 3.0f * 0.044715f * x * x)};
}

__device__ __forceinline__ f32x4_t mfma(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// A layer of the 16 samples, samples x features.  Rows of 68 floats: the 16
// samples' quadruples of one feature group, which a lane group reads as a
// K-step operand, cover all 64 banks once.
constexpr int kRow = kH + 4;
struct MlpLds {
    float x[kNS][32];  // inputs of the samples (25..31 zero)
    float h1[kNS][kRow], h2[kNS][kRow], d1[kNS][kRow], d2[kNS][kRow];
    float w3[kOut][kH];
};

// One workgroup of four wavefronts per 16 samples at a time, wavefront mt on
// the 16 features 16 mt .. 16 mt + 15 of each layer: lane (g, r) holds
// features 16 mt + 4 g + i of sample r, hands them to the other wavefronts
// through LDS, and keeps its share of the weights, in both directions, in
// registers over the samples the workgroup takes (b = blockIdx, then every
// gridDim-th 16).  Every product and sum runs in the order in which one
// wavefront per 16 samples ran it.
//
// Bound by the latency of a chain (weights, two layers of dependent matrix
// products and tanh, and back): a batch of 4096 is one workgroup per compute
// unit.  One wavefront per 16 samples, weights staged through LDS: training
// (forward) 40 (18) us at a batch of 4096, 130 (67) at 40000; this form 11
// (5.5) and 50 (18).
//
// grad_rows: per 16 samples kNParam floats; loss_rows: per 16 samples one
// double; out (forward only, may be null): batch x 2.  With TRAIN == false
// only the forward pass runs.
//
// kBlkPerCu: workgroups resident per compute unit.  Training takes 208
// registers, so two; at four it spills (batch 4096 16.7 us, 40000 59).
constexpr int kBlkThreads = 256;
template <bool TRAIN>
constexpr int kBlkPerCu = TRAIN ? 2 : 4;
template <bool TRAIN>
__global__ __launch_bounds__(kBlkThreads, kBlkPerCu<TRAIN>) void mlp_block_kernel(
    const float* __restrict__ w, const float* __restrict__ x, const float* __restrict__ y, int64_t batch, float inv_b,
    float* __restrict__ out, float* __restrict__ grad_rows, double* __restrict__ loss_rows) {
    __shared__ MlpLds L;
    const int t = threadIdx.x, l = t % 64, r = l % 16, g = l / 16;
    const int mt = __builtin_amdgcn_readfirstlane(t / 64);
    const int f0 = 16 * mt + 4 * g;  // the lane's first feature
    const int64_t nb = (batch + kNS - 1) / kNS;
    auto quad = [&](int off) { return *reinterpret_cast<const f32x4_t*>(w + off); };

    // the wavefront's weights (layer 3's, which every wavefront takes whole, in
    // LDS): rows 16 mt + r of W1 and W2 (forward), columns 16 mt + r of W2
    // (backward)
    float w1[kKin / 4], w2t[4][4];
    f32x4_t w2[4];
#pragma unroll
    for (int ks = 0; ks < kKin / 4; ++ks) {
        const int k = 4 * ks + g;
        w1[ks] = k < kIn ? w[oW1 + (16 * mt + r) * kIn + k] : 0.f;
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) w2[kt] = quad(oW2 + (16 * mt + r) * kH + 16 * kt + 4 * g);
    if constexpr (TRAIN) {
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) w2t[kt][i] = w[oW2 + (16 * kt + 4 * g + i) * kH + 16 * mt + r];
    }
    const f32x4_t b1 = quad(ob1 + f0), b2 = quad(ob2 + f0);
    const float b3[kOut] = {w[ob3], w[ob3 + 1]};
    if (t < kOut * kH) L.w3[t / kH][t % kH] = w[oW3 + t];

    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t s0 = b * kNS;
        for (int i = t; i < kNS * 32; i += kBlkThreads) {
            const int n = i / 32, k = i % 32;
            L.x[n][k] = (k < kIn && s0 + n < batch) ? x[(s0 + n) * kIn + k] : 0.f;
        }
        __syncthreads();

        // ---- forward
        f32x4_t acc = b1;
#pragma unroll
        for (int ks = 0; ks < kKin / 4; ++ks) acc = mfma(w1[ks], L.x[r][4 * ks + g], acc);
        f32x4_t h, gd1, gd2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Gelu a = gelu(acc[i]);
            h[i] = a.v;
            gd1[i] = a.d;
        }
        *reinterpret_cast<f32x4_t*>(&L.h1[r][f0]) = h;
        __syncthreads();
        acc = b2;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(&L.h1[r][16 * kt + 4 * g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = mfma(w2[kt][i], v[i], acc);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Gelu a = gelu(acc[i]);
            h[i] = a.v;
            gd2[i] = a.d;
        }
        *reinterpret_cast<f32x4_t*>(&L.h2[r][f0]) = h;
        __syncthreads();
        // layer 3 on the vector units, on every wavefront: the lane group's 16
        // features, then the four lane groups of a sample summed pairwise (the
        // same order on every lane)
        f32x4_t h2[4];
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) h2[kt] = *reinterpret_cast<const f32x4_t*>(&L.h2[r][16 * kt + 4 * g]);
        float o[kOut];
#pragma unroll
        for (int c = 0; c < kOut; ++c) {
            float p = 0.f;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const f32x4_t w3 = *reinterpret_cast<const f32x4_t*>(&L.w3[c][16 * kt + 4 * g]);
#pragma unroll
                for (int i = 0; i < 4; ++i) p = __builtin_fmaf(w3[i], h2[kt][i], p);
            }
            p += __shfl_xor(p, 16, 64);
            p += __shfl_xor(p, 32, 64);
            o[c] = b3[c] + p;
        }
        const int64_t s = s0 + r;
        const bool real = s < batch;
        if constexpr (!TRAIN) {
            if (out && mt == 0 && g == 0 && real) {
                out[s * kOut] = o[0];
                out[s * kOut + 1] = o[1];
            }
            // (the next samples' inputs and h1 are read by no wavefront that is
            // still here: all have passed the barrier after h2)
            continue;
        }

        // ---- loss and backward
        const float e0 = real ? o[0] - y[s * kOut] : 0.f;
        const float e1 = real ? o[1] - y[s * kOut + 1] : 0.f;
        const float d30 = 2.0f * e0 * inv_b, d31 = 2.0f * e1 * inv_b;
        {
            const f32x4_t wa = *reinterpret_cast<const f32x4_t*>(&L.w3[0][f0]);
            const f32x4_t wb = *reinterpret_cast<const f32x4_t*>(&L.w3[1][f0]);
            f32x4_t d;
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = (wa[i] * d30 + wb[i] * d31) * gd2[i];
            *reinterpret_cast<f32x4_t*>(&L.d2[r][f0]) = d;
        }
        __syncthreads();
        // d1 = (W2^T d2) * gelu'(z1)
        acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(&L.d2[r][16 * kt + 4 * g]);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = mfma(w2t[kt][i], v[i], acc);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = acc[i] * gd1[i];
        *reinterpret_cast<f32x4_t*>(&L.d1[r][f0]) = acc;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // (read back below by other lanes of this wavefront)
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---- the gradient rows of these samples: K = the 16 samples
        float* G = grad_rows + b * kNParam;
        // dW2 [64 x 64] = d2 H1^T, this wavefront's 16 rows
        float a2[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a2[ks] = L.d2[4 * ks + g][16 * mt + r];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = mfma(a2[ks], L.h1[4 * ks + g][16 * nt + r], acc);
#pragma unroll
            for (int i = 0; i < 4; ++i) G[oW2 + (f0 + i) * kH + 16 * nt + r] = acc[i];
        }
        // dW1 [64 x 25] = d1 X^T (N-tiles of 16 inputs); d1 of this
        // wavefront's features, which it wrote itself
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a2[ks] = L.d1[4 * ks + g][16 * mt + r];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = mfma(a2[ks], L.x[4 * ks + g][16 * nt + r], acc);
            const int k = 16 * nt + r;
            if (k < kIn)
#pragma unroll
                for (int i = 0; i < 4; ++i) G[oW1 + (f0 + i) * kIn + k] = acc[i];
        }
        __syncthreads();  // d1 of every feature
        // dW3 [2 x 64] = d3 H2^T (wavefronts 0, 1) and the bias rows
        // (wavefronts 2, 3): sums over samples in order; d3 of sample n in lane n
        if (mt < 2) {
            const float d3 = mt == 0 ? d30 : d31;
            float a = 0.f, bs = 0.f;
#pragma unroll
            for (int n = 0; n < kNS; ++n) {
                const float dn = __shfl(d3, n, 64);
                a = __builtin_fmaf(dn, L.h2[n][l], a);
                bs += dn;
            }
            G[oW3 + mt * kH + l] = a;
            if (l == 0) G[ob3 + mt] = bs;
        } else {
            float bs = 0.f;
            const float(*d)[kRow] = mt == 2 ? L.d1 : L.d2;
#pragma unroll
            for (int n = 0; n < kNS; ++n) bs += d[n][l];
            G[(mt == 2 ? ob1 : ob2) + l] = bs;
        }
        // the samples' loss share: squared errors in sample order
        if (mt == 3) {
            const double se = (double)e0 * e0 + (double)e1 * e1;
            double a = 0.0;
#pragma unroll
            for (int n = 0; n < kNS; ++n) a += __shfl(se, n, 64);
            if (l == 0) loss_rows[b] = a;
        }
        __syncthreads();  // every value of these samples has been read
    }
}

// The gradient as the sum of the blocks' rows, in a fixed order: row b belongs
// to sum b mod 16, each taken in ascending order by a thread of its own (16
// loads each at a batch of 4096); sum 4 u + q is the u-th of quarter q, the
// four of a quarter are added pairwise and the four quarters are added
// pairwise again.  A workgroup takes 32 parameters, whole 128-byte lines: 187
// of them and one for the loss.  (64 parameters and four sums per thread, 94
// workgroups: 11.2 us at a batch of 4096; this form 4.4.)
// With adam != 0 the Adam update of the weights follows.  The last block sums
// the loss shares (thread t the rows t mod 256, then a pairwise tree) into
// *loss (divided by the batch size).
constexpr int kRedParams = 32, kRedSums = 16;
constexpr int kRedBlocks = (kNParam + kRedParams - 1) / kRedParams + 1;
__global__ __launch_bounds__(kRedParams* kRedSums) void mlp_reduce_kernel(
    const float* __restrict__ grad_rows, const double* __restrict__ loss_rows, int nblk, int64_t batch,
    float* __restrict__ grad, double* __restrict__ loss, int adam, float* __restrict__ w, float* __restrict__ m,
    float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    __shared__ float part[kRedSums][kRedParams];
    const int t = threadIdx.x;
    if (blockIdx.x == kRedBlocks - 1) {
        __shared__ double lsum[256];
        if (t < 256) {
            double a = 0.0;
            for (int b = t; b < nblk; b += 256) a += loss_rows[b];
            lsum[t] = a;
        }
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (t < h) lsum[t] += lsum[t + h];
            __syncthreads();
        }
        if (t == 0) loss[0] = lsum[0] / (double)batch;
        return;
    }
    const int sum = t / kRedParams, pl = t % kRedParams;
    const int p = blockIdx.x * kRedParams + pl;
    float acc = 0.f;
    if (p < kNParam) {
        // eight rows in flight
        int b = sum;
        const float* row = grad_rows + (int64_t)b * kNParam + p;
        constexpr int64_t kStep = (int64_t)kRedSums * kNParam;
        for (; b + 7 * kRedSums < nblk; b += 8 * kRedSums, row += 8 * kStep) {
            float in[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) in[u] = row[u * kStep];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += in[u];
        }
        for (; b < nblk; b += kRedSums, row += kStep) acc += row[0];
    }
    part[sum][pl] = acc;
    __syncthreads();
    if (sum != 0 || p >= kNParam) return;
    float quarter[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) quarter[q] = (part[q][pl] + part[4 + q][pl]) + (part[8 + q][pl] + part[12 + q][pl]);
    const float gp = (quarter[0] + quarter[1]) + (quarter[2] + quarter[3]);
    grad[p] = gp;
    if (!adam) return;
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    w[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

}  // namespace

struct lbac_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    float *w = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
    float* grad_rows = nullptr;   // per block of 16 samples: its share of the gradient
    double* loss_rows = nullptr;  // per block: its share of the loss
    double* loss = nullptr;
    double* host_loss = nullptr;
    int64_t cap = 0;
    int64_t t = 0;
    std::string err;
};

namespace {

int mfail(lbac_mlp* h, int code, const std::string& msg) {
    if (h) h->err = msg;
    return code;
}

#define MHIP(h, call)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (call);                                                                         \
        if (e_ != hipSuccess) return mfail(h, LBAC_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int64_t blocks_of(int64_t batch) { return (batch + kNS - 1) / kNS; }
// Workgroups of the block kernel: what a device of 256 compute units keeps
// resident, each taking several 16 samples beyond that.
template <bool TRAIN>
unsigned grid_of(int64_t batch) {
    return (unsigned)std::min<int64_t>(blocks_of(batch), 256 * kBlkPerCu<TRAIN>);
}

int ensure(lbac_mlp* h, int64_t batch) {
    const int64_t nb = blocks_of(batch);
    if (nb <= h->cap) return LBAC_OK;
    (void)hipFree(h->grad_rows);
    (void)hipFree(h->loss_rows);
    h->grad_rows = nullptr;
    h->loss_rows = nullptr;
    h->cap = 0;
    MHIP(h, hipMalloc(&h->grad_rows, sizeof(float) * kNParam * nb));
    MHIP(h, hipMalloc(&h->loss_rows, sizeof(double) * nb));
    h->cap = nb;
    return LBAC_OK;
}

// Gradient of the loss into h->g and the loss into h->loss; with lr > 0 also
// the Adam update of the weights.
int gradient_step(lbac_mlp* h, const float* x, const float* y, int64_t batch, float lr) {
    if (batch > ((int64_t)1 << 31) * kNS) return mfail(h, LBAC_EINVAL, "batch too large");
    int rc = ensure(h, batch);
    if (rc != LBAC_OK) return rc;
    const int nb = (int)blocks_of(batch);
    hipLaunchKernelGGL(mlp_block_kernel<true>, dim3(grid_of<true>(batch)), dim3(kBlkThreads), 0, h->stream, h->w, x, y, batch,
                       1.0f / (float)batch, (float*)nullptr, h->grad_rows, h->loss_rows);
    float c1 = 1.f, c2 = 1.f;
    if (lr > 0.f) {
        h->t += 1;
        c1 = (float)(1.0 - std::pow(0.9, (double)h->t));
        c2 = (float)(1.0 - std::pow(0.999, (double)h->t));
    }
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3(kRedBlocks), dim3(kRedParams * kRedSums), 0, h->stream,
                       h->grad_rows,
                       h->loss_rows, nb, batch, h->g, h->loss, lr > 0.f ? 1 : 0, h->w, h->m, h->v, lr, 0.9f, 0.999f,
                       1e-8f, c1, c2);
    MHIP(h, hipGetLastError());
    return LBAC_OK;
}

}  // namespace

extern "C" {

int lbac_mlp_create(const float* init, void* stream, lbac_mlp** out) {
    if (!out || !init) return LBAC_EINVAL;
    *out = nullptr;
    for (int i = 0; i < kNParam; ++i)
        if (!std::isfinite(init[i])) return LBAC_EINVAL;
    lbac_mlp* h = new (std::nothrow) lbac_mlp();
    if (!h) return LBAC_ENOMEM;
    auto bail = [&](int code) {
        lbac_mlp_free(h);
        return code;
    };
    if (hipGetDevice(&h->device) != hipSuccess) return bail(LBAC_EDEVICE);
    if (stream) {
        h->stream = (hipStream_t)stream;
    } else {
        if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess) return bail(LBAC_EDEVICE);
        h->own_stream = true;
    }
    const size_t pb = sizeof(float) * kNParam;
    if (hipMalloc(&h->w, pb) != hipSuccess || hipMalloc(&h->g, pb) != hipSuccess ||
        hipMalloc(&h->m, pb) != hipSuccess || hipMalloc(&h->v, pb) != hipSuccess ||
        hipMalloc(&h->loss, sizeof(double)) != hipSuccess ||
        hipHostMalloc((void**)&h->host_loss, sizeof(double), hipHostMallocDefault) != hipSuccess)
        return bail(LBAC_ENOMEM);
    std::vector<float> zero(kNParam, 0.f);
    if (hipMemcpyAsync(h->w, init, pb, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemcpyAsync(h->m, zero.data(), pb, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemcpyAsync(h->v, zero.data(), pb, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipStreamSynchronize(h->stream) != hipSuccess)
        return bail(LBAC_EDEVICE);
    *out = h;
    return LBAC_OK;
}

int lbac_mlp_free(lbac_mlp* h) {
    if (!h) return LBAC_OK;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    (void)hipFree(h->w);
    (void)hipFree(h->g);
    (void)hipFree(h->m);
    (void)hipFree(h->v);
    (void)hipFree(h->grad_rows);
    (void)hipFree(h->loss_rows);
    (void)hipFree(h->loss);
    if (h->host_loss) (void)hipHostFree(h->host_loss);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
    return LBAC_OK;
}

int lbac_mlp_get_weights(lbac_mlp* h, float* out) {
    if (!h || !out) return LBAC_EINVAL;
    MHIP(h, hipMemcpyAsync(out, h->w, sizeof(float) * kNParam, hipMemcpyDeviceToHost, h->stream));
    MHIP(h, hipStreamSynchronize(h->stream));
    return LBAC_OK;
}

int lbac_mlp_set_weights(lbac_mlp* h, const float* in) {
    if (!h || !in) return LBAC_EINVAL;
    MHIP(h, hipMemcpyAsync(h->w, in, sizeof(float) * kNParam, hipMemcpyHostToDevice, h->stream));
    MHIP(h, hipStreamSynchronize(h->stream));
    return LBAC_OK;
}

int lbac_mlp_forward(lbac_mlp* h, const float* x_dev, int64_t batch, float* out_dev) {
    if (!h || !x_dev || !out_dev || batch < 1) return LBAC_EINVAL;
    if (batch > ((int64_t)1 << 31) * kNS) return mfail(h, LBAC_EINVAL, "batch too large");
    hipLaunchKernelGGL(mlp_block_kernel<false>, dim3(grid_of<false>(batch)), dim3(kBlkThreads), 0, h->stream, h->w, x_dev,
                       (const float*)nullptr, batch, 1.0f / (float)batch, out_dev, (float*)nullptr, (double*)nullptr);
    MHIP(h, hipGetLastError());
    return LBAC_OK;
}

int lbac_mlp_loss_grad(lbac_mlp* h, const float* x_dev, const float* y_dev, int64_t batch, double* loss,
                       float* grad) {
    if (!h || !x_dev || !y_dev || batch < 1) return LBAC_EINVAL;
    int rc = gradient_step(h, x_dev, y_dev, batch, 0.f);
    if (rc != LBAC_OK) return rc;
    if (grad) MHIP(h, hipMemcpyAsync(grad, h->g, sizeof(float) * kNParam, hipMemcpyDeviceToHost, h->stream));
    MHIP(h, hipMemcpyAsync(h->host_loss, h->loss, sizeof(double), hipMemcpyDeviceToHost, h->stream));
    MHIP(h, hipStreamSynchronize(h->stream));
    if (loss) *loss = *h->host_loss;
    return LBAC_OK;
}

int lbac_mlp_train_step(lbac_mlp* h, const float* x_dev, const float* y_dev, int64_t batch, float lr, double* loss) {
    if (!h || !x_dev || !y_dev || batch < 1 || !(lr > 0.f)) return LBAC_EINVAL;
    int rc = gradient_step(h, x_dev, y_dev, batch, lr);
    if (rc != LBAC_OK) return rc;
    if (loss) {
        MHIP(h, hipMemcpyAsync(h->host_loss, h->loss, sizeof(double), hipMemcpyDeviceToHost, h->stream));
        MHIP(h, hipStreamSynchronize(h->stream));
        *loss = *h->host_loss;
    }
    return LBAC_OK;
}

const char* lbac_mlp_last_error(lbac_mlp* h) { return h ? h->err.c_str() : "no network"; }

}  // extern "C"
