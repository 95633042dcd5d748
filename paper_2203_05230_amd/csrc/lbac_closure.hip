// Training data for the learned closure, computed on the GPU from a fine
// field (for example lbac_phi_device of a run r times finer):
//   phi_c  = mean of each r x r block of phi_f                      (restriction)
//   target = mean_block(r S_f n_f) - S_c(phi_c) n_c(phi_c)          (flux the fine field
//            carries, per coarse lattice unit, minus the flux the coarse scheme computes)
// with S n the sharpening flux of Eq. (6), (7), (13) (isotropic gradient of
// psi, regulariser delta), and one sample per coarse node of the interface
// band theta < clip(phi_c) < 1 - theta: the 5x5 neighbourhood of phi_c
// (dy = -2..2 outer, dx = -2..2 inner, periodic) and the target, optionally
// with its 7 images under the symmetries of the square (neighbourhood
// permuted, target vector transformed).  Samples are written in row-major
// node order, so the output is deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <string>

#include "lbac.h"

namespace {

__device__ __forceinline__ int wrapi(int a, int n) {
    int r = a % n;
    return r < 0 ? r + n : r;
}

__device__ __forceinline__ double clip(double p) { return p < 0.0 ? 0.0 : (p > 1.0 ? 1.0 : p); }

__device__ __forceinline__ double psi_of(double p, double eps, double delta) {
    const double pc = clip(p);
    return eps * log((pc + delta) / (1.0 - pc + delta));
}

// S n at a node: p its phi, ps(dx, dy) the psi of the node dx, dy away (FP64,
// correctly rounded functions)
template <typename Psi>
__device__ __forceinline__ void flux_of(double p, Psi ps, double eps, double delta, double& fx, double& fy) {
    const double gx = (ps(1, 0) - ps(-1, 0)) / 3.0 + ((ps(1, 1) - ps(-1, 1)) + (ps(1, -1) - ps(-1, -1))) / 12.0;
    const double gy = (ps(0, 1) - ps(0, -1)) / 3.0 + ((ps(1, 1) + ps(-1, 1)) - (ps(1, -1) + ps(-1, -1))) / 12.0;
    const double inv = 1.0 / (sqrt(gx * gx + gy * gy) + delta);
    const double pc = clip(p);
    const double S = (pc + delta) * (1.0 - pc + delta) / (eps * (1.0 + 2.0 * delta) * (1.0 + 2.0 * delta));
    fx = S * gx * inv;
    fy = S * gy * inv;
}

// S n at node (i, j) of a periodic double field
__device__ void flux_at(const double* phi, int nx, int ny, int i, int j, double eps, double delta, double& fx,
                        double& fy) {
    double ps[3][3];
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx)
            ps[dy + 1][dx + 1] = psi_of(phi[(int64_t)wrapi(j + dy, ny) * nx + wrapi(i + dx, nx)], eps, delta);
    flux_of(phi[(int64_t)j * nx + i], [&](int dx, int dy) { return ps[dy + 1][dx + 1]; }, eps, delta, fx, fy);
}

// Coarse phi and block mean of r S_f n_f for r <= kTileR: a workgroup per tile of
// whole coarse nodes, at most kTileW fine columns and max(r, kTileH) fine rows.
// psi of every fine node (and of one around the tile) is formed once and
// shared through LDS, the flux of every fine node by a thread of its own, and
// a thread per coarse node sums its r x r values in the order of
// restrict_kernel below.  Bound by the logarithms (1.3 per fine node, where
// restrict_kernel takes 9, one coarse node's after another): a 512^2 field at
// r = 4 takes 46 us there, 8 here.
constexpr int kTileW = 32, kTileH = 8, kTileR = 16, kTileT = 256;
__global__ __launch_bounds__(kTileT) void restrict_tile_kernel(const double* __restrict__ phif, int nxf, int nyf, int r,
                                                               double eps_f, double delta, double* __restrict__ phic,
                                                               double* __restrict__ tx, double* __restrict__ ty) {
    constexpr int W = kTileW + 2, HM = kTileR;
    __shared__ double p[(HM + 2) * W], ps[(HM + 2) * W];  // with one node around the tile
    __shared__ double fx[HM * kTileW], fy[HM * kTileW];
    const int nxc = nxf / r, nyc = nyf / r;
    const int cx = kTileW / r, cy = max(1, kTileH / r);  // coarse nodes of a tile
    const int i0 = blockIdx.x * cx, j0 = blockIdx.y * cy;
    const int nc = min(cx, nxc - i0), mc = min(cy, nyc - j0);
    const int w = nc * r, h = mc * r;  // fine nodes of this tile
    const int t = threadIdx.x;
    for (int k = t; k < (w + 2) * (h + 2); k += kTileT) {
        const int y = k / (w + 2), x = k % (w + 2);
        const double v = phif[(int64_t)wrapi(j0 * r + y - 1, nyf) * nxf + wrapi(i0 * r + x - 1, nxf)];
        p[y * W + x] = v;
        ps[y * W + x] = psi_of(v, eps_f, delta);
    }
    __syncthreads();
    for (int k = t; k < w * h; k += kTileT) {
        const int y = k / w, x = k % w, o = (y + 1) * W + x + 1;
        flux_of(p[o], [&](int dx, int dy) { return ps[o + dy * W + dx]; }, eps_f, delta, fx[y * kTileW + x],
                fy[y * kTileW + x]);
    }
    __syncthreads();
    for (int k = t; k < nc * mc; k += kTileT) {
        const int y = k / nc, x = k % nc;
        double sp = 0.0, sx = 0.0, sy = 0.0;
        for (int b = 0; b < r; ++b)
            for (int a = 0; a < r; ++a) {
                const int fj = y * r + b, fi = x * r + a;
                sp += p[(fj + 1) * W + fi + 1];
                sx += fx[fj * kTileW + fi];
                sy += fy[fj * kTileW + fi];
            }
        const double inv = 1.0 / (double)(r * r);
        const int64_t o = (int64_t)(j0 + y) * nxc + i0 + x;
        phic[o] = sp * inv;
        tx[o] = r * sx * inv;
        ty[o] = r * sy * inv;
    }
}

// The same for any r, a thread per coarse node (a tile of larger r does not fit LDS).
__global__ void restrict_kernel(const double* __restrict__ phif, int nxf, int nyf, int r, double eps_f, double delta,
                                double* __restrict__ phic, double* __restrict__ tx, double* __restrict__ ty) {
    const int nxc = nxf / r, nyc = nyf / r;
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (i >= nxc || j >= nyc) return;
    double sp = 0.0, sx = 0.0, sy = 0.0;
    for (int b = 0; b < r; ++b)
        for (int a = 0; a < r; ++a) {
            const int fi = i * r + a, fj = j * r + b;
            sp += phif[(int64_t)fj * nxf + fi];
            double fx, fy;
            flux_at(phif, nxf, nyf, fi, fj, eps_f, delta, fx, fy);
            sx += fx;
            sy += fy;
        }
    const double inv = 1.0 / (double)(r * r);
    phic[(int64_t)j * nxc + i] = sp * inv;
    tx[(int64_t)j * nxc + i] = r * sx * inv;
    ty[(int64_t)j * nxc + i] = r * sy * inv;
}

__device__ __forceinline__ bool in_band(double p, float theta) {
    const double pc = p < 0.0 ? 0.0 : (p > 1.0 ? 1.0 : p);
    return pc > (double)theta && pc < 1.0 - (double)theta;
}

// per coarse row: number of band nodes
__global__ void count_kernel(const double* __restrict__ phic, int nxc, float theta, int* __restrict__ rows) {
    __shared__ int sh[256];
    const int j = blockIdx.x;
    int c = 0;
    for (int i = threadIdx.x; i < nxc; i += blockDim.x) c += in_band(phic[(int64_t)j * nxc + i], theta) ? 1 : 0;
    sh[threadIdx.x] = c;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) rows[j] = sh[0];
}

// Exclusive prefix sum of the row counts, one workgroup: each thread takes a
// run of rows, and the runs' sums are scanned in LDS.  (One thread's loop took
// 15 us at 128 rows; 3 like this.)
constexpr int kScanT = 1024;
__global__ __launch_bounds__(kScanT) void scan_kernel(int* __restrict__ rows, int nyc, long long* __restrict__ total) {
    __shared__ long long sum[kScanT];
    const int t = threadIdx.x, n = (nyc + kScanT - 1) / kScanT;
    const int first = min(t * n, nyc), last = min(first + n, nyc);
    long long s = 0;
    for (int j = first; j < last; ++j) s += rows[j];
    sum[t] = s;
    __syncthreads();
    for (int h = 1; h < kScanT; h *= 2) {
        const long long v = t >= h ? sum[t - h] : 0;
        __syncthreads();
        sum[t] += v;
        __syncthreads();
    }
    long long at = sum[t] - s;
    for (int j = first; j < last; ++j) {
        const int c = rows[j];
        rows[j] = (int)at;
        at += c;
    }
    if (t == kScanT - 1) total[0] = sum[t];
}

// the 8 symmetries of the square as integer matrices (a b; c d) acting on (dx, dy)
__constant__ int kD4[8][4] = {{1, 0, 0, 1},  {0, -1, 1, 0}, {-1, 0, 0, -1}, {0, 1, -1, 0},
                              {-1, 0, 0, 1}, {1, 0, 0, -1}, {0, 1, 1, 0},   {0, -1, -1, 0}};

// A workgroup per coarse row: the row's band nodes (the first kEmitNodes of
// them) listed in order by ballots; then, kEmitChunk nodes at a time, their
// neighbourhoods and psi read and their targets formed in LDS, and the
// samples' values written by consecutive threads.  Bound by that chain, with
// a few dozen nodes in a row.  (The list by one thread's loop, a target per
// image and a sample per thread before: 26 us for a 128^2 coarse field with
// all images, 9 like this.)
constexpr int kEmitT = 512, kEmitNodes = 1024, kEmitChunk = 128;
__global__ __launch_bounds__(kEmitT) void emit_kernel(const double* __restrict__ phic, const double* __restrict__ tfx,
                                                      const double* __restrict__ tfy, int nxc, int nyc, double eps_c,
                                                      double delta, float theta, const int* __restrict__ rows,
                                                      int copies, float* __restrict__ X, float* __restrict__ Y,
                                                      long long base, long long capacity) {
    constexpr int kWaves = kEmitT / 64;
    __shared__ int order[kEmitNodes];
    __shared__ float st[kEmitChunk][25];
    __shared__ double ps[kEmitChunk][9], tgt[kEmitChunk][2];
    __shared__ int wcount[2][kWaves];
    const int j = blockIdx.x, t = threadIdx.x, wv = t / 64;
    int nband = 0;
    for (int i0 = 0, par = 0; i0 < nxc && nband < kEmitNodes; i0 += kEmitT, par ^= 1) {
        const int i = i0 + t;
        const bool in = i < nxc && in_band(phic[(int64_t)j * nxc + i], theta);
        const unsigned long long m = __ballot(in);
        if (t % 64 == 0) wcount[par][wv] = __popcll(m);
        __syncthreads();
        int at = nband, all = nband;
        for (int k = 0; k < kWaves; ++k) {
            at += k < wv ? wcount[par][k] : 0;
            all += wcount[par][k];
        }
        at += __popcll(m & ((1ull << (t % 64)) - 1));
        if (in && at < kEmitNodes) order[at] = i;
        nband = min(all, kEmitNodes);
    }
    for (int n0 = 0; n0 < nband; n0 += kEmitChunk) {
        const int nn = min(kEmitChunk, nband - n0);
        __syncthreads();  // (the list; the previous chunk's values have been written)
        auto value = [&](int n, int dx, int dy) {
            return phic[(int64_t)wrapi(j + dy, nyc) * nxc + wrapi(order[n0 + n] + dx, nxc)];
        };
        for (int e = t; e < nn * 25; e += kEmitT) st[e / 25][e % 25] = (float)value(e / 25, e % 5 - 2, e % 25 / 5 - 2);
        for (int e = t; e < nn * 9; e += kEmitT)
            ps[e / 9][e % 9] = psi_of(value(e / 9, e % 3 - 1, e % 9 / 3 - 1), eps_c, delta);
        __syncthreads();
        for (int n = t; n < nn; n += kEmitT) {
            double cfx, cfy;
            flux_of(value(n, 0, 0), [&](int dx, int dy) { return ps[n][3 * dy + dx + 4]; }, eps_c, delta, cfx, cfy);
            const int64_t o = (int64_t)j * nxc + order[n0 + n];
            tgt[n][0] = tfx[o] - cfx;
            tgt[n][1] = tfy[o] - cfy;
        }
        __syncthreads();
        const long long first = base + ((long long)rows[j] + n0) * copies;
        const int ns = nn * copies;
        // image: X'(p) = X(T^-1 p) with T^-1 = T^T; target' = T target
        for (int e = t; e < ns * 25; e += kEmitT) {
            const int s = e / 25, k = e % 25, g = s % copies;
            const int dy = k / 5 - 2, dx = k % 5 - 2;
            const int sx = kD4[g][0] * dx + kD4[g][2] * dy, sy = kD4[g][1] * dx + kD4[g][3] * dy;
            if (first + s < capacity) X[first * 25 + e] = st[s / copies][(sy + 2) * 5 + sx + 2];
        }
        for (int s = t; s < ns; s += kEmitT) {
            const int g = s % copies;
            const double tx = tgt[s / copies][0], ty = tgt[s / copies][1];
            if (first + s >= capacity) continue;
            Y[(first + s) * 2] = (float)(kD4[g][0] * tx + kD4[g][1] * ty);
            Y[(first + s) * 2 + 1] = (float)(kD4[g][2] * tx + kD4[g][3] * ty);
        }
    }
}

}  // namespace

// Workspace of lbac_closure_extract_noalloc: a file-scope device array, one
// copy per GPU, held until the process ends.  Host code never uses its name
// as an address (that is a host-side stand-in): the device address comes
// from hipGetSymbolAddress, once per device, with that device current.
constexpr size_t kNoAllocScratchBytes = size_t(8) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch[kMaxDevices];
std::mutex g_scratch_mu;

// The current device's address of `scratch`, or nullptr on a HIP error.
void* scratch_ptr() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void* p = g_scratch[dev].load(std::memory_order_acquire);
    if (p) return p;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch[dev].load(std::memory_order_relaxed);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch[dev].store(p, std::memory_order_release);
    }
    return p;
}

int64_t workspace_bytes(int32_t nxf, int32_t nyf, int32_t r) {
    if (r < 1 || nxf < r || nyf < r) return -1;
    const int64_t nc = (int64_t)(nxf / r) * (nyf / r);
    return (int64_t)(3 * nc * sizeof(double) + (nyf / r + 64) * sizeof(int) + 64);
}

// The extraction with a given workspace (device memory of workspace_bytes).
int extract(const double* phi_f_dev, int32_t nxf, int32_t nyf, int32_t r, double eps_f, double eps_c, double delta,
            float theta, int32_t augment, void* workspace, float* x_dev, float* y_dev, int64_t base, int64_t capacity,
            int64_t* count, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int nxc = nxf / r, nyc = nyf / r;
    const int64_t nc = (int64_t)nxc * nyc;
    double* phic = (double*)workspace;
    double* tx = phic + nc;
    double* ty = tx + nc;
    int* rows = (int*)(ty + nc);
    long long* total = (long long*)(rows + ((nyc + 63) / 64) * 64);
    if (r <= kTileR) {
        const int cx = kTileW / r, cy = std::max(1, kTileH / r);
        hipLaunchKernelGGL(restrict_tile_kernel, dim3((nxc + cx - 1) / cx, (nyc + cy - 1) / cy), dim3(kTileT), 0, s,
                           phi_f_dev, nxf, nyf, r, eps_f, delta, phic, tx, ty);
    } else {
        hipLaunchKernelGGL(restrict_kernel, dim3((nxc + 127) / 128, nyc), dim3(128), 0, s, phi_f_dev, nxf, nyf, r,
                           eps_f, delta, phic, tx, ty);
    }
    hipLaunchKernelGGL(count_kernel, dim3(nyc), dim3(256), 0, s, phic, nxc, theta, rows);
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanT), 0, s, rows, nyc, total);
    const int copies = augment ? 8 : 1;
    if (x_dev && y_dev && capacity > base)
        hipLaunchKernelGGL(emit_kernel, dim3(nyc), dim3(kEmitT), 0, s, phic, tx, ty, nxc, nyc, eps_c, delta, theta,
                           rows, copies, x_dev, y_dev, (long long)base, (long long)capacity);
    long long host_total = 0;
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&host_total, total, sizeof(long long), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return LBAC_EDEVICE;
    *count = host_total * copies;
    return LBAC_OK;
}

int check_args(const double* phi_f_dev, int32_t nxf, int32_t nyf, int32_t r, double eps_f, double eps_c,
               double delta, float theta, int64_t base, int64_t* count) {
    if (!phi_f_dev || !count || r < 1 || nxf % r || nyf % r || nxf / r < 5 || nyf / r < 5) return LBAC_EINVAL;
    if (!(eps_f > 0.0) || !(eps_c > 0.0) || !(delta >= 0.0) || !(theta >= 0.f) || !(theta < 0.5f) || base < 0)
        return LBAC_EINVAL;
    if (nxf / r > 1024 * 16) return LBAC_EINVAL;
    return LBAC_OK;
}

}  // namespace

extern "C" {

int64_t lbac_closure_workspace_bytes(int32_t nxf, int32_t nyf, int32_t r) { return workspace_bytes(nxf, nyf, r); }

int lbac_closure_extract(const double* phi_f_dev, int32_t nxf, int32_t nyf, int32_t r, double eps_f, double eps_c,
                         double delta, float theta, int32_t augment, void* workspace, float* x_dev, float* y_dev,
                         int64_t base, int64_t capacity, int64_t* count, void* stream) {
    const int rc = check_args(phi_f_dev, nxf, nyf, r, eps_f, eps_c, delta, theta, base, count);
    if (rc != LBAC_OK || !workspace) return LBAC_EINVAL;
    return extract(phi_f_dev, nxf, nyf, r, eps_f, eps_c, delta, theta, augment, workspace, x_dev, y_dev, base,
                   capacity, count, stream);
}

int lbac_closure_extract_noalloc(const double* phi_f_dev, int32_t nxf, int32_t nyf, int32_t r, double eps_f,
                                 double eps_c, double delta, float theta, int32_t augment, float* x_dev, float* y_dev,
                                 int64_t base, int64_t capacity, int64_t* count, void* stream) {
    const int rc = check_args(phi_f_dev, nxf, nyf, r, eps_f, eps_c, delta, theta, base, count);
    if (rc != LBAC_OK) return rc;
    if (workspace_bytes(nxf, nyf, r) > (int64_t)kNoAllocScratchBytes) return LBAC_EINVAL;
    void* ws = scratch_ptr();
    if (!ws) return LBAC_EDEVICE;
    return extract(phi_f_dev, nxf, nyf, r, eps_f, eps_c, delta, theta, augment, ws, x_dev, y_dev, base, capacity,
                   count, stream);
}

}  // extern "C"
