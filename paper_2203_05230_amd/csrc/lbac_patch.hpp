// The step on patches: the form for grids whose strips cannot fill the device,
// and in FP64, which has no multi-step strips, for any grid.
//
// A strip-marching tile (lbac_kernels.hpp) works through its rows one after
// another, about 1 us per row whatever the grid, so on a grid of a few hundred
// rows the march itself is the time: the device is nearly idle and latency
// bound.  Here a block takes a patch of PW x PH nodes, loads it once grown by
// H = RC S nodes on each side, and advances it S steps with one thread per
// node (or a few), all rows at once: per step two barriers and one pass of
// the node arithmetic.  The populations of the grown patch stay in LDS (each
// node's rest population in its thread's register); the region a step updates
// shrinks by RC on each side, and the last step stores the patch.  Neighbouring
// patches compute the 2H rows and columns they share both; on an idle device
// that costs nothing, and in FP64 less than moving the state at every step: 384
// and 1470 us per step at 4096^2 and 8192^2, 322 and 1341 with the conventional
// model, where the one-step strips take 564 and 2112 (543 and 1945).
//
// Every node helper, its order of operations and its rounding are those of
// the strip kernels, so the results are the same bit for bit.
#pragma once

#include <algorithm>

#include "lbac_internal.hpp"
#include "lbac_kernels.hpp"

namespace lbac {

template <int S, int PW, int PH, bool CL>
struct PatchGeom {
    static constexpr int RC = CL ? 3 : 2;  // columns and rows one step reaches (the closure's network: 5x5 of phi)
    static constexpr int H = RC * S;
    static constexpr int GW = PW + 2 * H, GH = PH + 2 * H;  // the grown patch
    static constexpr int N = GW * GH;
};

template <typename R, int S, int PW, int PH, bool CL>
struct PatchLds {
    static constexpr int N = PatchGeom<S, PW, PH, CL>::N;
    R f[8][N];  // moving populations 1..8 of every node of the grown patch
    R ps[N];    // psi
};
template <int S, int PW, int PH>
struct PatchLds<float, S, PW, PH, true> {
    static constexpr int N = PatchGeom<S, PW, PH, true>::N;
    float f[8][N];
    float ps[N];
    float phr[N];             // phi (the network's input)
    int tab[N];               // the band nodes of the step's update, in any order
    float cor[N][2];          // their corrections
    uint32_t count[S];        // how many, per step
    alignas(16) uint16_t w[kClWN];  // the network, packed
    float b[kClBN];
};

// a wrapped into [0, n): one step of n at most away unless the grid is smaller
// than the grown patch (near: uniform)
__device__ __forceinline__ int wrap_near(int a, int n, bool near) {
    if (!near) return wrap_idx(a, n);
    return a < 0 ? a + n : (a >= n ? a - n : a);
}

// NT threads, NPT nodes per thread (node i of thread l: l + i NT of the grown
// patch, row by row, so that neighbouring lanes hold neighbouring columns).
template <typename R, int ST, int MODEL, int S, int PW, int PH, int NT, bool CL, bool LOOP = false>
__device__ __forceinline__ void patch_steps(const StepArgs& a, int x0, int y0, PatchLds<R, S, PW, PH, CL>& lds) {
    static_assert(!CL || (sizeof(R) == 4 && ST == ST_PLAIN && MODEL == MODEL_IMPROVED), "closure: FP32 plain storage");
    static_assert(ST == ST_PLAIN || S == 1, "16-bit storage is rounded once per launch: one step");
    using G = PatchGeom<S, PW, PH, CL>;
    constexpr int RC = G::RC, H = G::H, GW = G::GW, GH = G::GH, N = G::N;
    constexpr int NPT = (N + NT - 1) / NT;
    const int l = threadIdx.x;
    const bool nearx = a.nx >= GW, neary = a.ny >= GH;
    const Io<R, ST> io(a);

    int lx[NPT], ly[NPT];
    uint32_t off[NPT];
    R v[NPT][9];             // own post-collision populations
    R Ax[NPT], Bx[NPT], Ay[NPT], By[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int n = min(l + i * NT, N - 1);
        lx[i] = n % GW - H;
        ly[i] = n / GW - H;
        const int gx = wrap_near(x0 + lx[i], a.nx, nearx), gy = wrap_near(y0 + ly[i], a.ny, neary);
        off[i] = (uint32_t)gy * (uint32_t)a.pitch + (uint32_t)gx;
        io.load(off[i], v[i]);
        if constexpr (sizeof(R) == 4) {
            Ax[i] = a.vtabf[gx];
            Bx[i] = a.vtabf[a.nx + gx];
            Ay[i] = a.vtabf[2 * a.nx + gy];
            By[i] = a.vtabf[2 * a.nx + a.ny + gy];
        } else {
            Ax[i] = R(a.vtab[gx]);
            Bx[i] = R(a.vtab[a.nx + gx]);
            Ay[i] = R(a.vtab[2 * a.nx + gy]);
            By[i] = R(a.vtab[2 * a.nx + a.ny + gy]);
        }
    }
    if constexpr (CL) {
        if (l < S) lds.count[l] = 0;
    }
    R rest[NPT], P[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int n = l + i * NT;
        if (n < N) {
#pragma unroll
            for (int q = 1; q < 9; ++q) lds.f[q - 1][n] = v[i][q];
        }
        rest[i] = v[i][0];
        P[i] = Io<R, ST>::kShifted ? v[i][0] : sum9(v[i]);
    }
    // (LOOP: the steps stay a loop, and the lane index opaque: what they share,
    // addresses above all, held across them takes more registers than two
    // blocks of the list kernel have)
#pragma unroll(LOOP ? 1 : S)
    for (int k = 0; k < S; ++k) {
        int l = threadIdx.x;
        if constexpr (LOOP) asm volatile("" : "+v"(l));
        const NodeConst<R> kc(a, k);
        R fp[NPT][9], phi[NPT];
        lds_barrier();
        // ---- phi (Eq. (12)) and psi (Eq. (13)) one node beyond what the step updates
        const int ma = RC * (S - k) - 1;
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int n = l + i * NT;
            if (n < N && lx[i] >= -ma && lx[i] < PW + ma && ly[i] >= -ma && ly[i] < PH + ma) {
                fp[i][0] = rest[i];
#pragma unroll
                for (int q = 1; q < 9; ++q) fp[i][q] = lds.f[q - 1][n - cy(q) * GW - cx(q)];
                R s;
                if constexpr (Io<R, ST>::kShifted) s = shifted_phi(v[i][0], fp[i], v[i]);
                else s = sum9(fp[i]);
                phi[i] = s;
                lds.ps[n] = normal_source<R, MODEL>(s, kc);
                if constexpr (CL) lds.phr[n] = s;
            }
        }
        lds_barrier();
        // ---- update
        const int mb = RC * (S - 1 - k);
        int slot[NPT];  // closure: the node's place in the list of band nodes, or -1
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int n = l + i * NT;
            const bool in = n < N && lx[i] >= -mb && lx[i] < PW + mb && ly[i] >= -mb && ly[i] < PH + mb;
            const bool mine = in && x0 + lx[i] < a.nx && y0 + ly[i] < a.ny;  // the last step stores it
            R out[9];
            slot[i] = -1;
            if (in) {
                R gx, gy, Gx, Gy;
                const R* p = &lds.ps[n];
                iso_gradient(p[1], p[-1], p[GW], p[-GW], p[GW + 1], p[GW - 1], p[1 - GW], p[-1 - GW], gx, gy);
                const R uxr = Ax[i] * Ay[i], uyr = Bx[i] * By[i];
                flux_bracket<R, MODEL>(gx, gy, phi[i], kc.first ? phi[i] : P[i], kc.s_now * uxr, kc.s_now * uyr,
                                       kc.s_old * uxr, kc.s_old * uyr, kc, Gx, Gy);
                collide(fp[i], phi[i], kc.s_now * uxr, kc.s_now * uyr, Gx, Gy, kc, out);
            }
            if constexpr (CL) {
                const float pc = clip01(phi[i]);
                const bool band = in && pc > a.cl_theta && pc < 1.0f - a.cl_theta;
                const uint64_t m = __ballot(band);
                if (m) {
                    const int lane = l % kWave;
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&lds.count[k], (uint32_t)__popcll(m));
                    base = __builtin_amdgcn_readfirstlane(base);
                    if (band) {
                        slot[i] = (int)base + __popcll(m & ((1ull << lane) - 1ull));
                        lds.tab[slot[i]] = n;
                    }
                }
            }
            // (a band node goes through LDS on the last step too: its
            // correction is added below, and the network has the registers
            // to itself)
            const bool later = CL && slot[i] >= 0;
            if (k == S - 1) io.store(mine && !later, off[i], out, phi[i]);
            if (in && (k < S - 1 || later)) {
#pragma unroll
                for (int q = 1; q < 9; ++q) lds.f[q - 1][n] = out[q];
                rest[i] = out[0];
                P[i] = sum9(out);
            }
        }
        if constexpr (CL) {
            // The network on the block's band nodes, 16 to a wavefront at a
            // time: a wavefront's own few would each take a whole 16-sample
            // pass (5 us per step at 16 wavefronts per block; packed, 2 to 3)
            lds_barrier();
            const int count = (int)lds.count[k], lane = l % kWave;
            for (int s0 = l / kWave * 16; s0 < count; s0 += NT / kWave * 16) {
                const int s = s0 + lane % 16, g = lane / 16;
                const bool on = s < count;
                const int c = on ? lds.tab[s] : 0;
                auto xfrag = [&](int) {
                    u16x8_t x;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int kk = 8 * g + e;
                        x[e] = on && kk < 25 ? bf16_bits(lds.phr[c + (kk / 5 - 2) * GW + kk % 5 - 2]) : (uint16_t)0;
                    }
                    return __builtin_bit_cast(bf16x8_t, x);
                };
                float ccx, ccy;
                closure_mlp(lds.w, lds.b, xfrag, 0xffffull, ccx, ccy);
                if (g == 0 && on) {
                    lds.cor[s][0] = ccx;
                    lds.cor[s][1] = ccy;
                }
            }
            if (count) lds_barrier();  // (the same count on every wavefront)
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
                const int n = l + i * NT;
                if (slot[i] < 0) continue;
                float f[9];
#pragma unroll
                for (int q = 1; q < 9; ++q) f[q] = lds.f[q - 1][n];
                closure_correct(f, phi[i], kc.kforce, lds.cor[slot[i]][0], lds.cor[slot[i]][1]);
                if (k == S - 1) {
                    io.store(x0 + lx[i] < a.nx && y0 + ly[i] < a.ny, off[i], f, phi[i]);
                } else {
#pragma unroll
                    for (int q = 1; q < 9; ++q) lds.f[q - 1][n] = f[q];
                    rest[i] = f[0];
                    P[i] = sum9(f);
                }
            }
        }
    }
}

// The closure's network into LDS (seen after the next barrier).
template <int NT, typename Lds>
__device__ __forceinline__ void patch_network(const StepArgs& a, Lds& lds) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cl_w);
    uint32_t* dst = reinterpret_cast<uint32_t*>(lds.w);
    for (int i = threadIdx.x; i < kClWN / 2; i += NT) dst[i] = src[i];
    for (int i = threadIdx.x; i < kClBN; i += NT) lds.b[i] = a.cl_b[i];
}

// Every patch of the grid, one per block.
template <typename R, int ST, int MODEL, int S, int PW, int PH, int NT, bool CL>
__global__ __launch_bounds__(NT) void patch_kernel(StepArgs a) {
    __shared__ PatchLds<R, S, PW, PH, CL> lds;
    const int tile = xcd_tile(blockIdx.x, a.nbx * a.nby, a.n_xcd);
    if constexpr (CL) patch_network<NT>(a, lds);
    patch_steps<R, ST, MODEL, S, PW, PH, NT, CL>(a, (tile % a.nbx) * PW, (tile / a.nbx) * PH, lds);
}

// The listed patches (closure), each block several in turn.
template <int S, int PW, int PH, int NT>
__global__ __launch_bounds__(NT) void patch_list_kernel(StepArgs a) {
    __shared__ PatchLds<float, S, PW, PH, true> lds;
    patch_network<NT>(a, lds);
    const int n = (int)a.cl_count[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) closure_seen(a, (uint32_t)n, PW * PH);
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int tile = a.cl_list[i];
        patch_steps<float, ST_PLAIN, MODEL_IMPROVED, S, PW, PH, NT, true, true>(a, (tile % a.cl_npx) * PW, (tile / a.cl_npx) * PH,
                                                                          lds);
        lds_barrier();  // the LDS is filled again by the next patch
    }
}

}  // namespace lbac

// ---------------------------------------------------------------------------
// host side: the shapes that are built, the rule that chooses one, the launches

namespace {

using namespace lbac;

// A shape: S steps of patches of pw x ph nodes.  first, more: microseconds of
// a launch of at most 256 patches (one per CU) and of every further 256,
// fitted to launches back to back on an MI355X.  They rank the shapes against
// each other and against the strip kernels.  conv: the same relative to the
// other shapes with the conventional model, whose step without logarithms
// leaves less to gain from fewer shared nodes.
struct Shape {
    int S, pw, ph;
    float first, more, conv = 1.f;
};

// FP32: measured at 64^2 to 4096^2 (for example 1.24 us per step with six
// steps of 8 x 8 at 64^2, 1.62 with four of 16 x 16 at 256^2, 2.93 with four
// of 32 x 16 at 512^2, 2.4, 5.4 and 8.9 with four of 48 x 16 at 400^2, 768^2 and
// 1024^2; the best of the strip shapes take 6.9, 7.4, 8.1 and, at 1024^2, 12.6).
constexpr Shape kF32[] = {{6, 8, 8, 7.5f, 3.7f},   {4, 16, 16, 6.4f, 2.8f}, {6, 24, 24, 14.3f, 11.4f},
                          {4, 32, 16, 7.8f, 4.1f}, {3, 52, 20, 8.3f, 5.2f}, {2, 24, 24, 5.4f, 2.2f},
                          {4, 48, 16, 9.8f, 5.3f}, {1, 28, 28, 5.0f, 2.1f}};
// FP64 is bound by its instructions where a SIMD has more than a wavefront or
// two, so small patches and just enough threads for the grown patch pay
// (us per step: 1.97 with three steps of 4 x 4 at 64^2, 2.37 with three of 8 x
// 8 at 100^2, 2.83 with four of 12 x 8 at 150^2, 3.14 with three of 13 x 13
// at 200^2, 6.2, 8.8 and 25 with two of 24 x 16, one node per thread of twelve
// wavefronts, at 400^2, 512^2 and 1024^2, where three of 52 x 20 and two of 24 x
// 24 had taken 6.9, 9.6 and 31; with only four steps of 8 x 8 or 16 x 16 before, 2.41,
// 2.55, 3.37, 3.50 and 9.0; the best one-step strips 7.2 at 64^2, 9.8 at
// 200^2, 37 and 522).
constexpr Shape kF64[] = {{3, 4, 4, 5.9f, 1.65f},   {3, 8, 8, 7.f, 3.1f},     {4, 12, 8, 11.f, 5.7f},
                          {3, 13, 13, 9.3f, 5.f},   {3, 16, 16, 10.5f, 7.5f}, {2, 16, 16, 7.5f, 4.2f},
                          {3, 20, 20, 11.1f, 9.1f}, {2, 24, 24, 9.9f, 8.3f},  {3, 52, 20, 19.7f, 20.f},
                          {2, 24, 16, 8.4f, 4.5f, 1.25f}, {1, 28, 28, 6.6f, 6.f}};
// 16-bit storage: one step, since a launch rounds once (us per step, and
// the best strips: 3.3 and 4.0 at 64^2, 3.8 and 4.4 at 200^2, 6.2 and 6.7 at
// 512^2, 12.6 and 14.8 at 1024^2, 22 and 26 at 1536^2, 36 and 39 at 2048^2; only
// 28 x 28 before, 4.3, 4.6, 7.0, 16.2, 28.5 and 49.  Where the state no longer
// stays in the last-level cache the strips win: 105 and 103 at 3000^2, 176 and
// 151 at 4096^2).
constexpr Shape kF16[] = {{1, 12, 12, 3.3f, 0.48f}, {1, 28, 12, 3.6f, 0.9f}, {1, 60, 28, 5.7f, 3.2f}};

// FP32 with the closure, a disk's edge in the field (5.2, 6.6, 7.3 and 12.8 us
// per step at 128^2, 200^2, 256^2 and 512^2; with four steps of 8 x 8, three of
// 14 x 14 and two of 20 x 20 before, 5.7, 7.9, 8.1 and 14.3; the two-pass
// launches at their best 17.8 at 128^2, 17.7 at 512^2 and 21.7 at 1024^2).
constexpr Shape kCl[] = {{2, 8, 8, 10.5f, 2.4f},  {2, 14, 14, 13.f, 4.2f},  {2, 16, 16, 14.f, 5.7f},
                         {2, 20, 20, 15.f, 6.5f}, {1, 16, 16, 8.4f, 1.9f}, {2, 52, 20, 24.f, 8.5f},
                         {1, 26, 26, 9.8f, 3.f}};

template <typename R, int ST, int MODEL, int S, int PW, int PH, int NT, bool CL = false>
hipError_t go(StepArgs a, hipStream_t s) {
    a.nbx = (a.nx + PW - 1) / PW;
    a.nby = (a.ny + PH - 1) / PH;
    a.n_xcd = lbac_host::kXcds;
    hipLaunchKernelGGL((patch_kernel<R, ST, MODEL, S, PW, PH, NT, CL>), dim3(a.nbx * a.nby), dim3(NT), 0, s, a);
    return hipGetLastError();
}

template <int MODEL>
hipError_t go_f32(int shape, const StepArgs& a, hipStream_t s) {
    switch (shape) {
    case 0:
        return go<float, ST_PLAIN, MODEL, 6, 8, 8, 1024>(a, s);
    case 1:
        return go<float, ST_PLAIN, MODEL, 4, 16, 16, 1024>(a, s);
    case 2:
        return go<float, ST_PLAIN, MODEL, 6, 24, 24, 768>(a, s);
    case 3:
        return go<float, ST_PLAIN, MODEL, 4, 32, 16, 768>(a, s);
    case 4:
        return go<float, ST_PLAIN, MODEL, 3, 52, 20, 1024>(a, s);
    case 5:
        return go<float, ST_PLAIN, MODEL, 2, 24, 24, 1024>(a, s);
    case 6:
        return go<float, ST_PLAIN, MODEL, 4, 48, 16, 1024>(a, s);
    default:
        return go<float, ST_PLAIN, MODEL, 1, 28, 28, 1024>(a, s);
    }
}

template <int MODEL>
hipError_t go_f64(int shape, const StepArgs& a, hipStream_t s) {
    switch (shape) {
    case 0:
        return go<double, ST_PLAIN, MODEL, 3, 4, 4, 256>(a, s);
    case 1:
        return go<double, ST_PLAIN, MODEL, 3, 8, 8, 448>(a, s);
    case 2:
        return go<double, ST_PLAIN, MODEL, 4, 12, 8, 704>(a, s);
    case 3:
        return go<double, ST_PLAIN, MODEL, 3, 13, 13, 640>(a, s);
    case 4:
        return go<double, ST_PLAIN, MODEL, 3, 16, 16, 832>(a, s);
    case 5:
        return go<double, ST_PLAIN, MODEL, 2, 16, 16, 576>(a, s);
    case 6:
        return go<double, ST_PLAIN, MODEL, 3, 20, 20, 1024>(a, s);
    case 7:
        return go<double, ST_PLAIN, MODEL, 2, 24, 24, 1024>(a, s);
    case 8:
        return go<double, ST_PLAIN, MODEL, 3, 52, 20, 1024>(a, s);
    case 9:
        return go<double, ST_PLAIN, MODEL, 2, 24, 16, 768>(a, s);
    default:
        return go<double, ST_PLAIN, MODEL, 1, 28, 28, 1024>(a, s);
    }
}

template <int ST, int MODEL>
hipError_t go_f16(int shape, const StepArgs& a, hipStream_t s) {
    switch (shape) {
    case 0:
        return go<float, ST, MODEL, 1, 12, 12, 256>(a, s);
    case 1:
        return go<float, ST, MODEL, 1, 28, 12, 512>(a, s);
    default:
        return go<float, ST, MODEL, 1, 60, 28, 1024>(a, s);
    }
}

hipError_t go_cl(int shape, const StepArgs& a, hipStream_t s) {
    switch (shape) {
    case 0:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 2, 8, 8, 448, true>(a, s);
    case 1:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 2, 14, 14, 704, true>(a, s);
    case 2:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 2, 16, 16, 832, true>(a, s);
    case 3:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 2, 20, 20, 1024, true>(a, s);
    case 4:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 1, 16, 16, 512, true>(a, s);
    case 5:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 2, 52, 20, 1024, true>(a, s);
    default:
        return go<float, ST_PLAIN, MODEL_IMPROVED, 1, 26, 26, 1024, true>(a, s);
    }
}

// The closure in two passes over large grids: the plain S-step strips, which
// mark the patches near the interface band, then the marked patches again
// with the network, from the same input.  The band is thin (0.1% of the nodes
// of the benchmark's disk at 8192^2), so nearly all of the grid runs at the
// plain kernel's speed; before, every tile ran a kernel with the network
// inside, at two wavefronts per SIMD.
constexpr int kMarkBlocks = 512;

// The strips and the list of the marked patches (a: completed for the patches).
template <int S>
hipError_t go_marks(const lbac_ctx* h, StepArgs& a, int bx) {
    a.cl_npx = (a.nx + kMarkW - 1) / kMarkW;
    const int np = a.cl_npx * ((a.ny + kMarkH<S> - 1) / kMarkH<S>);
    const hipError_t e = lbac_host::launch_stepS_band(S, a, bx, h->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(closure_list_kernel, dim3((np + 2047) / 2048), dim3(256), 0, h->stream, a.cl_flags, np,
                       const_cast<int32_t*>(a.cl_list), a.cl_count);
    return hipGetLastError();
}

template <int S>
hipError_t go_split(const lbac_ctx* h, StepArgs a, int bx) {
    const hipError_t e = go_marks<S>(h, a, bx);
    if (e != hipSuccess) return e;
    const int np = a.cl_npx * ((a.ny + kMarkH<S> - 1) / kMarkH<S>);
    hipLaunchKernelGGL((patch_list_kernel<S, kMarkW, kMarkH<S>, 512>), dim3(std::min(np, kMarkBlocks)), dim3(512), 0,
                       h->stream, a);
    return hipGetLastError();
}

template <int N>
const Shape* all(const Shape (&t)[N], int& n) {
    n = N;
    return t;
}
const Shape* shapes_of(const lbac_ctx* h, int& n) {
    if (h->closure) return all(kCl, n);
    if (h->storage != ST_PLAIN) return all(kF16, n);
    return h->p.precision == LBAC_F64 ? all(kF64, n) : all(kF32, n);
}

}  // namespace

lbac_host::PatchPlan lbac_host::plan_patch(const lbac_ctx* h, int64_t left) {
    PatchPlan best{-1, 0, 0.f};
    int n = 0;
    const Shape* t = shapes_of(h, n);
    // the state read and written once per launch bounds short launches on large
    // grids: 4 TB/s from HBM, about 6 where both buffers stay in the last-level
    // cache (FP64, one step at 1024^2: 151 MB in 25 us)
    const float state = 1e-6f * (float)((int64_t)h->p.nx * h->p.ny) * state_bytes(h);  // MB
    // The closure's patches share three nodes a step on each side, so they read
    // more than the state once it no longer stays in the cache (4096^2, one step
    // of 26 x 26: 382 us).  And where there are several to a CU they wait for the
    // network of the last ones, the longer the wider the band is: its width goes
    // with log(1 / theta), and from theta = 0.02 to 1e-4 two steps of 52 x 20 take
    // 285 -> 520 us per step at 4096^2 and 81 -> 189 at 2048^2, one of 26 x 26 382
    // -> 501 and 100 -> 160, the one-step strips 293 -> 297 and 105 -> 107.
    const float tail = h->closure ? std::max(1.f, -0.256f * std::log(h->cl_theta + 1e-10f)) : 1.f;
    const bool conv = h->p.model == LBAC_MODEL_CONVENTIONAL;
    // FP64 without the logarithms: 9.9, 17.2 and 25 us for one step of 28 x 28 at 600^2, 768^2 and 1024^2, where the
    // table gives 12.6, 24.6 and 36.6; the strips, whose costs are the model's own, take 21, 27 and 33
    const float conv_all = h->p.precision == LBAC_F64 ? 0.7f : 1.f;
    for (int i = 0; i < n; ++i) {
        if (t[i].S > left) continue;
        const int64_t tiles = (int64_t)((h->p.nx + t[i].pw - 1) / t[i].pw) * ((h->p.ny + t[i].ph - 1) / t[i].ph);
        // on long grids a few rows high the network runs on every image of a row a patch covers, while a strip
        // marches no more rows than there are (all of 37197 x 1 in the band: 82 us per step with patches of 26 x 26,
        // 38 with one-step strips)
        const int64_t rows = (int64_t)((h->p.ny + t[i].ph - 1) / t[i].ph) * t[i].ph;
        if (h->closure && tiles > 256 && rows > (t[i].S == 1 ? 4 : 2) * (int64_t)h->p.ny) continue;
        const float wait = t[i].S == 1 ? std::min(0.6f + 0.4f * tail, 1.35f) : std::min(tail, 2.2f);
        float cost = t[i].first + (float)((tiles + 255) / 256 - 1) * t[i].more * wait;
        if (conv) cost *= t[i].conv * conv_all;
        const int halo = h->closure ? 6 * t[i].S : 0;
        const float moved = state * (1.f + (float)((t[i].pw + halo) * (t[i].ph + halo)) / (float)(t[i].pw * t[i].ph));
        const float us = std::max(cost, moved / (2.f * state < 256.f ? 6.f : 4.f)) / (float)t[i].S;
        if (best.shape < 0 || us < best.us) best = {i, t[i].S, us};
    }
    return best;
}

hipError_t lbac_host::launch_patch(const lbac_ctx* h, int src, int32_t k, const PatchPlan& p) {
    const StepArgs a = make_args(h, src, k);
    const bool conv = h->p.model == LBAC_MODEL_CONVENTIONAL;
    if (h->closure) return go_cl(p.shape, a, h->stream);
    switch (h->p.precision) {
    case LBAC_F64:
        return conv ? go_f64<MODEL_CONVENTIONAL>(p.shape, a, h->stream) : go_f64<MODEL_IMPROVED>(p.shape, a, h->stream);
    case LBAC_F32:
        return conv ? go_f32<MODEL_CONVENTIONAL>(p.shape, a, h->stream) : go_f32<MODEL_IMPROVED>(p.shape, a, h->stream);
    case LBAC_F32_F16STORE:
        return conv ? go_f16<ST_F16, MODEL_CONVENTIONAL>(p.shape, a, h->stream)
                    : go_f16<ST_F16, MODEL_IMPROVED>(p.shape, a, h->stream);
    default:
        return conv ? go_f16<ST_BF16, MODEL_CONVENTIONAL>(p.shape, a, h->stream)
                    : go_f16<ST_BF16, MODEL_IMPROVED>(p.shape, a, h->stream);
    }
}

hipError_t lbac_host::launch_split(const lbac_ctx* h, const StepArgs& a, int S) {
    return S == 3 ? go_split<3>(h, a, h->bx) : go_split<2>(h, a, h->bx);
}

hipError_t lbac_host::launch_look(const lbac_ctx* h, StepArgs a, int bx) {
    const hipError_t e = go_marks<3>(h, a, bx);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(closure_seen_kernel, dim3(1), dim3(1), 0, h->stream, a, (uint32_t)(kMarkW * kMarkH<3>));
    return hipGetLastError();
}

size_t lbac_host::mark_count(int nx, int ny) {
    static_assert(kMarkH<3> <= kMarkH<2>, "the lower patches are the more");
    return (size_t)((nx + kMarkW - 1) / kMarkW) * ((ny + kMarkH<3> - 1) / kMarkH<3>);
}
