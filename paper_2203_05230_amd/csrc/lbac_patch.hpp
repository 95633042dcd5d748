// The step on patches: the form for grids whose strips cannot fill the device.
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
// that costs nothing.
//
// Every node helper, its order of operations and its rounding are those of
// the strip kernels, so the results are the same bit for bit.
#pragma once

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
    int tab[16][kWave];       // per wavefront: its band nodes
    uint16_t w[kClWN];        // the network, packed
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
template <typename R, int ST, int MODEL, int S, int PW, int PH, int NT, bool CL>
__global__ __launch_bounds__(NT) void patch_kernel(StepArgs a) {
    static_assert(!CL || (sizeof(R) == 4 && ST == ST_PLAIN && MODEL == MODEL_IMPROVED), "closure: FP32 plain storage");
    static_assert(ST == ST_PLAIN || S == 1, "16-bit storage is rounded once per launch: one step");
    using G = PatchGeom<S, PW, PH, CL>;
    constexpr int RC = G::RC, H = G::H, GW = G::GW, GH = G::GH, N = G::N;
    constexpr int NPT = (N + NT - 1) / NT;
    __shared__ PatchLds<R, S, PW, PH, CL> lds;
    const int tile = xcd_tile(blockIdx.x, a.nbx * a.nby, a.n_xcd);
    const int x0 = (tile % a.nbx) * PW, y0 = (tile / a.nbx) * PH;
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
        const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cl_w);
        uint32_t* dst = reinterpret_cast<uint32_t*>(lds.w);
        for (int i = l; i < kClWN / 2; i += NT) dst[i] = src[i];
        for (int i = l; i < kClBN; i += NT) lds.b[i] = a.cl_b[i];
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
#pragma unroll
    for (int k = 0; k < S; ++k) {
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
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int n = l + i * NT;
            const bool in = n < N && lx[i] >= -mb && lx[i] < PW + mb && ly[i] >= -mb && ly[i] < PH + mb;
            R out[9];
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
                // the network on the wavefront's band nodes, packed into a list
                const float pc = clip01(phi[i]);
                const bool band = in && pc > a.cl_theta && pc < 1.0f - a.cl_theta;
                const uint64_t m = __ballot(band);
                if (m) {
                    const int lane = l % kWave, slot = __popcll(m & ((1ull << lane) - 1ull)), count = __popcll(m);
                    int* tab = lds.tab[l / kWave];
                    if (band) tab[slot] = n;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
                    auto xfrag = [&](int nt) {
                        const int s = 16 * nt + lane % 16, g = lane / 16;
                        const bool on = s < count;
                        const int c = on ? tab[s] : 0;
                        u16x8_t x;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int kk = 8 * g + e;
                            x[e] = on && kk < 25 ? bf16_bits(lds.phr[c + (kk / 5 - 2) * GW + kk % 5 - 2]) : (uint16_t)0;
                        }
                        return __builtin_bit_cast(bf16x8_t, x);
                    };
                    float ccx, ccy;
                    closure_mlp(lds.w, lds.b, xfrag, count >= 64 ? ~0ull : (1ull << count) - 1ull, ccx, ccy);
                    const float vx = __shfl(ccx, slot & (kWave - 1), kWave), vy = __shfl(ccy, slot & (kWave - 1), kWave);
                    if (band) closure_correct(out, phi[i], kc.kforce, vx, vy, false);
                    __builtin_amdgcn_wave_barrier();  // the list is rewritten by the next step
                }
            }
            if (k == S - 1) {
                io.store(in && x0 + lx[i] < a.nx && y0 + ly[i] < a.ny, off[i], out, phi[i]);
            } else if (in) {
#pragma unroll
                for (int q = 1; q < 9; ++q) lds.f[q - 1][n] = out[q];
                rest[i] = out[0];
                P[i] = sum9(out);
            }
        }
    }
}

}  // namespace lbac
