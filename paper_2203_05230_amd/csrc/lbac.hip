// Host side of the lbac library: context, memory layout, launches, graph
// replay, autotuning, reductions and the C ABI declared in include/lbac.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "lbac_internal.hpp"
#include "lbac_patch.hpp"

using namespace lbac;
using namespace lbac_host;

namespace lbac_host {

int fail(lbac_ctx* h, int code, const std::string& msg) {
    if (h) h->err = msg;
    return code;
}

void* dev_alloc(lbac_ctx* h, size_t bytes) {
    if (h->has_alloc) return h->alloc.alloc(bytes, h->alloc.user);
    void* ptr = nullptr;
    if (hipMalloc(&ptr, bytes) != hipSuccess) return nullptr;
    return ptr;
}

void dev_free(lbac_ctx* h, void* ptr) {
    if (!ptr) return;
    if (h->has_alloc)
        h->alloc.free(ptr, h->alloc.user);
    else
        (void)hipFree(ptr);
}

}  // namespace lbac_host

namespace {

void drop_graphs(lbac_ctx* h) {
    for (int i = 0; i < 2; ++i) {
        if (h->gexec[i]) (void)hipGraphExecDestroy(h->gexec[i]);
        h->gexec[i] = nullptr;
        h->gexec_chunk[i] = 0;
    }
}

// What the closure changes: the launches of a context whose shape nobody set.
void drop_plans(lbac_ctx* h) {
    for (Launch& l : h->plans) l.S = 0;
    drop_graphs(h);
}

// The closure's buffers: all of them, or (after this) none.
void free_closure(lbac_ctx* h) {
    for (void* p : {(void*)h->cl_param, (void*)h->cl_w, (void*)h->cl_b, (void*)h->cl_mask, (void*)h->cl_list,
                    (void*)h->cl_count, (void*)h->cl_flags})
        dev_free(h, p);
    h->cl_param = nullptr;
    h->cl_w = nullptr;
    h->cl_b = nullptr;
    h->cl_mask = nullptr;
    h->cl_list = nullptr;
    h->cl_count = nullptr;
    h->cl_flags = nullptr;
}

void release(lbac_ctx* h) {
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    drop_graphs(h);
    for (int i = 0; i < 2; ++i) {
        dev_free(h, h->pop[i]);
        dev_free(h, h->phis[i]);
    }
    dev_free(h, h->vtab);
    dev_free(h, h->vtabf);
    dev_free(h, h->t_dev);
    dev_free(h, h->tfac);
    dev_free(h, h->rows);
    dev_free(h, h->red5);
    dev_free(h, h->dtmp);
    free_closure(h);
    if (h->host5) (void)hipHostFree(h->host5);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
}

// Separable velocity tables: u = s(t) Ax[x] Ay[y], v = s(t) Bx[x] By[y].
void build_velocity(const lbac_params& p, std::vector<double>& tab) {
    const int nx = p.nx, ny = p.ny;
    tab.assign(2 * (size_t)nx + 2 * (size_t)ny, 0.0);
    double* Ax = tab.data();
    double* Bx = Ax + nx;
    double* Ay = Bx + nx;
    double* By = Ay + ny;
    const double PI = 3.14159265358979323846;
    for (int i = 0; i < nx; ++i) {
        const double X = i + 0.5, x = X / nx;
        const double sx = std::sin(PI * x);
        switch (p.vel_kind) {
        case LBAC_VEL_VORTEX:
            Ax[i] = -p.U * sx * sx;
            Bx[i] = p.U * std::sin(2.0 * PI * x);
            break;
        case LBAC_VEL_VORTEX_PAPER:
            Ax[i] = p.U * sx * sx;
            Bx[i] = -p.U * std::sin(2.0 * PI * x);
            break;
        case LBAC_VEL_ROTATION:
            Ax[i] = -p.omega;
            Bx[i] = p.omega * (X - p.cx);
            break;
        case LBAC_VEL_UNIFORM:
            Ax[i] = p.ux;
            Bx[i] = p.uy;
            break;
        default:
            break;
        }
    }
    for (int j = 0; j < ny; ++j) {
        const double Y = j + 0.5, y = Y / ny;
        const double sy = std::sin(PI * y);
        switch (p.vel_kind) {
        case LBAC_VEL_VORTEX:
        case LBAC_VEL_VORTEX_PAPER:
            Ay[j] = std::sin(2.0 * PI * y);
            By[j] = sy * sy;
            break;
        case LBAC_VEL_ROTATION:
            Ay[j] = Y - p.cy;
            By[j] = 1.0;
            break;
        case LBAC_VEL_UNIFORM:
            Ay[j] = 1.0;
            By[j] = 1.0;
            break;
        default:
            break;
        }
    }
}

double time_period(const lbac_params& p) {
    return (p.vel_kind == LBAC_VEL_VORTEX || p.vel_kind == LBAC_VEL_VORTEX_PAPER) ? p.period_T : 0.0;
}

}  // namespace

float lbac_host::state_bytes(const lbac_ctx* h) {
    return (float)(h->nplanes * h->elem_bytes + (h->storage == ST_PLAIN ? 0 : 4));
}

StepArgs lbac_host::make_args(const lbac_ctx* h, int src, int32_t k) {
    StepArgs a{};
    a.src = h->pop[src];
    a.dst = h->pop[1 - src];
    a.src_phi = h->phis[src];
    a.dst_phi = h->phis[1 - src];
    a.plane_stride = h->plane_stride;
    a.pitch = h->pitch;
    a.nx = h->p.nx;
    a.ny = h->p.ny;
    a.strip_h = h->strip_h;
    a.vtab = h->vtab;
    a.vtabf = h->vtabf;
    a.vrowf = h->vtabf + 2 * h->p.nx + 2 * h->p.ny;
    a.t_dev = h->t_dev;
    a.tfac = h->tfac;
    a.k = k;
    a.period_T = time_period(h->p);
    a.eps = h->p.eps;
    a.tau = h->p.tau;
    a.delta = h->p.delta;
    a.psi_scale = a.eps * 0.69314718055994530942;
    a.s_scale = 1.0 / (a.eps * (1.0 + 2.0 * a.delta) * (1.0 + 2.0 * a.delta));
    a.omega = 1.0 / a.tau;
    a.kforce = 1.0 - 0.5 / a.tau;
    a.keep = 1.0 - 1.0 / a.tau;
    a.cl_w = h->cl_w;
    a.cl_b = h->cl_b;
    a.cl_theta = h->cl_theta;
    a.cl_mask = h->closure ? h->cl_mask : nullptr;
    a.cl_words = h->cl_words;
    if (h->closure) {
        // a b at theta, less a hundred times what FP32 rounding can take from it: of a band node's a and b each is
        // above theta + delta but for its own rounding (1 - phi is exact from 1/2 on), whatever theta is.  (An
        // absolute slack of 1e-7 let every node pass for theta + delta below that: 2048^2 at theta = 5e-8 took 325
        // us per step instead of the 170 of one-step launches.)
        const double th = h->cl_theta;
        a.cl_ab = th + a.delta > 1e-30 ? (float)((th + a.delta) * (1.0 - th + a.delta) * (1.0 - 1e-5)) : -1.f;
        a.cl_flags = h->cl_flags;
        a.cl_list = h->cl_list;
        a.cl_count = h->cl_count;
        a.cl_seen = h->cl_seen;
    }
    return a;
}

namespace {

template <typename R, int ST, int MODEL>
hipError_t launch_step_bx(StepArgs a, int variant, int bx, hipStream_t s) {
    a.nby = (a.ny + a.strip_h - 1) / a.strip_h;
    a.n_xcd = kXcds;
    if (variant == LBAC_KERNEL_BLOCK || variant == LBAC_KERNEL_BLOCK_DEEP) {
        // one block of bx column threads plus one halo wavefront per bx-column tile
        a.nbx = (a.nx + bx - 1) / bx;
        dim3 grid(a.nbx * a.nby);
        const bool deep = variant == LBAC_KERNEL_BLOCK_DEEP;
        switch (bx) {
        case 64:
            if (deep)
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 64, 2>), grid, dim3(block_threads<64>()), 0, s, a);
            else
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 64, 1>), grid, dim3(block_threads<64>()), 0, s, a);
            break;
        case 128:
            if (deep)
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 128, 2>), grid, dim3(block_threads<128>()), 0, s, a);
            else
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 128, 1>), grid, dim3(block_threads<128>()), 0, s, a);
            break;
        default:
            if (deep)
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 256, 2>), grid, dim3(block_threads<256>()), 0, s, a);
            else
                hipLaunchKernelGGL((step_kernel_lds<R, ST, MODEL, 256, 1>), grid, dim3(block_threads<256>()), 0, s, a);
            break;
        }
        return hipGetLastError();
    }
    // bx / 64 wavefronts per block, each owning one 60-column tile
    const int wpb = bx / kWave;
    a.nbx = (a.nx + kTileW - 1) / kTileW;
    dim3 grid(((a.nbx + wpb - 1) / wpb) * a.nby);
    switch (wpb) {
    case 1:
        hipLaunchKernelGGL((step_kernel<R, ST, MODEL, 1>), grid, dim3(64), 0, s, a);
        break;
    case 2:
        hipLaunchKernelGGL((step_kernel<R, ST, MODEL, 2>), grid, dim3(128), 0, s, a);
        break;
    default:
        hipLaunchKernelGGL((step_kernel<R, ST, MODEL, 4>), grid, dim3(256), 0, s, a);
        break;
    }
    return hipGetLastError();
}

template <typename R, int ST>
hipError_t launch_step_m(const lbac_ctx* h, const StepArgs& a, int variant, int bx) {
    if (h->p.model == LBAC_MODEL_CONVENTIONAL)
        return launch_step_bx<R, ST, MODEL_CONVENTIONAL>(a, variant, bx, h->stream);
    return launch_step_bx<R, ST, MODEL_IMPROVED>(a, variant, bx, h->stream);
}

// Tile widths of the one-step block kernels.
bool one_step_bx(int bx) { return bx == 64 || bx == 128 || bx == 256; }

// Tile widths of the S-step kernels: multiples of 32 columns from 64 to 320,
// and 240 (the widest tile whose grown columns, bx + 4S at S = 3, fill four
// wavefronts; tiles that start off a 128-byte line of the storage, every
// other one in FP32, give their head columns to the halo wavefront).
bool stepS_bx(int bx) { return (bx >= 64 && bx <= 320 && bx % 32 == 0) || bx == 240; }

hipError_t launch_step(const lbac_ctx* h, int src, int32_t k) {
    StepArgs a = make_args(h, src, k);
    // one-step launches of the S-step variants use the deep block kernel, at a
    // tile width it has (the others exist for the S-step kernels only)
    const int var1 =
        h->variant == LBAC_KERNEL_FUSED2 || h->variant == LBAC_KERNEL_FUSED3 ? LBAC_KERNEL_BLOCK_DEEP : h->variant;
    const int bx1 = one_step_bx(h->bx) ? h->bx : 256;
    if (h->closure) {
        // FP32 plain storage.  The block variants write the band masks; then the
        // band list is rebuilt and the correction pass adds the network's flux
        // correction at the listed nodes.
        const int variant = var1 == LBAC_KERNEL_WAVE ? LBAC_KERNEL_BLOCK : var1;
        const hipError_t e = h->p.model == LBAC_MODEL_CONVENTIONAL
                                 ? launch_step_bx<float, ST_PLAIN, MODEL_CONVENTIONAL>(a, variant, bx1, h->stream)
                                 : launch_step_bx<float, ST_PLAIN, MODEL_IMPROVED>(a, variant, bx1, h->stream);
        if (e != hipSuccess) return e;
        const int64_t nwords = (int64_t)h->p.ny * h->cl_words;
        hipLaunchKernelGGL(closure_reset_kernel, dim3(1), dim3(64), 0, h->stream, h->cl_count);
        hipLaunchKernelGGL(closure_scan_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, h->stream,
                           h->cl_mask, nwords, h->cl_words, h->p.nx, h->cl_list, h->cl_count);
        hipLaunchKernelGGL(closure_apply_kernel, dim3(kClosureBlocks), dim3(kClWaves * kWave), 0, h->stream, a,
                           h->cl_list, h->cl_count);
        return hipGetLastError();
    }
    switch (h->p.precision) {
    case LBAC_F64:
        return launch_step_m<double, ST_PLAIN>(h, a, var1, bx1);
    case LBAC_F32:
        return launch_step_m<float, ST_PLAIN>(h, a, var1, bx1);
    case LBAC_F32_F16STORE:
        return launch_step_m<float, ST_F16>(h, a, var1, bx1);
    default:
        return launch_step_m<float, ST_BF16>(h, a, var1, bx1);
    }
}

// Whether the S-step variants can take the run: FP32 collision, and with the
// closure on FP32 storage and the improved model.
bool stepS_allowed(const lbac_ctx* h) {
    if (h->p.precision == LBAC_F64) return false;
    return !h->closure || h->p.model == LBAC_MODEL_IMPROVED;
}

// Tile width of the one-step kernels by default: full-width blocks when the grid allows.
int default_bx(int nx) { return nx >= 256 ? 256 : (nx >= 128 ? 128 : 64); }

// Steps one launch takes: S with the S-step variants, else 1.
int launch_steps_of(const lbac_ctx* h) {
    if (!stepS_allowed(h)) return 1;
    return h->variant == LBAC_KERNEL_FUSED2 ? 2 : (h->variant == LBAC_KERNEL_FUSED3 ? 3 : 1);
}

// What a row of a strip takes in a launch of `tiles` S-step tiles (us): up to
// three run on a CU at once, 768 in all; a started round counts half.
float stepS_row(int64_t tiles) {
    const int64_t rounds = (tiles + 767) / 768;
    return tiles <= 256 ? 0.35f : (tiles <= 512 ? 0.455f : (tiles <= 768 ? 0.65f
           : 0.31f * ((float)tiles / 768.f + (float)rounds)));
}

// Rows of the strips when `rows` are asked for: the kernel marches whole
// periods of Q rows, so the nearest multiple (at least one); but the multiple
// above where the one below would add a strip that it does not (200 rows in
// one strip become 198 and 2) and the added tiles find no room beside the
// others.  Three steps on 128-column tiles, us per step with the nearest and
// with these: 2048^2 in strips of 128 53 and 47, 8192^2 in strips of 512 457
// and 361; where all run at once the shorter strips are the faster.
int stepS_height(int nx, int ny, int bx, int rows, int Q) {
    const int h = std::max(Q, (rows + Q / 2) / Q * Q), high = h + Q;
    auto strips = [&](int r) { return (ny + r - 1) / r; };
    auto us = [&](int r) { return stepS_row((int64_t)((nx + bx - 1) / bx) * strips(r)) * (float)(r + 14); };
    return h < rows && strips(high) == strips(rows) && us(high) < us(h) ? high : h;
}

// One S-step launch with tiles of bx columns.
template <int MODEL, int S, int ST, bool BAND = false>
hipError_t launch_stepS_m(StepArgs a, int bx, hipStream_t s) {
    using L = TileSRows<S>;
    a.strip_h = stepS_height(a.nx, a.ny, bx, a.strip_h, L::kPeriod);
    a.nby = (a.ny + a.strip_h - 1) / a.strip_h;
    a.n_xcd = kXcds;
    a.tile_w = bx;
    a.nbx = (a.nx + bx - 1) / bx;
    const dim3 grid(a.nbx * a.nby), block((bx + 4 * S + 63) / 64 * 64);
    hipLaunchKernelGGL((stepS_kernel_lds<MODEL, S, ST, BAND>), grid, block, L::bytes(bx), s, a);
    return hipGetLastError();
}

template <int ST>
hipError_t launch_stepS_st(const lbac_ctx* h, const StepArgs& a, int S) {
    const bool conv = h->p.model == LBAC_MODEL_CONVENTIONAL;
    if (S == 3)
        return conv ? launch_stepS_m<MODEL_CONVENTIONAL, 3, ST>(a, h->bx, h->stream)
                    : launch_stepS_m<MODEL_IMPROVED, 3, ST>(a, h->bx, h->stream);
    return conv ? launch_stepS_m<MODEL_CONVENTIONAL, 2, ST>(a, h->bx, h->stream)
                : launch_stepS_m<MODEL_IMPROVED, 2, ST>(a, h->bx, h->stream);
}

// Steps k .. k + S - 1 of the current run in one launch, from pop[src] into pop[1 - src].
hipError_t launch_stepS(const lbac_ctx* h, int src, int32_t k, int S) {
    const StepArgs a = make_args(h, src, k);
    if (h->closure) return launch_split(h, a, S);
    switch (h->p.precision) {
    case LBAC_F32_F16STORE:
        return launch_stepS_st<ST_F16>(h, a, S);
    case LBAC_F32_BF16STORE:
        return launch_stepS_st<ST_BF16>(h, a, S);
    default:
        return launch_stepS_st<ST_PLAIN>(h, a, S);
    }
}

// What a row of a one-step strip costs: a strip takes its rows and the
// pipeline's four, each alone + busy k microseconds with k tiles on a CU, of
// which `resident` run at once; never less than the state read and written
// once at 4.75 TB/s.  The 256-column FP64 tile (five wavefronts, bound by their
// instructions) takes as long again for every further tile, so that a height
// whose tiles divide evenly among the 256 CUs is worth more than many tiles;
// FP32 tiles wait for loads and share a CU better.  Fitted to heights of 4 to
// 64 on seventeen grids from 4096 x 64 to 8192 x 4096 and 16 x 65536; the
// choice is within 15% of the best of them (9% but for one), and no slower
// than strips of 64.  us per step, strips of 64, of about 1024 tiles whatever
// the type (the earlier rule) and these: FP64 65536 x 16 43, 63 and 43 (16 rows),
// 2048^2 140, 159 and 140 (64), 3000 x 2000 273, 261 and 208 (48); FP32 3000 x
// 2000 104, 108 and 96 (48); FP16 storage 3000^2 115, 112 and 92 (48).
struct RowCost {
    float alone, busy;
    int resident;
};
RowCost one_step_row(const lbac_ctx* h, int bx) {
    const int w = bx == 256 ? 0 : (bx == 128 ? 1 : 2);
    constexpr RowCost f32[] = {{0.58f, 0.39f, 5}, {0.70f, 0.17f, 10}, {0.74f, 0.09f, 16}};
    constexpr RowCost f64[] = {{0.f, 1.92f, 2}, {0.84f, 0.57f, 5}, {1.03f, 0.26f, 9}};
    constexpr RowCost f64_conv[] = {{0.f, 1.46f, 2}, {0.65f, 0.46f, 5}, {0.78f, 0.20f, 9}};
    if (h->p.precision != LBAC_F64) return f32[w];
    return h->p.model == LBAC_MODEL_CONVENTIONAL ? f64_conv[w] : f64[w];
}

// The default shape of the strip kernels, for grids the patch kernels leave to
// them, and an estimate of its time per step in microseconds (as PatchPlan's).
//
// Three steps per launch (FP32 storage): 224 columns and the strip height of
// the least estimate.  A strip costs its rows and the pipeline's 14, each 0.35
// us where every CU has one tile at most, 0.455 with two, 0.65 with three (the
// device's 768 at once), beyond that 0.62 per round of 768, a started round
// counting half; never less than the state read and written once at 4.76 TB/s.
// Measured with the chosen strips: 17.5 us per step at 1536^2 (24 rows), 25.4
// at 2048^2 (42; 30 rows 27.2, 48 27.3), 37.8 at 3001 x 2210 (42), 93.5 at
// 4096^2 and 341 at 8192^2 (42); the best of 72 shapes 16.5, 25.4, 36.6, 91.4.
//
// One step: the height of the least estimate by RowCost.
float default_strips(const lbac_ctx* h, bool three, int& variant, int& bx, int& strip_h) {
    const int nx = h->p.nx, ny = h->p.ny;
    const float mnodes = 1e-6f * (float)((int64_t)nx * ny);
    if (three) {
        variant = LBAC_KERNEL_FUSED3;
        bx = 224;
        const int64_t nbx = (nx + bx - 1) / bx;
        float best = 1e30f;
        for (int sh : {42, 36, 48, 30, 54, 24, 60, 18, 12}) {
            const float us = std::max(stepS_row(nbx * ((ny + sh - 1) / sh)) * (float)(sh + 14), 5.04f * mnodes);
            if (us < best) {
                best = us;
                strip_h = std::min(sh, ny);
            }
        }
        // with the closure: the marks, their list, and the marked patches of an interface across the grid
        return h->closure ? best + 15.f + 3.f * std::sqrt(mnodes) : best;
    }
    variant = LBAC_KERNEL_BLOCK;
    bx = default_bx(nx);
    const int64_t nbx = (nx + bx - 1) / bx;
    const RowCost rc = one_step_row(h, bx);
    const float mem = mnodes * 2.f * state_bytes(h) / 4.75f;
    float best = 1e30f;
    for (int sh : {64, 48, 32, 24, 16, 12, 8, 6, 4}) {
        const int64_t k = (nbx * ((ny + sh - 1) / sh) + 255) / 256;
        const float row = rc.alone * (float)((k + rc.resident - 1) / rc.resident) + rc.busy * (float)k;
        const float us = std::max(row * (float)(std::min(sh, ny) + 4), mem) + 3.f;
        if (us < best) {
            best = us;
            strip_h = std::min(sh, ny);
        }
    }
    return h->closure ? best + 17.f + 9.f * std::sqrt(mnodes) : best;
}

// Whether the closure's band is wide: the last look at it, or two-pass launch,
// marked more than three sixteenths of a grid on which that matters.  Two-pass
// launches are for thin bands: they compute a patch they mark again, with two
// to three times the band nodes of one step.  One-step patches over the whole
// grid, a single pass whose network takes no node twice, are the faster from
// about there on (the closure's 4096^2, us per step: a disk, 1% marked, 119 in
// two passes, 382 in patches, 293 in one-step strips; rows of drops, all
// marked, a third of the nodes in the band, 1969, 696 and 1579; every node in
// the band 3251, 1174 and 3387; three steps with the network inside the strips
// had taken 1156 and 2293 at the last two).  Below 2^19 nodes only a caller
// chooses two passes, and gains by them at any band (512^2, every node in it: 82
// us per step, with the network inside the strips 445).
constexpr int64_t kLookNodes = int64_t(1) << 19;
constexpr int kLookSteps = 256;  // a wide band is looked at again after so many steps (0.3 ms at 4096^2)
bool look_grid(const lbac_ctx* h) {
    return h->p.model == LBAC_MODEL_IMPROVED && (int64_t)h->p.nx * h->p.ny >= kLookNodes;
}
bool wide_band(const lbac_ctx* h) {
    return h->closure && look_grid(h) && (!h->shape_set || launch_steps_of(h) > 1) &&
           16 * (int64_t)__atomic_load_n(h->cl_seen, __ATOMIC_RELAXED) > 3 * (int64_t)h->p.nx * h->p.ny;
}

// The next launch of a run with `left` steps to go: the shape that was set,
// or, where nobody set one, the faster of the patch kernels and the strip
// kernels (made once per context: the estimates take as long as a launch's own
// host work); patches of one step where the closure's band is wide.  Results
// do not depend on the choice (16-bit storage takes one step per launch here,
// as its rounding depends on the steps of a launch).
Launch plan_launch(lbac_ctx* h, int64_t left) {
    const bool wide = wide_band(h);
    if (h->shape_set && !wide) {
        const int S = launch_steps_of(h);
        return {false, {}, S > 1 && left >= S ? S : 1, h->variant, h->bx, h->strip_h};
    }
    Launch& l = h->plans[wide ? 0 : std::min<int64_t>(left, kPlanSteps)];
    if (l.S == 0) {
        const bool three = !wide && h->p.precision == LBAC_F32 && left >= 3 && (!h->closure || look_grid(h));
        l.patch = false;
        l.S = three ? 3 : 1;
        const float strips = default_strips(h, three, l.variant, l.bx, l.strip_h);
        // (the closure with the conventional model: one-step launches only)
        if (!h->closure || h->p.model == LBAC_MODEL_IMPROVED) {
            const PatchPlan p = plan_patch(h, wide ? 1 : left);
            if (p.shape >= 0 && (wide || p.us < strips)) {
                l.patch = true;
                l.p = p;
                l.S = p.S;
            }
        }
    }
    if (h->shape_set) return l;
    h->variant = l.variant;
    h->bx = l.bx;
    h->strip_h = l.strip_h;
    return l;
}

hipError_t do_launch(const lbac_ctx* h, const Launch& l, int src, int32_t k) {
    if (l.patch) return launch_patch(h, src, k, l.p);
    return l.S > 1 ? launch_stepS(h, src, k, l.S) : launch_step(h, src, k);
}

void launch_set_time(const lbac_ctx* h, int64_t t) {
    hipLaunchKernelGGL(set_time_kernel, dim3(1), dim3(kTimeThreads), 0, h->stream, h->t_dev, h->tfac,
                       time_period(h->p), t);
}

// Looks at the closure's band: marks the patches of pop[src] as three steps of
// the strips do (into the other buffer, which the next launch overwrites), for
// *cl_seen.
hipError_t look(lbac_ctx* h, int src) {
    int variant, bx;
    StepArgs a = make_args(h, src, 0);
    default_strips(h, true, variant, bx, a.strip_h);
    h->cl_since = 0;
    return launch_look(h, a, bx);
}
hipError_t look_again(lbac_ctx* h, int src) {
    return wide_band(h) && h->cl_since >= kLookSteps ? look(h, src) : hipSuccess;
}

// Queues `n` steps from pop[src], several per launch where the plan allows and
// single steps for the rest, and the advance of the step counter.  The
// counter (and the table of time factors with it) moves after every
// kTimeFactors steps at the latest.  *flips gets the number of launches
// (buffer swaps).  look: look at a wide band again when it is time.
hipError_t launch_steps(lbac_ctx* h, int src, int64_t n, int64_t* flips, bool look) {
    int64_t f = 0;
    hipError_t e = hipSuccess;
    int32_t k = 0;  // steps queued since the counter moved
    auto advance = [&]() {
        hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(kTimeThreads), 0, h->stream, h->t_dev, h->tfac,
                           time_period(h->p), (int64_t)k);
        k = 0;
        return hipGetLastError();
    };
    for (int64_t left = n; left > 0 && e == hipSuccess;) {
        const Launch l = plan_launch(h, left);
        if (k + l.S > kTimeFactors) e = advance();
        if (look && k == 0 && e == hipSuccess) e = look_again(h, src ^ (int)(f & 1));
        if (e == hipSuccess) e = do_launch(h, l, src ^ (int)(f & 1), k);
        k += l.S;
        h->cl_since += l.S;
        left -= l.S;
        ++f;
    }
    if (e == hipSuccess && k > 0) e = advance();
    *flips = f;
    return e;
}

template <typename R, int ST>
hipError_t launch_aux_t(const lbac_ctx* h, int which, const StepArgs& a, double* out, const double* ref,
                        const double* phi0) {
    dim3 g2((a.nx + 255) / 256, a.ny);
    switch (which) {
    case 0:
        hipLaunchKernelGGL((init_kernel<R, ST>), g2, dim3(256), 0, h->stream, a, phi0);
        break;
    case 1:
        hipLaunchKernelGGL((phi_kernel<R, ST>), g2, dim3(256), 0, h->stream, a, out);
        break;
    default:
        hipLaunchKernelGGL((row_sums_kernel<R, ST>), dim3(a.ny), dim3(kRedThreads), 0, h->stream, a, ref,
                           static_cast<R*>(h->rows));
        hipLaunchKernelGGL((reduce_rows_kernel<R>), dim3(1), dim3(kRedThreads), 0, h->stream,
                           static_cast<const R*>(h->rows), a.ny, h->red5);
        break;
    }
    return hipGetLastError();
}

hipError_t launch_aux(const lbac_ctx* h, int which, const StepArgs& a, double* out, const double* ref,
                      const double* phi0) {
    switch (h->p.precision) {
    case LBAC_F64:
        return launch_aux_t<double, ST_PLAIN>(h, which, a, out, ref, phi0);
    case LBAC_F32:
        return launch_aux_t<float, ST_PLAIN>(h, which, a, out, ref, phi0);
    case LBAC_F32_F16STORE:
        return launch_aux_t<float, ST_F16>(h, which, a, out, ref, phi0);
    default:
        return launch_aux_t<float, ST_BF16>(h, which, a, out, ref, phi0);
    }
}

int validate(const lbac_params* p, std::string& why) {
    if (!p) return why = "params is NULL", LBAC_EINVAL;
    // at most 2^27 nodes: every padded plane then stays below 2 GiB, which the
    // kernels' 32-bit byte offsets and buffer ranges rely on
    if (p->nx < 1 || p->ny < 1 || p->nx > 65536 || p->ny > 65536 || (int64_t)p->nx * p->ny > (1ll << 27))
        return why = "grid size out of range (1 <= nx, ny <= 65536, nx * ny <= 2^27)", LBAC_EINVAL;
    if (!(p->tau > 0.5) || !std::isfinite(p->tau)) return why = "tau must exceed 1/2", LBAC_EINVAL;
    if (!(p->eps > 0.0) || !std::isfinite(p->eps)) return why = "eps must be positive", LBAC_EINVAL;
    if (!(p->delta >= 0.0) || !std::isfinite(p->delta)) return why = "delta must be >= 0", LBAC_EINVAL;
    if (p->vel_kind < LBAC_VEL_ZERO || p->vel_kind > LBAC_VEL_VORTEX_PAPER) return why = "bad vel_kind", LBAC_EINVAL;
    if ((p->vel_kind == LBAC_VEL_VORTEX || p->vel_kind == LBAC_VEL_VORTEX_PAPER) && !(p->period_T > 0.0))
        return why = "vortex needs period_T > 0", LBAC_EINVAL;
    if (p->precision < LBAC_F64 || p->precision > LBAC_F32_BF16STORE) return why = "bad precision", LBAC_EINVAL;
    if (p->model != LBAC_MODEL_IMPROVED && p->model != LBAC_MODEL_CONVENTIONAL) return why = "bad model", LBAC_EINVAL;
    if (p->alloc && (!p->alloc->alloc || !p->alloc->free)) return why = "allocator without alloc/free", LBAC_EINVAL;
    std::vector<double> tab;
    build_velocity(*p, tab);
    double ma = 0, mb = 0, mc = 0, md = 0;
    for (int i = 0; i < p->nx; ++i) {
        ma = std::max(ma, std::fabs(tab[i]));
        mb = std::max(mb, std::fabs(tab[p->nx + i]));
    }
    for (int j = 0; j < p->ny; ++j) {
        mc = std::max(mc, std::fabs(tab[2 * (size_t)p->nx + j]));
        md = std::max(md, std::fabs(tab[2 * (size_t)p->nx + p->ny + j]));
    }
    if (!std::isfinite(ma * mc + mb * md) || ma * mc + mb * md >= 1.0 / 3.0)
        return why = "velocity too large: max |u| + |v| must stay below 1/3", LBAC_EINVAL;
    return LBAC_OK;
}

}  // namespace

hipError_t lbac_host::launch_stepS_band(int S, StepArgs a, int bx, hipStream_t s) {
    return S == 3 ? launch_stepS_m<MODEL_IMPROVED, 3, ST_PLAIN, true>(a, bx, s)
                  : launch_stepS_m<MODEL_IMPROVED, 2, ST_PLAIN, true>(a, bx, s);
}

int lbac_host::create(const lbac_params* p, const double* phi0, bool phi0_on_device, lbac_ctx** out) {
    if (!out) return LBAC_EINVAL;
    *out = nullptr;
    std::string why;
    int rc = validate(p, why);
    if (rc != LBAC_OK) return rc;
    if (!phi0) return LBAC_EINVAL;
    const size_t n = (size_t)p->nx * p->ny;
    if (!phi0_on_device)
        for (size_t i = 0; i < n; ++i)
            if (!std::isfinite(phi0[i])) return LBAC_EINVAL;

    lbac_ctx* h = new (std::nothrow) lbac_ctx();
    if (!h) return LBAC_ENOMEM;
    h->p = *p;
    if (p->alloc) {
        h->alloc = *p->alloc;
        h->has_alloc = true;
    }
    h->p.alloc = nullptr;
    if (hipGetDevice(&h->device) != hipSuccess) {
        delete h;
        return LBAC_EDEVICE;
    }
    auto bail = [&](int code) {
        release(h);
        delete h;
        return code;
    };
    if (p->stream) {
        h->stream = (hipStream_t)p->stream;
    } else {
        if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess) return bail(LBAC_EDEVICE);
        h->own_stream = true;
    }
    h->storage = p->precision == LBAC_F64 || p->precision == LBAC_F32 ? ST_PLAIN
                 : (p->precision == LBAC_F32_F16STORE ? ST_F16 : ST_BF16);
    h->elem_bytes = p->precision == LBAC_F64 ? 8 : (p->precision == LBAC_F32 ? 4 : 2);
    h->nplanes = h->storage == ST_PLAIN ? 9 : 8;
    // rows are an odd multiple of 256 bytes apart: with a power-of-two row
    // pitch, rows processed at the same time by different strips and XCDs
    // land on the same HBM channels
    {
        const int unit = 256 / h->elem_bytes;
        h->pitch = (p->nx + unit - 1) / unit * unit;
        if ((h->pitch / unit) % 2 == 0) h->pitch += unit;
    }
    h->plane_stride = (int64_t)h->pitch * p->ny + kPlanePadBytes / h->elem_bytes;
    h->bx = h->unset_bx = default_bx(p->nx);
    h->strip_h = h->unset_strip_h = std::min(64, p->ny);
    const size_t pop_bytes = (size_t)h->plane_stride * h->nplanes * h->elem_bytes;
    const size_t phis_bytes = ((size_t)h->pitch * p->ny + 64) * sizeof(float);
    for (int i = 0; i < 2; ++i) {
        h->pop[i] = dev_alloc(h, pop_bytes);
        if (!h->pop[i]) return bail(LBAC_ENOMEM);
        if (h->storage != ST_PLAIN) {
            h->phis[i] = (float*)dev_alloc(h, phis_bytes);
            if (!h->phis[i]) return bail(LBAC_ENOMEM);
        }
    }
    std::vector<double> tab;
    build_velocity(h->p, tab);
    h->vtab = (double*)dev_alloc(h, tab.size() * sizeof(double));
    std::vector<float> tabf(tab.begin(), tab.end());
    for (int j = 0; j < p->ny; ++j)  // the row factors again, as pairs
        for (int c = 0; c < 2; ++c) tabf.push_back(tabf[2 * (size_t)p->nx + (size_t)c * p->ny + j]);
    h->vtabf = (float*)dev_alloc(h, tabf.size() * sizeof(float));
    h->t_dev = (int64_t*)dev_alloc(h, 64);
    h->tfac = (double*)dev_alloc(h, (kTimeFactors + 1) * sizeof(double));
    h->rows = dev_alloc(h, 10 * sizeof(double) * (size_t)p->ny);  // five compensated pairs per row
    h->red5 = (double*)dev_alloc(h, 64);
    h->dtmp = (double*)dev_alloc(h, n * sizeof(double));
    if (!h->vtab || !h->vtabf || !h->t_dev || !h->tfac || !h->rows || !h->red5 || !h->dtmp) return bail(LBAC_ENOMEM);
    if (hipHostMalloc((void**)&h->host5, 8 * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        h->host5 = nullptr;
        return bail(LBAC_ENOMEM);
    }
    h->cl_seen = reinterpret_cast<uint32_t*>(h->host5 + 7);
    *h->cl_seen = 0;
    if (hipMemcpyAsync(h->vtab, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice, h->stream) !=
            hipSuccess ||
        hipMemcpyAsync(h->vtabf, tabf.data(), tabf.size() * sizeof(float), hipMemcpyHostToDevice, h->stream) !=
            hipSuccess)
        return bail(LBAC_EDEVICE);
    const double* src0 = phi0;
    if (!phi0_on_device) {
        if (hipMemcpyAsync(h->dtmp, phi0, n * sizeof(double), hipMemcpyHostToDevice, h->stream) != hipSuccess)
            return bail(LBAC_EDEVICE);
        src0 = h->dtmp;
    }
    launch_set_time(h, 0);
    StepArgs a = make_args(h, 1, 0);  // dst = pop[0]
    if (launch_aux(h, 0, a, nullptr, nullptr, src0) != hipSuccess) return bail(LBAC_EDEVICE);
    if (hipStreamSynchronize(h->stream) != hipSuccess) return bail(LBAC_EDEVICE);
    h->cur = 0;
    h->t = 0;
    *out = h;
    return LBAC_OK;
}

void lbac_host::destroy(lbac_ctx* h) {
    if (!h) return;
    DeviceGuard g(h->device);
    release(h);
    delete h;
}

namespace {

int capture_graph(lbac_ctx* h, int parity) {
    const bool wide = wide_band(h);
    if (h->gexec[parity] && h->gexec_chunk[parity] == h->graph_chunk && h->gexec_wide[parity] == wide) return LBAC_OK;
    if (h->gexec[parity]) {
        (void)hipGraphExecDestroy(h->gexec[parity]);
        h->gexec[parity] = nullptr;
    }
    HIPCHK(h, hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal));
    int64_t flips = 0;
    hipError_t e = launch_steps(h, parity, h->graph_chunk, &flips, false);
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(h->stream, &g);
    if (e != hipSuccess || e2 != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return fail(h, LBAC_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e != hipSuccess ? e : e2));
    }
    hipGraphExec_t ge = nullptr;
    e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return fail(h, LBAC_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(e));
    h->gexec[parity] = ge;
    h->gexec_chunk[parity] = h->graph_chunk;
    h->gexec_wide[parity] = wide;
    h->gexec_flips[parity] = (int)(flips & 1);
    return LBAC_OK;
}

// Runs the row-sum and row-reduce kernels; results land in host5[0..4].
int reduce5(lbac_ctx* h, const double* ref_dev) {
    StepArgs a = make_args(h, h->cur, 0);
    HIPCHK(h, launch_aux(h, 2, a, nullptr, ref_dev, nullptr));
    HIPCHK(h, hipMemcpyAsync(h->host5, h->red5, 5 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(h, hipStreamSynchronize(h->stream));
    return LBAC_OK;
}

}  // namespace

extern "C" {

void lbac_default_params(lbac_params* p, int32_t nx, int32_t ny) {
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->nx = nx;
    p->ny = ny;
    p->eps = 1.0;
    p->tau = 0.8;
    p->delta = 1e-10;
    p->vel_kind = LBAC_VEL_VORTEX;
    p->U = 0.02;
    p->period_T = 2000.0;
    p->cx = 0.5 * nx;
    p->cy = 0.5 * ny;
    p->precision = LBAC_F64;
    p->model = LBAC_MODEL_IMPROVED;
}

int lbac_init(const lbac_params* p, const double* phi0, lbac_ctx** out) { return create(p, phi0, false, out); }

int lbac_init_device(const lbac_params* p, const double* phi0_device, lbac_ctx** out) {
    return create(p, phi0_device, true, out);
}

int lbac_free(lbac_ctx* h) {
    if (!h) return LBAC_OK;
    if (h->in_batch) return fail(h, LBAC_ESTATE, "context belongs to a batch; free the batch");
    destroy(h);
    return LBAC_OK;
}

int lbac_step(lbac_ctx* h, int64_t n) {
    if (!h) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    if (n < 0) return fail(h, LBAC_EINVAL, "negative step count");
    DeviceGuard g(h->device);
    if (!g.ok) return fail(h, LBAC_EDEVICE, "hipSetDevice failed");
    int64_t done = 0;
    if (h->graph_chunk > 0) {
        while (n - done >= h->graph_chunk) {
            int rc = capture_graph(h, h->cur);
            if (rc != LBAC_OK) return rc;
            HIPCHK(h, look_again(h, h->cur));
            HIPCHK(h, hipGraphLaunch(h->gexec[h->cur], h->stream));
            h->cl_since += h->graph_chunk;
            done += h->graph_chunk;
            h->t += h->graph_chunk;
            h->cur ^= h->gexec_flips[h->cur];  // parity of the chunk's launches
        }
    }
    const int64_t r = n - done;
    if (r > 0) {
        int64_t flips = 0;
        HIPCHK(h, launch_steps(h, h->cur, r, &flips, true));
        h->cur ^= (int)(flips & 1);
        h->t += r;
    }
    return LBAC_OK;
}

int lbac_phi_device(lbac_ctx* h, double* out_device) {
    if (!h || !out_device) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    DeviceGuard g(h->device);
    StepArgs a = make_args(h, h->cur, 0);
    HIPCHK(h, launch_aux(h, 1, a, out_device, nullptr, nullptr));
    return LBAC_OK;
}

int lbac_phi(lbac_ctx* h, double* out) {
    if (!h || !out) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    DeviceGuard g(h->device);
    int rc = lbac_phi_device(h, h->dtmp);
    if (rc != LBAC_OK) return rc;
    HIPCHK(h, hipMemcpyAsync(out, h->dtmp, sizeof(double) * (size_t)h->p.nx * h->p.ny, hipMemcpyDeviceToHost,
                             h->stream));
    HIPCHK(h, hipStreamSynchronize(h->stream));
    return LBAC_OK;
}

int lbac_mass(lbac_ctx* h, double* out) {
    if (!h || !out) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    DeviceGuard g(h->device);
    int rc = reduce5(h, nullptr);
    if (rc != LBAC_OK) return rc;
    *out = h->host5[0];
    if (!std::isfinite(*out)) return fail(h, LBAC_ENONFINITE, "mass is not finite");
    return LBAC_OK;
}

int lbac_shape_error(lbac_ctx* h, const double* ref, double* e1, double* e2) {
    if (!h || !ref) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    DeviceGuard g(h->device);
    const size_t n = (size_t)h->p.nx * h->p.ny;
    HIPCHK(h, hipMemcpyAsync(h->dtmp, ref, n * sizeof(double), hipMemcpyHostToDevice, h->stream));
    int rc = reduce5(h, h->dtmp);
    if (rc != LBAC_OK) return rc;
    const double* r = h->host5;
    const double v1 = r[1] / r[2], v2 = std::sqrt(r[3] / r[4]);
    if (e1) *e1 = v1;
    if (e2) *e2 = v2;
    if (!std::isfinite(v1) || !std::isfinite(v2)) return fail(h, LBAC_ENONFINITE, "shape error is not finite");
    return LBAC_OK;
}

int lbac_time(lbac_ctx* h, int64_t* t) {
    if (!h || !t) return LBAC_EINVAL;
    *t = h->t;
    return LBAC_OK;
}

int lbac_get_state(lbac_ctx* h, void* buf, size_t* bytes) {
    if (!h || !bytes) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    const size_t plane = (size_t)h->pitch * h->p.ny * h->elem_bytes;
    const size_t phib = h->storage == ST_PLAIN ? 0 : (size_t)h->pitch * h->p.ny * sizeof(float);
    const size_t need = 64 + plane * h->nplanes + phib;
    if (!buf) {
        *bytes = need;
        return LBAC_OK;
    }
    if (*bytes < need) return fail(h, LBAC_EINVAL, "state buffer too small");
    DeviceGuard g(h->device);
    unsigned char* b = (unsigned char*)buf;
    std::memset(b, 0, 64);
    uint64_t magic = kStateMagic;
    int32_t hdr[4] = {h->p.nx, h->p.ny, h->p.precision, h->nplanes};
    std::memcpy(b, &magic, 8);
    std::memcpy(b + 8, hdr, 16);
    std::memcpy(b + 24, &h->t, 8);
    unsigned char* d = b + 64;
    for (int q = 0; q < h->nplanes; ++q) {
        HIPCHK(h, hipMemcpyAsync(d + q * plane, (char*)h->pop[h->cur] + (size_t)q * h->plane_stride * h->elem_bytes,
                                 plane, hipMemcpyDeviceToHost, h->stream));
    }
    if (phib) HIPCHK(h, hipMemcpyAsync(d + h->nplanes * plane, h->phis[h->cur], phib, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(h, hipStreamSynchronize(h->stream));
    *bytes = need;
    return LBAC_OK;
}

int lbac_set_state(lbac_ctx* h, const void* buf, size_t bytes) {
    if (!h || !buf) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    const size_t plane = (size_t)h->pitch * h->p.ny * h->elem_bytes;
    const size_t phib = h->storage == ST_PLAIN ? 0 : (size_t)h->pitch * h->p.ny * sizeof(float);
    const size_t need = 64 + plane * h->nplanes + phib;
    if (bytes < need) return fail(h, LBAC_EINVAL, "state blob too small");
    const unsigned char* b = (const unsigned char*)buf;
    uint64_t magic;
    int32_t hdr[4];
    int64_t t;
    std::memcpy(&magic, b, 8);
    std::memcpy(hdr, b + 8, 16);
    std::memcpy(&t, b + 24, 8);
    if (magic != kStateMagic || hdr[0] != h->p.nx || hdr[1] != h->p.ny || hdr[2] != h->p.precision ||
        hdr[3] != h->nplanes || t < 0)
        return fail(h, LBAC_EINVAL, "state blob does not match this context");
    DeviceGuard g(h->device);
    const unsigned char* d = b + 64;
    for (int q = 0; q < h->nplanes; ++q)
        HIPCHK(h, hipMemcpyAsync((char*)h->pop[h->cur] + (size_t)q * h->plane_stride * h->elem_bytes, d + q * plane,
                                 plane, hipMemcpyHostToDevice, h->stream));
    if (phib) HIPCHK(h, hipMemcpyAsync(h->phis[h->cur], d + h->nplanes * plane, phib, hipMemcpyHostToDevice, h->stream));
    launch_set_time(h, t);
    HIPCHK(h, hipGetLastError());
    if (h->closure && look_grid(h)) HIPCHK(h, look(h, h->cur));
    HIPCHK(h, hipStreamSynchronize(h->stream));
    h->t = t;
    return LBAC_OK;
}

int lbac_set_launch(lbac_ctx* h, int32_t variant, int32_t bx, int32_t strip_h) {
    if (!h) return LBAC_EINVAL;
    if (variant < LBAC_KERNEL_BLOCK || variant > LBAC_KERNEL_FUSED3) return fail(h, LBAC_EINVAL, "unknown kernel variant");
    if ((variant == LBAC_KERNEL_FUSED2 || variant == LBAC_KERNEL_FUSED3) && h->p.precision == LBAC_F64)
        return fail(h, LBAC_EINVAL, "the multi-step variants need FP32 collision (LBAC_F32 or a 16-bit storage)");
    const int S = variant == LBAC_KERNEL_FUSED2 ? 2 : (variant == LBAC_KERNEL_FUSED3 ? 3 : 1);
    if (!(S == 1 ? one_step_bx(bx) : stepS_bx(bx)))
        return fail(h, LBAC_EINVAL, "bx must be 64, 128 or 256 (with the multi-step variants any multiple of 32 from "
                                    "64 to 320, or 240)");
    if (strip_h < 1) return fail(h, LBAC_EINVAL, "strip_h must be >= 1");
    h->variant = variant;
    h->bx = bx;
    h->strip_h = std::min(strip_h, h->p.ny);
    h->shape_set = true;
    drop_graphs(h);
    return LBAC_OK;
}

int lbac_get_launch(lbac_ctx* h, int32_t* variant, int32_t* bx, int32_t* strip_h) {
    if (!h) return LBAC_EINVAL;
    // a context whose shape nobody set reports the shape of creation, which
    // lbac_set_launch accepts
    if (variant) *variant = h->shape_set ? h->variant : h->unset_variant;
    if (bx) *bx = h->shape_set ? h->bx : h->unset_bx;
    if (strip_h) *strip_h = h->shape_set ? h->strip_h : h->unset_strip_h;
    return LBAC_OK;
}

int lbac_autotune(lbac_ctx* h, int32_t steps, double* us_per_step) {
    if (!h || steps < 1) return LBAC_EINVAL;
    if (h->failed) return fail(h, LBAC_ESTATE, "the batch run of this instance timed out; its state is undefined");
    DeviceGuard g(h->device);
    const int bxs[10] = {64, 96, 128, 160, 192, 224, 240, 256, 288, 320};
    // strip heights: multiples of 8 up to 256 and powers of two up to 512 (the
    // count of tiles against the workgroups resident at once decides how full
    // the last round of tiles is, so heights between the powers of two can
    // win), and ny split into k equal strips (so that a grid whose tiles all
    // fit on the device at once marches long strips in step)
    std::vector<int> hs;
    for (int sh = 8; sh <= 256; sh += 8) hs.push_back(std::min(sh, h->p.ny));
    hs.push_back(std::min(512, h->p.ny));
    for (int k = 1; k <= 32; ++k) hs.push_back((h->p.ny + k - 1) / k);
    std::sort(hs.begin(), hs.end());
    hs.erase(std::unique(hs.begin(), hs.end()), hs.end());
    hipEvent_t e0, e1;
    HIPCHK(h, hipEventCreate(&e0));
    HIPCHK(h, hipEventCreate(&e1));
    const int keep_bx = h->bx, keep_h = h->strip_h, keep_v = h->variant;
    const bool keep_set = h->shape_set;
    int best_bx = keep_bx, best_h = keep_h, best_v = keep_v;
    float best = 1e30f;
    hipError_t e = hipSuccess;
    // mean ms per step of one(), which takes S steps per launch
    auto time_ms = [&](auto&& one, int S) {
        for (int w = 0; w < 2 && e == hipSuccess; ++w) e = one();
        if (e == hipSuccess) e = hipEventRecord(e0, h->stream);
        for (int s = 0; s < steps && e == hipSuccess; ++s) e = one();
        if (e == hipSuccess) e = hipEventRecord(e1, h->stream);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        return ms / (float)S;
    };
    const int last_var = stepS_allowed(h) ? LBAC_KERNEL_FUSED3 : LBAC_KERNEL_BLOCK_DEEP;
    for (int var = LBAC_KERNEL_BLOCK; var <= last_var && e == hipSuccess; ++var)
    for (int bx : bxs) {
        const int S = var == LBAC_KERNEL_FUSED2 ? 2 : (var == LBAC_KERNEL_FUSED3 ? 3 : 1);
        if (bx > 64 && bx / 2 >= h->p.nx) continue;
        if (S == 1 ? !one_step_bx(bx) : !stepS_bx(bx)) continue;
        int last = 0;
        for (int sh : hs) {
            // (heights that come to the same launch are timed once)
            const int run = S == 1 ? sh : stepS_height(h->p.nx, h->p.ny, bx, sh, S == 2 ? TileSRows<2>::kPeriod : TileSRows<3>::kPeriod);
            if (run == last) continue;
            last = run;
            h->variant = var;
            h->bx = bx;
            h->strip_h = std::min(sh, h->p.ny);
            // repeated launches from pop[cur] into the scratch buffer: the state
            // is untouched; an S-step launch counts as S steps
            const int S = launch_steps_of(h);
            auto one = [&]() { return S > 1 ? launch_stepS(h, h->cur, 0, S) : launch_step(h, h->cur, 0); };
            const float ms = time_ms(one, S);
            if (e != hipSuccess) break;
            if (ms < best) {
                best = ms;
                best_v = var;
                best_bx = bx;
                best_h = h->strip_h;
            }
        }
        if (e != hipSuccess) break;
    }
    // The launches a context makes whose shape nobody set (the patch kernels on
    // small grids).  Where they win, the context keeps making them, and
    // lbac_get_launch gives the fastest of the shapes that can be set, for a
    // caller that sets it on another context.
    bool set = true;
    if (e == hipSuccess) {
        h->shape_set = false;
        const Launch l = plan_launch(h, INT32_MAX);
        const float ms = time_ms([&]() { return do_launch(h, l, h->cur, 0); }, l.S);
        if (e == hipSuccess && ms < best) {
            best = ms;
            set = false;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    h->shape_set = set;
    h->variant = best_v;
    h->bx = best_bx;
    h->strip_h = best_h;
    if (!set) {
        h->unset_variant = best_v;
        h->unset_bx = best_bx;
        h->unset_strip_h = best_h;
    }
    drop_graphs(h);
    if (e != hipSuccess) {
        h->shape_set = keep_set;
        h->variant = keep_v;
        h->bx = keep_bx;
        h->strip_h = keep_h;
        return fail(h, LBAC_EDEVICE, std::string("autotune: ") + hipGetErrorString(e));
    }
    if (us_per_step) *us_per_step = 1000.0 * best / steps;
    return LBAC_OK;
}

int lbac_set_graph_chunk(lbac_ctx* h, int32_t chunk) {
    if (!h) return LBAC_EINVAL;
    if (chunk < 0 || (chunk & 1)) return fail(h, LBAC_EINVAL, "graph chunk must be an even number >= 0");
    h->graph_chunk = chunk;
    drop_graphs(h);
    return LBAC_OK;
}

int lbac_set_closure(lbac_ctx* h, const float* params, float theta) {
    if (!h) return LBAC_EINVAL;
    DeviceGuard g(h->device);
    if (!params) {
        h->closure = false;
        drop_plans(h);
        return LBAC_OK;
    }
    if (h->p.precision != LBAC_F32) return fail(h, LBAC_EINVAL, "the learned closure runs with LBAC_F32 only");
    if (h->in_batch) return fail(h, LBAC_EINVAL, "the learned closure is not available for batch instances");
    if (!(theta >= 0.f) || !(theta < 0.5f)) return fail(h, LBAC_EINVAL, "theta must lie in [0, 0.5)");
    for (int i = 0; i < LBAC_MLP_NPARAM; ++i)
        if (!std::isfinite(params[i])) return fail(h, LBAC_EINVAL, "non-finite closure parameter");
    if (!h->cl_param) {
        h->cl_param = (float*)dev_alloc(h, sizeof(float) * LBAC_MLP_NPARAM);
        h->cl_w = (uint16_t*)dev_alloc(h, sizeof(uint16_t) * kClWN);
        h->cl_b = (float*)dev_alloc(h, sizeof(float) * kClBN);
        h->cl_words = (h->p.nx + 63) / 64;
        h->cl_mask = (uint64_t*)dev_alloc(h, sizeof(uint64_t) * (size_t)h->cl_words * h->p.ny);
        h->cl_list = (int32_t*)dev_alloc(h, sizeof(int32_t) * (size_t)h->p.nx * h->p.ny);
        h->cl_count = (uint32_t*)dev_alloc(h, 256);
        const size_t marks = (mark_count(h->p.nx, h->p.ny) + 7) / 8 * 8;
        h->cl_flags = (uint8_t*)dev_alloc(h, marks);
        if (!h->cl_param || !h->cl_w || !h->cl_b || !h->cl_mask || !h->cl_list || !h->cl_count || !h->cl_flags) {
            free_closure(h);  // a later call starts over, rather than run without the missing ones
            return fail(h, LBAC_ENOMEM, "closure buffers");
        }
        const hipError_t e = hipMemsetAsync(h->cl_flags, 0, marks, h->stream);
        if (e != hipSuccess) free_closure(h);
        HIPCHK(h, e);
    }
    HIPCHK(h, hipMemcpyAsync(h->cl_param, params, sizeof(float) * LBAC_MLP_NPARAM, hipMemcpyHostToDevice, h->stream));
    hipLaunchKernelGGL(closure_pack_kernel, dim3((64 * 64 + 255) / 256), dim3(256), 0, h->stream, h->cl_param, h->cl_w,
                       h->cl_b);
    HIPCHK(h, hipGetLastError());
    h->closure = true;
    h->cl_theta = theta;
    drop_plans(h);
    hipError_t e = look_grid(h) ? look(h, h->cur) : hipSuccess;
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) h->closure = false;
    HIPCHK(h, e);
    return LBAC_OK;
}

int lbac_copy_ceiling(lbac_ctx* h, int32_t launches, double* us_per_launch) {
    if (!h || launches < 1 || !us_per_launch) return LBAC_EINVAL;
    DeviceGuard g(h->device);
    // copies pop[cur] into the other buffer, which the next step overwrites anyway
    StepArgs a = make_args(h, h->cur, 0);
    a.n_xcd = kXcds;
    hipEvent_t e0, e1;
    HIPCHK(h, hipEventCreate(&e0));
    HIPCHK(h, hipEventCreate(&e1));
    hipError_t e = hipSuccess;
    float best = 1e30f;
    for (int sh : {8, 16, 32, 64}) {
        a.strip_h = std::min(sh, a.ny);
        a.nby = (a.ny + a.strip_h - 1) / a.strip_h;
        const dim3 grid(((a.nx + 255) / 256) * a.nby), block(256);
        auto launch = [&]() {
            // plain storage: 9 planes; shifted storage: 8 16-bit planes plus the FP32 phi* plane
            if (h->elem_bytes == 8)
                hipLaunchKernelGGL((pattern_copy_kernel<uint64_t, 9>), grid, block, 0, h->stream, a);
            else if (h->elem_bytes == 4)
                hipLaunchKernelGGL((pattern_copy_kernel<uint32_t, 9>), grid, block, 0, h->stream, a);
            else
                hipLaunchKernelGGL((pattern_copy_kernel<uint16_t, 8>), grid, block, 0, h->stream, a);
            return hipGetLastError();
        };
        e = launch();
        if (e == hipSuccess) e = hipEventRecord(e0, h->stream);
        for (int k = 0; k < launches && e == hipSuccess; ++k) e = launch();
        if (e == hipSuccess) e = hipEventRecord(e1, h->stream);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess) break;
        best = std::min(best, ms);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return fail(h, LBAC_EDEVICE, std::string("copy ceiling: ") + hipGetErrorString(e));
    *us_per_launch = 1000.0 * best / launches;
    return LBAC_OK;
}

int lbac_bytes_per_node(lbac_ctx* h, double* bytes) {
    if (!h || !bytes) return LBAC_EINVAL;
    // read and write of every stored value once per launch
    *bytes = 2.0 * (h->nplanes * h->elem_bytes + (h->storage == ST_PLAIN ? 0 : 4));
    return LBAC_OK;
}

int lbac_steps_per_launch(lbac_ctx* h, int32_t* steps) {
    if (!h || !steps) return LBAC_EINVAL;
    *steps = h->shape_set ? launch_steps_of(h) : plan_launch(h, INT32_MAX).S;
    return LBAC_OK;
}

void* lbac_stream(lbac_ctx* h) { return h ? (void*)h->stream : nullptr; }

const char* lbac_strerror(int code) {
    switch (code) {
    case LBAC_OK:
        return "ok";
    case LBAC_EINVAL:
        return "invalid argument";
    case LBAC_ENOMEM:
        return "out of memory";
    case LBAC_EDEVICE:
        return "device error";
    case LBAC_ENONFINITE:
        return "non-finite result";
    case LBAC_ESTATE:
        return "invalid state";
    default:
        return "unknown status";
    }
}

const char* lbac_last_error(lbac_ctx* h) { return h ? h->err.c_str() : "no context"; }

}  // extern "C"
