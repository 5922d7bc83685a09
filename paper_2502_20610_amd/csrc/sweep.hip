// Sweeps of one grid: kernels and launches (the tile itself is in sweep_tile.h,
// the plan of a pass in sweep_plan.cpp).
#include <math.h>

#include <algorithm>
#include <new>

#include "sweep_tile.h"

namespace fdtd {
namespace {

template <int T, int R, int W, int MODE, bool WHOLE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void sweep_kernel(
    const SweepArgs A)
{
    __shared__ Lds<T, R, W, MODE> S;
    int xcd, slot, per_xcd;
    if (!place(A, xcd, slot, per_xcd)) return;  // whole block
    sweep_tile<T, R, W, MODE, WHOLE, kUpdate>(A, HookArgs{}, S, xcd, slot, per_xcd);
}
#define V(T, R, W, M) sweep_kernel<T, R, W, M, false>,
#define VW(T, W, M) sweep_kernel<T, 1, W, M, true>,
void (*const kKernels[])(const SweepArgs) = {FDTD_SWEEP_SHAPES(V, VW)};
#undef V
#undef VW

}  // namespace

int sweep::mode_of(const fdtd_ctx* c)
{
    const bool tab = c->use_mat && c->mat_id8 && c->ntab8 > 0;
    return c->ca[0] ? (tab ? kLossyTable : kLossy) : (tab ? kTable : kArrays);
}

struct SweepState {
    int cus = 0;
    int mode = -1;
    Pass pass[kMaxT + 1];    // the plan of a pass of T steps, for `mode`
    bool fused = false;      // a pass of one step as a launch of the fused step
    int hooked_mode = -1;
    Pass forward[kMaxT + 1], reverse[kMaxT + 1];  // of the adjoint's passes
    unsigned* pace = nullptr;
    int pace_words = 0;  // of one of the two alternating halves: enough for any mode
    int turn = 0;
    int steps = 0, blocks = 0, tiles = 0;  // of the last call's longest pass
};

namespace {

// (the two halves of the progress marks are cleared here once; after that
// every pass clears the half of the next one)
__global__ void clear_words(unsigned* p, int n)
{
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) p[q] = 0u;
}

int state(fdtd_ctx* ctx)
{
    if (!ctx->sweep) {
        ctx->sweep = new (std::nothrow) SweepState();
        if (!ctx->sweep) return fail(ctx, FDTD_ENOMEM, "sweep: host allocation failed");
    }
    SweepState* S = ctx->sweep;
    if (S->cus == 0) {
        int v = 0;
        hipError_t e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, ctx->device);
        if (e != hipSuccess) return hip_fail(ctx, e, "sweep: device attribute");
        S->cus = std::max(1, v);
    }
    return FDTD_OK;
}

// The passes for the coefficients the context has now.
int plan_passes(fdtd_ctx* ctx)
{
    int rc = state(ctx);
    if (rc) return rc;
    SweepState* S = ctx->sweep;
    const int mode = mode_of(ctx);
    const int N[3] = {ctx->nx, ctx->ny, ctx->nz};
    if (S->mode == mode) return FDTD_OK;
    for (int T = 1; T <= kMaxT; ++T) S->pass[T] = plan_pass(N, mode, kUpdate, T, S->cus);
    // a pass of one step is the fused step's launch where that is the faster
    // (256^3 arrays 245 / 345 us, 128^3 conductive arrays 32 / 52)
    S->fused = one_step_us(N, ctx->ca[0] != nullptr) < alone_us(S->pass[1], N, S->cus);
    S->mode = mode;
    return FDTD_OK;
}

// (its blocks read every source on every plane)
bool one_step_launch(const fdtd_ctx* ctx) { return ctx->sweep->fused && ctx->dev_sources_n <= 8; }

int plan(fdtd_ctx* ctx)
{
    int rc = plan_passes(ctx);
    if (rc) return rc;
    SweepState* S = ctx->sweep;
    const int N[3] = {ctx->nx, ctx->ny, ctx->nz};
    // Blocks are kept in step where the state is past 1 GiB: 512^3, T = 5,
    // 225 -> 256 G cell updates/s, 1024 x 1024 x 512 255 -> 269; at 256^3,
    // one round of blocks, 202 against 205.  The marks are allocated once, for
    // whatever coefficients the context is given later.
    if (!S->pace && 24.0 * (double)ctx->ncell > 1.0737e9 && !stream_capturing(ctx)) {
        const long long words = most_mark_words(N, S->cus);
        if (words > 0 && words < (1 << 24)) {
            if (hipMalloc(&S->pace, 2 * (size_t)words * sizeof(unsigned)) != hipSuccess) {
                (void)hipGetLastError();
                S->pace = nullptr;  // (only a matter of speed)
            } else {
                S->pace_words = (int)words;
                hipLaunchKernelGGL(clear_words, dim3(64), dim3(256), 0, ctx->stream, S->pace, 2 * (int)words);
            }
        }
    }
    return FDTD_OK;
}

// Number of passes that advance n steps (0: none fits): as few as the cheapest
// split takes, lengths within one of each other, the longer ones first; an
// even number when `even`.
int64_t split(const Pass* pass, int64_t n, bool even)
{
    double best = 1e300;
    int64_t bp = 0;
    for (int T = 1; T <= kMaxT; ++T) {
        if (!pass[T].s) continue;
        int64_t p = (n + T - 1) / T;
        if (even && (p & 1)) ++p;
        if (p > n) continue;
        const int t = (int)(n / p);
        const int64_t longer = n % p;
        if (t + (longer ? 1 : 0) > kMaxT || !pass[t].s || (longer && !pass[t + 1].s)) continue;
        const double us = (double)(p - longer) * pass[t].us + (longer ? (double)longer * pass[t + 1].us : 0.0);
        if (us < best) {
            best = us;
            bp = p;
        }
    }
    return bp;
}

unsigned blocks_of(const Pass& P) { return (unsigned)((P.ntiles + kXCD - 1) / kXCD * kXCD); }

void launch_pass(const fdtd_ctx* ctx, const Pass& P, SweepArgs& A, const HookArgs* K = nullptr)
{
    A.gz = P.gz;
    A.gy = P.gy;
    A.xchunk = P.xchunk;
    A.ntiles = (int)P.ntiles;
    if (K)
        hipLaunchKernelGGL(hooked_kernel_of(P.index), dim3(blocks_of(P)), dim3(64 * P.s->W), 0, ctx->stream, A, *K);
    else
        hipLaunchKernelGGL(kKernels[P.index], dim3(blocks_of(P)), dim3(64 * P.s->W), 0, ctx->stream, A);
}

}  // namespace

SweepArgs sweep::base_args(const fdtd_ctx* ctx)
{
    SweepArgs A{};
    A.cH = ctx->cH;
    A.nx = ctx->nx;
    A.ny = ctx->ny;
    A.nz = ctx->nz;
    for (int c = 0; c < 3; ++c) {
        A.cE[c] = ctx->coef[c];
        A.ca[c] = ctx->ca[c];
    }
    return A;
}

// A plane must fit a buffer descriptor with room for the dropped offset, and
// many sources need their index of planes.
bool sweep_supported(const fdtd_ctx* ctx)
{
    if (ctx->dev_sources_n > kListedSources && ctx->nx > kMaxIndexedPlanes) return false;
    // (FP16 storage: with the coefficients' exact values in a table)
    return (ctx->storage == FDTD_FP32 || mode_of(ctx) == kTable) && (uint64_t)ctx->ny * (uint64_t)ctx->nz * 4u < (uint64_t)kDropped;
}

bool sweep_ready(fdtd_ctx* ctx)
{
    if (!ctx->use_sweeps || !sweep_supported(ctx)) return false;
    const bool half = ctx->storage == FDTD_FP16_STORAGE;
    bool have = true;
    for (int c = 0; c < 6; ++c) have = have && ctx->alt[c] && (!half || ctx->wide[c]);
    if (have) return true;
    // A scheme that can do without the second field set takes it only where
    // three quarters of the free memory stay free.  FP16 storage, which is there
    // to hold larger grids, takes its two FP32 sets (48 B per cell next to 23 of
    // its own) from a sixteenth: on an empty device up to 370 M cells.
    if (stream_capturing(ctx)) return false;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (half ? 48.0 * (double)ctx->ncell > 0.0625 * (double)free_b : 24.0 * (double)ctx->ncell > 0.25 * (double)free_b)
        return false;
    if (sweep_prepare(ctx) == FDTD_OK) return true;
    sweep_give_back(ctx);
    return false;
}

void sweep_give_back(fdtd_ctx* ctx)
{
    (void)hipStreamSynchronize(ctx->stream);
    for (int c = 0; c < 6; ++c) {
        if (ctx->alt[c]) (void)hipFree(ctx->alt[c]);
        if (ctx->wide[c]) (void)hipFree(ctx->wide[c]);
        ctx->alt[c] = ctx->wide[c] = nullptr;
    }
}

int sweep_prepare(fdtd_ctx* ctx)
{
    const size_t bytes = (size_t)ctx->ncell * sizeof(float);
    for (int c = 0; c < 6; ++c)
        for (float** p : {&ctx->alt[c], &ctx->wide[c]}) {
            if (*p || (p == &ctx->wide[c] && ctx->storage == FDTD_FP32)) continue;
            hipError_t e = hipMalloc(p, bytes);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                *p = nullptr;
                return fail(ctx, FDTD_ENOMEM, "the second field set does not fit");
            }
        }
    return plan(ctx);
}

namespace {

// n steps from `now` into `other` and back; the pointers trade places with
// every pass, so `now` holds the state in the end.
int run(fdtd_ctx* ctx, float* now[6], float* other[6], int64_t n, int kernel, bool even)
{
    SweepState* S = ctx->sweep;
    const int64_t passes = split(S->pass, n, even && n > 1);
    if (passes == 0) return fail(ctx, FDTD_EUNSUPPORTED, "sweep: no pass fits this call");
    SweepArgs A = base_args(ctx);
    A.id = ctx->mat_id8;
    A.tab = ctx->mat_tab8;
    A.ntab = ctx->ntab8;
    A.src = ctx->dev_sources;
    A.nsrc = ctx->dev_sources_n;
    const int t0 = (int)(n / passes);
    const int64_t longer = n % passes;
    {
        const Pass& P = S->pass[t0 + (longer ? 1 : 0)];
        S->steps = t0 + (longer ? 1 : 0);
        S->tiles = (int)P.ntiles;
        S->blocks = (int)blocks_of(P);
    }
    for (int64_t p = 0; p < passes; ++p) {
        const int T = t0 + (p < longer ? 1 : 0);
        const Pass& P = S->pass[T];
        for (int c = 0; c < 6; ++c) {
            A.in[c] = now[c];
            A.out[c] = other[c];
        }
        A.step = ctx->step_count;
        const bool one = T == 1 && ctx->storage == FDTD_FP32 && one_step_launch(ctx);
        const bool paced = S->pace && !one && mark_words(P) <= S->pace_words;
        A.pace = paced ? S->pace + (size_t)S->turn * S->pace_words : nullptr;
        A.pace_next = paced ? S->pace + (size_t)(S->turn ^ 1) * S->pace_words : nullptr;
        A.pace_words = S->pace_words;
        if (paced) S->turn ^= 1;
        PendingTiming t;
        timing_begin(ctx, kernel, &t);
        int rc = FDTD_OK;
        if (one)
            rc = fused_one_step(ctx, now, other);
        else
            launch_pass(ctx, P, A);
        timing_end(ctx, &t);
        if (rc) return rc;
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "launch(sweep)");
        for (int c = 0; c < 6; ++c) std::swap(now[c], other[c]);
        ctx->step_count += T;
    }
    return FDTD_OK;
}

}  // namespace

bool sweeps_too_thin(const fdtd_ctx* ctx, int64_t n)
{
    bool periodic = false;
    for (int d = 0; d < 3; ++d) periodic = periodic || ctx->cfg.bc[d] == FDTD_BC_PERIODIC;
    const bool half = ctx->storage == FDTD_FP16_STORAGE;
    // (FP16 storage converts the state both ways in a dozen launches of their
    // own: two steps on periodic 32^3 72 us persistent, 83 swept; closed 128 / 81)
    if (half && periodic && n == 2) return true;
    const int N[3] = {ctx->nx, ctx->ny, ctx->nz};
    return thin_for_sweeps(N, periodic, mode_of(ctx), half, n);
}

bool sweeps_beat_in_place(fdtd_ctx* ctx, int64_t n)
{
    if (plan_passes(ctx) != FDTD_OK) return false;
    const SweepState* S = ctx->sweep;
    const int N[3] = {ctx->nx, ctx->ny, ctx->nz};
    const int64_t passes = split(S->pass, n, n > 1);
    if (passes == 0) return false;
    auto pass_us = [&](int T) {
        const double us = alone_us(S->pass[T], N, S->cus);
        return T == 1 && one_step_launch(ctx) ? std::min(us, one_step_us(N, ctx->ca[0] != nullptr)) : us;
    };
    const int t = (int)(n / passes);
    const int64_t longer = n % passes;
    const double us = (double)(passes - longer) * pass_us(t) + (longer ? (double)longer * pass_us(t + 1) : 0.0);
    return us <= 1.1 * in_place_us(N, ctx->ca[0] != nullptr, n);
}

int sweep_steps(fdtd_ctx* ctx, int64_t n, int kernel, bool even)
{
    int rc = sweep_prepare(ctx);
    if (rc) return rc;
    return run(ctx, ctx->field, ctx->alt, n, kernel, even);
}

// The binary16 arrays are read and written once per band, as the persistent
// launch does; the conversions move 72 B per cell and band.
int sweep_half_steps(fdtd_ctx* ctx, int64_t n, int64_t band, int kernel)
{
    int rc = sweep_prepare(ctx);
    if (rc) return rc;
    for (int64_t done = 0; done < n; done += band) {
        const int64_t k = std::min(band, n - done);
        if ((rc = widen_fields(ctx, ctx->wide)) || (rc = run(ctx, ctx->wide, ctx->alt, k, kernel, false)) ||
            (rc = narrow_fields(ctx, ctx->wide)))
            return rc;
    }
    return FDTD_OK;
}

bool sweep_hooked_ready(fdtd_ctx* ctx)
{
    if (!sweep_ready(ctx) || state(ctx) != FDTD_OK) return false;
    SweepState* S = ctx->sweep;
    const int mode = ctx->ca[0] ? kLossy : kArrays;
    if (S->hooked_mode != mode) {
        const int N[3] = {ctx->nx, ctx->ny, ctx->nz};
        for (int T = 1; T <= kMaxT; ++T) {
            S->forward[T] = plan_pass(N, mode, kForward, T, S->cus);
            S->reverse[T] = plan_pass(N, mode, kReverse, T, S->cus);
        }
        S->hooked_mode = mode;
    }
    return true;
}

namespace {

HookArgs hook_args(const SweepHooks& h)
{
    HookArgs K{};
    for (int a = 0; a < 3; ++a) {
        K.dlo[a] = h.des_lo[a];
        K.dn[a] = h.des_n[a];
        K.mlo[a] = h.mon_lo[a];
        K.mn[a] = h.mon_n[a];
    }
    K.comp = h.comp;
    K.F = h.F;
    return K;
}

void hook_phase(HookArgs* K, const SweepHooks& h, int l, int64_t n)
{
    const double th = h.omega * (double)n * h.dt;
    K->cr[l] = cos(th);
    K->ci[l] = -sin(th);
}

}  // namespace

int sweep_forward(fdtd_ctx* ctx, const SweepHooks& h, int64_t n0, int64_t n, bool record, int64_t first)
{
    if (n == 0) return FDTD_OK;
    SweepState* S = ctx->sweep;
    const int64_t passes = split(S->forward, n, false);
    if (passes == 0) return fail(ctx, FDTD_EUNSUPPORTED, "adjoint: no pass fits this run");
    SweepArgs A = base_args(ctx);
    A.src = ctx->dev_sources;
    A.nsrc = ctx->dev_sources_n;
    HookArgs K = hook_args(h);
    K.stride = (ctx->ca[0] ? 6 : 3) * (long long)h.des_n[0] * h.des_n[1] * h.des_n[2];
    int64_t done = 0;
    for (int64_t p = 0; p < passes; ++p) {
        const int T = (int)(n / passes) + (p < n % passes ? 1 : 0);
        for (int l = 0; l < T; ++l) hook_phase(&K, h, l, n0 + done + l + 1);
        K.hist = record ? h.hist + (first + done) * K.stride : nullptr;
        for (int c = 0; c < 6; ++c) {
            A.in[c] = ctx->field[c];
            A.out[c] = ctx->alt[c];
        }
        A.step = ctx->step_count;
        PendingTiming t;
        timing_begin(ctx, FDTD_KERNEL_PLAIN_FUSED, &t);
        launch_pass(ctx, S->forward[T], A, &K);
        timing_end(ctx, &t);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "launch(adjoint forward sweep)");
        for (int c = 0; c < 6; ++c) std::swap(ctx->field[c], ctx->alt[c]);
        ctx->step_count += T;
        done += T;
    }
    return FDTD_OK;
}

int sweep_reverse(fdtd_ctx* ctx, const SweepHooks& h, float* lam[6], float* lam2[6], int64_t n0, int64_t n)
{
    SweepState* S = ctx->sweep;
    const int64_t passes = split(S->reverse, n, false);
    if (passes == 0) return fail(ctx, FDTD_EUNSUPPORTED, "adjoint: no pass fits this run");
    SweepArgs A = base_args(ctx);
    HookArgs K = hook_args(h);
    K.stride = 3 * (long long)h.des_n[0] * h.des_n[1] * h.des_n[2];
    int64_t left = n;
    for (int64_t p = 0; p < passes; ++p) {
        const int T = (int)(n / passes) + (p < n % passes ? 1 : 0);
        for (int l = 0; l < T; ++l) hook_phase(&K, h, l, n0 + left - l);
        K.hist = h.back + (n - left) * K.stride;
        for (int c = 0; c < 6; ++c) {
            A.in[c] = lam[c];
            A.out[c] = lam2[c];
        }
        launch_pass(ctx, S->reverse[T], A, &K);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "launch(adjoint reverse sweep)");
        for (int c = 0; c < 6; ++c) std::swap(lam[c], lam2[c]);
        left -= T;
    }
    return FDTD_OK;
}

void sweep_shape(const fdtd_ctx* ctx, int* steps, int* blocks, int* tiles)
{
    *steps = ctx->sweep->steps;
    *blocks = ctx->sweep->blocks;
    *tiles = ctx->sweep->tiles;
}

void sweep_release(fdtd_ctx* ctx)
{
    if (!ctx->sweep) return;
    if (ctx->sweep->pace) (void)hipFree(ctx->sweep->pace);
    delete ctx->sweep;
    ctx->sweep = nullptr;
}

}  // namespace fdtd
