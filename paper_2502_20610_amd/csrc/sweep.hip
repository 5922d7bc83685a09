// Sweeps of one grid: kernels, the plan of a pass, launches (the tile itself is
// in sweep_tile.h).
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
#define V(T, R, W, M) {T, R, W, M, false, kUpdate, sweep_kernel<T, R, W, M, false>, nullptr}
#define VW(T, W, M) {T, 1, W, M, true, kUpdate, sweep_kernel<T, 1, W, M, true>, nullptr}
#define VW4(W, M) VW(1, W, M), VW(2, W, M), VW(3, W, M), VW(4, W, M)
#define V2(R, W, M) V(1, R, W, M), V(2, R, W, M)
#define V3(R, W, M) V2(R, W, M), V(3, R, W, M)
#define V4(R, W, M) V3(R, W, M), V(4, R, W, M)
#define V5(R, W, M) V4(R, W, M), V(5, R, W, M)
const Variant kVariants[] = {
    V5(3, 12, kTable),      V4(2, 16, kTable),     V4(1, 16, kTable),
    V4(3, 12, kLossyTable), V5(2, 16, kLossyTable), V4(1, 16, kLossyTable),
    V4(4, 8, kArrays),      V3(2, 16, kArrays), V4(1, 16, kArrays),
    V3(3, 8, kLossy),       V2(2, 16, kLossy), V4(1, 16, kLossy),
    VW4(16, kTable),        VW4(16, kArrays),    VW4(16, kLossyTable), VW4(16, kLossy),
};
#undef V
#undef VW
#undef VW4
#undef V2
#undef V3
#undef V4
#undef V5

}  // namespace

int sweep::mode_of(const fdtd_ctx* c)
{
    const bool tab = c->use_mat && c->mat_id8 && c->ntab8 > 0;
    return c->ca[0] ? (tab ? kLossyTable : kLossy) : (tab ? kTable : kArrays);
}

namespace {
int in_bytes(int mode) { return 24 + (mode == kArrays ? 12 : mode == kLossy ? 24 : 1); }
}  // namespace

bool sweep::fits_cache(int mode, double cells) { return (24.0 + in_bytes(mode)) * cells <= 256e6; }

double sweep::round_us(int mode, int rows, int T, int xc, bool cached)
{
    const double level = 0.11 + 0.29 * rows / 16.0;
    const double bytes = rows * 64.0 * in_bytes(mode) + (rows - 2 * T) * (64 - 2 * T) * 24.0;
    // (level l starts at iteration 2l)
    const double compute = 0.45 * (xc + 2 * T) + level * (T * (T + 1) + (double)xc * T);
    return std::max(compute, bytes / (cached ? 2.2 * 17600.0 : 17600.0) * (xc + 2 * T));
}

namespace {

// The best pass of T steps by a model of a block's time, fitted to passes
// measured from 32^3 to 1024 x 1024 x 512 (within 20%): 3 us for the launch;
// per iteration 0.45 us and, for each level that runs, 0.11 us + 0.29 us per 16
// rows; or the time the loads and stores of the iterations take at 17.6 KB/us
// per CU (4.5 TB/s in all; 2.2 times that where everything sits in the
// Infinity Cache), if that is longer; the last round of blocks counts in full.
// Where a pass does not fill the device, fewer blocks leave room for another
// context's (three contexts in turn, 48^3: chunks of one plane 3.3 us per step,
// of two 2.1, and 4.4 for either alone): the blocks of a full device count 0.6 more.
Pass plan_pass(const fdtd_ctx* c, int mode, int hook, int T, int cus)
{
    Pass best;
    const bool cached = fits_cache(mode, (double)c->ncell);
    int nv = (int)(sizeof(kVariants) / sizeof(kVariants[0]));
    const Variant* vs = hook == kUpdate ? kVariants : hooked_variants(&nv);
    for (int i = 0; i < nv; ++i) {
        const Variant& v = vs[i];
        if (v.T != T || v.mode != mode || v.hook != hook || (v.whole && c->nz != 64)) continue;
        const int rows = v.R * v.W, vz = v.whole ? 64 : 64 - 2 * T, vy = rows - 2 * T;
        Pass p;
        p.v = &v;
        p.gz = (c->nz + vz - 1) / vz;
        p.gy = (c->ny + vy - 1) / vy;
        const long long base = (long long)p.gz * p.gy;
        int last = 0;
        for (int q = 1; q <= std::min(c->nx, 1024); ++q) {
            const int xc = (c->nx + q - 1) / q;
            if (xc == last) continue;
            last = xc;
            const long long nt = base * ((c->nx + xc - 1) / xc);
            const double us = ((double)((nt + cus - 1) / cus) * round_us(mode, rows, T, xc, cached) + 3.0) *
                              (1.0 + 0.6 * std::min(1.0, (double)nt / cus));
            if (us < p.us) {
                p.us = us;
                p.xchunk = xc;
                p.ntiles = nt;
            }
            if (nt > 64LL * cus) break;
        }
        if (p.us < best.us) best = p;
    }
    return best;
}

}  // namespace

struct SweepState {
    int cus = 0;
    int mode = -1;
    Pass pass[kMaxT + 1];    // the plan of a pass of T steps, for `mode`
    int hooked_mode = -1;
    Pass forward[kMaxT + 1], reverse[kMaxT + 1];  // of the adjoint's passes
    unsigned* pace = nullptr;
    int pace_words = 0;  // of one of the two alternating halves
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

int plan(fdtd_ctx* ctx)
{
    int rc = state(ctx);
    if (rc) return rc;
    SweepState* S = ctx->sweep;
    const int mode = mode_of(ctx);
    if (S->mode != mode) {
        for (int T = 1; T <= kMaxT; ++T) S->pass[T] = plan_pass(ctx, mode, kUpdate, T, S->cus);
        S->mode = mode;
    }
    // Blocks are kept in step where the state is past 1 GiB: 512^3, T = 5,
    // 225 -> 256 G cell updates/s, 1024 x 1024 x 512 255 -> 269; at 256^3,
    // one round of blocks, 202 against 205.
    if (!S->pace && 24.0 * (double)ctx->ncell > 1.0737e9 && !stream_capturing(ctx)) {
        long long words = 0;
        for (int T = 1; T <= kMaxT; ++T) {
            const Pass& p = S->pass[T];
            if (!p.v) continue;
            const long long groups = ((p.ntiles + kXCD - 1) / kXCD + kPaceGroup - 1) / kPaceGroup * kXCD;
            words = std::max(words, groups * ((p.xchunk + 2 * T) / kPacePlanes + 1));
        }
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
        if (!pass[T].v) continue;
        int64_t p = (n + T - 1) / T;
        if (even && (p & 1)) ++p;
        if (p > n) continue;
        const int t = (int)(n / p);
        const int64_t longer = n % p;
        if (t + (longer ? 1 : 0) > kMaxT || !pass[t].v || (longer && !pass[t + 1].v)) continue;
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
        hipLaunchKernelGGL(P.v->hooked, dim3(blocks_of(P)), dim3(64 * P.v->W), 0, ctx->stream, A, *K);
    else
        hipLaunchKernelGGL(P.v->kern, dim3(blocks_of(P)), dim3(64 * P.v->W), 0, ctx->stream, A);
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

// A plane must fit a buffer descriptor with room for the dropped offset.
bool sweep_supported(const fdtd_ctx* ctx)
{
    // (FP16 storage: with the coefficients' exact values in a table)
    return (ctx->storage == FDTD_FP32 || mode_of(ctx) == kTable) && (uint64_t)ctx->ny * (uint64_t)ctx->nz * 4u < (uint64_t)kDropped;
}

bool sweep_ready(fdtd_ctx* ctx)
{
    if (!sweep_supported(ctx)) return false;
    const bool half = ctx->storage == FDTD_FP16_STORAGE;
    bool have = true;
    for (int c = 0; c < 6; ++c) have = have && ctx->alt[c] && (!half || ctx->wide[c]);
    if (have) return true;
    // a scheme that can do without the second field set takes it only where
    // three quarters of the free memory stay free
    if (stream_capturing(ctx)) return false;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if ((half ? 48.0 : 24.0) * (double)ctx->ncell > 0.25 * (double)free_b) return false;
    if (sweep_prepare(ctx) == FDTD_OK) return true;
    for (int c = 0; c < 6; ++c) {
        if (ctx->alt[c]) (void)hipFree(ctx->alt[c]);
        if (ctx->wide[c]) (void)hipFree(ctx->wide[c]);
        ctx->alt[c] = ctx->wide[c] = nullptr;
    }
    return false;
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
                return fail(ctx, FDTD_ENOMEM, "fused plain step: second field set does not fit");
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
        A.pace = S->pace ? S->pace + (size_t)S->turn * S->pace_words : nullptr;
        A.pace_next = S->pace ? S->pace + (size_t)(S->turn ^ 1) * S->pace_words : nullptr;
        A.pace_words = S->pace_words;
        S->turn ^= 1;
        PendingTiming t;
        timing_begin(ctx, kernel, &t);
        launch_pass(ctx, P, A);
        timing_end(ctx, &t);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "launch(sweep)");
        for (int c = 0; c < 6; ++c) std::swap(now[c], other[c]);
        ctx->step_count += T;
    }
    return FDTD_OK;
}

}  // namespace

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
        for (int T = 1; T <= kMaxT; ++T) {
            S->forward[T] = plan_pass(ctx, mode, kForward, T, S->cus);
            S->reverse[T] = plan_pass(ctx, mode, kReverse, T, S->cus);
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
        launch_pass(ctx, S->forward[T], A, &K);
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
