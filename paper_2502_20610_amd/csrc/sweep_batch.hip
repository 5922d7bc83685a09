// Sweeps of several grids in one launch per pass (fdtd_step_batch).
//
// Small grids leave most of the device idle in a launch of their own, and a
// launch costs as much as their pass.  Here the tiles of all grids of the
// batch make one launch; a block finds its grid in a table.  The tile itself
// is that of one grid's sweep (sweep_tile.h).
#include <string.h>

#include <algorithm>
#include <new>

#include "sweep_tile.h"

namespace fdtd {
namespace {

// Records read through the constant address space: a block's record is the
// same for all its lanes and comes through the scalar cache.
template <typename T>
using Const = const __attribute__((address_space(4))) T;

template <int T, int R, int W, int MODE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void batch_kernel(
    const SweepArgs* sims, const int2* blocks, long long steps_done)
{
    static_assert(sizeof(SweepArgs) % 4 == 0, "read by words");
    __shared__ Lds<T, R, W, MODE> S;
    Const<int>* const b = (Const<int>*)(const void*)(blocks + blockIdx.x);
    const int sim = b[0], tile = b[1];
    union {
        SweepArgs A;
        unsigned words[sizeof(SweepArgs) / 4];
    } u;
    Const<unsigned>* const w = (Const<unsigned>*)(const void*)(sims + sim);
#pragma unroll
    for (unsigned q = 0; q < sizeof(SweepArgs) / 4; ++q) u.words[q] = w[q];
    SweepArgs A = u.A;
    A.step += steps_done;
    sweep_tile<T, R, W, MODE, false, kUpdate>(A, HookArgs{}, S, 0, tile, A.ntiles);
}

struct BatchShape {
    int T, R, W, mode;
    void (*kern)(const SweepArgs*, const int2*, long long);
};
#define S(T, R, W, M) {T, R, W, M, batch_kernel<T, R, W, M>}
#define S4(R, W, M) S(1, R, W, M), S(2, R, W, M), S(3, R, W, M), S(4, R, W, M)
const BatchShape kShapes[] = {
    S4(1, 16, kTable), S4(2, 16, kTable), S4(1, 16, kArrays), S4(4, 8, kArrays),
    S4(1, 16, kLossyTable), S4(2, 16, kLossyTable), S4(1, 16, kLossy),
};
#undef S
#undef S4

constexpr int kMaxBatchT = 4;

// One pass of T steps over every grid of the batch.
struct BatchPass {
    const BatchShape* s = nullptr;
    int xcap = 0;  // planes of a chunk, at most
    double us = 1e300;
};

int chunk(int nx, int cap)
{
    const int q = (nx + cap - 1) / cap;
    return (nx + q - 1) / q;
}

long long tiles(const fdtd_ctx* c, const BatchShape& s, int cap, int* gz, int* gy, int* xc)
{
    const int vz = 64 - 2 * s.T, vy = s.R * s.W - 2 * s.T;
    *gz = (c->nz + vz - 1) / vz;
    *gy = (c->ny + vy - 1) / vy;
    *xc = chunk(c->nx, cap);
    return (long long)*gz * *gy * ((c->nx + *xc - 1) / *xc);
}

// The shape and chunk length that take the least by the model of a block's
// time: all blocks of all grids in whole rounds of one per CU, each as long as
// its longest block, or as long as an even spread and one more block.  (16
// grids of 16 to 64 cells an axis, 64 steps: the model takes 4 steps, 32 rows
// and chunks of 8, the fastest measured, 690 us; spreads alone, without whole
// rounds, took 3 steps and 800 us.)
BatchPass plan(fdtd_ctx* const* cs, int n, int mode, int T, int cus)
{
    double cells = 0.0;
    for (int i = 0; i < n; ++i) cells += (double)cs[i]->ncell;
    const bool cached = fits_cache(mode, cells);
    BatchPass best;
    for (const BatchShape& s : kShapes) {
        if (s.T != T || s.mode != mode) continue;
        for (int cap = 1; cap <= 512; cap += std::max(1, cap / 4)) {
            long long nt = 0;
            int longest = 0;
            double work = 0.0;
            for (int i = 0; i < n; ++i) {
                int gz, gy, xc;
                const long long k = tiles(cs[i], s, cap, &gz, &gy, &xc);
                nt += k;
                longest = std::max(longest, xc);
                work += (double)k * round_us(mode, s.R * s.W, T, xc, cached);
            }
            const double block = round_us(mode, s.R * s.W, T, longest, cached);
            const double us = std::min((double)((nt + cus - 1) / cus) * block, work / cus + block) + 3.0;
            if (us < best.us && nt < (1 << 20)) {
                best.us = us;
                best.s = &s;
                best.xcap = cap;
            }
        }
    }
    return best;
}

template <typename T>
bool reserve(T** host, T** dev, size_t* cap, size_t n)
{
    if (n <= *cap) return true;
    if (*host) (void)hipHostFree(*host);
    if (*dev) (void)hipFree(*dev);
    *host = nullptr;
    *dev = nullptr;
    *cap = 0;
    if (hipHostMalloc(host, n * sizeof(T), hipHostMallocDefault) != hipSuccess || hipMalloc(dev, n * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    *cap = n;
    return true;
}

}  // namespace

// Tables of the last batch led by a context (staged through pinned memory).
struct SweepBatch {
    SweepArgs *h_sims = nullptr, *d_sims = nullptr;
    int2 *h_blocks = nullptr, *d_blocks = nullptr;
    size_t cap_sims = 0, cap_blocks = 0;
    hipEvent_t copied = nullptr;  // the staging may be written again
};

void sweep_batch_release(fdtd_ctx* ctx)
{
    SweepBatch* B = ctx->sweep_batch;
    if (!B) return;
    if (B->copied) (void)hipEventSynchronize(B->copied);
    if (B->h_sims) (void)hipHostFree(B->h_sims);
    if (B->h_blocks) (void)hipHostFree(B->h_blocks);
    if (B->d_sims) (void)hipFree(B->d_sims);
    if (B->d_blocks) (void)hipFree(B->d_blocks);
    if (B->copied) (void)hipEventDestroy(B->copied);
    delete B;
    ctx->sweep_batch = nullptr;
}

int sweep_batch_steps(fdtd_ctx* const* cs, int n, int64_t nsteps, bool* done)
{
    *done = false;
    fdtd_ctx* lead = cs[0];
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, lead->device);
    if (e != hipSuccess) return hip_fail(lead, e, "sweep batch: device attribute");
    // the table form when every member has it (two grids of 256^3, 20 steps: both
    // with a table 3.99 ms, one 4.50, none 4.52; one persistent launch 4.67 to 5.0)
    int mode = mode_of(lead);
    for (int i = 1; i < n; ++i)
        if (mode_of(cs[i]) != mode) mode = lead->ca[0] ? kLossy : kArrays;
    // an even number of passes: the state ends in the arrays it started from
    BatchPass pass[kMaxBatchT + 1];
    for (int T = 1; T <= kMaxBatchT; ++T) pass[T] = plan(cs, n, mode, T, std::max(1, cus));
    int64_t passes = 0;
    double best = 1e300;
    for (int T = 1; T <= kMaxBatchT; ++T) {
        int64_t p = (nsteps + T - 1) / T;
        p += p & 1;
        if (p > nsteps) continue;
        const int t = (int)(nsteps / p);
        const int64_t longer = nsteps % p;
        if (t + (longer ? 1 : 0) > kMaxBatchT || !pass[t].s || (longer && !pass[t + 1].s)) continue;
        const double us = (double)(p - longer) * pass[t].us + (longer ? (double)longer * pass[t + 1].us : 0.0);
        if (us < best) {
            best = us;
            passes = p;
        }
    }
    if (passes == 0) return FDTD_OK;
    const int t = (int)(nsteps / passes);
    const int64_t longer = nsteps % passes;
    if (!lead->sweep_batch) {
        lead->sweep_batch = new (std::nothrow) SweepBatch();
        if (!lead->sweep_batch) return fail(lead, FDTD_ENOMEM, "sweep batch: host allocation failed");
    }
    SweepBatch* B = lead->sweep_batch;
    if (!B->copied && (e = hipEventCreateWithFlags(&B->copied, hipEventDisableTiming)) != hipSuccess)
        return hip_fail(lead, e, "hipEventCreate");
    if ((e = hipEventSynchronize(B->copied)) != hipSuccess) return hip_fail(lead, e, "hipEventSynchronize");
    // records: [length of pass (t, t + 1)][direction (home -> alt, back)][grid];
    // block tables per length
    size_t nblocks[2] = {0, 0};
    for (int k = 0; k < 2; ++k) {
        const BatchPass& P = pass[t + k <= kMaxBatchT ? t + k : t];
        if ((k == 1 && !longer) || !P.s) continue;
        for (int i = 0; i < n; ++i) {
            int gz, gy, xc;
            nblocks[k] += (size_t)tiles(cs[i], *P.s, P.xcap, &gz, &gy, &xc);
        }
    }
    if (!reserve(&B->h_sims, &B->d_sims, &B->cap_sims, (size_t)4 * n) ||
        !reserve(&B->h_blocks, &B->d_blocks, &B->cap_blocks, nblocks[0] + nblocks[1]))
        return fail(lead, FDTD_ENOMEM, "sweep batch: tables");
    size_t at = 0;
    for (int k = 0; k < 2; ++k) {
        if (nblocks[k] == 0) continue;
        const BatchPass& P = pass[t + k];
        for (int i = 0; i < n; ++i) {
            const fdtd_ctx* c = cs[i];
            SweepArgs A = base_args(c);
            A.id = c->mat_id8;
            A.tab = c->mat_tab8;
            A.ntab = c->ntab8;
            A.src = c->dev_sources;
            A.nsrc = c->dev_sources_n;
            A.step = c->step_count;
            A.ntiles = (int)tiles(c, *P.s, P.xcap, &A.gz, &A.gy, &A.xchunk);
            for (int d = 0; d < 2; ++d) {
                for (int q = 0; q < 6; ++q) {
                    A.in[q] = d ? c->alt[q] : c->field[q];
                    A.out[q] = d ? c->field[q] : c->alt[q];
                }
                memcpy(&B->h_sims[(size_t)(2 * k + d) * n + i], &A, sizeof(A));
            }
            for (int b = 0; b < A.ntiles; ++b) B->h_blocks[at++] = make_int2(i, b);
        }
    }
    // after every member's earlier work, on the lead's stream
    hipStream_t st = lead->stream;
    hipEvent_t ev = nullptr;
    for (int i = 1; i < n && e == hipSuccess; ++i) {
        if (cs[i]->stream == st) continue;
        if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) break;
        if ((e = hipEventRecord(ev, cs[i]->stream)) == hipSuccess) e = hipStreamWaitEvent(st, ev, 0);
        (void)hipEventDestroy(ev);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(B->d_sims, B->h_sims, (size_t)4 * n * sizeof(SweepArgs), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(B->d_blocks, B->h_blocks, at * sizeof(int2), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipEventRecord(B->copied, st);
    if (e != hipSuccess) return hip_fail(lead, e, "sweep batch set-up");
    long long steps = 0;
    for (int64_t p = 0; p < passes; ++p) {
        const int k = p < longer ? 1 : 0;
        const BatchShape& s = *pass[t + k].s;
        PendingTiming tm;
        timing_begin(lead, FDTD_KERNEL_SYSTOLIC, &tm);
        hipLaunchKernelGGL(s.kern, dim3((unsigned)nblocks[k]), dim3(64 * s.W), 0, st,
                           (const SweepArgs*)(B->d_sims + (size_t)(2 * k + (int)(p & 1)) * n),
                           (const int2*)(B->d_blocks + (k ? nblocks[0] : 0)), steps);
        timing_end(lead, &tm);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(lead, e, "launch(sweep batch)");
        steps += t + k;
    }
    // the members' streams continue after the passes
    bool others = false;
    for (int i = 1; i < n; ++i) others = others || cs[i]->stream != st;
    if (others && (e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) == hipSuccess) {
        e = hipEventRecord(ev, st);
        for (int i = 1; i < n && e == hipSuccess; ++i)
            if (cs[i]->stream != st) e = hipStreamWaitEvent(cs[i]->stream, ev, 0);
        (void)hipEventDestroy(ev);
    }
    if (e != hipSuccess) return hip_fail(lead, e, "sweep batch completion");
    for (int i = 0; i < n; ++i) {
        cs[i]->step_count += nsteps;
        cs[i]->sys_band = t + (longer ? 1 : 0);
        cs[i]->sys_grid = cs[i]->sys_tickets = (int)nblocks[longer ? 1 : 0];
        cs[i]->sys_ring_slots = 0;
    }
    *done = true;
    return FDTD_OK;
}

}  // namespace fdtd
