// Material indices: of a lossless grid (FP32 or FP16 storage) into a table of
// (cEx, cEy, cEz), of a conductive one into a table of (cE, ca).
//
// The E update of Section 2 multiplies by the per-cell coefficients cE_c
// (the structural fields of Section 4).  Grids built from a few materials
// (boxes of a few permittivities, PEC walls) hold only a few distinct
// triples (cEx, cEy, cEz) per cell.  The systolic scheme then streams a
// 4-byte index per cell instead of the triple (12 bytes, or the 6 of
// binary16 with FP16 storage, which also had to travel on face rings) and
// looks the triple up in a table of at most kMaxMaterials entries: the
// coefficient values, and so every result, are the same bits as with the
// arrays.
//
// The distinct triples are found on the device in rounds.  Each round
// classifies every cell against the triples known so far (a hash table in
// LDS, keyed on the three bit patterns); cells that match get their index,
// and unmatched triples are reported, up to kCand distinct ones per round.
// The host adds the new triples and runs another round until every cell
// matches, or gives up once there are more than kMaxMaterials.  Entry 0 is always (+0, +0, +0):
// the value that positions outside the grid read.
#include <string.h>

#include <algorithm>

#include <vector>

#include "fdtd_internal.h"

namespace fdtd {

namespace {

constexpr int kSlots = 1024;  // hash slots (at most kMaxMaterials used)
constexpr int kCand = 256;    // unmatched entries reported per round
constexpr int kReports = 16;  // of them by one wavefront
constexpr int kThreads = 256;

// N words of a key: the bits of (cEx, cEy, cEz), with conductivity of
// (cax, cay, caz) too
template <int N>
__host__ __device__ inline unsigned slot_of(const unsigned* k)
{
    unsigned h = (k[0] * 0x9E3779B1u) ^ (k[1] * 0x85EBCA77u) ^ (k[2] * 0xC2B2AE3Du);
    if (N == 6) h ^= (k[N - 3] * 0x27D4EB2Fu) ^ (k[N - 2] * 0x165667B1u) ^ (k[N - 1] * 0xD3A2646Du);
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 13;
    return h & (kSlots - 1);
}

struct Arrays {
    const void* a[6];  // cE, then ca
};

// keys: kSlots x N words (an entry's bits), idx: kSlots entries (-1 empty).
// Cells that match get their index (ids: 4 bytes, may be null; ids8: 1 byte,
// may be null).  Unmatched entries are reported into a table of kCand slots
// keyed by a hash of the entry: each wavefront reports up to kReports distinct
// ones per launch (at most one atomic compare-and-swap each, no waiting), so a
// round finds up to kCand new entries (with 64 slots and four reports a
// conductive shell of 35 M cells took 15 ms to set up instead of 8); cand[0] is set when any cell did not match.
// cand layout: [0] flag, [1 .. kCand] slot keys, then kCand entries.
// With H16 the coefficients are binary16 (FP16 storage) and the entry is
// that of their exact FP32 values.
template <bool H16, int N>
__global__ __launch_bounds__(kThreads) void classify_kernel(Arrays A, long long n,
                                                            const unsigned* __restrict__ keys,
                                                            const int* __restrict__ idx,
                                                            unsigned* __restrict__ ids,
                                                            uint8_t* __restrict__ ids8,
                                                            unsigned* __restrict__ cand)
{
    __shared__ unsigned s_key[kSlots][N];
    __shared__ int s_idx[kSlots];
    auto bits = [&](const void* base, long long p) -> unsigned {
        if (H16) return __float_as_uint((float)__builtin_bit_cast(_Float16, ((const uint16_t*)base)[p]));
        return __float_as_uint(((const float*)base)[p]);
    };
    for (int i = threadIdx.x; i < kSlots; i += kThreads) {
#pragma unroll
        for (int q = 0; q < N; ++q) s_key[i][q] = keys[N * i + q];
        s_idx[i] = idx[i];
    }
    __syncthreads();
    int reports = 0;  // wave-uniform: distinct entries this wavefront reported
    const long long nr = (n + kThreads - 1) / kThreads * kThreads;  // every lane runs every pass
    for (long long p0 = (long long)blockIdx.x * kThreads; p0 < nr; p0 += (long long)gridDim.x * kThreads) {
        const long long p = p0 + threadIdx.x;
        const bool in = p < n;
        unsigned k[N];
#pragma unroll
        for (int q = 0; q < N; ++q) k[q] = 0u;
        int found = -1;
        if (in) {
#pragma unroll
            for (int q = 0; q < N; ++q) k[q] = bits(A.a[q], p);
            unsigned s = slot_of<N>(k);
            // the table is at most a quarter full, so an empty slot ends every probe
            for (int probe = 0; probe < kSlots; ++probe) {
                const int id = s_idx[s];
                if (id < 0) break;
                bool same = true;
#pragma unroll
                for (int q = 0; q < N; ++q) same = same && s_key[s][q] == k[q];
                if (same) {
                    found = id;
                    break;
                }
                s = (s + 1) & (kSlots - 1);
            }
            if (ids) ids[p] = found >= 0 ? (unsigned)found : 0u;
            if (ids8) ids8[p] = found >= 0 ? (uint8_t)found : (uint8_t)0;
        }
        unsigned long long miss = __ballot(in && found < 0);
        if (miss && (threadIdx.x & 63) == __ffsll((long long)miss) - 1) cand[0] = 1u;
        while (miss && reports < kReports) {
            const int lead = __ffsll((long long)miss) - 1;
            unsigned t[N];
            bool same = true;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                t[q] = __shfl(k[q], lead, 64);
                same = same && k[q] == t[q];
            }
            if ((int)(threadIdx.x & 63) == lead) {
                const unsigned h = (slot_of<N>(t) * 0x9E3779B9u) | 1u;  // never 0 (free)
                const unsigned q = h % (unsigned)kCand;
                // (a slot once claimed stays claimed: most find it so without an atomic)
                const unsigned prev = __hip_atomic_load(&cand[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                          ? h : atomicCAS(&cand[1 + q], 0u, h);
                if (prev == 0u) {
                    unsigned* d = cand + 1 + kCand + N * q;
#pragma unroll
                    for (int c = 0; c < N; ++c) d[c] = t[c];
                }
            }
            // lanes holding the same entry are covered by that report
            miss &= __ballot(!same);
            ++reports;
        }
        // (a wavefront that could not report all it met leaves the rest to the
        // next round: 400 x 380 x 300 conductive cells, all different, set in 1.7
        // -> 1.2 ms)
        if (miss) break;
    }
}

int grid_blocks(int64_t n)
{
    const int64_t b = (n + kThreads - 1) / kThreads;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 2048));
}

}  // namespace

void release_material_ids(fdtd_ctx* ctx)
{
    for (void* p : {(void*)ctx->mat_id, (void*)ctx->mat_tab, (void*)ctx->mat_id8, (void*)ctx->mat_tab8})
        if (p) (void)hipFree(p);
    ctx->mat_id = nullptr;
    ctx->mat_tab = nullptr;
    ctx->mat_id8 = nullptr;
    ctx->mat_tab8 = nullptr;
    ctx->nmat = 0;
    ctx->ntab8 = 0;
}

namespace {

template <typename T>
bool ensure(T** p, size_t n)
{
    if (*p || hipMalloc(p, n * sizeof(T)) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}

// Finds the distinct entries of N words and the index of every cell; leaves
// *count = 0 when there are more than kMaxMaterials.
template <int N>
int find_entries(fdtd_ctx* ctx, uint32_t* ids, uint8_t* ids8, std::vector<unsigned>* table, int* count)
{
    *count = 0;
    hipError_t e;
    // one buffer, one copy per round: keys, indices, candidates
    const size_t ncand = 1 + kCand + N * kCand;  // flag, slot keys, entries
    const size_t words = (size_t)kSlots * N + kSlots + ncand;
    unsigned* d_keys = nullptr;
    if ((e = hipMalloc(&d_keys, words * sizeof(unsigned))) != hipSuccess) {
        (void)hipGetLastError();
        // (a conductive grid did without the table, and can)
        return N == 6 ? FDTD_OK : fail(ctx, FDTD_ENOMEM, "material table: scratch allocation failed");
    }
    int* d_idx = (int*)(d_keys + kSlots * N);
    unsigned* d_cand = (unsigned*)(d_idx + kSlots);
    const bool h16 = ctx->storage == FDTD_FP16_STORAGE;
    Arrays A{};
    for (int q = 0; q < 3; ++q) {
        A.a[q] = h16 ? (const void*)ctx->coef16[q] : (const void*)ctx->coef[q];
        A.a[3 + q] = ctx->ca[q];
    }
    std::vector<unsigned>& tab = *table;
    tab.assign(N, 0u);  // entry 0: all +0
    std::vector<unsigned> up(words), cand(ncand);
    unsigned* const keys = up.data();
    int* const idx = (int*)(keys + kSlots * N);
    bool ok = false;
    e = hipSuccess;
    for (int round = 0; round <= kMaxMaterials && e == hipSuccess; ++round) {
        const int nm = (int)tab.size() / N;
        std::fill(up.begin(), up.end(), 0u);
        std::fill(idx, idx + kSlots, -1);
        for (int m = 0; m < nm; ++m) {
            unsigned s = slot_of<N>(&tab[N * m]);
            while (idx[s] >= 0) s = (s + 1) & (kSlots - 1);
            idx[s] = m;
            for (int q = 0; q < N; ++q) keys[N * s + q] = tab[N * m + q];
        }
        if ((e = hipMemcpyAsync(d_keys, up.data(), words * sizeof(unsigned), hipMemcpyHostToDevice, ctx->stream)) !=
            hipSuccess)
            break;
        const auto kern = N == 6 ? classify_kernel<false, N> : h16 ? classify_kernel<true, N> : classify_kernel<false, N>;
        hipLaunchKernelGGL(kern, dim3(grid_blocks(ctx->ncell)), dim3(kThreads), 0, ctx->stream, A,
                           (long long)ctx->ncell, d_keys, d_idx, ids, ids8, d_cand);
        if ((e = hipGetLastError()) != hipSuccess) break;
        if ((e = hipMemcpyAsync(cand.data(), d_cand, cand.size() * sizeof(unsigned), hipMemcpyDeviceToHost,
                                ctx->stream)) != hipSuccess ||
            (e = hipStreamSynchronize(ctx->stream)) != hipSuccess)
            break;
        if (cand[0] == 0) {
            ok = true;
            break;
        }
        for (int i = 0; i < kCand && (int)tab.size() / N <= kMaxMaterials; ++i) {
            if (cand[1 + i] == 0) continue;  // slot not claimed
            const unsigned* t = &cand[1 + kCand + N * i];
            bool have = false;
            for (size_t m = 0; m < tab.size() / N && !have; ++m) have = std::equal(t, t + N, &tab[N * m]);
            if (!have) tab.insert(tab.end(), t, t + N);
        }
        if ((int)tab.size() / N > kMaxMaterials) break;  // too many: the per-cell arrays serve
    }
    (void)hipFree(d_keys);
    if (e != hipSuccess) return hip_fail(ctx, e, "material table");
    if (ok) *count = (int)tab.size() / N;
    return FDTD_OK;
}

}  // namespace

int build_material_ids(fdtd_ctx* ctx)
{
    ctx->nmat = 0;
    ctx->ntab8 = 0;
    const bool lossy = ctx->ca[0] != nullptr;
    // (the table of a conductive grid is a matter of speed: none in a captured
    // stream, which can neither allocate nor be waited for)
    if (lossy && stream_capturing(ctx)) return FDTD_OK;
    const size_t nc = (size_t)ctx->ncell;
    const int N = lossy ? 6 : 3;
    if (lossy) {
        // (the systolic scheme streams a conductive grid's arrays)
        if (ctx->mat_id) (void)hipFree(ctx->mat_id);
        if (ctx->mat_tab) (void)hipFree(ctx->mat_tab);
        ctx->mat_id = nullptr;
        ctx->mat_tab = nullptr;
    }
    if (!lossy && (!ensure(&ctx->mat_id, nc) || !ensure(&ctx->mat_tab, (size_t)kMaxMaterials * 3)))
        return FDTD_OK;  // no room: the per-cell arrays serve
    const bool bytes = ensure(&ctx->mat_id8, nc) && ensure(&ctx->mat_tab8, (size_t)kMaxMaterials * 6);
    if (lossy && !bytes) return FDTD_OK;
    std::vector<unsigned> tab;
    int count = 0;
    int rc = lossy ? find_entries<6>(ctx, nullptr, ctx->mat_id8, &tab, &count)
                   : find_entries<3>(ctx, ctx->mat_id, bytes ? ctx->mat_id8 : nullptr, &tab, &count);
    if (rc) return rc;
    if (count > 0) {
        tab.resize((size_t)kMaxMaterials * N, 0u);
        hipError_t e = hipSuccess;
        if (!lossy)
            e = hipMemcpyAsync(ctx->mat_tab, tab.data(), tab.size() * sizeof(unsigned), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess && bytes)
            e = hipMemcpyAsync(ctx->mat_tab8, tab.data(), tab.size() * sizeof(unsigned), hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) return hip_fail(ctx, e, "material table");
        ctx->nmat = lossy ? 0 : count;
        ctx->ntab8 = bytes ? count : 0;
    } else {
        // too many materials: the per-cell arrays serve, the indices go
        release_material_ids(ctx);
    }
    return FDTD_OK;
}

}  // namespace fdtd
