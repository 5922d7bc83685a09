// Sweep: T whole steps of the Yee update in one pass over the grid.
//
// A step of Section 2 (E half-step, sources, H half-step) reads and writes the
// whole state, so a scheme of one launch per step runs at the rate of device
// memory: 60 B per cell update at best.  A sweep advances T steps between one
// read and one write.  It is the paper's x-t traversal (Section 3: the work
// moves along the x-t diagonal) inside one workgroup, with overlapping tiles
// in place of face exchange: nothing passes between workgroups.
//
// A block of W wavefronts covers 64 lanes (z) x W R rows (y; R per lane) and
// streams along x over a chunk of planes.  In iteration `it` plane `it` enters
// and level l (step l of the pass) updates E on plane it - l and then H on
// plane it - l - 1, in place; after level T - 1 plane it - T is finished and
// stored to the other field set.  Planes live in T + 2 register slots (the
// last one is being loaded); the loop is unrolled over the slots, so a plane
// never moves.  Every level costs one layer on each side: a tile stores its
// inner 64 - 2T lanes and W R - 2T rows, a chunk loads 2T planes more than it
// stores.  Neighbour values: x from registers, z by wavefront DPP shifts, y
// from the lane's own rows and, between wavefronts, through LDS (H of level l
// is exchanged behind the level's barrier; E is read an iteration after it is
// written, double-buffered).  All index arithmetic is modulo the grid, as in
// the plain kernels, and a wall is a zero coefficient.  The operations on a
// cell and their order are those of the plain step, so the result is the same
// FP32 value bit for bit.
//
// What bounds it: on grids beyond the Infinity Cache, device memory.  With the
// update left out the loads and stores alone take 97% of a pass (512^3, T = 4,
// 4.5 TB/s through the L2).  So the tile is the largest that the registers
// hold, coefficients come as a 1-byte index into a table in LDS wherever the
// grid has at most 256 materials (25 instead of 36 B in per cell; the indices
// of planes in flight are parked in LDS), stores bypass the caches, and blocks
// of one XCD are kept in step (below) so that the halos of neighbouring tiles
// meet in its L2.
#include <algorithm>
#include <new>

#include "fdtd_internal.h"

namespace fdtd {
namespace {

constexpr int kXCD = 8;          // XCDs of the device
constexpr int kPaceGroup = 32;   // blocks an XCD runs at once (one per CU)
constexpr int kPacePlanes = 4;   // planes between two progress marks
constexpr unsigned kDropped = 0x80000000u;  // a buffer offset past every plane: the access is dropped

enum { kArrays = 0, kLossy = 1, kTable = 2, kLossyTable = 3 };

struct SweepArgs {
    const float* in[6];
    float* out[6];
    const float* cE[3];
    const float* ca[3];
    const uint8_t* id;
    const float* tab;  // ntab x (cE) or (cE, ca)
    int ntab;
    float cH;
    int nx, ny, nz;
    int gz, gy, ntiles, xchunk;
    const DevSource* src;
    int nsrc;
    long long step;
    unsigned* pace;       // progress marks of this pass (null: not kept in step)
    unsigned* pace_next;  // those of the next pass, cleared by this one
    int pace_words;
};

__device__ __forceinline__ void lds_barrier()
{
    // LDS only: loads and stores of planes stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The value of lane - 1 and lane + 1: a wavefront shift, or a rotation where
// the wavefront is the whole z axis.
template <bool WHOLE>
__device__ __forceinline__ float from_below(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), WHOLE ? 0x13C : 0x138,
                                                                 0xf, 0xf, true));
}
template <bool WHOLE>
__device__ __forceinline__ float from_above(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), WHOLE ? 0x134 : 0x130,
                                                                 0xf, 0xf, true));
}

__device__ __forceinline__ int wrap(int v, int n)
{
    const int m = v % n;
    return m < 0 ? m + n : m;
}

template <int T, int R, int W, int MODE, bool WHOLE>
__device__ __forceinline__ void sweep_tile(const SweepArgs& A, int block, int nblocks)
{
    static_assert(W * R > 2 * T && 64 > 2 * T, "the tile keeps at least one cell");
    constexpr int NS = T + 2;
    constexpr bool TAB = MODE == kTable || MODE == kLossyTable;
    constexpr bool LOSSY = MODE == kLossy || MODE == kLossyTable;
    constexpr int NC = LOSSY ? 6 : 3;  // coefficients per cell
    constexpr int NP = (R + 3) / 4;    // words of packed indices per plane and lane
    constexpr int kList = 64;          // sources a block keeps at hand
    __shared__ float2 hx_[T == 1 ? 2 : 1][T][W][64];
    __shared__ float2 ex_[2][T][W][64];
    __shared__ float4 tab_[TAB ? kMaxMaterials : 1];
    __shared__ float4 tabA_[MODE == kLossyTable ? kMaxMaterials : 1];
    __shared__ unsigned ids_[TAB ? T : 1][NP][64 * W];
    __shared__ int list_[kList];
    __shared__ int nlist_;
    // launch order is dealt round the XCDs; tiles are contiguous per XCD
    const int per_xcd = nblocks / kXCD, xcd = block % kXCD, slot = block / kXCD;
    const int tile = xcd * per_xcd + slot;
    if (A.pace_next) {
        const int each = (A.pace_words + nblocks - 1) / nblocks;
        for (int q = threadIdx.x; q < each; q += 64 * W)
            if (block * each + q < A.pace_words) A.pace_next[block * each + q] = 0u;
    }
    if (tile >= A.ntiles) return;  // whole block
    const int tz = tile % A.gz, ty = (tile / A.gz) % A.gy, tx = tile / (A.gz * A.gy);
    const int L = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k0 = WHOLE ? 0 : tz * (64 - 2 * T) - T, j0 = ty * (W * R - 2 * T) - T;
    const int x0 = tx * A.xchunk, x1 = min(A.nx, x0 + A.xchunk);
    const int nit = x1 - x0 + 2 * T;
    const int k = wrap(k0 + L, A.nz);
    const bool kown = WHOLE || (L >= T && L < 64 - T && k0 + L < A.nz);
    unsigned off[R];            // byte offset of the lane's cell in a plane
    unsigned long long own[R];  // lanes that store row r
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int rr = w * R + r;
        off[r] = ((unsigned)wrap(j0 + rr, A.ny) * (unsigned)A.nz + (unsigned)k) * 4u;
        own[r] = __ballot(kown && rr >= T && rr < W * R - T && j0 + rr < A.ny);
    }
    const unsigned pbytes = (unsigned)A.ny * (unsigned)A.nz * 4u;
    constexpr int CS = TAB ? 1 : NS, CR = TAB ? 1 : R, CC = TAB ? 1 : NC;
    float E[NS][R][3], H[NS][R][3], C[CS][CR][CC];
    unsigned ci[R];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) E[s][r][c] = H[s][r][c] = 0.f;
#pragma unroll
    for (int s = 0; s < CS; ++s)
#pragma unroll
        for (int r = 0; r < CR; ++r)
#pragma unroll
            for (int c = 0; c < CC; ++c) C[s][r][c] = 0.f;
    // descriptors cover one plane: 32-bit offsets whatever the grid's size
    auto rsrc = [&](const void* base, int plane, unsigned bytes) {
        const char* p = (const char*)base + (unsigned long long)(unsigned)plane * bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), (short)0, (int)bytes, 0x00020000);
    };
    auto ld = [&](const void* base, int plane, unsigned o) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc(base, plane, pbytes), (int)o, 0, 0));
    };
    int pin = wrap(x0 - T, A.nx);  // grid plane of the next load
    auto load = [&](int s) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) H[s][r][c] = ld(A.in[3 + c], pin, off[r]);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) E[s][r][c] = ld(A.in[c], pin, off[r]);
        if (TAB) {
            const auto ri = rsrc(A.id, pin, pbytes >> 2);
#pragma unroll
            for (int r = 0; r < R; ++r)
                ci[r] = (unsigned char)__builtin_amdgcn_raw_buffer_load_b8(ri, (int)(off[r] >> 2), 0, 0);
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    C[s % CS][r % CR][c % CC] = ld(c < 3 ? A.cE[c % 3] : A.ca[c % 3], pin, off[r]);
        }
        pin = pin + 1 == A.nx ? 0 : pin + 1;
    };
    load(0);
    if (TAB) {
        for (int q = threadIdx.x; q < A.ntab; q += 64 * W) {
            const float* t = A.tab + q * NC;
            tab_[q] = make_float4(t[0], t[1], t[2], 0.f);
            if (MODE == kLossyTable) tabA_[q] = make_float4(t[NC - 3], t[NC - 2], t[NC - 1], 0.f);
        }
#pragma unroll
        for (int d = 0; d < T; ++d)
#pragma unroll
            for (int q = 0; q < NP; ++q) ids_[d][q][threadIdx.x] = 0u;
    }
    // the sources this block meets, in table order (several on one cell add up
    // in the same order as in any other scheme)
    int nhit = 0;
    if (A.nsrc > 0) {
        if (w == 0) {
            int n = 0;
            for (int b = 0; b < A.nsrc; b += 64) {
                const int q = b + L;
                bool hit = false;
                if (q < A.nsrc) {
                    const DevSource s = A.src[q];
                    hit = wrap(s.k - k0, A.nz) < 64 && wrap(s.j - j0, A.ny) < W * R &&
                          wrap(s.i - (x0 - T), A.nx) < nit && A.step + T > s.first && A.step < s.first + s.len;
                }
                const unsigned long long m = __ballot(hit);
                const int at = n + __popcll(m & ((1ull << L) - 1));
                if (hit && at < kList) list_[at] = q;
                n += __popcll(m);
            }
            if (L == 0) nlist_ = n;
        }
        __syncthreads();
        nhit = __builtin_amdgcn_readfirstlane(nlist_);
    }
    // lane e of every wavefront holds the plane of entry e
    int lsi = -1;
    if (nhit > 0 && nhit <= kList && L < nhit) lsi = A.src[list_[L]].i;
    // Blocks of one XCD in step: each marks its progress every few planes, and
    // one that is ahead of the slowest of its group rests a little.  Nothing
    // depends on it: a mark is read once, never waited for.
    const int group = xcd * ((per_xcd + kPaceGroup - 1) / kPaceGroup) + slot / kPaceGroup;
    const int members = min(kPaceGroup, min(per_xcd, A.ntiles - xcd * per_xcd) - slot / kPaceGroup * kPaceGroup);
    unsigned* const marks = A.pace + (size_t)group * ((A.xchunk + 2 * T) / kPacePlanes + 1);
    unsigned seen = 0;
    int pe = wrap(x0 - T, A.nx);  // grid plane of iteration `it`
    int ring = 0;                 // slot of the index ring that holds plane `it`
    if (TAB) __syncthreads();
    for (int base = 0; base < nit; base += NS) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int it = base + u;
            if (it >= nit) break;
            const int par = it & 1;
            unsigned pk[NP];
            if (TAB) {
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    pk[q] = ci[4 * q];
#pragma unroll
                    for (int r = 1; r < 4; ++r)
                        if (4 * q + r < R) pk[q] |= ci[4 * q + r < R ? 4 * q + r : 0] << (8 * r);
                    ids_[ring][q][threadIdx.x] = pk[q];
                }
            }
            if (it + 1 < nit) load((u + 1) % NS);
            if (A.pace && threadIdx.x == 0) {
                constexpr int P = kPacePlanes;
                if (it % P == 0 && it >= 2 * P && (int)seen < members)
                    for (int q = 0; q < 4; ++q) __builtin_amdgcn_s_sleep(16);
                if (it % P == P - 1) {
                    unsigned* p = marks + it / P;
                    __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (it >= 2 * P - 1) seen = __hip_atomic_load(p - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            hx_[T == 1 ? par : 0][0][w][L] = make_float2(H[u][R - 1][0], H[u][R - 1][2]);
#pragma unroll
            for (int l = 0; l < T; ++l) {
                const int s0 = (u - l + NS) % NS, s1 = (u - l - 1 + NS) % NS;
                // until it = 2l no stored value depends on level l
                if (it < 2 * l) break;
                if (TAB && l > 0) {
                    const int q0 = ring - l < 0 ? ring - l + T : ring - l;
#pragma unroll
                    for (int q = 0; q < NP; ++q) pk[q] = ids_[q0][q][threadIdx.x];
                }
                lds_barrier();
                const float2 hl = hx_[T == 1 ? par : 0][l][w == 0 ? 0 : w - 1][L];
                const float2 eu = ex_[par ^ 1][l][w == W - 1 ? w : w + 1][L];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float hx = H[s0][r][0], hy = H[s0][r][1], hz = H[s0][r][2];
                    const float hx_jm = r ? H[s0][r - 1][0] : hl.x, hz_jm = r ? H[s0][r - 1][2] : hl.y;
                    const float hx_km = from_below<WHOLE>(hx), hy_km = from_below<WHOLE>(hy);
                    const float hy_im = H[s1][r][1], hz_im = H[s1][r][2];
                    float cx, cy, cz;
                    float ex = E[s0][r][0], ey = E[s0][r][1], ez = E[s0][r][2];
                    if (TAB) {
                        const unsigned id = pk[r / 4] >> (8 * (r % 4)) & 255u;
                        const float4 t = tab_[id];
                        cx = t.x;
                        cy = t.y;
                        cz = t.z;
                        if (MODE == kLossyTable) {
                            const float4 a = tabA_[id];
                            ex = a.x * ex;
                            ey = a.y * ey;
                            ez = a.z * ez;
                        }
                    } else {
                        const float* cc = C[s0 % CS][r % CR];
                        cx = cc[0];
                        cy = cc[1 % CC];
                        cz = cc[2 % CC];
                        if (LOSSY) {
                            ex = cc[3 % CC] * ex;
                            ey = cc[4 % CC] * ey;
                            ez = cc[5 % CC] * ez;
                        }
                    }
                    E[s0][r][0] = (ex + cx * (hz - hz_jm)) - cx * (hy - hy_km);
                    E[s0][r][1] = (ey + cy * (hx - hx_km)) - cy * (hz - hz_im);
                    E[s0][r][2] = (ez + cz * (hy - hy_im)) - cz * (hx - hx_jm);
                }
                if (nhit > 0) {
                    const int pl = wrap(pe - l, A.nx);
                    auto add = [&](int q) {
                        const DevSource s = A.src[q];
                        const long long m = A.step + l - s.first;
                        if (s.i != pl || m < 0 || m >= s.len) return;
                        const float v = s.wave[m];
                        const unsigned cell = ((unsigned)s.j * (unsigned)A.nz + (unsigned)s.k) * 4u;
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            if (off[r] == cell) {
                                E[s0][r][0] = s.comp == 0 ? E[s0][r][0] + v : E[s0][r][0];
                                E[s0][r][1] = s.comp == 1 ? E[s0][r][1] + v : E[s0][r][1];
                                E[s0][r][2] = s.comp == 2 ? E[s0][r][2] + v : E[s0][r][2];
                            }
                    };
                    if (nhit <= kList) {
                        unsigned long long m = __ballot(lsi == pl);
                        while (m) {
                            const int e = __ffsll((long long)m) - 1;
                            m &= m - 1;
                            add(__builtin_amdgcn_readfirstlane(list_[e]));
                        }
                    } else {
                        for (int q = 0; q < A.nsrc; ++q) add(q);
                    }
                }
                ex_[par][l][w][L] = make_float2(E[s0][0][0], E[s0][0][2]);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float ex = E[s1][r][0], ey = E[s1][r][1], ez = E[s1][r][2];
                    const float ex_jp = r < R - 1 ? E[s1][r + 1 < R ? r + 1 : r][0] : eu.x;
                    const float ez_jp = r < R - 1 ? E[s1][r + 1 < R ? r + 1 : r][2] : eu.y;
                    const float ey_kp = from_above<WHOLE>(ey), ex_kp = from_above<WHOLE>(ex);
                    const float ey_ip = E[s0][r][1], ez_ip = E[s0][r][2];
                    H[s1][r][0] = (H[s1][r][0] - A.cH * (ez_jp - ez)) + A.cH * (ey_kp - ey);
                    H[s1][r][1] = (H[s1][r][1] - A.cH * (ex_kp - ex)) + A.cH * (ez_ip - ez);
                    H[s1][r][2] = (H[s1][r][2] - A.cH * (ey_ip - ey)) + A.cH * (ex_jp - ex);
                }
                if (l + 1 < T) hx_[0][l + 1 < T ? l + 1 : 0][w][L] = make_float2(H[s1][R - 1][0], H[s1][R - 1][2]);
            }
            if (it >= 2 * T) {
                const int s = (u - T + NS) % NS;
                const int plane = x0 + it - 2 * T;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const unsigned so = __builtin_amdgcn_inverse_ballot_w64(own[r]) ? off[r] : kDropped;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, E[s][r][c]),
                                                              rsrc(A.out[c], plane, pbytes), (int)so, 0, 2);
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, H[s][r][c]),
                                                              rsrc(A.out[3 + c], plane, pbytes), (int)so, 0, 2);
                    }
                }
            }
            pe = pe + 1 == A.nx ? 0 : pe + 1;
            ring = ring + 1 == T ? 0 : ring + 1;
        }
    }
}

template <int T, int R, int W, int MODE, bool WHOLE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void sweep_kernel(
    const SweepArgs A)
{
    sweep_tile<T, R, W, MODE, WHOLE>(A, (int)blockIdx.x, (int)gridDim.x);
}

// Tile shapes: T steps per pass, R rows per lane, W wavefronts.
struct Variant {
    int T, R, W, mode;
    bool whole;  // for grids whose z axis is one wavefront
    void (*kern)(const SweepArgs);
};
#define V(T, R, W, M) {T, R, W, M, false, sweep_kernel<T, R, W, M, false>}
#define VW(T, W, M) {T, 1, W, M, true, sweep_kernel<T, 1, W, M, true>}
#define VW4(W, M) VW(1, W, M), VW(2, W, M), VW(3, W, M), VW(4, W, M)
#define V2(R, W, M) V(1, R, W, M), V(2, R, W, M)
#define V3(R, W, M) V2(R, W, M), V(3, R, W, M)
#define V4(R, W, M) V3(R, W, M), V(4, R, W, M)
#define V5(R, W, M) V4(R, W, M), V(5, R, W, M)
const Variant kVariants[] = {
    V5(2, 16, kTable),      V4(1, 16, kTable),
    V5(2, 16, kLossyTable), V4(1, 16, kLossyTable),
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


// One pass of T steps over a grid: the tile shape and the split of x.
struct Pass {
    const Variant* v = nullptr;
    int xchunk = 0, gz = 0, gy = 0;
    long long ntiles = 0;
    double us = 1e300;  // estimated
};

constexpr int kMaxT = 5;
constexpr double kCacheBytes = 256e6;  // Infinity Cache

int mode_of(const fdtd_ctx* c)
{
    const bool tab = c->use_mat && c->mat_id8 && c->ntab8 > 0;
    return c->ca[0] ? (tab ? kLossyTable : kLossy) : (tab ? kTable : kArrays);
}

// The fastest pass of T steps by a model of the time of one iteration of a
// block, fitted to measured passes from 64^3 to 1024 x 1024 x 512: with all
// CUs busy a block takes 0.5 us + 0.2 us per level + 0.125 us per level and 8
// rows, or the time its loads and stores take at 17.6 KB/us per CU (4.5 TB/s
// in all; 2.2 times that where the state sits in the Infinity Cache),
// whichever is longer; a chunk's 2T extra planes and the last round of blocks
// count in full.
Pass plan_pass(const fdtd_ctx* c, int mode, int T, int cus)
{
    Pass best;
    const int in_bytes = 24 + (mode == kArrays ? 12 : mode == kLossy ? 24 : 1);
    const bool cached = 24.0 * (double)c->ncell <= kCacheBytes;
    for (const Variant& v : kVariants) {
        if (v.T != T || v.mode != mode || (v.whole && c->nz != 64)) continue;
        const int rows = v.R * v.W, vz = v.whole ? 64 : 64 - 2 * T, vy = rows - 2 * T;
        Pass p;
        p.v = &v;
        p.gz = (c->nz + vz - 1) / vz;
        p.gy = (c->ny + vy - 1) / vy;
        const long long base = (long long)p.gz * p.gy;
        const double compute = 0.5 + T * (0.2 + rows / 64.0);
        const double memory = (rows * 64.0 * in_bytes + vy * vz * 24.0) / (cached ? 2.2 * 17600.0 : 17600.0);
        const double iter = std::max(compute, memory);
        int last = 0;
        for (int q = 1; q <= std::min(c->nx, 1024); ++q) {
            const int xc = (c->nx + q - 1) / q;
            if (xc == last) continue;
            last = xc;
            const long long nt = base * ((c->nx + xc - 1) / xc);
            const double us = (double)((nt + cus - 1) / cus) * (xc + 2 * T + 1) * iter + 5.0;
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
    Pass pass[kMaxT + 1];  // the plan of a pass of T steps, for `mode`
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

bool capturing(const fdtd_ctx* ctx)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

int plan(fdtd_ctx* ctx)
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
    const int mode = mode_of(ctx);
    if (S->mode != mode) {
        for (int T = 1; T <= kMaxT; ++T) S->pass[T] = plan_pass(ctx, mode, T, S->cus);
        S->mode = mode;
    }
    // Blocks are kept in step where the state is past 1 GiB: 512^3, T = 5,
    // 225 -> 256 G cell updates/s, 1024 x 1024 x 512 255 -> 269; at 256^3,
    // one round of blocks, 202 against 205.
    if (!S->pace && 24.0 * (double)ctx->ncell > 1.0737e9 && !capturing(ctx)) {
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

// Steps of the passes that advance n steps: as few as the cheapest split
// takes, lengths within one of each other, an even number of them when `even`.
int split(const SweepState* S, int64_t n, bool even, int64_t* passes)
{
    double best = 1e300;
    int64_t bp = 0;
    for (int T = 1; T <= kMaxT; ++T) {
        if (!S->pass[T].v) continue;
        int64_t p = (n + T - 1) / T;
        if (even && (p & 1)) ++p;
        if (p > n) continue;
        const int t = (int)(n / p);
        const int64_t longer = n % p;
        if (t + (longer ? 1 : 0) > kMaxT || !S->pass[t].v || (longer && !S->pass[t + 1].v)) continue;
        const double us = (double)(p - longer) * S->pass[t].us + (longer ? (double)longer * S->pass[t + 1].us : 0.0);
        if (us < best) {
            best = us;
            bp = p;
        }
    }
    *passes = bp;
    return bp > 0;
}

}  // namespace

// A plane must fit a buffer descriptor with room for the dropped offset.
bool sweep_supported(const fdtd_ctx* ctx)
{
    return ctx->storage == FDTD_FP32 && (uint64_t)ctx->ny * (uint64_t)ctx->nz * 4u < (uint64_t)kDropped;
}

bool sweep_ready(fdtd_ctx* ctx)
{
    if (!sweep_supported(ctx)) return false;
    bool have = true;
    for (int c = 0; c < 6; ++c) have = have && ctx->alt[c];
    if (have) return true;
    // a scheme that can do without the second field set takes it only where
    // three quarters of the free memory stay free
    if (capturing(ctx)) return false;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (24.0 * (double)ctx->ncell > 0.25 * (double)free_b) return false;
    if (sweep_prepare(ctx) == FDTD_OK) return true;
    for (int c = 0; c < 6; ++c) {
        if (ctx->alt[c]) (void)hipFree(ctx->alt[c]);
        ctx->alt[c] = nullptr;
    }
    return false;
}

int sweep_prepare(fdtd_ctx* ctx)
{
    const size_t bytes = (size_t)ctx->ncell * sizeof(float);
    for (int c = 0; c < 6; ++c)
        if (!ctx->alt[c]) {
            hipError_t e = hipMalloc(&ctx->alt[c], bytes);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                ctx->alt[c] = nullptr;
                return fail(ctx, FDTD_ENOMEM, "fused plain step: second field set does not fit");
            }
        }
    return plan(ctx);
}

int sweep_steps(fdtd_ctx* ctx, int64_t n, int kernel, bool even)
{
    int rc = sweep_prepare(ctx);
    if (rc) return rc;
    SweepState* S = ctx->sweep;
    int64_t passes = 0;
    if (!split(S, n, even && n > 1, &passes)) return fail(ctx, FDTD_EUNSUPPORTED, "sweep: no pass fits this call");
    SweepArgs A;
    A.cH = ctx->cH;
    A.nx = ctx->nx;
    A.ny = ctx->ny;
    A.nz = ctx->nz;
    for (int c = 0; c < 3; ++c) {
        A.cE[c] = ctx->coef[c];
        A.ca[c] = ctx->ca[c];
    }
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
        S->blocks = (int)((P.ntiles + kXCD - 1) / kXCD * kXCD);
    }
    for (int64_t p = 0; p < passes; ++p) {
        const int T = t0 + (p < longer ? 1 : 0);
        const Pass& P = S->pass[T];
        A.gz = P.gz;
        A.gy = P.gy;
        A.xchunk = P.xchunk;
        A.ntiles = (int)P.ntiles;
        for (int c = 0; c < 6; ++c) {
            A.in[c] = ctx->field[c];
            A.out[c] = ctx->alt[c];
        }
        A.step = ctx->step_count;
        A.pace = S->pace ? S->pace + (size_t)S->turn * S->pace_words : nullptr;
        A.pace_next = S->pace ? S->pace + (size_t)(S->turn ^ 1) * S->pace_words : nullptr;
        A.pace_words = S->pace_words;
        S->turn ^= 1;
        const unsigned blocks = (unsigned)((P.ntiles + kXCD - 1) / kXCD * kXCD);
        PendingTiming t;
        timing_begin(ctx, kernel, &t);
        hipLaunchKernelGGL(P.v->kern, dim3(blocks), dim3(64 * P.v->W), 0, ctx->stream, A);
        timing_end(ctx, &t);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(ctx, e, "launch(sweep)");
        for (int c = 0; c < 6; ++c) std::swap(ctx->field[c], ctx->alt[c]);
        ctx->step_count += T;
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
