// The tile of a sweep (sweep.hip, sweep_adjoint.hip, sweep_batch.hip).
//
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
#pragma once

#include "fdtd_internal.h"
#include "sweep_plan.h"

namespace fdtd {
namespace sweep {

constexpr unsigned kDropped = 0x80000000u;  // a buffer offset past every plane: the access is dropped

// Level l of a pass is step n + l (forward) or n - l (reverse).  A cell of the
// design box, and in the forward run of the monitor box, belongs to the lane
// that stores it; it adds to the transform once per level, in the order of the
// levels, by adds that return nothing.  The records only leave the kernel, so
// no level waits for memory.
struct HookArgs {
    int dlo[3], dn[3], mlo[3], mn[3];
    int comp;
    double cr[kMaxT], ci[kMaxT];  // exp(-i omega n dt) of the levels
    double* F;
    float* hist;       // the record of level 0 (null: none)
    long long stride;  // from the record of a level to that of the next
};

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
    // ordered by plane; more of them than a block keeps at hand are followed by
    // the first one of each plane (nx + 1 ints)
    const DevSource* src;
    int nsrc;
    long long step;
    unsigned* pace;       // progress marks of this pass (null: not kept in step)
    unsigned* pace_next;  // those of the next pass, cleared by this one
    int pace_words;
};

// The kernels of the adjoint's passes, in the order of their shapes
// (sweep_adjoint.hip).
using HookedKernel = void (*)(const SweepArgs, const HookArgs);
HookedKernel hooked_kernel_of(int index);
// Coefficients a context's sweeps read.
int mode_of(const fdtd_ctx* c);
SweepArgs base_args(const fdtd_ctx* ctx);

}  // namespace sweep

using namespace sweep;

namespace {

template <int T, int R, int W, int MODE>
struct Lds {
    static constexpr bool TAB = MODE == kTable || MODE == kLossyTable;
    static constexpr int kList = kListedSources;  // sources a block keeps at hand
    float2 hx0[2][W][64];                  // (Hx, Hz) of a wavefront's top row, level 0
    float2 hx[T > 1 ? T - 1 : 1][W][64];   // and levels 1 ..
    float2 ex[2][T][W][64];
    float4 tab[TAB ? kMaxMaterials : 1];
    float4 tabA[MODE == kLossyTable ? kMaxMaterials : 1];
    unsigned ids[TAB ? T : 1][(R + 3) / 4][64 * W];
    // a source: its plane and byte offset in it; bits 0..1 its component,
    // bit 8 + l whether it has a sample for level l; the samples
    int plane[kList], cell[kList], what[kList];
    float sample[T][kList];
    int nlist;
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

template <int T, int R, int W, int MODE, bool WHOLE, int HOOK>
__device__ __forceinline__ void sweep_tile(const SweepArgs& A, const HookArgs& K,
                                           Lds<T, R, W, MODE>& S, int xcd, int slot, int per_xcd)
{
    static_assert(W * R > 2 * T && 64 > 2 * T, "the tile keeps at least one cell");
    static_assert(HOOK == kUpdate || MODE == kArrays || MODE == kLossy, "the hooks read the arrays");
    constexpr bool BOXES = HOOK == kForward || HOOK == kReverse;
    constexpr bool BACK = HOOK == kReverse || HOOK == kTransposed;
    constexpr int NS = T + 2;
    constexpr bool TAB = MODE == kTable || MODE == kLossyTable;
    constexpr bool LOSSY = MODE == kLossy || MODE == kLossyTable;
    constexpr int NC = LOSSY ? 6 : 3;  // coefficients per cell
    constexpr int NP = (R + 3) / 4;    // words of packed indices per plane and lane
    constexpr int kList = Lds<T, R, W, MODE>::kList;
    const int tile = xcd * per_xcd + slot;
    const int tz = tile % A.gz, ty = (tile / A.gz) % A.gy, tx = tile / (A.gz * A.gy);
    const int L = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int k0 = WHOLE ? 0 : tz * (64 - 2 * T) - T, j0 = ty * (W * R - 2 * T) - T;
    const int x0 = tx * A.xchunk, x1 = min(A.nx, x0 + A.xchunk);
    const int nit = x1 - x0 + 2 * T;
    const int k = wrap(k0 + L, A.nz);
    // the lanes and rows that the tile stores
    const unsigned long long kown = __ballot(WHOLE || (L >= T && L < 64 - T && k0 + L < A.nz));
    auto jown = [&](int r) { return w * R + r >= T && w * R + r < W * R - T && j0 + w * R + r < A.ny; };
    // Byte offsets of the lane's cells in a plane.  The tile that fills the
    // registers adds a scalar offset per row to one of the lane instead (with
    // an offset per row it spills, and a spill waits for the planes in flight:
    // 256^3 74 -> 93 us per step; where there is room the scalar offsets cost
    // up to 8%).
    constexpr bool SOFF = T == 5 && R == 3;
    unsigned vo[SOFF ? 1 : R], so[SOFF ? R : 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int rr = w * R + r;
        const unsigned row = (unsigned)wrap(j0 + rr, A.ny) * (unsigned)A.nz * 4u;
        vo[SOFF ? 0 : r] = (unsigned)k * 4u + (SOFF ? 0u : row);
        so[SOFF ? r : 0] = SOFF ? row : 0u;
    }
    const unsigned pbytes = (unsigned)A.ny * (unsigned)A.nz * 4u;
    // the lane's cells in the design and monitor boxes: index within a plane of
    // the box, or -1 (not there; the design box and the forward run's monitor
    // count a cell where it is stored, the reverse run's monitor samples go to
    // every copy of a cell)
    constexpr int BR = BOXES ? R : 1;
    int qd[BR], qm[BR];
    if (BOXES) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int j = wrap(j0 + w * R + r, A.ny), jd = j - K.dlo[1], kd = k - K.dlo[2];
            const int jm = j - K.mlo[1], km = k - K.mlo[2];
            const bool mine = (kown >> L & 1) && jown(r), meets = mine || HOOK == kReverse;
            qd[r % BR] = mine && jd >= 0 && jd < K.dn[1] && kd >= 0 && kd < K.dn[2] ? jd * K.dn[2] + kd : -1;
            qm[r % BR] = meets && jm >= 0 && jm < K.mn[1] && km >= 0 && km < K.mn[2] ? jm * K.mn[2] + km : -1;
        }
    }
    const long long ndes = BOXES ? (long long)K.dn[0] * K.dn[1] * K.dn[2] : 0;
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
    auto ld = [&](const void* base, int plane, int r) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc(base, plane, pbytes), (int)vo[SOFF ? 0 : r], (int)so[SOFF ? r : 0], 0));
    };
    int pin = wrap(x0 - T, A.nx);  // grid plane of the next load
    auto load = [&](int s) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) H[s][r][c] = ld(A.in[3 + c], pin, r);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) E[s][r][c] = ld(A.in[c], pin, r);
        if (TAB) {
            const auto ri = rsrc(A.id, pin, pbytes >> 2);
#pragma unroll
            for (int r = 0; r < R; ++r)
                ci[r] = (unsigned char)__builtin_amdgcn_raw_buffer_load_b8(ri, (int)(vo[SOFF ? 0 : r] >> 2), (int)(so[SOFF ? r : 0] >> 2), 0);
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    C[s % CS][r % CR][c % CC] = ld(c < 3 ? A.cE[c % 3] : A.ca[c % 3], pin, r);
        }
        pin = pin + 1 == A.nx ? 0 : pin + 1;
    };
    load(0);
    if (TAB) {
        for (int q = threadIdx.x; q < A.ntab; q += 64 * W) {
            const float* t = A.tab + q * NC;
            S.tab[q] = make_float4(t[0], t[1], t[2], 0.f);
            if (MODE == kLossyTable) S.tabA[q] = make_float4(t[NC - 3], t[NC - 2], t[NC - 1], 0.f);
        }
#pragma unroll
        for (int d = 0; d < T; ++d)
#pragma unroll
            for (int q = 0; q < NP; ++q) S.ids[d][q][threadIdx.x] = 0u;
    }
    // the sources this block meets, in table order (several on one cell add up
    // in the same order as in any other scheme); of many, only those of its
    // planes are looked at, and no more once there are too many
    int nhit = 0;
    if (A.nsrc > 0) {
        if (w == 0) {
            int n = 0, b0 = 0, b1 = A.nsrc, rest = 0;
            if (A.nsrc > kList && nit < A.nx) {
                const int* const at = (const int*)(A.src + A.nsrc);
                const int first = wrap(x0 - T, A.nx), end = first + nit;
                b0 = at[first];
                b1 = at[min(end, A.nx)];
                rest = end > A.nx ? at[end - A.nx] : 0;
            }
            for (int b = b0; n <= kList; b += 64) {
                if (b >= b1) {
                    // (a chunk that passes the last plane goes on at the first)
                    if (rest == 0) break;
                    b = 0;
                    b1 = rest;
                    rest = 0;
                }
                const int q = b + L;
                bool hit = false;
                if (q < b1) {
                    const DevSource s = A.src[q];
                    hit = wrap(s.k - k0, A.nz) < 64 && wrap(s.j - j0, A.ny) < W * R &&
                          wrap(s.i - (x0 - T), A.nx) < nit && A.step + T > s.first && A.step - s.first < s.len;
                }
                const unsigned long long m = __ballot(hit);
                const int at = n + __popcll(m & ((1ull << L) - 1));
                if (hit && at < kList) {
                    const DevSource s = A.src[q];
                    int what = s.comp;
#pragma unroll
                    for (int l = 0; l < T; ++l) {
                        const long long i = A.step + l - s.first;
                        if (i < 0 || i >= s.len) continue;
                        what |= 256 << l;
                        S.sample[l][at] = s.wave[i];
                    }
                    S.plane[at] = s.i;
                    S.cell[at] = (int)(((unsigned)s.j * (unsigned)A.nz + (unsigned)s.k) * 4u);
                    S.what[at] = what;
                }
                n += __popcll(m);
            }
            if (L == 0) S.nlist = n;
        }
        __syncthreads();
        nhit = __builtin_amdgcn_readfirstlane(S.nlist);
    }
    // lane e of every wavefront holds the plane of entry e
    const int lsi = nhit <= kList && L < nhit ? S.plane[L] : -1;
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
                    S.ids[ring][q][threadIdx.x] = pk[q];
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
            S.hx0[par][w][L] = make_float2(H[u][R - 1][0], H[u][R - 1][2]);
#pragma unroll
            for (int l = 0; l < T; ++l) {
                const int s0 = (u - l + NS) % NS, s1 = (u - l - 1 + NS) % NS;
                // Until it = 2l no stored value depends on level l.  (An
                // iteration may then have one barrier alone: what level 0 and
                // the E rows exchange alternates between two buffers.)
                if (it < 2 * l) break;
                if (TAB && l > 0) {
                    const int q0 = ring - l < 0 ? ring - l + T : ring - l;
#pragma unroll
                    for (int q = 0; q < NP; ++q) pk[q] = S.ids[q0][q][threadIdx.x];
                }
                lds_barrier();
                const float2 hl = l == 0 ? S.hx0[par][w == 0 ? 0 : w - 1][L] : S.hx[l > 0 ? l - 1 : 0][w == 0 ? 0 : w - 1][L];
                const float2 eu = S.ex[par ^ 1][l][w == W - 1 ? w : w + 1][L];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float hx = H[s0][r][0], hy = H[s0][r][1], hz = H[s0][r][2];
                    const float hx_jm = r ? H[s0][r - 1][0] : hl.x, hz_jm = r ? H[s0][r - 1][2] : hl.y;
                    const float hx_km = from_below<WHOLE>(hx), hy_km = from_below<WHOLE>(hy);
                    const float hy_im = H[s1][r][1], hz_im = H[s1][r][2];
                    if (HOOK == kForward && K.hist) {
                        const int p = it - l, id = x0 + p - T - K.dlo[0];
                        if (p >= T && p < nit - T && id >= 0 && id < K.dn[0] && qd[r % BR] >= 0) {
                            float* o = K.hist + l * K.stride + (long long)id * K.dn[1] * K.dn[2] + qd[r % BR];
                            o[0] = (hz - hz_jm) - (hy - hy_km);
                            o[ndes] = (hx - hx_km) - (hz - hz_im);
                            o[2 * ndes] = (hy - hy_im) - (hx - hx_jm);
                            if (LOSSY) {
                                o[3 * ndes] = E[s0][r][0];
                                o[4 * ndes] = E[s0][r][1];
                                o[5 * ndes] = E[s0][r][2];
                            }
                        }
                    }
                    if (BACK) {
                        const float* cc = C[s0 % CS][r % CR];
                        const float dx = (hz - hz_jm) - (hy - hy_km), dy = (hx - hx_km) - (hz - hz_im),
                                    dz = (hy - hy_im) - (hx - hx_jm);
                        E[s0][r][0] = (LOSSY ? cc[3 % CC] * E[s0][r][0] : E[s0][r][0]) - A.cH * dx;
                        E[s0][r][1] = (LOSSY ? cc[4 % CC] * E[s0][r][1] : E[s0][r][1]) - A.cH * dy;
                        E[s0][r][2] = (LOSSY ? cc[5 % CC] * E[s0][r][2] : E[s0][r][2]) - A.cH * dz;
                        continue;
                    }
                    float cx, cy, cz;
                    float ex = E[s0][r][0], ey = E[s0][r][1], ez = E[s0][r][2];
                    if (TAB) {
                        const unsigned id = pk[r / 4] >> (8 * (r % 4)) & 255u;
                        const float4 t = S.tab[id];
                        cx = t.x;
                        cy = t.y;
                        cz = t.z;
                        if (MODE == kLossyTable) {
                            const float4 a = S.tabA[id];
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
                    auto add = [&](int c, unsigned cell, float v) {
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            if (SOFF ? vo[0] == cell - so[SOFF ? r : 0] : vo[SOFF ? 0 : r] == cell) {
                                E[s0][r][0] = c == 0 ? E[s0][r][0] + v : E[s0][r][0];
                                E[s0][r][1] = c == 1 ? E[s0][r][1] + v : E[s0][r][1];
                                E[s0][r][2] = c == 2 ? E[s0][r][2] + v : E[s0][r][2];
                            }
                    };
                    if (nhit <= kList) {
                        unsigned long long m = __ballot(lsi == pl);
                        while (m) {
                            const int e = __ffsll((long long)m) - 1;
                            m &= m - 1;
                            const int what = S.what[e];
                            if (what >> (8 + l) & 1) add(what & 3, (unsigned)S.cell[e], S.sample[l][e]);
                        }
                    } else {
                        // Too many to keep: those of this plane.  (Through the
                        // whole table, 4096 sources on a plane of 64^3 took
                        // 5500 us per step, this way 147.)
                        const int* const at = (const int*)(A.src + A.nsrc) + pl;
                        for (int q = at[0]; q < at[1]; ++q) {
                            const DevSource s = A.src[q];
                            const long long i = A.step + l - s.first;
                            if (i >= 0 && i < s.len)
                                add(s.comp, ((unsigned)s.j * (unsigned)A.nz + (unsigned)s.k) * 4u, s.wave[i]);
                        }
                    }
                }
                if (BOXES) {
                    const int p = it - l, im = wrap(pe - l, A.nx) - K.mlo[0], id = x0 + p - T - K.dlo[0];
                    const bool mine = p >= T && p < nit - T;
                    if ((mine || HOOK == kReverse) && im >= 0 && im < K.mn[0])
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            if (qm[r % BR] < 0) continue;
                            double* f = K.F + 2 * ((long long)im * K.mn[1] * K.mn[2] + qm[r % BR]);
                            if (HOOK == kForward) {
                                const double e = (double)(K.comp == 0 ? E[s0][r][0] : K.comp == 1 ? E[s0][r][1] : E[s0][r][2]);
                                unsafeAtomicAdd(f, e * K.cr[l]);
                                unsafeAtomicAdd(f + 1, e * K.ci[l]);
                            } else {
                                const double v = 2.0 * (f[0] * K.cr[l] + f[1] * K.ci[l]);
#pragma unroll
                                for (int c = 0; c < 3; ++c)
                                    E[s0][r][c] = K.comp == c ? (float)((double)E[s0][r][c] + v) : E[s0][r][c];
                            }
                        }
                    if (HOOK == kReverse && mine && id >= 0 && id < K.dn[0])
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            if (qd[r % BR] < 0) continue;
                            float* o = K.hist + l * K.stride + (long long)id * K.dn[1] * K.dn[2] + qd[r % BR];
#pragma unroll
                            for (int c = 0; c < 3; ++c) o[c * ndes] = E[s0][r][c];
                        }
                }
                if (BACK) {
                    // H += CE(w), w = cE (.) E: the neighbours exchange w
                    const float* c0 = C[s0 % CS][0];
                    S.ex[par][l][w][L] = make_float2(c0[0] * E[s0][0][0], c0[2 % CC] * E[s0][0][2]);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        constexpr int last = R - 1;
                        const int rn = r < last ? r + 1 : r;
                        const float* c1 = C[s1 % CS][r % CR];
                        const float* cn = C[s1 % CS][rn % CR];
                        const float* cp = C[s0 % CS][r % CR];
                        const float wx = c1[0] * E[s1][r][0], wy = c1[1 % CC] * E[s1][r][1], wz = c1[2 % CC] * E[s1][r][2];
                        const float wx_jp = r < last ? cn[0] * E[s1][rn][0] : eu.x;
                        const float wz_jp = r < last ? cn[2 % CC] * E[s1][rn][2] : eu.y;
                        const float wy_kp = from_above<WHOLE>(wy), wx_kp = from_above<WHOLE>(wx);
                        const float wy_ip = cp[1 % CC] * E[s0][r][1], wz_ip = cp[2 % CC] * E[s0][r][2];
                        H[s1][r][0] += (wz_jp - wz) - (wy_kp - wy);
                        H[s1][r][1] += (wx_kp - wx) - (wz_ip - wz);
                        H[s1][r][2] += (wy_ip - wy) - (wx_jp - wx);
                    }
                    if (l + 1 < T) S.hx[l + 1 < T ? l : 0][w][L] = make_float2(H[s1][R - 1][0], H[s1][R - 1][2]);
                    continue;
                }
                S.ex[par][l][w][L] = make_float2(E[s0][0][0], E[s0][0][2]);
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
                if (l + 1 < T) S.hx[l + 1 < T ? l : 0][w][L] = make_float2(H[s1][R - 1][0], H[s1][R - 1][2]);
            }
            if (it >= 2 * T) {
                const int s = (u - T + NS) % NS;
                const int plane = x0 + it - 2 * T;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const unsigned sr = __builtin_amdgcn_inverse_ballot_w64(jown(r) ? kown : 0ull) ? vo[SOFF ? 0 : r] : kDropped;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, E[s][r][c]),
                                                              rsrc(A.out[c], plane, pbytes), (int)sr, (int)so[SOFF ? r : 0], 2);
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, H[s][r][c]),
                                                              rsrc(A.out[3 + c], plane, pbytes), (int)sr, (int)so[SOFF ? r : 0], 2);
                    }
                }
            }
            pe = pe + 1 == A.nx ? 0 : pe + 1;
            ring = ring + 1 == T ? 0 : ring + 1;
        }
    }
}

// The block's place: launch order is dealt round the XCDs, tiles are
// contiguous per XCD.  Clears its share of the next pass's progress marks.
// False: no tile for it.
__device__ __forceinline__ bool place(const SweepArgs& A, int& xcd, int& slot, int& per_xcd)
{
    per_xcd = (int)gridDim.x / kXCD;
    xcd = (int)blockIdx.x % kXCD;
    slot = (int)blockIdx.x / kXCD;
    if (A.pace_next) {
        const int each = (A.pace_words + (int)gridDim.x - 1) / (int)gridDim.x;
        for (int q = threadIdx.x; q < each; q += (int)blockDim.x)
            if ((int)blockIdx.x * each + q < A.pace_words) A.pace_next[(int)blockIdx.x * each + q] = 0u;
    }
    return xcd * per_xcd + slot < A.ntiles;
}

}  // namespace
}  // namespace fdtd
