// Host-side plan of a sweep (see sweep_plan.h).
#include "sweep_plan.h"

#include <algorithm>

namespace fdtd {
namespace sweep {

namespace {

#define V(T, R, W, M) {T, R, W, M, false, kUpdate},
#define VW(T, W, M) {T, 1, W, M, true, kUpdate},
#define VH(T, R, W, M) {T, R, W, M, false, kForward}, {T, R, W, M, false, kReverse},
const Shape kShapes[] = {FDTD_SWEEP_SHAPES(V, VW)};
const Shape kHookedShapes[] = {FDTD_SWEEP_HOOKED_SHAPES(VH)};
#undef V
#undef VW
#undef VH

int in_bytes(int mode) { return 24 + (mode == kArrays ? 12 : mode == kLossy ? 24 : 1); }

}  // namespace

bool fits_cache(int mode, double cells) { return (24.0 + in_bytes(mode)) * cells <= 256e6; }

namespace {

// As round_us for tiles of `rows` rows that touch `met` rows and `lanes` lanes
// of the grid.
double tile_us(int mode, int rows, int T, int xc, bool cached, int met, int lanes)
{
    const double level = 0.11 + 0.29 * rows / 16.0;
    const double out = (double)std::max(1, std::min(met, rows - 2 * T)) * std::min(lanes, 64 - 2 * T);
    const double bytes = (double)met * lanes * in_bytes(mode) + out * 24.0;
    // (level l starts at iteration 2l)
    const double compute = 0.45 * (xc + 2 * T) + level * (T * (T + 1) + (double)xc * T);
    return std::max(compute, bytes / (cached ? 2.2 * 17600.0 : 17600.0) * (xc + 2 * T));
}

}  // namespace

double round_us(int mode, int rows, int T, int xc, bool cached)
{
    return tile_us(mode, rows, T, xc, cached, rows, 64);
}

// The model of a block's time, fitted to passes measured from 32^3 to 1024 x
// 1024 x 512 (within 20%): 3 us for the launch; per iteration 0.45 us and, for
// each level that runs, 0.11 us + 0.29 us per 16 rows; or the time the loads
// and stores of the iterations take at 17.6 KB/us per CU (4.5 TB/s in all; 2.2
// times that where everything sits in the Infinity Cache), if that is longer;
// the last round of blocks counts in full.  Where a pass does not fill the
// device, fewer blocks leave room for another context's (three contexts in
// turn, 48^3: chunks of one plane 3.3 us per step, of two 2.1, and 4.4 for
// either alone): the blocks of a full device count 0.6 more.
Pass plan_pass(const int N[3], int mode, int hook, int T, int cus)
{
    Pass best;
    const bool cached = fits_cache(mode, (double)N[0] * N[1] * N[2]);
    const Shape* const all = hook == kUpdate ? kShapes : kHookedShapes;
    const int n = (int)(hook == kUpdate ? sizeof(kShapes) : sizeof(kHookedShapes)) / (int)sizeof(Shape);
    for (int i = 0; i < n; ++i) {
        const Shape& v = all[i];
        if (v.T != T || v.mode != mode || v.hook != hook || (v.whole && N[2] != 64)) continue;
        const int rows = v.R * v.W, vz = v.whole ? 64 : 64 - 2 * T, vy = rows - 2 * T;
        Pass p;
        p.s = &v;
        p.index = i;
        p.gz = (N[2] + vz - 1) / vz;
        p.gy = (N[1] + vy - 1) / vy;
        const long long base = (long long)p.gz * p.gy;
        int last = 0;
        for (int q = 1; q <= std::min(N[0], 1024); ++q) {
            const int xc = (N[0] + q - 1) / q;
            if (xc == last) continue;
            last = xc;
            const long long nt = base * ((N[0] + xc - 1) / xc);
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

double alone_us(const Pass& p, const int N[3], int cus)
{
    const int rows = p.s->R * p.s->W;
    const bool cached = fits_cache(p.s->mode, (double)N[0] * N[1] * N[2]);
    const double round = tile_us(p.s->mode, rows, p.s->T, p.xchunk, cached, std::min(rows, N[1] + 8), std::min(64, N[2] + 16));
    return ((double)((p.ntiles + cus - 1) / cus) * round + 3.0) * (1.0 + 0.2 * std::min(1.0, (double)p.ntiles / cus));
}

double in_place_us(const int N[3], bool lossy, long long n)
{
    // 84 B per cell (96 with conductivity) at 4.7 TB/s, 6.3 where the arrays stay
    // in the Infinity Cache; 0.235 ns per row of 64 lanes in blocks of four rows;
    // 11 us where launches queue, 7 in a replayed graph
    const double cells = (double)N[0] * N[1] * N[2];
    const double rate = (lossy ? 48.0 : 36.0) * cells <= 256e6 ? 6.3e6 : 4.7e6;
    const double waves = (double)N[0] * ((N[1] + 3) / 4 * 4) * ((N[2] + 63) / 64);
    return (double)n * std::max(n < 16 ? 11.0 : 7.0, 5.0 + std::max(waves * 0.000235, (lossy ? 96.0 : 84.0) * cells / rate));
}

double one_step_us(const int N[3], bool lossy)
{
    // 256^3 247 us (conductive 277), 384^3 749 (876), 512^3 1921 (2317); 64^3 and
    // below 22 (5); thin along z 0.55 (0.33) ns per row of 64 lanes
    const double cells = (double)N[0] * N[1] * N[2];
    const double waves = (double)N[0] * ((N[1] + 6) / 7 * 8) * ((N[2] + 63) / 64);
    return lossy ? std::max(4.0 + 72.0 * cells / 4.3e6, waves * 0.00033) : std::max(25.0 + 60.0 * cells / 4.2e6, waves * 0.00055);
}

// A wavefront of a sweep is 64 lanes of z, a tile of the persistent launch 15
// cells; that launch pays for filling its pipeline of tiles, so what counts is
// its area times the steps.  Persistent / sweep in us, materials in a table
// (as arrays): 1024 x 1024 x 4, 20 steps 3170 / 3570 (3400 / 3850), x 16 4130 /
// 4670 (4490 / 5680), x 24 5280 / 4720 (5360 / 5430); 512 x 512 x 8, 20 steps
// 1280 / 1190, 64 steps 3380 / 4350; 1024 x 1024 x 8, 5 steps 1660 / 1310;
// 1500 x 1500 x 20, 12 steps 5360 / 6900 (5580 / 8390).
// Periodic axes have no pipeline to fill, and that launch is the faster in short
// calls: 1024 x 1024 x 1 with periodic y, 5 steps 630 / 815 us, x 16 1320 / 1430
// (x 4 830 / 750); 20 steps 1.16 to 1.34 times as long as sweeps.
bool thin_for_sweeps(const int N[3], bool periodic, int mode, bool half, long long n)
{
    const double area = (double)N[0] * N[1] * (double)n;
    const int nz = N[2];
    if (periodic) return nz <= 16 && n <= 8 && (double)N[0] * N[1] >= 262144.0;
    if (mode == kLossyTable) return nz <= 8 && n >= 12 && area >= 16e6;
    if (nz > (n > 24 ? (mode == kArrays ? 8 : 16) : (mode == kTable ? 24 : 28))) return false;
    if (nz < 6) return n >= 12 && area >= 10e6;
    return area >= ((mode == kLossy || half) && n >= 20 && nz <= 16 ? 4e6 : 10e6);
}

long long mark_words(const Pass& p)
{
    if (!p.s) return 0;
    const long long groups = ((p.ntiles + kXCD - 1) / kXCD + kPaceGroup - 1) / kPaceGroup * kXCD;
    return groups * ((p.xchunk + 2 * p.s->T) / kPacePlanes + 1);
}

long long most_mark_words(const int N[3], int cus)
{
    long long words = 0;
    for (int mode = 0; mode < kModes; ++mode)
        for (int T = 1; T <= kMaxT; ++T) words = std::max(words, mark_words(plan_pass(N, mode, kUpdate, T, cus)));
    return words;
}

}  // namespace sweep
}  // namespace fdtd
