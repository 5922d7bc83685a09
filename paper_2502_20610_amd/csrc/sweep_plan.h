// Host-side plan of a sweep (sweep.hip): the tile shapes there are, the pass of
// T steps that a model of its time picks, and the progress marks a pass needs.
// Plain C++ (no HIP types), so that it also builds for the host alone.
#pragma once

namespace fdtd {
namespace sweep {

constexpr int kXCD = 8;         // XCDs of the device
constexpr int kPaceGroup = 32;  // blocks an XCD runs at once (one per CU)
constexpr int kPacePlanes = 4;  // planes between two progress marks
constexpr int kMaxT = 5;        // steps of a pass

// What a sweep reads as coefficients.
enum { kArrays = 0, kLossy = 1, kTable = 2, kLossyTable = 3, kModes = 4 };
// What a pass computes: the update; the update with what the forward run of
// the adjoint takes from it (monitor transform, design-box history); the
// transposed half-steps of the reverse run,
//   lE = A (.) lE - cH CH(lH),  lH += CE(cE (.) lE),
// with the monitor samples of the step added to lE and lE recorded over the
// design box, or without either.  A block that meets neither box runs the
// plain form of its pass.
enum { kUpdate = 0, kForward = 1, kReverse = 2, kTransposed = 3 };

// Tile shapes: T steps per pass, R rows per lane, W wavefronts; `whole` for
// grids whose z axis is one wavefront.  V(T, R, W, mode) and VW(T, W, mode)
// are the plain sweeps, VH(T, R, W, mode) the adjoint's, forward and reverse.
#define FDTD_SWEEP_V2(V, R, W, M) V(1, R, W, M) V(2, R, W, M)
#define FDTD_SWEEP_V3(V, R, W, M) FDTD_SWEEP_V2(V, R, W, M) V(3, R, W, M)
#define FDTD_SWEEP_V4(V, R, W, M) FDTD_SWEEP_V3(V, R, W, M) V(4, R, W, M)
#define FDTD_SWEEP_V5(V, R, W, M) FDTD_SWEEP_V4(V, R, W, M) V(5, R, W, M)
#define FDTD_SWEEP_VW4(VW, W, M) VW(1, W, M) VW(2, W, M) VW(3, W, M) VW(4, W, M)
#define FDTD_SWEEP_SHAPES(V, VW)                                                                            \
    FDTD_SWEEP_V5(V, 3, 12, kTable) FDTD_SWEEP_V4(V, 2, 16, kTable) FDTD_SWEEP_V4(V, 1, 16, kTable)         \
    FDTD_SWEEP_V4(V, 3, 12, kLossyTable) FDTD_SWEEP_V5(V, 2, 16, kLossyTable)                               \
    FDTD_SWEEP_V4(V, 1, 16, kLossyTable)                                                                    \
    FDTD_SWEEP_V4(V, 4, 8, kArrays) FDTD_SWEEP_V3(V, 2, 16, kArrays) FDTD_SWEEP_V4(V, 1, 16, kArrays)       \
    FDTD_SWEEP_V3(V, 3, 8, kLossy) FDTD_SWEEP_V2(V, 2, 16, kLossy) FDTD_SWEEP_V4(V, 1, 16, kLossy)          \
    FDTD_SWEEP_VW4(VW, 16, kTable) FDTD_SWEEP_VW4(VW, 16, kArrays) FDTD_SWEEP_VW4(VW, 16, kLossyTable)      \
    FDTD_SWEEP_VW4(VW, 16, kLossy)
#define FDTD_SWEEP_HOOKED_SHAPES(VH)                                                                        \
    FDTD_SWEEP_V4(VH, 1, 16, kArrays) VH(2, 4, 8, kArrays) VH(3, 4, 8, kArrays)                             \
    FDTD_SWEEP_V3(VH, 1, 16, kLossy) VH(2, 3, 8, kLossy) VH(3, 3, 8, kLossy)

struct Shape {
    int T, R, W, mode;
    bool whole;
    int hook;
};

// One pass of T steps over a grid: the tile shape and the split of x.
struct Pass {
    const Shape* s = nullptr;
    int index = -1;  // of the shape's kernel in its list
    int xchunk = 0, gz = 0, gy = 0;
    long long ntiles = 0;
    double us = 1e300;  // estimated
};

bool fits_cache(int mode, double cells);
// Time of one round of blocks of `rows` rows over xc planes, us: the larger of
// what the levels and what the memory take.
double round_us(int mode, int rows, int T, int xc, bool cached);

// The best pass of T steps over a grid of N cells per axis on `cus` CUs
// (s null: no shape has that T).
Pass plan_pass(const int N[3], int mode, int hook, int T, int cus);

// Estimates by which a call chooses between sweeps and a scheme's own launches
// (fitted to both sides measured in turn on 340 thin, short and ordinary calls;
// the choice is right or within 4% of it on all but five, the worst 0.79):
// a pass alone on the device, counting what its tiles touch of a thin grid;
// n steps of two launches each, in place; one step in one launch (plain.hip).
double alone_us(const Pass& p, const int N[3], int cus);
double in_place_us(const int N[3], bool lossy, long long n);
double one_step_us(const int N[3], bool lossy);

// Whether the persistent launch is the faster of the two on a grid that is thin
// along z (`periodic` along any axis), in a call of n steps.
bool thin_for_sweeps(const int N[3], bool periodic, int mode, bool half, long long n);

// Words of progress marks that a pass of this plan addresses, and the most that
// any plan of the grid does, whatever coefficients the context is given.
long long mark_words(const Pass& p);
long long most_mark_words(const int N[3], int cus);

}  // namespace sweep
}  // namespace fdtd
