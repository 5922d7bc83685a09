// Host checks of the sweep's plan (sweep_plan.cpp): every tile shape splits the
// grid without gaps, and no block addresses progress marks past the ones that
// are allocated once per context, whatever coefficients it is given.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "sweep_plan.h"

using namespace fdtd::sweep;

static int failures = 0;
#define CHECK(c, ...)                 \
    do {                              \
        if (!(c)) {                   \
            std::printf(__VA_ARGS__); \
            std::printf("\n");        \
            ++failures;               \
        }                             \
    } while (0)

// The largest index + 1 that any block of the pass marks (the kernel's
// arithmetic, block by block).
static long long words_addressed(const Pass& p, int nx)
{
    const int T = p.s->T;
    const long long blocks = (p.ntiles + kXCD - 1) / kXCD * kXCD, per_xcd = blocks / kXCD;
    long long top = 0;
    for (long long b = 0; b < blocks; ++b) {
        const long long xcd = b % kXCD, slot = b / kXCD, tile = xcd * per_xcd + slot;
        if (tile >= p.ntiles) continue;
        const long long tx = tile / ((long long)p.gz * p.gy);
        const int x0 = (int)tx * p.xchunk, nit = std::min(nx, x0 + p.xchunk) - x0 + 2 * T;
        CHECK(x0 < nx, "an empty chunk");
        const long long group = xcd * ((per_xcd + kPaceGroup - 1) / kPaceGroup) + slot / kPaceGroup;
        const long long marks = group * ((p.xchunk + 2 * T) / kPacePlanes + 1);
        top = std::max(top, marks + (nit - 1) / kPacePlanes + 1);
    }
    return top;
}

int main()
{
    int grids[][3] = {{1, 1, 1},       {64, 64, 64},      {63, 17, 130},   {256, 256, 256},  {356, 356, 356},
                      {400, 400, 400}, {512, 512, 512},   {512, 448, 384}, {1024, 1024, 512}, {1024, 1024, 1024},
                      {7, 2600, 2600}, {2600, 7, 2600},   {2600, 2600, 7}, {100000, 21, 23}, {3, 3, 5000000},
                      {0, 0, 0},       {0, 0, 0},         {0, 0, 0},       {0, 0, 0},        {0, 0, 0}};
    std::srand(5);
    for (auto& g : grids)
        if (g[0] == 0)
            for (int d = 0; d < 3; ++d) g[d] = 16 + std::rand() % 700;
    for (const auto& N : grids)
        for (int cus : {256, 304, 64}) {
            const long long held = most_mark_words(N, cus);
            for (int hook : {kUpdate, kForward, kReverse})
                for (int mode = 0; mode < kModes; ++mode)
                    for (int T = 1; T <= kMaxT; ++T) {
                        const Pass p = plan_pass(N, mode, hook, T, cus);
                        if (!p.s) continue;
                        const int vz = p.s->whole ? 64 : 64 - 2 * T, vy = p.s->R * p.s->W - 2 * T;
                        const long long chunks = (N[0] + p.xchunk - 1) / p.xchunk;
                        CHECK(p.s->T == T && p.s->mode == mode && p.s->hook == hook, "another shape than asked for");
                        CHECK((long long)p.gz * vz >= N[2] && (long long)p.gy * vy >= N[1] && vy > 0, "rows or lanes left out");
                        CHECK(p.ntiles == chunks * p.gz * p.gy, "%lld tiles", p.ntiles);
                        CHECK(!p.s->whole || N[2] == 64, "a whole-axis tile on %d lanes", N[2]);
                        if (hook != kUpdate || p.ntiles > 2000000) continue;
                        const long long need = words_addressed(p, N[0]);
                        CHECK(need <= mark_words(p), "%dx%dx%d mode %d T %d: %lld words addressed, %lld counted", N[0],
                              N[1], N[2], mode, T, need, mark_words(p));
                        CHECK(need <= held, "%dx%dx%d mode %d T %d: %lld words addressed, %lld held", N[0], N[1], N[2],
                              mode, T, need, held);
                    }
        }
    if (failures) return 1;
    std::printf("sweep plan checks passed\n");
    return 0;
}
