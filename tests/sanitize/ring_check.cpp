// Host check of the systolic plan's distance bound (plan.cpp): never below the
// largest producer -> consumer distance of the plan itself.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "plan.h"

using namespace fdtd::plan;

int main()
{
    std::srand(3);
    int bad = 0;
    for (int q = 0; q < 220; ++q) {
        int N[3], per[3], W[3] = {q % 3 == 0 ? 11 : q % 3 == 1 ? 15 : 19, 15, 15};
        for (int d = 0; d < 3; ++d) {
            N[d] = q < 40 ? 1 + std::rand() % 20 : 16 + std::rand() % (q < 200 ? 150 : 500);
            per[d] = N[d] >= 16 && std::rand() % 3 == 0;
        }
        const int K = 1 + std::rand() % 64, nsteps = 1 + std::rand() % 200;
        Plan p;
        Merged m;
        std::string err;
        const Plan* one = &p;
        if (!build(N, per, W, nsteps, std::min(K, nsteps), &p, &err) || !merge(&one, 1, &m, &err)) return 2;
        const long long bound = distance_bound(N, per, W, std::min(K, nsteps));
        if (bound < m.D) {
            std::printf("%dx%dx%d per %d%d%d K %d steps %d: D %d, bound %lld\n", N[0], N[1], N[2], per[0], per[1], per[2],
                        K, nsteps, m.D, bound);
            ++bad;
        }
    }
    // the largest grid: the automatic band's rings do not fit, and the bound says so
    const int N[3] = {1024, 1024, 1024}, per[3] = {0, 0, 0}, W[3] = {19, 15, 15};
    const double bytes = (double)(distance_bound(N, per, W, 64) + 1024) * 64 * 6 * 1280;
    if (bytes < 4294967296.0) ++bad;
    if (bad) return 1;
    std::printf("ring checks passed\n");
    return 0;
}
