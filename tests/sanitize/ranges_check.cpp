// Host check of writable_at_once (ranges.h) against a byte-by-byte count.
#include <cstdio>
#include <cstdlib>

#include "ranges.h"

int main()
{
    std::srand(1);
    int yes = 0, bad = 0;
    for (int q = 0; q < 200000; ++q) {
        // up to four arrays of 4..16 bytes in allocations on a strip of 160 bytes
        const int m = 1 + std::rand() % 4;
        const size_t bytes = 4 * (1 + std::rand() % 4);
        uintptr_t dst[6], base[6];
        size_t size[6];
        int count[512] = {};
        bool want = true;
        for (int a = 0; a < m; ++a) {
            base[a] = 40 * a + 4 * (std::rand() % 3);
            size[a] = 4 * (std::rand() % 9);
            dst[a] = base[a] + (std::rand() % 4 ? 4 * (std::rand() % 6) : std::rand() % 24);
            if (std::rand() % 8 == 0 && a) {  // the allocation of another one
                base[a] = base[a - 1];
                size[a] = size[a - 1];
            }
            want = want && dst[a] % 4 == 0;
            for (size_t t = 0; t < bytes; ++t) {
                const uintptr_t p = dst[a] + t;
                want = want && p >= base[a] && p < base[a] + size[a] && ++count[p] == 1;
            }
        }
        yes += want;
        bad += fdtd::writable_at_once(dst, base, size, m, bytes) != want;
    }
    // no allocation, and one that ends with the address space
    const uintptr_t top[1] = {~(uintptr_t)0 - 7}, at[1] = {~(uintptr_t)0 - 63};
    const size_t none[1] = {0}, whole[1] = {64};
    bad += fdtd::writable_at_once(top, at, none, 1, 4);
    bad += !fdtd::writable_at_once(top, at, whole, 1, 8);
    bad += fdtd::writable_at_once(top, at, whole, 1, 12);
    if (bad || yes < 1000) return 1;
    std::printf("range checks passed\n");
    return 0;
}
