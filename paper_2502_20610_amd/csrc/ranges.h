// Address ranges of caller arrays.  Plain C++ (also built for the host alone).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace fdtd {

// Whether one kernel may write m arrays of `bytes` bytes at dst side by side:
// whole floats, each inside its allocation [base, base + size), none meeting
// another (copies in turn take any arrays, the last one written last).
inline bool writable_at_once(const uintptr_t* dst, const uintptr_t* base, const size_t* size, int m, size_t bytes)
{
    for (int a = 0; a < m; ++a) {
        if (dst[a] % sizeof(float) || dst[a] < base[a] || size[a] < bytes || dst[a] - base[a] > size[a] - bytes)
            return false;
        for (int b = 0; b < a; ++b)
            if (dst[a] < dst[b] ? dst[b] - dst[a] < bytes : dst[a] - dst[b] < bytes) return false;
    }
    return true;
}

}  // namespace fdtd
