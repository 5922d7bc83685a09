// The adjoint's passes: sweeps with hooks (sweep_tile.h).
#include "sweep_tile.h"

namespace fdtd {
namespace {

// Whether [start, start + len) meets [lo, lo + n), indices modulo N.
__device__ __forceinline__ bool meets(int start, int len, int lo, int n, int N)
{
    return n > 0 && (wrap(start - lo, N) < n || wrap(lo - start, N) < len);
}

template <int T, int R, int W, int MODE, int HOOK>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void hooked_kernel(
    const SweepArgs A, const HookArgs K)
{
    __shared__ Lds<T, R, W, MODE> S;
    int xcd, slot, per_xcd;
    if (!place(A, xcd, slot, per_xcd)) return;  // whole block
    const int tile = xcd * per_xcd + slot;
    const int k0 = tile % A.gz * (64 - 2 * T) - T, j0 = tile / A.gz % A.gy * (W * R - 2 * T) - T;
    const int x0 = tile / (A.gz * A.gy) * A.xchunk, nit = min(A.nx, x0 + A.xchunk) - x0 + 2 * T;
    auto box = [&](const int* lo, const int* n) {
        return meets(x0 - T, nit, lo[0], n[0], A.nx) && meets(j0, W * R, lo[1], n[1], A.ny) && meets(k0, 64, lo[2], n[2], A.nz);
    };
    if (box(K.dlo, K.dn) || box(K.mlo, K.mn))
        sweep_tile<T, R, W, MODE, false, HOOK>(A, K, S, xcd, slot, per_xcd);
    else
        sweep_tile<T, R, W, MODE, false, HOOK == kReverse ? kTransposed : kUpdate>(A, K, S, xcd, slot, per_xcd);
}
#define VH(T, R, W, M) hooked_kernel<T, R, W, M, kForward>, hooked_kernel<T, R, W, M, kReverse>,
const HookedKernel kKernels[] = {FDTD_SWEEP_HOOKED_SHAPES(VH)};
#undef VH

}  // namespace

HookedKernel sweep::hooked_kernel_of(int index) { return kKernels[index]; }

}  // namespace fdtd
