// What the brick kernels share (stage_brick.hip, adjoint_brick.hip): index arithmetic.
#pragma once

#include <hip/hip_runtime.h>

#include "pf_cell.h"

namespace pf {

// e / D for 0 <= e < 2^13 and a constant D: a 24-bit product and a shift, which run at the full
// rate (the general sequence takes a quarter-rate 32-bit product). With M = floor(2^19 / D) + 1
// the error e (M D - 2^19) / 2^19 stays below 1 for small e, and the product below 2^32 (exact()
// checks the whole range in a static assertion at each use).
template <int D>
struct SmallDiv {
    static constexpr unsigned M = (1u << 19) / D + 1u;
    static constexpr bool exact(unsigned e, unsigned n)
    {
        for (; e < n; ++e)
            if (((e * M) >> 19) != e / D) return false;
        return true;
    }
    static __device__ __forceinline__ int div(int e) { return (int)(__umul24((unsigned)e, M) >> 19); }
};

// An index within one period, or one mirror image, of [0, n) (FAST), or any index: wrapped into it,
// or reflected at its walls.
template <bool FAST>
__device__ __forceinline__ int brick_wrap(int v, int n)
{
    return FAST ? wrap1(v, n) : wrapn(v, n);
}
template <bool FAST>
__device__ __forceinline__ int brick_mirror(int v, int n)
{
    return FAST ? (v < 0 ? -1 - v : (v >= n ? 2 * n - 1 - v : v)) : reflectn(v, n);
}

}  // namespace pf
