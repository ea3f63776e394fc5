// What the brick kernels share (stage_brick.hip, stage_brick1.hip, adjoint_brick.hip): index arithmetic,
// and the frame of the two single-stage kernels.
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

// A brick of BX x BY x BZ cells, a thread to each cell, with a halo of two cells in LDS: the frame of
// the single-stage kernels (one forward stage, one reverse stage). Beside the arithmetic of its cells
// such a kernel mostly finds addresses, and where other work shares the device, so that no compute unit
// idles, that is paid in full (vector issue bounds it then: alone, latency does). So everything along z
// is scalar (a wave's elements lie in few planes, its own cells in one), the offsets to a cell's
// neighbours are differences instead of products, and bricks whose halo stays inside the plane wrap
// nothing; a lane keeps its column of the input from piece to piece. us per step alone / each of three at
// once on streams, every index in vector registers and the halo in pieces of 64 elements -> here:
// RK3 96^3 FP32 26.1 / 18.0 -> 23.1 / 14.9, FP64 32.6 / 25.6 -> 30.7 / 22.7; RK4 with walls on x and z 96^3
// FP32 38.6 / 26.4 -> 33.5 / 22.0, FP64 49.4 / 43.2 -> 44.3 / 37.9.
template <int BX, int BY, int BZ, bool WALLS, bool FAST>
struct BrickFrame {
    static constexpr int NT = BX * BY * BZ, NW = NT / 64;
    static constexpr int IX = BX + 4, IY = BY + 4, IZ = BZ + 4, IXY = IX * IY, IS = IXY * IZ;
    // an input plane in pieces of RP whole rows, a lane to each element: PP per plane, NL per wave
    static constexpr int RP = 64 / IX, PP = IY / RP, NL = (PP * IZ + NW - 1) / NW;
    static constexpr int NH = 2 * (BY * BZ + BX * BZ + BX * BY), NHS = (NH + NT - 1) / NT;
    static_assert(NT % 64 == 0 && BX * BY % 64 == 0, "a wave's own cells lie in one plane");
    static_assert(IY % RP == 0, "whole pieces");
    static_assert(SmallDiv<IX>::exact(0, 64), "the small division is exact over its range");

    // An index of an axis: wrapped into it, or reflected at its walls. Within one period or image
    // (FAST) both are (v ^ flip) + lo below 0 and (v ^ flip) + hi from n up, with flip = -1 at walls
    // (~v = -1 - v) and the three in scalar registers.
    struct Axis {
        int n, flip, lo, hi;
        __device__ __forceinline__ Axis(int n_, bool wall)
            : n(n_), flip(wall ? -1 : 0), lo(wall ? 0 : n_), hi(wall ? 2 * n_ : -n_)
        {
        }
        __device__ __forceinline__ int map(int v) const
        {
            if constexpr (!FAST) return flip ? reflectn(v, n) : wrapn(v, n);
            const int t = WALLS ? v ^ flip : v;
            const int r = v < 0 ? t + lo : v;  // one select after the other: no branches
            return v >= n ? t + hi : r;
        }
    };
    int nx, ny, nz, i0, j0, k0;
    bool wx, wy, wz, inner;  // inner: the halo stays inside the plane
    Axis ax, ay, az;
    size_t plane;  // cells of a plane
    int wave, lane;
    int x, y, z;  // the thread's cell in the brick (z: scalar)

    __device__ __forceinline__ BrickFrame(int nx_, int ny_, int nz_, int walls, int tiles_x, int tiles_y)
        : nx(nx_), ny(ny_), nz(nz_), wx(WALLS && (walls & 1)), wy(WALLS && (walls & 2)), wz(WALLS && (walls & 4)),
          ax(nx_, wx), ay(ny_, wy), az(nz_, wz), plane((size_t)nx_ * ny_)
    {
        int b = xcd_tile_order(blockIdx.x, gridDim.x);
        const int ti = b % tiles_x;
        b /= tiles_x;
        i0 = ti * BX;
        j0 = (b % tiles_y) * BY;
        k0 = (b / tiles_y) * BZ;
        inner = i0 >= 2 && i0 + BX + 2 <= nx && j0 >= 2 && j0 + BY + 2 <= ny;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        lane = threadIdx.x & 63;
        z = wave / (BX * BY / 64);
        const int t = (wave % (BX * BY / 64)) * 64 + lane;
        x = t % BX;
        y = t / BX;
    }
    // an element of a plane (gx < 2^20, gy < 2^16, a plane below 2^28 cells)
    __device__ __forceinline__ unsigned at(int gx, int gy) const { return __umul24((unsigned)gy, (unsigned)nx) + (unsigned)gx; }

    // f(s, element in LDS, element of the array as a scalar and a vector part) for the thread's elements
    template <typename F>
    __device__ __forceinline__ void for_input(F f) const
    {
        if (RP * IX < 64 && lane >= RP * IX) return;
        const int r = SmallDiv<IX>::div(lane), vx = i0 - 2 + lane - r * IX;
        auto go = [&](auto IN) {
            constexpr bool in = decltype(IN)::value != 0;
            const int gx = in ? vx : ax.map(vx);
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                const int p = wave * NL + s, zi = p / PP, row = (p - zi * PP) * RP;
                if (PP * IZ % NW != 0 && zi >= IZ) continue;
                const size_t base = az.map(k0 - 2 + zi) * plane;
                const int e = zi * IXY + row * IX + lane;
                if constexpr (in)
                    f(s, e, base + (size_t)(j0 - 2 + row) * nx, at(gx, r));
                else
                    f(s, e, base, at(gx, ay.map(j0 - 2 + row + r)));
            }
        };
        if (inner)
            go(IntC<1>());
        else
            go(IntC<0>());
    }
    // f(s, axis, x, y, z) for the thread's cells next to the brick, from the last thread down
    template <typename F>
    __device__ __forceinline__ void for_halo(F f) const
    {
        constexpr int EX = 2 * BY * BZ, EY = EX + 2 * BX * BZ;
        constexpr bool UNIFORM = EX % 64 == 0 && EY % 64 == 0 && NH % 64 == 0;  // a wave has one kind
#pragma unroll
        for (int s = 0; s < NHS; ++s) {
            const int eb = s * NT + (NW - 1 - wave) * 64, e = eb + 63 - lane, q = UNIFORM ? eb : e;
            if (q >= NH) continue;
            if (q < EX) {
                const int side = e >= BY * BZ, t = e - side * (BY * BZ);
                f(s, IntC<0>(), side ? BX : -1, t % BY, t / BY);
            } else if (q < EY) {
                const int r = e - EX, side = r >= BX * BZ, t = r - side * (BX * BZ);
                f(s, IntC<1>(), t % BX, side ? BY : -1, t / BX);
            } else {
                const int r = e - EY, side = r >= BX * BY, t = r - side * (BX * BY);
                f(s, IntC<2>(), t % BX, t / BX, side ? BZ : -1);
            }
        }
    }
};

}  // namespace pf
