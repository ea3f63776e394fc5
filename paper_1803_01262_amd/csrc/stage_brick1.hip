// One RK stage on bricks of cells (the per-stage form of small grids; see stage_brick.hip for two
// stages per launch and pf_tiled_body.h for the march).
//
// A workgroup owns a BX x BY x BZ brick, a thread to each cell: one round of loads (the stage input
// with a two-cell halo into LDS, everything else of the cell into registers), the sharpening
// products of the brick and of the cells next to it, one barrier, the flux divergence. Only the
// neighbours' sharpening products are evaluated again, one component each (16 x 8 x 4: 0.9 x the
// brick's cells). What bounds it: latency on small grids, then the cache traffic of the halo (3.75 x
// of one of its seven words; stage_takes_bricks has the line to the march). The same arithmetic in
// the same order, hence the same bits. WALLS: mirror reads on the walled axes, no velocity on their
// wall faces. NU: the non-uniform mesh (a.nu), as in the march.
#include "pf_brick.h"
#include "pf_internal.h"

namespace pf {

template <typename T, int BX, int BY, int BZ, bool WALLS, bool FAST, bool NU>
__global__ void __launch_bounds__(BX* BY* BZ) stage_brick_kernel(StageArgs<T> a, int tiles_x, int tiles_y)
{
    constexpr int NT = BX * BY * BZ;
    constexpr int IX = BX + 4, IY = BY + 4, IZ = BZ + 4, IXY = IX * IY, IS = IXY * IZ;
    constexpr int NL = (IS + NT - 1) / NT;
    constexpr int QXS = (BX + 2) * BY * BZ, QYS = BX * (BY + 2) * BZ, QZS = BX * BY * (BZ + 2);
    constexpr int NH = 2 * (BY * BZ + BX * BZ + BX * BY), NHS = (NH + NT - 1) / NT;
    static_assert(IS < 8192 && SmallDiv<IX>::exact(0, IS) && SmallDiv<IY>::exact(0, IY * IZ),
                  "the small divisions are exact over their ranges");
    __shared__ T sp[IS];
    __shared__ T sqx[QXS];
    __shared__ T sqy[QYS];
    __shared__ T sqz[QZS];

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    int b = xcd_tile_order(blockIdx.x, gridDim.x);
    const int ti = b % tiles_x;
    b /= tiles_x;
    const int i0 = ti * BX, j0 = (b % tiles_y) * BY, k0 = (b / tiles_y) * BZ;
    const int tid = threadIdx.x;
    const bool wx = WALLS && (a.walls & 1), wy = WALLS && (a.walls & 2), wz = WALLS && (a.walls & 4);
    auto mapx = [&](int v) { return wx ? brick_mirror<FAST>(v, nx) : brick_wrap<FAST>(v, nx); };
    auto mapy = [&](int v) { return wy ? brick_mirror<FAST>(v, ny) : brick_wrap<FAST>(v, ny); };
    auto mapz = [&](int v) { return wz ? brick_mirror<FAST>(v, nz) : brick_wrap<FAST>(v, nz); };
    constexpr unsigned ES = sizeof(T);
    const rsrc_t ry = plane_rsrc(a.y, (unsigned)((size_t)nx * ny * nz * ES));
    auto at = [&](int x, int y, int z) { return ((unsigned)(z * ny + y) * (unsigned)nx + (unsigned)x) * ES; };

    T py[NL];
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (IS % NT == 0 || e < IS) {
            const int row = SmallDiv<IX>::div(e), x = e - row * IX, z = SmallDiv<IY>::div(row), y = row - z * IY;
            py[s] = bload<T>(ry, at(mapx(i0 - 2 + x), mapy(j0 - 2 + y), mapz(k0 - 2 + z)));
        }
    }
    const int x = tid % BX, y = tid / BX % BY, z = tid / (BX * BY);
    const int i = i0 + x, j = j0 + y, k = k0 + z;
    const bool active = i < nx && j < ny && k < nz;
    const unsigned c = active ? at(i, j, k) : 0u;
    T u0 = T(0), u1 = T(0), v0 = T(0), v1 = T(0), w0 = T(0), w1 = T(0), b1 = T(0), b2 = T(0);
    if (active) {
        u0 = ldg(a.U, c);
        u1 = ldg(a.U, at(i + 1 == nx ? 0 : i + 1, j, k));
        v0 = ldg(a.V, c);
        v1 = ldg(a.V, at(i, j + 1 == ny ? 0 : j + 1, k));
        w0 = ldg(a.W, c);
        w1 = ldg(a.W, at(i, j, k + 1 == nz ? 0 : k + 1));
        if (a.out1) b1 = ldg(a.base1, c);
        if (a.out2) b2 = ldg(a.base2, c);
        if constexpr (WALLS) {  // velocities on wall faces (index 0 of a walled axis)
            if (wx && i == 0) u0 = T(0);
            if (wx && i == nx - 1) u1 = T(0);
            if (wy && j == 0) v0 = T(0);
            if (wy && j == ny - 1) v1 = T(0);
            if (wz && k == 0) w0 = T(0);
            if (wz && k == nz - 1) w1 = T(0);
        }
    }
    // non-uniform mesh: column col of the tables at cell v of an axis
    auto tab = [&](int axis, int v, int col) -> T {
        const int m = axis == 0 ? mapx(v) : axis == 1 ? mapy(v) : mapz(v);
        return a.nu[axis][m * kNuCols + col];
    };
    T sgx = a.inv_2dx, sgy = a.inv_2dx, sgz = a.inv_2dx;
    T nf[3][3], wd[3][3];  // per axis: 1/h, 1/distance across the low and the high face; the widths around
    if constexpr (NU) {
        const int v[3] = {i, j, k};
        sgx = tab(0, i, kNuInvSpan);
        sgy = tab(1, j, kNuInvSpan);
        sgz = tab(2, k, kNuInvSpan);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            nf[ax][0] = tab(ax, v[ax], kNuInvW);
            nf[ax][1] = tab(ax, v[ax], kNuInvDist);
            nf[ax][2] = tab(ax, v[ax] + 1, kNuInvDist);  // the low face of the next cell
#pragma unroll
            for (int d = 0; d < 3; ++d) wd[ax][d] = tab(ax, v[ax] - 1 + d, kNuWidth);
        }
    }
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (IS % NT == 0 || e < IS) sp[e] = py[s];
    }
    __syncthreads();

    const T d2 = a.delta2, hg = NU ? a.nu_hg : a.hg;
    auto sharpen = [&](int q, T cx, T cy, T cz, T g[3]) -> T {
        const T* p = sp + q;
        g[0] = grad1(p[1], p[-1], cx);
        g[1] = grad1(p[IX], p[-IX], cy);
        g[2] = grad1(p[IXY], p[-IXY], cz);
        return sharpen_factor(p[0], g[0], g[1], g[2], d2, hg);
    };
    const int o = (x + 2) + (y + 2) * IX + (z + 2) * IXY;
    {
        T g[3];
        const T fac = sharpen(o, sgx, sgy, sgz, g);
        sqx[(x + 1) + y * (BX + 2) + z * ((BX + 2) * BY)] = fac * g[0];
        sqy[x + (y + 1) * BX + z * (BX * (BY + 2))] = fac * g[1];
        sqz[tid + BX * BY] = fac * g[2];
    }
#pragma unroll
    for (int s = 0; s < NHS; ++s) {
        int e = s * NT + (NT - 1 - tid);
        if (e >= NH) continue;
        int hx, hy, hz, comp;  // the halo cell, relative to the brick
        if (e < 2 * BY * BZ) {
            const int side = e >= BY * BZ, t = e - side * (BY * BZ);
            comp = 0;
            hx = side ? BX : -1;
            hy = t % BY;
            hz = t / BY;
        } else if (e < 2 * BY * BZ + 2 * BX * BZ) {
            e -= 2 * BY * BZ;
            const int side = e >= BX * BZ, t = e - side * (BX * BZ);
            comp = 1;
            hx = t % BX;
            hy = side ? BY : -1;
            hz = t / BX;
        } else {
            e -= 2 * BY * BZ + 2 * BX * BZ;
            const int side = e >= BX * BY, t = e - side * (BX * BY);
            comp = 2;
            hx = t % BX;
            hy = t / BX;
            hz = side ? BZ : -1;
        }
        T cx = a.inv_2dx, cy = a.inv_2dx, cz = a.inv_2dx;
        if constexpr (NU) {
            cx = tab(0, i0 + hx, kNuInvSpan);
            cy = tab(1, j0 + hy, kNuInvSpan);
            cz = tab(2, k0 + hz, kNuInvSpan);
        }
        T g[3];
        const T fac = sharpen((hx + 2) + (hy + 2) * IX + (hz + 2) * IXY, cx, cy, cz, g);
        if (comp == 0)
            sqx[(hx + 1) + hy * (BX + 2) + hz * ((BX + 2) * BY)] = fac * g[0];
        else if (comp == 1)
            sqy[hx + (hy + 1) * BX + hz * (BX * (BY + 2))] = fac * g[1];
        else
            sqz[hx + hy * BX + (hz + 1) * (BX * BY)] = fac * g[2];
    }
    __syncthreads();
    if (!active) return;

    const T* p = sp + o;
    const T pc = p[0], xm = p[-1], xp = p[1], ym = p[-IX], yp = p[IX], zm = p[-IXY], zp = p[IXY];
    const T* QX = sqx + x + y * (BX + 2) + z * ((BX + 2) * BY);
    const T* QY = sqy + x + y * BX + z * (BX * (BY + 2));
    const T* QZ = sqz + tid;
    T f;
    if constexpr (NU) {
        // diffusive coefficients of the six faces: gamma eps_face / centre distance
        T exl = a.nu_ge, exh = a.nu_ge, eyl = a.nu_ge, eyh = a.nu_ge, ezl = a.nu_ge, ezh = a.nu_ge;
        if (a.nu_eps_mode == 1) {  // eps of a cell ~ its largest width
            const T hx = wd[0][1], hy = wd[1][1], hz = wd[2][1];
            const T mc = fmax(hx, fmax(hy, hz));
            const T hh = a.nu_ge * T(0.5);
            exl = hh * (fmax(wd[0][0], fmax(hy, hz)) + mc);
            exh = hh * (fmax(wd[0][2], fmax(hy, hz)) + mc);
            eyl = hh * (fmax(hx, fmax(wd[1][0], hz)) + mc);
            eyh = hh * (fmax(hx, fmax(wd[1][2], hz)) + mc);
            ezl = hh * (fmax(hx, fmax(hy, wd[2][0])) + mc);
            ezh = hh * (fmax(hx, fmax(hy, wd[2][2])) + mc);
        }
        f = cell_rhs_nu(face_sum(xm, pc), face_sum(pc, xp), face_sum(ym, pc), face_sum(pc, yp),
                        face_sum(zm, pc), face_sum(pc, zp), face_diff(xm, pc), face_diff(pc, xp),
                        face_diff(ym, pc), face_diff(pc, yp), face_diff(zm, pc), face_diff(pc, zp), QX[0],
                        QX[2], QY[0], QY[2 * BX], QZ[0], QZ[2 * BX * BY], u0, u1, v0, v1, w0, w1, a.nu_nhs,
                        exl * nf[0][1], exh * nf[0][2], eyl * nf[1][1], eyh * nf[1][2], ezl * nf[2][1],
                        ezh * nf[2][2], nf[0][0], nf[1][0], nf[2][0]);
    } else {
        f = cell_rhs(face_sum(xm, pc), face_sum(pc, xp), face_sum(ym, pc), face_sum(pc, yp), face_sum(zm, pc),
                     face_sum(pc, zp), face_diff(xm, pc), face_diff(pc, xp), face_diff(ym, pc),
                     face_diff(pc, yp), face_diff(zm, pc), face_diff(pc, zp), QX[0], QX[2], QY[0], QY[2 * BX],
                     QZ[0], QZ[2 * BX * BY], u0, u1, v0, v1, w0, w1, a.nhs, a.ge);
    }
    if (a.out1) stg<T>(a.out1, c, fma(a.c1, f, b1));
    if (a.out2) stg<T>(a.out2, c, fma(a.c2, f, b2));
}

template <typename T, int BX, int BY, int BZ, bool NU>
static hipError_t launch_stage_brick_shape(const StageArgs<T>& a, hipStream_t st)
{
    const int tx = (a.nx + BX - 1) / BX, ty = (a.ny + BY - 1) / BY, tz = (a.nz + BZ - 1) / BZ;
    const long long blocks = (long long)tx * ty * tz;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // within one period or mirror image: a brick reaches B + 2 cells beyond the domain at most
    const bool fast = a.nx >= BX + 2 && a.ny >= BY + 2 && a.nz >= BZ + 2;
    const auto k = !fast     ? stage_brick_kernel<T, BX, BY, BZ, true, false, NU>
                   : a.walls ? stage_brick_kernel<T, BX, BY, BZ, true, true, NU>
                             : stage_brick_kernel<T, BX, BY, BZ, false, true, NU>;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(BX * BY * BZ), 0, st, a, tx, ty);
    return hipGetLastError();
}

// Arrays of 4 GiB or more (32-bit offsets here), and one-plane grids on a uniform mesh (their plane
// kernel), take the tiled launch.
template <typename T, int BX, int BY, int BZ>
hipError_t launch_stage_brick(const StageArgs<T>& a, hipStream_t st)
{
    if (a.nx <= 0 || a.ny <= 0 || a.nz <= 0) return hipErrorInvalidValue;
    if (field_needs_big(a.nx, a.ny, a.nz, sizeof(T)) || (a.nz == 1 && !a.nu[0]))
        return a.nu[0] ? launch_stage_nu_march<T>(a, st) : launch_stage_tiled<T, 64, 4, 0, false, false>(a, st);
    return a.nu[0] ? launch_stage_brick_shape<T, BX, BY, BZ, true>(a, st)
                   : launch_stage_brick_shape<T, BX, BY, BZ, false>(a, st);
}

#define PF_STAGE_BRICK_INST(BX, BY, BZ)                                                          \
    template hipError_t launch_stage_brick<float, BX, BY, BZ>(const StageArgs<float>&, hipStream_t); \
    template hipError_t launch_stage_brick<double, BX, BY, BZ>(const StageArgs<double>&, hipStream_t);
PF_STAGE_BRICK_INST(16, 8, 4)

}  // namespace pf
