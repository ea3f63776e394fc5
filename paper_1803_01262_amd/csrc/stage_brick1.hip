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
    using Frame = BrickFrame<BX, BY, BZ, WALLS, FAST>;
    constexpr int IX = Frame::IX, IXY = Frame::IXY;
    __shared__ T sp[Frame::IS];
    __shared__ T sqx[(BX + 2) * BY * BZ];
    __shared__ T sqy[BX * (BY + 2) * BZ];
    __shared__ T sqz[BX * BY * (BZ + 2)];

    const Frame fr(a.nx, a.ny, a.nz, a.walls, tiles_x, tiles_y);
    constexpr unsigned ES = sizeof(T);
    T py[Frame::NL];
    fr.for_input([&](int s, int, size_t base, unsigned o) { py[s] = ldg(a.y + base, o * ES); });
    const int nx = a.nx, ny = a.ny, nz = a.nz, x = fr.x, y = fr.y, z = fr.z;
    const int i = fr.i0 + x, j = fr.j0 + y, k = fr.k0 + z;
    const bool active = i < nx && j < ny && k < nz;
    const unsigned c = fr.at(i, j) * ES;
    const size_t kp = k * fr.plane;
    T u0 = T(0), u1 = T(0), v0 = T(0), v1 = T(0), w0 = T(0), w1 = T(0), b1 = T(0), b2 = T(0);
    if (active) {
        u0 = ldg(a.U + kp, c);
        u1 = ldg(a.U + kp, i + 1 == nx ? c - (unsigned)(nx - 1) * ES : c + ES);
        v0 = ldg(a.V + kp, c);
        v1 = ldg(a.V + kp, j + 1 == ny ? (unsigned)i * ES : c + (unsigned)nx * ES);
        w0 = ldg(a.W + kp, c);
        w1 = ldg(a.W + (k + 1 == nz ? 0 : k + 1) * fr.plane, c);
        if (a.out1) b1 = ldg(a.base1 + kp, c);
        if (a.out2) b2 = ldg(a.base2 + kp, c);
        if constexpr (WALLS) {  // velocities on wall faces (index 0 of a walled axis)
            if (fr.wx && i == 0) u0 = T(0);
            if (fr.wx && i == nx - 1) u1 = T(0);
            if (fr.wy && j == 0) v0 = T(0);
            if (fr.wy && j == ny - 1) v1 = T(0);
            if (fr.wz && k == 0) w0 = T(0);
            if (fr.wz && k == nz - 1) w1 = T(0);
        }
    }
    // non-uniform mesh: the row of an axis' table at cell v (adjacent columns: one load)
    auto row = [&](int axis, int v) -> const T* {
        const int m = axis == 0 ? fr.ax.map(v) : axis == 1 ? fr.ay.map(v) : fr.az.map(v);
        return a.nu[axis] + m * kNuCols;
    };
    T sgx = a.inv_2dx, sgy = a.inv_2dx, sgz = a.inv_2dx;
    T nf[3][3], wd[3][3];  // per axis: 1/h, 1/distance across the low and the high face; the widths around
    if constexpr (NU) {
        const int v[3] = {i, j, k};
        T sg[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const T *lo = row(ax, v[ax] - 1), *me = row(ax, v[ax]), *hi = row(ax, v[ax] + 1);
            nf[ax][0] = me[kNuInvW];
            sg[ax] = me[kNuInvSpan];
            nf[ax][1] = me[kNuInvDist];
            wd[ax][1] = me[kNuWidth];
            nf[ax][2] = hi[kNuInvDist];  // the low face of the next cell
            wd[ax][2] = hi[kNuWidth];
            wd[ax][0] = lo[kNuWidth];
        }
        sgx = sg[0];
        sgy = sg[1];
        sgz = sg[2];
    }
    T hc[Frame::NHS][3];  // gradient coefficients at the thread's cells next to the brick
    if constexpr (NU)
        fr.for_halo([&](int s, auto, int hx, int hy, int hz) {
            hc[s][0] = row(0, fr.i0 + hx)[kNuInvSpan];
            hc[s][1] = row(1, fr.j0 + hy)[kNuInvSpan];
            hc[s][2] = row(2, fr.k0 + hz)[kNuInvSpan];
        });
    fr.for_input([&](int s, int e, size_t, unsigned) { sp[e] = py[s]; });
    __syncthreads();

    const T d2 = a.delta2, hg = NU ? a.nu_hg : a.hg;
    // the cell and its neighbours, for the products here and the fluxes below
    const T* p = sp + (x + 2) + (y + 2) * IX + (z + 2) * IXY;
    const T pc = p[0], xm = p[-1], xp = p[1], ym = p[-IX], yp = p[IX], zm = p[-IXY], zp = p[IXY];
    {
        const T gx = grad1(xp, xm, sgx), gy = grad1(yp, ym, sgy), gz = grad1(zp, zm, sgz);
        const T fac = sharpen_factor(pc, gx, gy, gz, d2, hg);
        sqx[(x + 1) + y * (BX + 2) + z * ((BX + 2) * BY)] = fac * gx;
        sqy[x + (y + 1) * BX + z * (BX * (BY + 2))] = fac * gy;
        sqz[x + y * BX + (z + 1) * (BX * BY)] = fac * gz;
    }
    fr.for_halo([&](int s, auto AXIS, int hx, int hy, int hz) {
        constexpr int axis = decltype(AXIS)::value;
        const T cx = NU ? hc[s][0] : a.inv_2dx, cy = NU ? hc[s][1] : a.inv_2dx, cz = NU ? hc[s][2] : a.inv_2dx;
        const T* h = sp + (hx + 2) + (hy + 2) * IX + (hz + 2) * IXY;
        const T g[3] = {grad1(h[1], h[-1], cx), grad1(h[IX], h[-IX], cy), grad1(h[IXY], h[-IXY], cz)};
        const T q = sharpen_factor(h[0], g[0], g[1], g[2], d2, hg) * g[axis];
        if constexpr (axis == 0)
            sqx[(hx + 1) + hy * (BX + 2) + hz * ((BX + 2) * BY)] = q;
        else if constexpr (axis == 1)
            sqy[hx + (hy + 1) * BX + hz * (BX * (BY + 2))] = q;
        else
            sqz[hx + hy * BX + (hz + 1) * (BX * BY)] = q;
    });
    __syncthreads();
    if (!active) return;

    const T* QX = sqx + x + y * (BX + 2) + z * ((BX + 2) * BY);
    const T* QY = sqy + x + y * BX + z * (BX * (BY + 2));
    const T* QZ = sqz + x + y * BX + z * (BX * BY);
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
    if (a.out1) stg<T>(a.out1 + kp, c, fma(a.c1, f, b1));
    if (a.out2) stg<T>(a.out2 + kp, c, fma(a.c2, f, b2));
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
