// One reverse stage on bricks of cells (see adjoint.hip for the transpose and its tiled march).
//
// The tiled march runs its planes one after the other and waits out a plane's memory latency in
// each; on small grids a launch is little else. Here a workgroup owns a BX x BY x BZ brick, a thread
// to each cell: one round of loads (the stage input and the cotangent with a two-cell halo into
// LDS, everything else of the cell into registers), the gradient cotangents of the brick and of the
// cells next to it, one barrier, the gather. Only the gradient cotangents of the neighbours are
// evaluated again (16 x 8 x 4: 1.9 x its cells, one component each), and the halo planes come from
// L2. What bounds it: latency on small grids, then the cache traffic of the halos (3.75 x of two of
// its fifteen words; adjoint_takes_bricks has the line). The same arithmetic in the same order as the other forms, hence the same
// bits. WALLS: mirror reads on the walled axes, as there.
#include "pf_brick.h"
#include "pf_internal.h"

namespace pf {

template <typename T, int BX, int BY, int BZ, bool WALLS, bool FAST>
__global__ void __launch_bounds__(BX* BY* BZ) adjoint_brick_kernel(AdjArgs<T> a, int tiles_x, int tiles_y)
{
    using Frame = BrickFrame<BX, BY, BZ, WALLS, FAST>;
    constexpr int IX = Frame::IX, IXY = Frame::IXY;
    __shared__ T sy[Frame::IS];
    __shared__ T sk[Frame::IS];
    __shared__ T sgx[(BX + 2) * BY * BZ];
    __shared__ T sgy[BX * (BY + 2) * BZ];
    __shared__ T sgz[BX * BY * (BZ + 2)];

    const Frame fr(a.nx, a.ny, a.nz, a.walls, tiles_x, tiles_y);
    constexpr unsigned ES = sizeof(T);
    T py[Frame::NL], pk[Frame::NL];
    fr.for_input([&](int s, int, size_t base, unsigned o) {
        py[s] = ldg(a.y + base, o * ES);
        pk[s] = ldg(a.kap_in + base, o * ES);
    });
    const int nx = a.nx, ny = a.ny, nz = a.nz, x = fr.x, y = fr.y, z = fr.z;
    const int i = fr.i0 + x, j = fr.j0 + y, k = fr.k0 + z;
    const bool active = i < nx && j < ny && k < nz;
    const unsigned c = fr.at(i, j) * ES;
    const size_t kp = k * fr.plane;
    T u0 = T(0), u1 = T(0), v0 = T(0), v1 = T(0), w0 = T(0), w1 = T(0), gu = T(0), gv = T(0), gw = T(0), lb = T(0),
      lp = T(0);
    if (active) {
        u0 = ldg(a.U + kp, c);
        u1 = ldg(a.U + kp, i + 1 == nx ? c - (unsigned)(nx - 1) * ES : c + ES);
        v0 = ldg(a.V + kp, c);
        v1 = ldg(a.V + kp, j + 1 == ny ? (unsigned)i * ES : c + (unsigned)nx * ES);
        w0 = ldg(a.W + kp, c);
        w1 = ldg(a.W + (k + 1 == nz ? 0 : k + 1) * fr.plane, c);
        if (a.gU) gu = ldg(a.gU + kp, c);
        if (a.gV) gv = ldg(a.gV + kp, c);
        if (a.gW) gw = ldg(a.gW + kp, c);
        if (a.lam_out) lb = ldg(a.lam_base + kp, c);
        if (a.kap_out) lp = ldg(a.lamp + kp, c);
    }
    fr.for_input([&](int s, int e, size_t, unsigned) {
        sy[e] = py[s];
        sk[e] = a.kap_scale * pk[s];
    });
    __syncthreads();

    const T inv_dx = a.inv_dx, inv_2dx = a.inv_2dx, d2 = a.delta2, hs = a.hs, hg = a.hg, ge = a.ge;
    // the cell at offset q: the cotangent's terms f of its six faces, its gradient cotangent gb and, as
    // the result, its local term
    auto cell = [&](int q, T f[6], T gb[3]) -> T {
        const T *Y = sy + q, *K = sk + q;
        const T kc = K[0];
        const T g[3] = {grad1(Y[1], Y[-1], inv_2dx), grad1(Y[IX], Y[-IX], inv_2dx), grad1(Y[IXY], Y[-IXY], inv_2dx)};
        f[0] = adj_face(K[-1], kc, inv_dx);
        f[1] = adj_face(kc, K[1], inv_dx);
        f[2] = adj_face(K[-IX], kc, inv_dx);
        f[3] = adj_face(kc, K[IX], inv_dx);
        f[4] = adj_face(K[-IXY], kc, inv_dx);
        f[5] = adj_face(kc, K[IXY], inv_dx);
        const T qb[3] = {-hg * (f[0] + f[1]), -hg * (f[2] + f[3]), -hg * (f[4] + f[5])};
        return adj_cell(Y[0], g, qb, d2, gb);
    };
    const int o = (x + 2) + (y + 2) * IX + (z + 2) * IXY;
    T f[6], gb[3];  // f: kept for the gather
    const T loc = cell(o, f, gb);
    sgx[(x + 1) + y * (BX + 2) + z * ((BX + 2) * BY)] = gb[0];
    sgy[x + (y + 1) * BX + z * (BX * (BY + 2))] = gb[1];
    sgz[x + y * BX + (z + 1) * (BX * BY)] = gb[2];
    fr.for_halo([&](int, auto AXIS, int hx, int hy, int hz) {
        constexpr int axis = decltype(AXIS)::value;
        T hf[6], hb[3];
        (void)cell((hx + 2) + (hy + 2) * IX + (hz + 2) * IXY, hf, hb);
        if constexpr (axis == 0)
            sgx[(hx + 1) + hy * (BX + 2) + hz * ((BX + 2) * BY)] = hb[0];
        else if constexpr (axis == 1)
            sgy[hx + (hy + 1) * BX + hz * (BX * (BY + 2))] = hb[1];
        else
            sgz[hx + hy * BX + (hz + 1) * (BX * BY)] = hb[2];
    });
    __syncthreads();
    if (!active) return;

    const T* Y = sy + o;
    const T* GX = sgx + x + y * (BX + 2) + z * ((BX + 2) * BY);
    const T* GY = sgy + x + y * BX + z * (BX * (BY + 2));
    const T* GZ = sgz + x + y * BX + z * (BX * BY);
    T ybar = loc;
    ybar = fma(f[0], fma(-hs, u0, ge), ybar);
    ybar = fma(f[1], fma(-hs, u1, -ge), ybar);
    if (a.gU) stg<T>(a.gU + kp, c, fma(-hs * (Y[-1] + Y[0]), f[0], gu));
    ybar = fma(GX[0] - GX[2], inv_2dx, ybar);
    ybar = fma(f[2], fma(-hs, v0, ge), ybar);
    ybar = fma(f[3], fma(-hs, v1, -ge), ybar);
    if (a.gV) stg<T>(a.gV + kp, c, fma(-hs * (Y[-IX] + Y[0]), f[2], gv));
    ybar = fma(GY[0] - GY[2 * BX], inv_2dx, ybar);
    ybar = fma(f[4], fma(-hs, w0, ge), ybar);
    ybar = fma(f[5], fma(-hs, w1, -ge), ybar);
    if (a.gW) stg<T>(a.gW + kp, c, fma(-hs * (Y[-IXY] + Y[0]), f[4], gw));
    ybar = fma(GZ[0] - GZ[2 * BX * BY], inv_2dx, ybar);
    if (a.lam_out) stg<T>(a.lam_out + kp, c, lb + ybar);
    if (a.kap_out) stg<T>(a.kap_out + kp, c, fma(a.ka, ybar, a.kb * lp));
}

template <typename T, int BX, int BY, int BZ>
static hipError_t launch_adjoint_brick_shape(const AdjArgs<T>& a, hipStream_t st)
{
    if (a.nx <= 0 || a.ny <= 0 || a.nz <= 0 || a.nu[0] || field_needs_big(a.nx, a.ny, a.nz, sizeof(T)))
        return hipErrorInvalidValue;
    const int tx = (a.nx + BX - 1) / BX, ty = (a.ny + BY - 1) / BY, tz = (a.nz + BZ - 1) / BZ;
    const long long blocks = (long long)tx * ty * tz;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // within one period or mirror image: a brick reaches B + 2 cells beyond the domain at most
    const bool fast = a.nx >= BX + 2 && a.ny >= BY + 2 && a.nz >= BZ + 2;
    const auto k = !fast     ? adjoint_brick_kernel<T, BX, BY, BZ, true, false>
                   : a.walls ? adjoint_brick_kernel<T, BX, BY, BZ, true, true>
                             : adjoint_brick_kernel<T, BX, BY, BZ, false, true>;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(BX * BY * BZ), 0, st, a, tx, ty);
    return hipGetLastError();
}

// 16x8x4 bricks were the fastest shape at every size from 32^3 to 160^3 (8x8x8, 16x8x8, 16x16x4,
// 32x8x4 and 16x4x4 were 0-60 % slower); large planes take 16x32x1 (the z halo of a 16x8x4 brick is
// copies of the one plane).
template <typename T>
hipError_t launch_adjoint_brick(const AdjArgs<T>& a, hipStream_t st)
{
    if (a.nz == 1 && (long long)a.nx * a.ny > 362LL * 362) return launch_adjoint_brick_shape<T, 16, 32, 1>(a, st);
    return launch_adjoint_brick_shape<T, 16, 8, 4>(a, st);
}
template hipError_t launch_adjoint_brick<float>(const AdjArgs<float>&, hipStream_t);
template hipError_t launch_adjoint_brick<double>(const AdjArgs<double>&, hipStream_t);

// Up to 15 bricks of 16x8x4 per compute unit, where neither a grid alone on the device nor one beside
// others loses more than the other gains (stage_takes_bricks; us per RK4 adjoint step alone / each of three
// at once on streams, march -> bricks: FP32 64x72x101 (936 bricks) 71.8 / 33.6 -> 46.0 / 28.0, 112x88x116
// (2233) 124.0 / 70.7 -> 80.4 / 59.8, 120^3 (3600) 133.6 / 104.3 -> 118.1 / 115.5, 128^3 (4096) 135.8 / 125.3 ->
// 123.6 / 152.7; FP64 85.9 / 68.8 -> 63.8 / 45.6, 172.3 / 149.7 -> 118.7 / 143.6, 211.5 / 221.4 -> 195.3 / 249.2,
// 126x120x128 (3840) 205.3 / 251.7 -> 196.0 / 283.0). One plane: us for the four reverse stages FP64 64^2 35.8 /
// 19.9, 512^2 81 / 47.
bool adjoint_takes_bricks(int nx, int ny, int nz)
{
    const long long bricks = (long long)((nx + 15) / 16) * ((ny + 7) / 8) * ((nz + 3) / 4);
    return nz == 1 || bricks <= 15LL * device_compute_units();
}

}  // namespace pf
