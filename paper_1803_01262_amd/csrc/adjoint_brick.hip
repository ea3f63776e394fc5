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
    constexpr int NT = BX * BY * BZ;
    constexpr int IX = BX + 4, IY = BY + 4, IZ = BZ + 4, IXY = IX * IY, IS = IXY * IZ;
    constexpr int NL = (IS + NT - 1) / NT;
    constexpr int GXS = (BX + 2) * BY * BZ, GYS = BX * (BY + 2) * BZ, GZS = BX * BY * (BZ + 2);
    constexpr int NH = 2 * (BY * BZ + BX * BZ + BX * BY), NHS = (NH + NT - 1) / NT;
    static_assert(IS < 8192 && SmallDiv<IX>::exact(0, IS) && SmallDiv<IY>::exact(0, IY * IZ),
                  "the small divisions are exact over their ranges");
    __shared__ T sy[IS];
    __shared__ T sk[IS];
    __shared__ T sgx[GXS];
    __shared__ T sgy[GYS];
    __shared__ T sgz[GZS];

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
    const unsigned whole = (unsigned)((size_t)nx * ny * nz * ES);
    const rsrc_t ry = plane_rsrc(a.y, whole), rk = plane_rsrc(a.kap_in, whole);
    auto at = [&](int x, int y, int z) { return ((unsigned)(z * ny + y) * (unsigned)nx + (unsigned)x) * ES; };

    T py[NL], pk[NL];
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (IS % NT == 0 || e < IS) {
            const int row = SmallDiv<IX>::div(e), x = e - row * IX, z = SmallDiv<IY>::div(row), y = row - z * IY;
            const unsigned off = at(mapx(i0 - 2 + x), mapy(j0 - 2 + y), mapz(k0 - 2 + z));
            py[s] = bload<T>(ry, off);
            pk[s] = bload<T>(rk, off);
        }
    }
    const int x = tid % BX, y = tid / BX % BY, z = tid / (BX * BY);
    const int i = i0 + x, j = j0 + y, k = k0 + z;
    const bool active = i < nx && j < ny && k < nz;
    const unsigned c = active ? at(i, j, k) : 0u;
    T u0 = T(0), u1 = T(0), v0 = T(0), v1 = T(0), w0 = T(0), w1 = T(0), gu = T(0), gv = T(0), gw = T(0), lb = T(0),
      lp = T(0);
    if (active) {
        u0 = ldg(a.U, c);
        u1 = ldg(a.U, at(i + 1 == nx ? 0 : i + 1, j, k));
        v0 = ldg(a.V, c);
        v1 = ldg(a.V, at(i, j + 1 == ny ? 0 : j + 1, k));
        w0 = ldg(a.W, c);
        w1 = ldg(a.W, at(i, j, k + 1 == nz ? 0 : k + 1));
        if (a.gU) gu = ldg(a.gU, c);
        if (a.gV) gv = ldg(a.gV, c);
        if (a.gW) gw = ldg(a.gW, c);
        if (a.lam_out) lb = ldg(a.lam_base, c);
        if (a.kap_out) lp = ldg(a.lamp, c);
    }
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (IS % NT == 0 || e < IS) {
            sy[e] = py[s];
            sk[e] = a.kap_scale * pk[s];
        }
    }
    __syncthreads();

    const T inv_dx = a.inv_dx, inv_2dx = a.inv_2dx, d2 = a.delta2, hs = a.hs, hg = a.hg, ge = a.ge;
    auto cell = [&](int q, T gb[3]) -> T {  // gbar and the local term of the cell at offset q
        const T *Y = sy + q, *K = sk + q;
        T g[3], qb[3];
        g[0] = grad1(Y[1], Y[-1], inv_2dx);
        g[1] = grad1(Y[IX], Y[-IX], inv_2dx);
        g[2] = grad1(Y[IXY], Y[-IXY], inv_2dx);
        qb[0] = -hg * (adj_face(K[-1], K[0], inv_dx) + adj_face(K[0], K[1], inv_dx));
        qb[1] = -hg * (adj_face(K[-IX], K[0], inv_dx) + adj_face(K[0], K[IX], inv_dx));
        qb[2] = -hg * (adj_face(K[-IXY], K[0], inv_dx) + adj_face(K[0], K[IXY], inv_dx));
        return adj_cell(Y[0], g, qb, d2, gb);
    };
    const int o = (x + 2) + (y + 2) * IX + (z + 2) * IXY;
    T gb[3];
    const T loc = cell(o, gb);
    sgx[(x + 1) + y * (BX + 2) + z * ((BX + 2) * BY)] = gb[0];
    sgy[x + (y + 1) * BX + z * (BX * (BY + 2))] = gb[1];
    sgz[tid + BX * BY] = gb[2];
#pragma unroll
    for (int s = 0; s < NHS; ++s) {
        int e = s * NT + (NT - 1 - tid);
        if (e >= NH) continue;
        T hb[3];
        if (e < 2 * BY * BZ) {
            const int side = e >= BY * BZ, t = e - side * (BY * BZ), hy = t % BY, hz = t / BY;
            (void)cell((side ? BX + 2 : 1) + (hy + 2) * IX + (hz + 2) * IXY, hb);
            sgx[(side ? BX + 1 : 0) + hy * (BX + 2) + hz * ((BX + 2) * BY)] = hb[0];
        } else if (e < 2 * BY * BZ + 2 * BX * BZ) {
            e -= 2 * BY * BZ;
            const int side = e >= BX * BZ, t = e - side * (BX * BZ), hx = t % BX, hz = t / BX;
            (void)cell((hx + 2) + (side ? BY + 2 : 1) * IX + (hz + 2) * IXY, hb);
            sgy[hx + (side ? BY + 1 : 0) * BX + hz * (BX * (BY + 2))] = hb[1];
        } else {
            e -= 2 * BY * BZ + 2 * BX * BZ;
            const int side = e >= BX * BY, t = e - side * (BX * BY), hx = t % BX, hy = t / BX;
            (void)cell((hx + 2) + (hy + 2) * IX + (side ? BZ + 2 : 1) * IXY, hb);
            sgz[t + (side ? BZ + 1 : 0) * (BX * BY)] = hb[2];
        }
    }
    __syncthreads();
    if (!active) return;

    const T *Y = sy + o, *K = sk + o;
    T ybar = loc;
    T lo = adj_face(K[-1], K[0], inv_dx), hi = adj_face(K[0], K[1], inv_dx);
    ybar = fma(lo, fma(-hs, u0, ge), ybar);
    ybar = fma(hi, fma(-hs, u1, -ge), ybar);
    if (a.gU) stg<T>(a.gU, c, fma(-hs * (Y[-1] + Y[0]), lo, gu));
    const T* GX = sgx + x + y * (BX + 2) + z * ((BX + 2) * BY);
    ybar = fma(GX[0] - GX[2], inv_2dx, ybar);
    lo = adj_face(K[-IX], K[0], inv_dx);
    hi = adj_face(K[0], K[IX], inv_dx);
    ybar = fma(lo, fma(-hs, v0, ge), ybar);
    ybar = fma(hi, fma(-hs, v1, -ge), ybar);
    if (a.gV) stg<T>(a.gV, c, fma(-hs * (Y[-IX] + Y[0]), lo, gv));
    const T* GY = sgy + x + y * BX + z * (BX * (BY + 2));
    ybar = fma(GY[0] - GY[2 * BX], inv_2dx, ybar);
    lo = adj_face(K[-IXY], K[0], inv_dx);
    hi = adj_face(K[0], K[IXY], inv_dx);
    ybar = fma(lo, fma(-hs, w0, ge), ybar);
    ybar = fma(hi, fma(-hs, w1, -ge), ybar);
    if (a.gW) stg<T>(a.gW, c, fma(-hs * (Y[-IXY] + Y[0]), lo, gw));
    const T* GZ = sgz + tid;
    ybar = fma(GZ[0] - GZ[2 * BX * BY], inv_2dx, ybar);
    if (a.lam_out) stg<T>(a.lam_out, c, lb + ybar);
    if (a.kap_out) stg<T>(a.kap_out, c, fma(a.ka, ybar, a.kb * lp));
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
// 32x8x4 and 16x4x4 were 0-60 % slower); large planes take 32x16x1 (the z halo of a 16x8x4 brick is
// copies of the one plane).
template <typename T>
hipError_t launch_adjoint_brick(const AdjArgs<T>& a, hipStream_t st)
{
    if (a.nz == 1 && (long long)a.nx * a.ny > 362LL * 362) return launch_adjoint_brick_shape<T, 32, 16, 1>(a, st);
    return launch_adjoint_brick_shape<T, 16, 8, 4>(a, st);
}
template hipError_t launch_adjoint_brick<float>(const AdjArgs<float>&, hipStream_t);
template hipError_t launch_adjoint_brick<double>(const AdjArgs<double>&, hipStream_t);

// us for the four reverse stages of an RK4 step, march / bricks: FP32 32^3 38.6 / 19.9, 64^3 42.4 /
// 23.7, 96^3 58.5 / 49.2, 128^3 100.2 / 98.2, 160^3 165 / 178; FP64 32^3 41.9 / 20.3, 64^3 53.6 /
// 31.8, 96^3 98.8 / 81.7, 112^3 146.6 / 117.9, 128^3 164 / 171, 160^3 380 / 454; one plane 64^2
// FP64 35.8 / 19.9, 512^2 81 / 47.
bool adjoint_takes_bricks(int nx, int ny, int nz, int dtype)
{
    const long long n = dtype == PF_F32 ? 128 : 120;
    return nz == 1 || (long long)nx * ny * nz <= n * n * n;
}

}  // namespace pf
