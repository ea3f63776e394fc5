// Two RK stages on a brick of cells (the fused variants of small grids).
//
// The z-marches (pf_fused_body.h) keep a large device busy with one column tile per workgroup, but
// every workgroup of a march runs its planes one after the other: on a small grid the chunks are a
// few planes long, most iterations are warm-up and the launch takes the latency of a dozen
// load-barrier-compute rounds however few cells there are. Here a workgroup owns a BX x BY x BZ
// brick and handles all of it at once: one round of loads, then four phases with a barrier between
// them,
//   q1  the sharpening products of the stage input,
//   E1  the middle stage value on the brick plus two cells on every side,
//   q2  the sharpening products of the middle stage,
//   E2  the outputs,
// each cell on a thread of its own. The halo is evaluated again by every brick that needs it (an
// 8 x 8 x 8 brick: 5.1 x its cells in q1, 3.4 x in E1), which costs nothing while compute units
// are idle. What bounds it: latency (launch, one load round, four barriers), then vector issue.
// 32^3 FP32 RK4 step from graphs: four per-stage launches 27.7 us, two brick launches 11.0 (auto_step_variant
// has the other sizes and the line to the marches).
//
// Same arguments, same arithmetic in the same order as the fused sweeps, hence the same bits.
// Regions in LDS, for a brick at (i0, j0, k0), halo on every side:
//   IN 4 cells; MID 2 cells; q1 along its own axis 3 cells and 2 across it; q2 1 cell along its
//   own axis only (over the space of q1).
// Threads: cell e of MID is the brick's own cell e for e < BX BY BZ (slot 0, kept from E1 to E2 in
// registers), then its ring cells. The q1 cells outside MID and the q2 cells outside the brick need
// one component each.
// WALLS (a.walls): the stage input and phi are read through mirror indices, velocities on wall
// faces count as zero, and a ghost cell of MID takes the value of its mirror partner: its thread
// evaluates E1 at the partner's place, so no copy and no further barrier. Exactly what the walled
// sweeps and the per-stage kernel read there.
#include <type_traits>

#include "pf_brick.h"
#include "pf_internal.h"

namespace pf {

template <typename T, int BX, int BY, int BZ>
struct BrickLayout {
    static constexpr int TS = BX * BY * BZ;
    static constexpr int IX = BX + 8, IY = BY + 8, IZ = BZ + 8, IS = IX * IY * IZ;
    static constexpr int MX = BX + 4, MY = BY + 4, MZ = BZ + 4, MXY = MX * MY, MS = MXY * MZ;
    static constexpr int Q1X = (BX + 6) * MY * MZ, Q1Y = MX * (BY + 6) * MZ, Q1Z = MX * MY * (BZ + 6);
    static constexpr int Q2X = (BX + 2) * BY * BZ, Q2Y = BX * (BY + 2) * BZ, Q2Z = BX * BY * (BZ + 2);
    static constexpr int NRING = MS - TS;
    static constexpr int NOUT = 2 * (MY * MZ + MX * MZ + MX * MY);
    static constexpr int NH2 = 2 * (BY * BZ + BX * BZ + BX * BY);
    static constexpr int QS = Q1X + Q1Y + Q1Z;
    static_assert(Q2X + Q2Y + Q2Z <= QS, "q2 reuses the space of q1");
    static constexpr size_t bytes = sizeof(T) * (size_t)(IS + MS + QS);
};

template <typename T, int BX, int BY, int BZ, int NT, bool SWEEP_B, bool WIDE, bool WALLS, bool FAST>
__global__ void __launch_bounds__(NT) brick_kernel(FusedArgs<T> a, int tiles_x, int tiles_y)
{
    static_assert(!(WALLS && WIDE), "mirror reads are element-wise");
    using L = BrickLayout<T, BX, BY, BZ>;
    constexpr int VEC = 16 / (int)sizeof(T);
    constexpr int IX = L::IX, IY = L::IY, IZ = L::IZ, IXY = IX * IY;
    constexpr int MX = L::MX, MY = L::MY, MZ = L::MZ, MXY = L::MXY, TS = L::TS;
    constexpr int NS = (L::MS + NT - 1) / NT;   // MID slots per thread, slot 0 the brick's own
    constexpr int NO = (L::NOUT + NT - 1) / NT;
    constexpr int NP = (WIDE ? L::IS / VEC : L::IS);
    constexpr int NL = (NP + NT - 1) / NT;
    static_assert(TS <= NT && TS % 64 == 0, "one thread per own cell, ring cells on waves of their own");
    static_assert(BX % VEC == 0 && 4 % VEC == 0, "rows of whole 16-byte pieces");
    static_assert(TS + L::NH2 <= 2 * NT, "at most two q2 slots");
    static_assert(L::IS < 8192, "the range of the small divisions");

    __shared__ __align__(16) T s_in[L::IS];
    __shared__ T s_mid[L::MS];
    __shared__ T s_q[L::QS];
    T* const q1x = s_q;
    T* const q1y = s_q + L::Q1X;
    T* const q1z = s_q + L::Q1X + L::Q1Y;
    T* const q2x = s_q;
    T* const q2y = s_q + L::Q2X;
    T* const q2z = s_q + L::Q2X + L::Q2Y;

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    int b = xcd_tile_order(blockIdx.x, gridDim.x);
    const int ti = b % tiles_x;
    b /= tiles_x;
    const int i0 = ti * BX, j0 = (b % tiles_y) * BY, k0 = (b / tiles_y) * BZ;
    const int tid = threadIdx.x;
    const T inv_2dx = a.inv_2dx, d2 = a.delta2, hg = a.hg, ge = a.ge;
    const bool wx = WALLS && (a.walls & 1), wy = WALLS && (a.walls & 2), wz = WALLS && (a.walls & 4);
    // an index of the brick lies at most 4 cells below the domain and B + 3 cells beyond its end:
    // within one period, or one mirror image, of an axis of B + 4 cells or more (FAST)
    auto per = [](int v, int n) { return brick_wrap<FAST>(v, n); };
    auto mir = [](int v, int n) { return brick_mirror<FAST>(v, n); };
    auto mapx = [&](int v) { return WALLS && wx ? mir(v, nx) : per(v, nx); };
    auto mapy = [&](int v) { return WALLS && wy ? mir(v, ny) : per(v, ny); };
    auto mapz = [&](int v) { return WALLS && wz ? mir(v, nz) : per(v, nz); };
    constexpr unsigned ES = sizeof(T);
    const unsigned whole = (unsigned)((size_t)nx * ny * nz * ES);
    const rsrc_t ry = plane_rsrc(a.y, whole), rphi = plane_rsrc(a.phi, whole),
                 racc = plane_rsrc(a.acc_in, whole), rU = plane_rsrc(a.U, whole),
                 rV = plane_rsrc(a.V, whole), rW = plane_rsrc(a.W, whole);
    auto at = [&](int x, int y, int z) { return ((unsigned)(z * ny + y) * (unsigned)nx + (unsigned)x) * ES; };

    // ---- loads: the stage input, then the velocities (and sweep B's bases) of the MID slots
    typedef typename std::conditional<WIDE, v4i_t, T>::type piece_t;
    piece_t pre[NL];
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (NP % NT == 0 || e < NP) {
            constexpr int PR = WIDE ? IX / VEC : IX;  // pieces of a row
            const int row = SmallDiv<PR>::div(e), g = e - row * PR, z = SmallDiv<IY>::div(row), y = row - z * IY;
            const unsigned off = at(mapx(i0 - 4 + g * (WIDE ? VEC : 1)), mapy(j0 - 4 + y), mapz(k0 - 4 + z));
            if constexpr (WIDE)
                pre[s] = __builtin_amdgcn_raw_buffer_load_b128(ry, (int)off, 0, 0);
            else
                pre[s] = bload<T>(ry, off);
        }
    }
    int lx[NS], ly[NS], lz[NS];
    // where E1 evaluates the slot: offsets into IN and the q1 planes (the slot's own cell, or a
    // ghost's mirror partner), and whether it does
    int em[NS], ex[NS], ey[NS], ez[NS];
    bool on[NS], ev[NS];
    unsigned c0 = 0;  // slot 0: byte offset of the own cell
    T u0[NS], u1[NS], v0[NS], v1[NS], w0[NS], w1[NS], base[NS], acc = T(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int e = tid + s * NT;
        on[s] = e < L::MS;
        if (!on[s]) continue;
        int x, y, z;
        if (e < TS) {
            x = e % BX + 2;
            y = e / BX % BY + 2;
            z = e / (BX * BY) + 2;
        } else {
            int r = e - TS;
            if (r < 4 * MXY) {  // two planes below and two above
                z = SmallDiv<MXY>::div(r);
                const int t = r - z * MXY;
                y = SmallDiv<MX>::div(t);
                x = t - y * MX;
                z = z < 2 ? z : BZ + z;
            } else if (r < 4 * MXY + 4 * MX * BZ) {  // two rows before and two after, per plane
                r -= 4 * MXY;
                z = SmallDiv<4 * MX>::div(r);
                const int t = r - z * (4 * MX);
                y = SmallDiv<MX>::div(t);
                x = t - y * MX;
                z += 2;
                y = y < 2 ? y : BY + y;
            } else {  // two cells left and two right, per row
                r -= 4 * MXY + 4 * MX * BZ;
                x = r & 3;
                y = (r >> 2) % BY + 2;
                z = (r >> 2) / BY + 2;
                x = x < 2 ? x : BX + x;
            }
        }
        lx[s] = x;
        ly[s] = y;
        lz[s] = z;
        const int ux = i0 - 2 + x, uy = j0 - 2 + y, uz = k0 - 2 + z;
        int vx = ux, vy = uy, vz = uz;
        ev[s] = true;
        if constexpr (WALLS) {
            // a ghost cell is evaluated at its mirror partner, which lies in MID wherever the
            // ghost is read for a cell of the domain; one further out feeds nothing stored
            vx = wx ? mir(ux, nx) : ux;
            vy = wy ? mir(uy, ny) : uy;
            vz = wz ? mir(uz, nz) : uz;
            x = vx - (i0 - 2);
            y = vy - (j0 - 2);
            z = vz - (k0 - 2);
            ev[s] = x >= 0 && x < MX && y >= 0 && y < MY && z >= 0 && z < MZ;
            if (!ev[s]) continue;
        }
        em[s] = (x + 2) + (y + 2) * IX + (z + 2) * IXY;
        ex[s] = x + y * (BX + 6) + z * ((BX + 6) * MY);
        ey[s] = x + y * MX + z * (MX * (BY + 6));
        ez[s] = x + y * MX + z * MXY;
        const int gx = per(vx, nx), gy = per(vy, ny), gz = per(vz, nz);
        const unsigned c = at(gx, gy, gz);
        if (s == 0) c0 = c;
        u0[s] = bload<T>(rU, c);
        u1[s] = bload<T>(rU, at(gx + 1 == nx ? 0 : gx + 1, gy, gz));
        v0[s] = bload<T>(rV, c);
        v1[s] = bload<T>(rV, at(gx, gy + 1 == ny ? 0 : gy + 1, gz));
        w0[s] = bload<T>(rW, c);
        w1[s] = bload<T>(rW, at(gx, gy, gz + 1 == nz ? 0 : gz + 1));
        if (SWEEP_B) {
            base[s] = bload<T>(rphi, c);
            if (s == 0 && tid < TS) acc = bload<T>(racc, c);
        }
        if constexpr (WALLS) {  // velocities on wall faces (index 0 of a walled axis)
            if (wx && gx == 0) u0[s] = T(0);
            if (wx && gx == nx - 1) u1[s] = T(0);
            if (wy && gy == 0) v0[s] = T(0);
            if (wy && gy == ny - 1) v1[s] = T(0);
            if (wz && gz == 0) w0[s] = T(0);
            if (wz && gz == nz - 1) w1[s] = T(0);
        }
    }
#pragma unroll
    for (int s = 0; s < NL; ++s) {
        const int e = tid + s * NT;
        if (NP % NT == 0 || e < NP) {
            if constexpr (WIDE)
                *reinterpret_cast<v4i_t*>(s_in + e * VEC) = pre[s];
            else
                s_in[e] = pre[s];
        }
    }
    __syncthreads();

    // ---- q1 on MID, and one component on the cells next to it
    auto sharpen = [&](const T* p, int sy, int sz, T g[3]) -> T {  // g and the factor at *p
        g[0] = grad1(p[1], p[-1], inv_2dx);
        g[1] = grad1(p[sy], p[-sy], inv_2dx);
        g[2] = grad1(p[sz], p[-sz], inv_2dx);
        return sharpen_factor(p[0], g[0], g[1], g[2], d2, hg);
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (!on[s]) continue;
        T g[3];
        const T fac = sharpen(s_in + (lx[s] + 2) + (ly[s] + 2) * IX + (lz[s] + 2) * IXY, IX, IXY, g);
        q1x[(lx[s] + 1) + ly[s] * (BX + 6) + lz[s] * ((BX + 6) * MY)] = fac * g[0];
        q1y[lx[s] + (ly[s] + 1) * MX + lz[s] * (MX * (BY + 6))] = fac * g[1];
        q1z[lx[s] + ly[s] * MX + (lz[s] + 1) * MXY] = fac * g[2];
    }
#pragma unroll
    for (int s = 0; s < NO; ++s) {
        // the threads without a last MID slot come first
        int e = s * NT + (NT - 1 - tid);
        if (e >= L::NOUT) continue;
        T g[3];
        if (e < 2 * MY * MZ) {
            const int side = e >= MY * MZ, t = e - side * (MY * MZ);
            const int z = SmallDiv<MY>::div(t), y = t - z * MY;
            const T fac = sharpen(s_in + (side ? BX + 6 : 1) + (y + 2) * IX + (z + 2) * IXY, IX, IXY, g);
            q1x[(side ? BX + 5 : 0) + y * (BX + 6) + z * ((BX + 6) * MY)] = fac * g[0];
        } else if (e < 2 * MY * MZ + 2 * MX * MZ) {
            e -= 2 * MY * MZ;
            const int side = e >= MX * MZ, t = e - side * (MX * MZ);
            const int z = SmallDiv<MX>::div(t), x = t - z * MX;
            const T fac = sharpen(s_in + (x + 2) + (side ? BY + 6 : 1) * IX + (z + 2) * IXY, IX, IXY, g);
            q1y[x + (side ? BY + 5 : 0) * MX + z * (MX * (BY + 6))] = fac * g[1];
        } else {
            e -= 2 * MY * MZ + 2 * MX * MZ;
            const int side = e >= MXY, t = e - side * MXY;
            const int y = SmallDiv<MX>::div(t), x = t - y * MX;
            const T fac = sharpen(s_in + (x + 2) + (y + 2) * IX + (side ? BZ + 6 : 1) * IXY, IX, IXY, g);
            q1z[x + y * MX + (side ? BZ + 5 : 0) * MXY] = fac * g[2];
        }
    }
    __syncthreads();

    // ---- E1: f at the stage input, the middle stage value on MID
    T f1_acc = T(0), own_phi = T(0);
    auto rhs = [&](const T* p, int sy, int sz, const T* qx, const T* qy, int qys, const T* qz, int qzs, int s,
                   T nhs) {
        const T pc = p[0], xm = p[-1], xp = p[1], ym = p[-sy], yp = p[sy], zm = p[-sz], zp = p[sz];
        return cell_rhs(face_sum(xm, pc), face_sum(pc, xp), face_sum(ym, pc), face_sum(pc, yp),
                        face_sum(zm, pc), face_sum(pc, zp), face_diff(xm, pc), face_diff(pc, xp),
                        face_diff(ym, pc), face_diff(pc, yp), face_diff(zm, pc), face_diff(pc, zp),
                        qx[0], qx[2], qy[0], qy[2 * qys], qz[0], qz[2 * qzs], u0[s], u1[s], v0[s],
                        v1[s], w0[s], w1[s], nhs, ge);
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (!on[s] || !ev[s]) continue;
        const T* p = s_in + em[s];
        const T f1 = rhs(p, IX, IXY, q1x + ex[s], q1y + ey[s], MX, q1z + ez[s], MXY, s, a.nhs1);
        const T pc = p[0];
        s_mid[lx[s] + ly[s] * MX + lz[s] * MXY] = fma(a.c_mid, f1, SWEEP_B ? base[s] : pc);
        if (s == 0) {
            own_phi = pc;
            f1_acc = fma(a.c_acc1, f1, SWEEP_B ? acc : pc);
        }
    }
    __syncthreads();

    // ---- q2 on the brick, and one component on the cells next to it
    const bool own = tid < TS;
    if (own) {
        T g[3];
        const int x = lx[0] - 2, y = ly[0] - 2, z = lz[0] - 2;
        const T fac = sharpen(s_mid + lx[0] + ly[0] * MX + lz[0] * MXY, MX, MXY, g);
        q2x[(x + 1) + y * (BX + 2) + z * ((BX + 2) * BY)] = fac * g[0];
        q2y[x + (y + 1) * BX + z * (BX * (BY + 2))] = fac * g[1];
        q2z[x + y * BX + (z + 1) * (BX * BY)] = fac * g[2];
    }
#pragma unroll
    for (int h = 0; h < (TS + L::NH2 > NT ? 2 : 1); ++h) {
        // threads above the brick's own first, then from the start
        int e = h == 0 ? tid - TS : (NT - TS) + tid;
        if (e < 0 || e >= L::NH2 || (h == 1 && e < NT - TS)) continue;
        T g[3];
        if (e < 2 * BY * BZ) {
            const int side = e >= BY * BZ, t = e - side * (BY * BZ), y = t % BY, z = t / BY;
            const T fac = sharpen(s_mid + (side ? BX + 2 : 1) + (y + 2) * MX + (z + 2) * MXY, MX, MXY, g);
            q2x[(side ? BX + 1 : 0) + y * (BX + 2) + z * ((BX + 2) * BY)] = fac * g[0];
        } else if (e < 2 * BY * BZ + 2 * BX * BZ) {
            e -= 2 * BY * BZ;
            const int side = e >= BX * BZ, t = e - side * (BX * BZ), x = t % BX, z = t / BX;
            const T fac = sharpen(s_mid + (x + 2) + (side ? BY + 2 : 1) * MX + (z + 2) * MXY, MX, MXY, g);
            q2y[x + (side ? BY + 1 : 0) * BX + z * (BX * (BY + 2))] = fac * g[1];
        } else {
            e -= 2 * BY * BZ + 2 * BX * BZ;
            const int side = e >= BX * BY, t = e - side * (BX * BY), x = t % BX, y = t / BX;
            const T fac = sharpen(s_mid + (x + 2) + (y + 2) * MX + (side ? BZ + 2 : 1) * MXY, MX, MXY, g);
            q2z[x + y * BX + (side ? BZ + 1 : 0) * (BX * BY)] = fac * g[2];
        }
    }
    __syncthreads();

    // ---- E2: f at the middle stage value, the outputs
    if (!own) return;
    const int x = lx[0] - 2, y = ly[0] - 2, z = lz[0] - 2;
    if (i0 + x >= nx || j0 + y >= ny || k0 + z >= nz) return;
    const T* p = s_mid + lx[0] + ly[0] * MX + lz[0] * MXY;
    const T f2 = rhs(p, MX, MXY, q2x + x + y * (BX + 2) + z * ((BX + 2) * BY),
                     q2y + x + y * BX + z * (BX * (BY + 2)), BX, q2z + x + y * BX + z * (BX * BY), BX * BY, 0,
                     a.nhs2);
    if (a.out_mid) bstore(plane_rsrc(a.out_mid, whole), c0, p[0]);
    if (!SWEEP_B) {
        bstore(plane_rsrc(a.out_y, whole), c0, fma(a.c_y2, f2, own_phi));
        if (a.out_phi) bstore(plane_rsrc(a.out_phi, whole), c0, own_phi);
    }
    if (SWEEP_B || a.out_acc) bstore(plane_rsrc(a.out_acc, whole), c0, fma(a.c_acc2, f2, f1_acc));
}

template <typename T, int BX, int BY, int BZ, int NT>
hipError_t launch_brick(const FusedArgs<T>& a, bool sweep_b, hipStream_t st)
{
    static_assert(BrickLayout<T, BX, BY, BZ>::bytes <= 160 * 1024, "the regions fit in LDS");
    using L = BrickLayout<T, BX, BY, BZ>;
    static_assert(SmallDiv<L::MXY>::exact(0, L::MS) && SmallDiv<L::MX>::exact(0, L::MXY) &&
                      SmallDiv<4 * L::MX>::exact(0, 4 * L::MX * BZ) && SmallDiv<L::MY>::exact(0, L::MY * L::MZ) &&
                      SmallDiv<L::MX>::exact(0, L::MX * L::MZ) && SmallDiv<L::IX>::exact(0, L::IS) &&
                      SmallDiv<L::IX * (int)sizeof(T) / 16>::exact(0, L::IS * (int)sizeof(T) / 16) &&
                      SmallDiv<L::IY>::exact(0, L::IY * L::IZ),
                  "the small divisions are exact over their ranges");
    if (a.nx <= 0 || a.ny <= 0 || a.nz <= 0) return hipErrorInvalidValue;
    // 32-bit offsets into whole arrays: larger fields take the marches
    if (field_needs_big(a.nx, a.ny, a.nz, sizeof(T))) return launch_fused<T, 32, 16, 0, false>(a, sweep_b, st);
    const int tx = (a.nx + BX - 1) / BX, ty = (a.ny + BY - 1) / BY, tz = (a.nz + BZ - 1) / BZ;
    const long long blocks = (long long)tx * ty * tz;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool fast = a.nx >= BX + 4 && a.ny >= BY + 4 && a.nz >= BZ + 4;
    const bool wide = fast && a.walls == 0 && a.nx % (16 / (int)sizeof(T)) == 0;
    using Kernel = void (*)(FusedArgs<T>, int, int);
    const Kernel k =
        sweep_b ? (wide                ? brick_kernel<T, BX, BY, BZ, NT, true, true, false, true>
                   : !fast             ? brick_kernel<T, BX, BY, BZ, NT, true, false, true, false>
                   : a.walls           ? brick_kernel<T, BX, BY, BZ, NT, true, false, true, true>
                                       : brick_kernel<T, BX, BY, BZ, NT, true, false, false, true>)
                : (wide                ? brick_kernel<T, BX, BY, BZ, NT, false, true, false, true>
                   : !fast             ? brick_kernel<T, BX, BY, BZ, NT, false, false, true, false>
                   : a.walls           ? brick_kernel<T, BX, BY, BZ, NT, false, false, true, true>
                                       : brick_kernel<T, BX, BY, BZ, NT, false, false, false, true>);
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(NT), 0, st, a, tx, ty);
    return hipGetLastError();
}

#define PF_BRICK_INST(T, BX, BY, BZ, NT) \
    template hipError_t launch_brick<T, BX, BY, BZ, NT>(const FusedArgs<T>&, bool, hipStream_t);
PF_BRICK_INST(float, 8, 8, 8, 1024)
PF_BRICK_INST(float, 8, 8, 4, 512)
PF_BRICK_INST(float, 16, 8, 8, 1024)
PF_BRICK_INST(double, 8, 8, 8, 1024)
PF_BRICK_INST(double, 8, 8, 4, 512)

}  // namespace pf
