// A whole Runge-Kutta step of a one-plane grid (nz = 1: the 2D problems of the paper) in one
// launch.
//
// A plane of 64^2 cells is a few workgroups' work, and a step in four launches (stage_tiled.hip:
// stage_plane_kernel) is four times the latency of one. Here a workgroup takes a 32 x 32 patch of
// the plane, a thread to each cell, and runs all stages on it in LDS: every stage is valid on two
// cells less on each side than the one before, so RK4 leaves 16 x 16 new cells of the patch
// (RK3 20 x 20, RK2 24 x 24). Field, velocities and accumulator of a cell stay in its thread's
// registers, only the stage value and its sharpening products pass through LDS: one round of loads
// and two barriers per stage. What bounds it: latency up to about one patch per compute unit
// (256^2 cells), then the halo cells evaluated again (RK4: a patch evaluates f at 2016 cells
// for 1024 in the plane's own four evaluations). us per RK4 step from graphs, four launches / this
// kernel: FP64 64^2 13.1 / 5.8, 256^2 14.9 / 6.4, 512^2 19.0 / 13.9, 1024^2 45.7 / 41.2, 2048^2
// 153.4 / 152.5, 4096^2 750 / 625; FP32 64^2 12.3 / 4.8, 512^2 16.2 / 10.0, 2048^2 108.3 / 104.3,
// 4096^2 499 / 429 (walls on x and y: 545 / 467), so it serves planes of every size.
//
// Same arithmetic in the same order as the stage launches, hence the same bits: the z-face sum is
// 2 phi, the z-difference and z-gradient are zero, both z-faces carry the cell's own q_z and W.
// WALLS: the patch's field is read through mirror indices; the thread of a ghost cell evaluates f at
// the ghost's mirror partner in the patch, so the ghost holds its partner's value in every stage,
// which is what the stage launches read there.
#include "pf_brick.h"
#include "pf_internal.h"

namespace pf {

template <typename T, int STAGES, bool WALLS, bool FAST>
__global__ void __launch_bounds__(1024) plane_step_kernel(PlaneStepArgs<T> a, int tiles_x)
{
    constexpr int P = 32, H = 2 * STAGES, B = P - 2 * H;
    __shared__ T s_y[2][P * P];
    __shared__ T s_qx[P * P];
    __shared__ T s_qy[P * P];

    const int nx = a.nx, ny = a.ny;
    const int bi = blockIdx.x % tiles_x, bj = blockIdx.x / tiles_x;
    const int lx = threadIdx.x % P, ly = threadIdx.x / P, o = threadIdx.x;
    const int ux = bi * B - H + lx, uy = bj * B - H + ly;
    const bool wx = WALLS && (a.walls & 1), wy = WALLS && (a.walls & 2), wz = WALLS && (a.walls & 4);
    // the patch reaches at most H + B cells beyond the plane's end: within one period, or one
    // mirror image, of an axis of P cells or more (FAST)
    auto per = [](int v, int n) { return brick_wrap<FAST>(v, n); };
    auto mir = [](int v, int n) { return brick_mirror<FAST>(v, n); };
    const int vx = wx ? mir(ux, nx) : ux, vy = wy ? mir(uy, ny) : uy;
    // where f is evaluated: the cell, or a ghost's partner (in the patch wherever it is needed)
    const int ex = vx - (bi * B - H), ey = vy - (bj * B - H);
    const bool in_patch = !WALLS || (ex >= 0 && ex < P && ey >= 0 && ey < P);
    const int gx = per(vx, nx), gy = per(vy, ny);
    const unsigned row = (unsigned)gy * (unsigned)nx, c = (row + (unsigned)gx) * (unsigned)sizeof(T);
    const T phi = ldg(a.phi, c);
    T u0 = ldg(a.U, c), u1 = ldg(a.U, (row + (unsigned)(gx + 1 == nx ? 0 : gx + 1)) * (unsigned)sizeof(T));
    T v0 = ldg(a.V, c),
      v1 = ldg(a.V, ((unsigned)(gy + 1 == ny ? 0 : gy + 1) * (unsigned)nx + (unsigned)gx) * (unsigned)sizeof(T));
    T w = ldg(a.W, c);
    if constexpr (WALLS) {  // velocities on wall faces (index 0 of a walled axis)
        if (wx && gx == 0) u0 = T(0);
        if (wx && gx == nx - 1) u1 = T(0);
        if (wy && gy == 0) v0 = T(0);
        if (wy && gy == ny - 1) v1 = T(0);
        if (wz) w = T(0);
    }
    s_y[0][o] = phi;
    __syncthreads();

    const int eo = in_patch ? ex + ey * P : o;
    T acc = phi;
    // RK4: y = phi + c_s f and acc += b_s f, the last stage acc + b f. RK3 (low storage): y2 from
    // phi, acc = phi + b f, then y3 and the new phi from acc. RK2: both from phi.
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        const T* y = s_y[s & 1];
        // q on one ring more than f needs: cells at least 2 s + 1 from the patch's edge
        T qz = T(0);
        if (lx >= 2 * s + 1 && lx < P - 2 * s - 1 && ly >= 2 * s + 1 && ly < P - 2 * s - 1) {
            const T pc = y[o];
            const T gxx = grad1(y[o + 1], y[o - 1], a.inv_2dx), gyy = grad1(y[o + P], y[o - P], a.inv_2dx);
            const T gz = grad1(pc, pc, a.inv_2dx);
            const T fac = sharpen_factor(pc, gxx, gyy, gz, a.delta2, a.hg);
            s_qx[o] = fac * gxx;
            s_qy[o] = fac * gyy;
            qz = fac * gz;
        }
        __syncthreads();
        const int m = 2 * s + 2;
        if (in_patch && lx >= m && lx < P - m && ly >= m && ly < P - m && ex >= m && ex < P - m && ey >= m &&
            ey < P - m) {
            const T pc = y[eo], xm = y[eo - 1], xp = y[eo + 1], ym = y[eo - P], yp = y[eo + P];
            const T sz = face_sum(pc, pc), dz = face_diff(pc, pc);
            const T f = cell_rhs(face_sum(xm, pc), face_sum(pc, xp), face_sum(ym, pc), face_sum(pc, yp), sz, sz,
                                 face_diff(xm, pc), face_diff(pc, xp), face_diff(ym, pc), face_diff(pc, yp), dz,
                                 dz, s_qx[eo - 1], s_qx[eo + 1], s_qy[eo - P], s_qy[eo + P], qz, qz, u0, u1, v0,
                                 v1, w, w, a.nhs[s], a.ge);
            if (s == STAGES - 1) {
                if (ux < nx && uy < ny)
                    stg<T>(a.out, c, fma(a.b[s], f, STAGES == 2 ? phi : acc));
            } else {
                s_y[(s + 1) & 1][o] = fma(a.c[s], f, STAGES == 3 && s == 1 ? acc : phi);
                if (STAGES == 4 || (STAGES == 3 && s == 0)) acc = fma(a.b[s], f, acc);
            }
        }
        if (s < STAGES - 1) __syncthreads();
    }
}

template <typename T>
hipError_t launch_plane_step(const PlaneStepArgs<T>& a, int stages, hipStream_t st)
{
    if (a.nx <= 0 || a.ny <= 0 || stages < 2 || stages > 4) return hipErrorInvalidValue;
    const int B = 32 - 4 * stages;
    const int tx = (a.nx + B - 1) / B, ty = (a.ny + B - 1) / B;
    const long long blocks = (long long)tx * ty;  // a plane is below 2^28 cells
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const bool fast = a.nx >= 32 && a.ny >= 32;
    using Kernel = void (*)(PlaneStepArgs<T>, int);
    auto pick = [&](auto SC) -> Kernel {
        constexpr int S = decltype(SC)::value;
        return !fast ? plane_step_kernel<T, S, true, false>
                     : (a.walls ? plane_step_kernel<T, S, true, true> : plane_step_kernel<T, S, false, true>);
    };
    const Kernel k = stages == 4 ? pick(IntC<4>()) : stages == 3 ? pick(IntC<3>()) : pick(IntC<2>());
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(1024), 0, st, a, tx);
    return hipGetLastError();
}
template hipError_t launch_plane_step<float>(const PlaneStepArgs<float>&, int, hipStream_t);
template hipError_t launch_plane_step<double>(const PlaneStepArgs<double>&, int, hipStream_t);

}  // namespace pf
