// State in and out of the device (gfx950): populations in FP64 and node
// positions in the caller's order, converted by the GPU straight into or out
// of the host's pinned staging chunks.
//
// Bound: the host's copy between the staging chunk and the caller's pageable
// array (the GPU's side, PCIe, runs beside it).  The conversion is here
// because the host's loop over 19 values per cell took 36 ms to put in and
// take out the field of a 64x48x40 box, and because copying the whole hi and
// lo arrays to read one droplet's nodes took 40 ms over 64 droplets.
#pragma once
#include "iblb_device.h"

namespace iblb {

// Moving-wall term of population i reflected at the lower (z = 0) or upper
// wall: 6 w_i rho0 (c_i . u_w).
__device__ __forceinline__ double wall_term(const BoxDev &B, int i, bool lower) {
    const double *u = B.uw + (lower ? 0 : 2);
    return 6.0 * w_of(i) * B.rho0 * (cx_of(i) * u[0] + cy_of(i) * u[1]);
}

template <int ST> __device__ __forceinline__ double decode(const void *f, int64_t k, double scale) {
    using T = typename Stor<ST>::T;
    const double v = (double)(typename Stor<ST>::R)((const T *)f)[k];
    return Stor<ST>::SCALED ? v / scale : v;
}
template <int ST> __device__ __forceinline__ void encode(void *f, int64_t k, double v, double scale) {
    using T = typename Stor<ST>::T;
    if constexpr (Stor<ST>::SCALED) v *= scale;
    ((T *)f)[k] = (T)(typename Stor<ST>::R)v;
}

// Elements e0 .. e0 + n - 1 of the window's populations [19][ez][ey][ex]
// (those that the next step pulls) into out[0 .. n).  The weight's product
// is rounded by itself before the sum: a fluid at rest reads w rho0 exactly.
template <int ST>
__global__ void __launch_bounds__(256) k_read_f(DevPtrs P, int box, int parity, Window W, double scale, int64_t e0, int n,
                                                double *out) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const BoxDev &B = P.boxes[box];
    const int nx = B.nx, ny = B.ny, nz = B.nz;
    const bool zper = B.zbc == 1;
    const int64_t wcells = (int64_t)W.ext[0] * W.ext[1] * W.ext[2], e = e0 + k;
    const int i = (int)(e / wcells);
    const int cell = (int)(e - (int64_t)i * wcells);
    const int wr = cell / W.ext[0], wx = cell - wr * W.ext[0], wz = wr / W.ext[1], wy = wr - wz * W.ext[1];
    const int x = wrapn(W.lo[0] + wx, nx), y = wrapn(W.lo[1] + wy, ny);
    const int z = zper ? wrapn(W.lo[2] + wz, nz) : W.lo[2] + wz;
    const int zs = z - cz_of(i);
    int64_t src;
    double wall = 0.0;
    if (!zper && (zs < 0 || zs >= nz)) {
        src = (int64_t)opp_of(i) * B.plane + ((int64_t)z * ny + y) * B.sx + x;
        wall = wall_term(B, i, zs < 0);
    } else {
        src = (int64_t)i * B.plane + ((int64_t)wrapn(zs, nz) * ny + wrapn(y - cy_of(i), ny)) * B.sx +
              wrapn(x - cx_of(i), nx);
    }
    const double dev = decode<ST>(B.f[parity], src, scale) + wall;
    const double rest = w_of(i) * B.rho0;
    out[k] = rest + dev;
}

// The inverse: elements e0 .. e0 + n - 1 of the whole box's populations into
// buffer set `to`.  Population i at x was streamed from x - c_i, or, where
// that lies in a wall, reflected: then it is the opposite one stored at x.
template <int ST>
__global__ void __launch_bounds__(256) k_write_f(DevPtrs P, int box, int to, double scale, int64_t e0, int n,
                                                 const double *in) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const BoxDev &B = P.boxes[box];
    const int nx = B.nx, ny = B.ny, nz = B.nz;
    const bool zper = B.zbc == 1;
    const int64_t cells = (int64_t)nx * ny * nz, e = e0 + k;
    const int i = (int)(e / cells);
    const int cell = (int)(e - (int64_t)i * cells);
    const int r = cell / nx, x = cell - r * nx, z = r / ny, y = r - z * ny;
    const int zs = z - cz_of(i);
    double v = in[k];
    int64_t dst;
    if (!zper && (zs < 0 || zs >= nz)) {
        dst = (int64_t)opp_of(i) * B.plane + ((int64_t)z * ny + y) * B.sx + x;
        v -= wall_term(B, i, zs < 0);
    } else {
        dst = (int64_t)i * B.plane + ((int64_t)wrapn(zs, nz) * ny + wrapn(y - cy_of(i), ny)) * B.sx +
              wrapn(x - cx_of(i), nx);
    }
    const double rest = w_of(i) * B.rho0;
    encode<ST>(B.f[to], dst, v - rest, scale);
}

// Elements e0 .. e0 + n - 1 of a droplet's positions [n_nodes][3] in the
// caller's node order.
template <typename R>
__global__ void __launch_bounds__(256) k_read_q(DevPtrs P, int node_off, int64_t e0, int n, double *out) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const int64_t e = e0 + k;
    const int u = (int)(e / 3), a = (int)(e - 3 * (int64_t)u);
    const int64_t j = (int64_t)a * P.Ntot + P.node_of[node_off + u];
    out[k] = (double)((const R *)P.qh)[j] + (double)((const R *)P.ql)[j];
}

hipError_t launch_read_f(const DevPtrs &P, int storage, int box, int parity, const Window &W, double scale, int64_t e0,
                         int n, double *out, hipStream_t s) {
    const dim3 grid((n + 255) / 256), block(256);
    switch (storage) {
    case 0: hipLaunchKernelGGL(k_read_f<0>, grid, block, 0, s, P, box, parity, W, scale, e0, n, out); break;
    case 1: hipLaunchKernelGGL(k_read_f<1>, grid, block, 0, s, P, box, parity, W, scale, e0, n, out); break;
    case 2: hipLaunchKernelGGL(k_read_f<2>, grid, block, 0, s, P, box, parity, W, scale, e0, n, out); break;
    default: hipLaunchKernelGGL(k_read_f<3>, grid, block, 0, s, P, box, parity, W, scale, e0, n, out); break;
    }
    return hipGetLastError();
}

hipError_t launch_write_f(const DevPtrs &P, int storage, int box, int to, double scale, int64_t e0, int n,
                          const double *in, hipStream_t s) {
    const dim3 grid((n + 255) / 256), block(256);
    switch (storage) {
    case 0: hipLaunchKernelGGL(k_write_f<0>, grid, block, 0, s, P, box, to, scale, e0, n, in); break;
    case 1: hipLaunchKernelGGL(k_write_f<1>, grid, block, 0, s, P, box, to, scale, e0, n, in); break;
    case 2: hipLaunchKernelGGL(k_write_f<2>, grid, block, 0, s, P, box, to, scale, e0, n, in); break;
    default: hipLaunchKernelGGL(k_write_f<3>, grid, block, 0, s, P, box, to, scale, e0, n, in); break;
    }
    return hipGetLastError();
}

hipError_t launch_read_q(const DevPtrs &P, bool f64, int node_off, int64_t e0, int n, double *out, hipStream_t s) {
    const dim3 grid((n + 255) / 256), block(256);
    if (f64) hipLaunchKernelGGL(k_read_q<double>, grid, block, 0, s, P, node_off, e0, n, out);
    else hipLaunchKernelGGL(k_read_q<float>, grid, block, 0, s, P, node_off, e0, n, out);
    return hipGetLastError();
}

}  // namespace iblb
