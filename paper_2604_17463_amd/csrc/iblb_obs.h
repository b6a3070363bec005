// Observables of the IBLB wetting step (gfx950): mass and largest bare
// velocity per box, and the mesh observables per droplet, in three launches
// whatever the number of boxes and droplets.  The results go straight to
// the host's pinned buffer.
//
// All sums are FP64 over fixed partitions and fixed trees, so a result does
// not depend on the launch or on what else the context holds.
//
// Bound: the read of the populations (first launch) and, for small boxes,
// the latency of three dependent launches.  The mesh sums are cut by
// triangle chunks because one workgroup per droplet, walking all its
// triangles twice, took 30 / 209 / 900 / 1,321 us at 642 / 10,242 / 40,962 /
// 59,292 nodes; now the first pass hides beside the populations' read and
// the other two launches take 10-13 and 8-9 us.  The boxes share one launch
// because 64 pairs of launches of 21 + 4.5 us took 1.6 ms for the 64 uneven
// boxes of 28 M cells; now 0.39 ms (5.5 TB/s).  256x256x128 in BF16: 133 ->
// 69 us (4.6 TB/s); 250x250x150 in FP32: 147 -> 132 us (5.4 TB/s).
#pragma once
#include "iblb_device.h"

namespace iblb {

namespace {

// Sum / minimum / maximum of NV values per thread over a workgroup of 256:
// the waves' shuffles, then the four wave results in order.  Every thread
// gets the result.  op[k]: 0 sum, 1 minimum, 2 maximum.
template <int NV, typename Op>
__device__ __forceinline__ void block_reduce256(double (&v)[NV], double (*sh)[NV], Op op) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v[k] = op(k, v[k], __shfl_xor(v[k], o, 64));
        if (lane == 0) sh[wave][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = op(k, op(k, sh[0][k], sh[1][k]), op(k, sh[2][k], sh[3][k]));
    __syncthreads();
}

struct SumOp {
    __device__ double operator()(int, double a, double b) const { return a + b; }
};

// First pass over a droplet's chunk: z range and sum of its share of the
// nodes, and of its triangles the volume (about the droplet's reference
// point), area and area-weighted centroid.
enum { P_ZMIN, P_ZMAX, P_MX, P_MY, P_MZ, P_VOL, P_AREA, P_CX, P_CY, P_CZ, NP1 };
struct Pass1Op {
    __device__ double operator()(int k, double a, double b) const {
        return k == P_ZMIN ? fmin(a, b) : (k == P_ZMAX ? fmax(a, b) : a + b);
    }
};
// Second pass: the volume moments about the node mean, then the sum and the
// number of the contact-plane crossings.
constexpr int NP2 = 12;
static_assert(NP1 == OBS_PASS1 && NP2 == OBS_PASS2, "partial sums per triangle chunk");

template <typename R> struct Pos {
    const R *qh, *ql;
    int N;
    __device__ __forceinline__ double operator()(int j, int a) const {
        return (double)qh[a * N + j] + (double)ql[a * N + j];
    }
};

template <typename R>
__device__ __forceinline__ void drop_pass1(const DevPtrs &P, int ci, double (*sh)[NP1]) {
    const TriChunk ch = P.chunks[ci];
    const DropDev &D = P.drops[ch.drop];
    const Pos<R> pos{(const R *)P.qh, (const R *)P.ql, P.Ntot};
    double v[NP1];
#pragma unroll
    for (int k = 0; k < NP1; ++k) v[k] = 0.0;
    v[P_ZMIN] = DBL_MAX;
    v[P_ZMAX] = -DBL_MAX;
    // this chunk's share of the nodes
    const int i = ci - D.chunk_off;
    const int k0 = (int)((int64_t)D.n_nodes * i / D.n_chunks), k1 = (int)((int64_t)D.n_nodes * (i + 1) / D.n_chunks);
    for (int k = k0 + (int)threadIdx.x; k < k1; k += 256) {
        const int j = D.node_off + k;
        const double z = pos(j, 2);
        v[P_ZMIN] = fmin(v[P_ZMIN], z);
        v[P_ZMAX] = fmax(v[P_ZMAX], z);
        v[P_MX] += pos(j, 0);
        v[P_MY] += pos(j, 1);
        v[P_MZ] += z;
    }
    const int t = ch.t0 + threadIdx.x;
    if (t < ch.t1) {
        double p[3][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int j = P.tri[3 * t + c];
#pragma unroll
            for (int a = 0; a < 3; ++a) p[c][a] = pos(j, a) - D.ref[a];
        }
        const double bc0 = p[1][1] * p[2][2] - p[1][2] * p[2][1];
        const double bc1 = p[1][2] * p[2][0] - p[1][0] * p[2][2];
        const double bc2 = p[1][0] * p[2][1] - p[1][1] * p[2][0];
        v[P_VOL] = (p[0][0] * bc0 + p[0][1] * bc1 + p[0][2] * bc2) / 6.0;
        double e1[3], e2[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            e1[a] = p[1][a] - p[0][a];
            e2[a] = p[2][a] - p[0][a];
        }
        const double n0 = e1[1] * e2[2] - e1[2] * e2[1];
        const double n1 = e1[2] * e2[0] - e1[0] * e2[2];
        const double n2 = e1[0] * e2[1] - e1[1] * e2[0];
        const double At = 0.5 * sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        v[P_AREA] = At;
        v[P_CX] = At * (p[0][0] + p[1][0] + p[2][0]) / 3.0;
        v[P_CY] = At * (p[0][1] + p[1][1] + p[2][1]) / 3.0;
        v[P_CZ] = At * (p[0][2] + p[1][2] + p[2][2]) / 3.0;
    }
    block_reduce256(v, sh, Pass1Op());
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NP1; ++k) P.obs_part1[(int64_t)ci * NP1 + k] = v[k];
}

// A droplet's first-pass result from its chunks' partials, the same in
// every workgroup that asks.
__device__ __forceinline__ void drop_totals(const DevPtrs &P, const DropDev &D, double (&v)[NP1], double (*sh)[NP1]) {
#pragma unroll
    for (int k = 0; k < NP1; ++k) v[k] = 0.0;
    v[P_ZMIN] = DBL_MAX;
    v[P_ZMAX] = -DBL_MAX;
    Pass1Op op;
    for (int i = threadIdx.x; i < D.n_chunks; i += 256) {
        const double *p = P.obs_part1 + (int64_t)(D.chunk_off + i) * NP1;
#pragma unroll
        for (int k = 0; k < NP1; ++k) v[k] = op(k, v[k], p[k]);
    }
    block_reduce256(v, sh, op);
}

// The moments of the enclosed volume about the node mean m (for the
// deformation index): over the tetrahedron (m, a, b, c) of each triangle,
// with p the corners relative to m, s = p_a + p_b + p_c and
// v = p_a . (p_b x p_c) / 6,
//   int dV = v,  int x dV = v s / 4,  int x x^T dV = v (sum p p^T + s s^T) / 20;
// and the edge crossings of the plane z = z_min + xi, each edge counted in
// the triangle that walks it from its lower node id.
template <typename R>
__device__ __forceinline__ void drop_pass2(const DevPtrs &P, int ci, double (*sh1)[NP1], double (*sh2)[NP2]) {
    const TriChunk ch = P.chunks[ci];
    const DropDev &D = P.drops[ch.drop];
    const Pos<R> pos{(const R *)P.qh, (const R *)P.ql, P.Ntot};
    const int t = ch.t0 + threadIdx.x;
    const bool on = t < ch.t1;
    int id[3] = {0, 0, 0};
    double q[3][3];
    if (on) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            id[c] = P.tri[3 * t + c];
#pragma unroll
            for (int a = 0; a < 3; ++a) q[c][a] = pos(id[c], a);
        }
    }
    double tot[NP1];
    drop_totals(P, D, tot, sh1);
    const double inv = (double)max(D.n_nodes, 1);
    const double mean[3] = {tot[P_MX] / inv, tot[P_MY] / inv, tot[P_MZ] / inv};
    const double c0 = tot[P_CX] / tot[P_AREA] + D.ref[0], c1 = tot[P_CY] / tot[P_AREA] + D.ref[1];
    const double zc = tot[P_ZMIN] + D.xi;
    double m[NP2];
#pragma unroll
    for (int k = 0; k < NP2; ++k) m[k] = 0.0;
    if (on) {
        double r[3][3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < 3; ++a) r[c][a] = q[c][a] - mean[a];
        const double v = (r[0][0] * (r[1][1] * r[2][2] - r[1][2] * r[2][1]) +
                          r[0][1] * (r[1][2] * r[2][0] - r[1][0] * r[2][2]) +
                          r[0][2] * (r[1][0] * r[2][1] - r[1][1] * r[2][0])) / 6.0;
        const double s[3] = {r[0][0] + r[1][0] + r[2][0], r[0][1] + r[1][1] + r[2][1],
                             r[0][2] + r[1][2] + r[2][2]};
        m[0] = v;
#pragma unroll
        for (int a = 0; a < 3; ++a) m[1 + a] = v * s[a] / 4.0;
        constexpr int I[6] = {0, 1, 2, 0, 0, 1}, J[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int e = 0; e < 6; ++e)
            m[4 + e] = v * (r[0][I[e]] * r[0][J[e]] + r[1][I[e]] * r[1][J[e]] + r[2][I[e]] * r[2][J[e]] +
                            s[I[e]] * s[J[e]]) / 20.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int d = (c + 1) % 3;
            if (id[c] > id[d]) continue;
            const double za = q[c][2], zb = q[d][2];
            if ((za < zc) == (zb < zc)) continue;
            const double f = (zc - za) / (zb - za);
            const double px = q[c][0] + f * (q[d][0] - q[c][0]) - c0;
            const double py = q[c][1] + f * (q[d][1] - q[c][1]) - c1;
            m[10] += sqrt(px * px + py * py);
            m[11] += 1.0;
        }
    }
    block_reduce256(m, sh2, SumOp());
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < NP2; ++k) P.obs_part2[(int64_t)ci * NP2 + k] = m[k];
}

// Mass and largest bare velocity of the current populations of one group of
// rows.  Each wave takes whole rows (row addressing in scalar registers,
// lanes along x).  The largest |j| / rho is found without a division per
// cell: |j|^2 rho_best^2 against |j_best|^2 rho^2; where those products could
// leave the range of FP64, by the quotient itself.  A negative density or one
// that is not a number gives no speed (the status word reports it).
template <int ST>
__device__ __forceinline__ void box_pass1(const DevPtrs &P, int gi, int parity, float inv, double (*sh)[2]) {
    using S = Stor<ST>;
    using R = typename S::R;
    const IBLB_CONST ObsGroup &G = ((const IBLB_CONST ObsGroup *)P.obs_groups)[gi];
    const IBLB_CONST BoxDev *B = (const IBLB_CONST BoxDev *)P.boxes + G.box;
    const int nx = B->nx, ny = B->ny, nz = B->nz, sx = B->sx;
    const bool zper = B->zbc == 1, moving = B->moving != 0;
    const double rho0 = B->rho0;
    R kw[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) kw[a] = (R)(6.0 * rho0 * B->uw[a]);
    const IBLB_GLOBAL char *src = (const IBLB_GLOBAL char *)B->f[parity];
    const uint64_t pb = (uint64_t)B->plane * sizeof(typename S::T);
    const int lane = threadIdx.x & 63, r1 = G.r1;
    double m = 0.0, bj = 0.0, br = 1.0;  // mass; |j|^2 and rho of the fastest cell
    double far = 0.0;                    // largest quotient
    for (int r = __builtin_amdgcn_readfirstlane(G.r0 + (int)(threadIdx.x >> 6)); r < r1; r += 4) {
        const int z = r / ny, y = r - z * ny;
        const RowAddr ra = row_addr(y, z, ny, nz, sx, zper, sizeof(typename S::T));
        for (int x = lane; x < nx; x += 64) {
            R g[Q];
            pull<ST>(src, pb, ra, x, nx, inv, g);
            if (moving && (ra.wlo || ra.whi)) wall_shift<R>(g, ra.wlo, ra.whi, kw);  // g holds unscaled deviations
            double dr = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                dr += (double)g[i];
                jx += cx_of(i) * (double)g[i];
                jy += cy_of(i) * (double)g[i];
                jz += cz_of(i) * (double)g[i];
            }
            m += dr;
            const double j2 = jx * jx + jy * jy + jz * jz, rho = rho0 + dr;
            if (j2 < 1e75 && rho < 1e75 && rho > 1e-75) {
                if (j2 * (br * br) > bj * (rho * rho)) {
                    bj = j2;
                    br = rho;
                }
            } else {
                far = fmax(far, sqrt(j2) / rho);
            }
        }
    }
    double v[2] = {m, fmax(sqrt(bj) / br, far)};
    block_reduce256(v, sh, [](int k, double a, double b) { return k == 0 ? a + b : fmax(a, b); });
    if (threadIdx.x == 0) {
        P.obs_part[2 * (int64_t)gi] = v[0];
        P.obs_part[2 * (int64_t)gi + 1] = v[1];
    }
}

}  // namespace

// First launch: the row groups of every box, then the triangle chunks of
// every droplet (both only read the state, so they run side by side).
template <int ST>
__global__ void __launch_bounds__(256) k_obs1(DevPtrs P, int parity, float inv) {
    __shared__ double sh[4][NP1];
    if ((int)blockIdx.x < P.n_obs_groups)
        box_pass1<ST>(P, blockIdx.x, parity, inv, (double(*)[2])sh);
    else
        drop_pass1<typename Stor<ST>::R>(P, blockIdx.x - P.n_obs_groups, sh);
}

// Second launch: the second pass over the triangle chunks; and per box the
// sum of its groups, written out with the status word.
template <typename R>
__global__ void __launch_bounds__(256) k_obs2(DevPtrs P, double *out) {
    __shared__ double sh1[4][NP1], sh2[4][NP2];
    if ((int)blockIdx.x < P.n_chunks) {
        drop_pass2<R>(P, blockIdx.x, sh1, sh2);
        return;
    }
    const int box = blockIdx.x - P.n_chunks;
    const BoxDev &B = P.boxes[box];
    double v[2] = {0.0, 0.0};
    for (int k = B.obs_begin + (int)threadIdx.x; k < B.obs_end; k += 256) {
        v[0] += P.obs_part[2 * (int64_t)k];
        v[1] = fmax(v[1], P.obs_part[2 * (int64_t)k + 1]);
    }
    block_reduce256(v, (double(*)[2])sh1, [](int k, double a, double b) { return k == 0 ? a + b : fmax(a, b); });
    if (threadIdx.x == 0) {
        double *o = out + (int64_t)P.n_drops * OBS_DROP + (int64_t)box * OBS_BOX;
        o[0] = B.cells_rho0 + v[0];
        o[1] = v[1];
        if (box == 0) out[(int64_t)P.n_drops * OBS_DROP + (int64_t)P.n_boxes * OBS_BOX] = (double)*P.status;
    }
}

// Third launch, one workgroup per droplet: its totals.
__global__ void __launch_bounds__(256) k_obs3(DevPtrs P, double *out) {
    __shared__ double sh1[4][NP1], sh2[4][NP2];
    const DropDev &D = P.drops[blockIdx.x];
    double m[NP2];
#pragma unroll
    for (int k = 0; k < NP2; ++k) m[k] = 0.0;
    for (int i = threadIdx.x; i < D.n_chunks; i += 256) {
        const double *p = P.obs_part2 + (int64_t)(D.chunk_off + i) * NP2;
#pragma unroll
        for (int k = 0; k < NP2; ++k) m[k] += p[k];
    }
    double tot[NP1];
    drop_totals(P, D, tot, sh1);
    block_reduce256(m, sh2, SumOp());
    if (threadIdx.x == 0) {
        double *o = out + (int64_t)blockIdx.x * OBS_DROP;
        o[0] = tot[P_VOL];
        o[1] = tot[P_AREA];
        o[2] = tot[P_ZMIN];
        o[3] = tot[P_ZMAX];
        o[4] = tot[P_CX] / tot[P_AREA] + D.ref[0];
        o[5] = tot[P_CY] / tot[P_AREA] + D.ref[1];
        o[6] = tot[P_CZ] / tot[P_AREA] + D.ref[2];
        o[7] = m[10];
        o[8] = m[11];
        for (int e = 0; e < 10; ++e) o[9 + e] = m[e];
    }
}

hipError_t launch_obs(const DevPtrs &P, int storage, int parity, float inv, double *out, hipStream_t s) {
    const dim3 block(256), g1(P.n_obs_groups + P.n_chunks), g2(P.n_chunks + P.n_boxes);
    switch (storage) {
    case 0: hipLaunchKernelGGL(k_obs1<0>, g1, block, 0, s, P, parity, inv); break;
    case 1: hipLaunchKernelGGL(k_obs1<1>, g1, block, 0, s, P, parity, inv); break;
    case 2: hipLaunchKernelGGL(k_obs1<2>, g1, block, 0, s, P, parity, inv); break;
    default: hipLaunchKernelGGL(k_obs1<3>, g1, block, 0, s, P, parity, inv); break;
    }
    if (storage == 0) hipLaunchKernelGGL(k_obs2<double>, g2, block, 0, s, P, out);
    else hipLaunchKernelGGL(k_obs2<float>, g2, block, 0, s, P, out);
    if (P.n_drops > 0) hipLaunchKernelGGL(k_obs3, dim3(P.n_drops), block, 0, s, P, out);
    return hipGetLastError();
}

}  // namespace iblb
