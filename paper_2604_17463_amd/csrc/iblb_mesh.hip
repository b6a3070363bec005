// Mesh kernels of the IBLB wetting step (gfx950): the launches of the mesh
// chain (its device code is in iblb_mesh_dev.h), the observables
// (iblb_obs.h) and the state's way in and out (iblb_io.h).
#include "iblb_io.h"
#include "iblb_mesh_dev.h"
#include "iblb_obs.h"

namespace iblb {

// LDS of the roles, sized at launch.  (Static LDS that allows few workgroups
// per compute unit makes the compiler claim VGPRs up to the count that allows
// no more waves than those: 97 instead of 80 for the move kernel, 169 instead
// of 112 for the node kernel, which then wait longer for room beside the bulk
// kernel's waves.)
extern __shared__ __align__(16) char lds[];

// LDS of a mesh launch: what the work needs, or more where the context holds
// the mesh kernels to fewer workgroups per compute unit (DevPtrs::mesh_lds).
static size_t lds_bytes(const DevPtrs &P, size_t need) { return need > (size_t)P.mesh_lds ? need : (size_t)P.mesh_lds; }

// Workgroups past the node blocks (with a viscosity contrast) clear this
// step's inside bits, which the next launch of the chain toggles.
template <typename R, int MODE>
__global__ void __launch_bounds__(256) k_move(DevPtrs P, int parity, double *Uout) {
    const int w = blockIdx.x;
    if (w >= P.nblk) {
        mask_clear_role(P, w - P.nblk, gridDim.x - P.nblk, parity);
        return;
    }
    move_role<R, MODE>(P, xcd_item(w, P.nblk), w == 0, parity, (MODE & MV_ADVECT) ? 1 : 0, Uout, lds);
}

// What follows the new positions: the volumes (or, when no droplet has a
// volume penalty, the whole node pass), the inside bits, the list of stamped
// tiles.
template <typename R, bool NODE, bool FEW, bool CONTRAST>
__global__ void __launch_bounds__(256) k_aux(DevPtrs P, int parity, int adv) {
    const int n0 = NODE ? P.nblk : P.n_chunks, n1 = CONTRAST ? P.n_chunks : 0;
    const int w = blockIdx.x;
    if (w < n0) {
        if constexpr (NODE) node_role<R, FEW, true>(P, xcd_item(w, n0), lds);
        else volume_role<R>(P, xcd_item(w, n0), (double *)lds);
    } else if (w < n0 + n1) {
        if constexpr (CONTRAST) inside_role<R>(P, w - n0, parity);
    } else {
        compact_role(P, w - n0 - n1, parity, *P.ctr + adv);
    }
}

// Many blocks: the kernel runs beside the bulk kernel, and its waves take
// the room that a bulk wave of 80 (16 bits) to 136 VGPRs (FP64) leaves.
template <typename R, bool FEW, bool SPREAD>
__global__ void __launch_bounds__(256) k_node(DevPtrs P) {
    node_role<R, FEW, SPREAD>(P, xcd_item(blockIdx.x, gridDim.x), lds);
}

template <typename R>
__global__ void __launch_bounds__(256) k_volume(DevPtrs P) {
    __shared__ double sv[256];
    volume_role<R>(P, xcd_item(blockIdx.x, gridDim.x), sv);
}

// V0 of each droplet = the same fixed-order sum the volume penalty uses.
__global__ void __launch_bounds__(64) k_set_v0(DevPtrs P) {
    DropDev *D = P.drops + blockIdx.x;
    const double V = droplet_partial_sum(P.tri_part, D->chunk_off, D->n_chunks, threadIdx.x);
    if (threadIdx.x == 0) D->V0 = V;
}

template <typename R>
__global__ void __launch_bounds__(256) k_inside(DevPtrs P, int slot) {
    inside_role<R>(P, blockIdx.x, slot);
}

__global__ void __launch_bounds__(256) k_mask_clear(DevPtrs P, int slot) {
    mask_clear_role(P, blockIdx.x, gridDim.x, slot);
}

__global__ void k_epoch(DevPtrs P) {
    if (threadIdx.x == 0) *P.ctr = *P.ctr + 1;
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------- launchers
template <typename R>
static hipError_t launch_move_t(const DevPtrs &P, int mode, int parity, double *Uout, hipStream_t s) {
    const dim3 block(256), grid(P.nblk), step(P.nblk + mask_clear_groups(P));
    switch (mode) {
    case MOVE_STEP: hipLaunchKernelGGL((k_move<R, MOVE_STEP>), step, block, lds_bytes(P, MOVE_LDS), s, P, parity, Uout); break;
    case MOVE_PLACE: hipLaunchKernelGGL((k_move<R, MOVE_PLACE>), step, block, lds_bytes(P, 0), s, P, parity, Uout); break;
    case MOVE_FLUSH: hipLaunchKernelGGL((k_move<R, MOVE_FLUSH>), grid, block, MOVE_LDS, s, P, parity, Uout); break;
    case MOVE_BINS: hipLaunchKernelGGL((k_move<R, MOVE_BINS>), grid, block, 0, s, P, parity, Uout); break;
    case MOVE_U: hipLaunchKernelGGL((k_move<R, MOVE_U>), grid, block, MOVE_LDS, s, P, parity, Uout); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_move(const DevPtrs &P, bool f64, int mode, int parity, double *Uout, hipStream_t s) {
    if (P.nblk == 0) return hipSuccess;
    return f64 ? launch_move_t<double>(P, mode, parity, Uout, s) : launch_move_t<float>(P, mode, parity, Uout, s);
}

template <typename R, bool CONTRAST>
static hipError_t launch_aux_t(const DevPtrs &P, int parity, int adv, hipStream_t s) {
    const dim3 grid((P.penalty ? P.n_chunks : P.nblk) + (CONTRAST ? P.n_chunks : 0) + compact_groups(P)), block(256);
    if (P.penalty) hipLaunchKernelGGL((k_aux<R, false, false, CONTRAST>), grid, block, lds_bytes(P, 256 * 8), s, P, parity, adv);
    else if (few_blocks(P)) hipLaunchKernelGGL((k_aux<R, true, true, CONTRAST>), grid, block, sizeof(NodeLds<R, true>), s, P, parity, adv);
    else hipLaunchKernelGGL((k_aux<R, true, false, CONTRAST>), grid, block, lds_bytes(P, sizeof(NodeLds<R, false>)), s, P,
                            parity, adv);
    return hipGetLastError();
}

hipError_t launch_aux(const DevPtrs &P, bool f64, int parity, int adv, hipStream_t s) {
    if (P.nblk == 0) return hipSuccess;
    if (P.contrast) return f64 ? launch_aux_t<double, true>(P, parity, adv, s) : launch_aux_t<float, true>(P, parity, adv, s);
    return f64 ? launch_aux_t<double, false>(P, parity, adv, s) : launch_aux_t<float, false>(P, parity, adv, s);
}

template <typename R>
static hipError_t launch_node_t(const DevPtrs &P, bool spread, hipStream_t s) {
    const dim3 grid(P.nblk), block(256);
    if (!spread) hipLaunchKernelGGL((k_node<R, false, false>), grid, block, sizeof(NodeLds<R, false>), s, P);
    else if (few_blocks(P)) hipLaunchKernelGGL((k_node<R, true, true>), grid, block, sizeof(NodeLds<R, true>), s, P);
    else hipLaunchKernelGGL((k_node<R, false, true>), grid, block,
                            lds_bytes(P, sizeof(NodeLds<R, false>)), s, P);
    return hipGetLastError();
}

hipError_t launch_node(const DevPtrs &P, bool f64, bool spread, hipStream_t s) {
    if (P.nblk == 0) return hipSuccess;
    return f64 ? launch_node_t<double>(P, spread, s) : launch_node_t<float>(P, spread, s);
}

hipError_t launch_volume(const DevPtrs &P, bool f64, hipStream_t s) {
    if (P.n_chunks == 0) return hipSuccess;
    if (f64) hipLaunchKernelGGL(k_volume<double>, dim3(P.n_chunks), dim3(256), 0, s, P);
    else hipLaunchKernelGGL(k_volume<float>, dim3(P.n_chunks), dim3(256), 0, s, P);
    return hipGetLastError();
}

hipError_t launch_set_v0(const DevPtrs &P, hipStream_t s) {
    if (P.n_drops == 0) return hipSuccess;
    hipLaunchKernelGGL(k_set_v0, dim3(P.n_drops), dim3(64), 0, s, P);
    return hipGetLastError();
}

hipError_t launch_mask_clear(const DevPtrs &P, int slot, hipStream_t s) {
    if (!P.contrast) return hipSuccess;
    hipLaunchKernelGGL(k_mask_clear, dim3(mask_clear_groups(P)), dim3(256), 0, s, P, slot);
    return hipGetLastError();
}

hipError_t launch_inside(const DevPtrs &P, bool f64, int slot, hipStream_t s) {
    if (P.n_chunks == 0) return hipSuccess;
    if (f64) hipLaunchKernelGGL(k_inside<double>, dim3(P.n_chunks), dim3(TRI_CHUNK), 0, s, P, slot);
    else hipLaunchKernelGGL(k_inside<float>, dim3(P.n_chunks), dim3(TRI_CHUNK), 0, s, P, slot);
    return hipGetLastError();
}

hipError_t launch_epoch(const DevPtrs &P, hipStream_t s) {
    hipLaunchKernelGGL(k_epoch, dim3(1), dim3(64), 0, s, P);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t g = (n + 255) / 256;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)(g < 4096 ? g : 4096)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

}  // namespace iblb
