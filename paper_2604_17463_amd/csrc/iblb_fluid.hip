// Fluid kernels of the IBLB wetting step (gfx950): the bulk fused
// pull-stream / moments / BGK-Guo collision with the body force only, over
// every cell outside this step's stamped band tiles; the band kernel, which
// gathers the spread interface force for each stamped tile and does the
// collision of its 64 cells with it.  The two write disjoint cells and run
// side by side.
#include "iblb_mesh_dev.h"

#include <algorithm>

namespace iblb {

// ------------------------------------------------------------------- bulk
// Every cell of every box with F = body force, except (SKIP) the cells of
// the band tiles this step's node pass stamped: the band kernel owns those
// (it adds the spread force) and runs beside this kernel, so each cell is
// pulled, collided and stored once per step.  A workgroup takes a row group
// (rows, or one segment of threads_x cells of rows longer than that; the
// segments of a row go to workgroups on one XCD, so the lines at their ends
// are fetched once); threads stride along x so the +-1 shifted loads of a
// row stay inside the workgroup or its XCD.  UROW: each wavefront lies in one row
// (threads_x a multiple of 64), so the row addressing is wave-uniform and
// lives in scalar registers.  NT: the populations are written with
// streaming stores (they are read again only in the next step; pays off
// once the two population buffers exceed the last-level cache).  EXT: some
// box has a viscosity contrast or a moving wall (the plain variant carries
// none of their registers).  Without SKIP the kernel is the plain
// stream-collide of every cell (boxes without droplets, timing).
// NTM: 0 plain stores, 1 streaming, 2 as `nt` says.
// EARLY: the rows run before this step's stamps are known, and a speed that
// only cells outside the band may not have is left to fast_role
// (DevPtrs::fast_tile), under the epoch that the stamps will carry.
template <int ST, bool UROW, int NTM, int CPT, bool EXT, bool SKIP, bool PADW, bool EARLY = false>
__device__ __forceinline__ void bulk_rows(const DevPtrs &P, const IBLB_CONST RowGroup &rg, int tx, int ty, int BX,
                                          int BY, int parity, int epoch, int full_u, float scale, float inv, int nt) {
    using S = Stor<ST>;
    using R = typename S::R;
    constexpr uint32_t EB = sizeof(typename S::T);
    // 2-byte storage goes through buffer resources (scalar row offsets, one
    // per-lane offset per access); 4- and 8-byte storage measured faster with
    // plain global addressing (us per step, buffer and global: 250x250x150
    // FP32 292 and 290, 64 boxes of 128x128x64 971 and 962, 256x256x128 FP64
    // 494 and 482)
    constexpr bool BUF = UROW && EB == 2;
    const IBLB_CONST BoxDev *B = (const IBLB_CONST BoxDev *)P.boxes + rg.box;
    const int nx = B->nx, ny = B->ny, nz = B->nz, sx = B->sx;
    const bool zper = B->zbc == 1;
    const uint64_t pb = (uint64_t)B->plane * EB;
    const IBLB_GLOBAL char *__restrict__ src = (const IBLB_GLOBAL char *)B->f[parity];
    IBLB_GLOBAL char *__restrict__ dst = (IBLB_GLOBAL char *)B->f[parity ^ 1];
    const R omega = (R)B->omega, guo = (R)B->guo, rho0 = (R)B->rho0;
    const R omega_in = (R)B->omega_in, guo_in = (R)B->guo_in;
    const bool contrast = B->contrast != 0, moving = B->moving != 0;
    const IBLB_GLOBAL uint64_t *mask = (const IBLB_GLOBAL uint64_t *)B->mask[parity];
    const IBLB_GLOBAL int32_t *stamp = (const IBLB_GLOBAL int32_t *)B->stamp[parity];
    const int tnx = B->tnx, tny = B->tny;
    const bool skip_box = SKIP && B->blk_end > B->blk_begin;  // only boxes holding droplets
    const R gx = (R)B->g[0], gy = (R)B->g[1], gz = (R)B->g[2];
    IBLB_GLOBAL R *__restrict__ uf = (IBLB_GLOBAL R *)B->ufull;
    const uint64_t plane = (uint64_t)B->plane;
    const PopRes rs = pop_res((const void *)src, pb), rd = pop_res((const void *)dst, pb);
    // row r = z * ny + y, stepped by BY without a division per row; a
    // thread takes CPT rows (BY apart) at a time, with the loads of all
    // of them issued before the first collision.  UROW: a row group has at
    // most BY * CPT rows of at most BX cells (padding included), so both
    // loops are left after one pass: what the compiler moved in front of
    // them, 38 plane and row addresses above all, outgrew the scalar
    // registers and was kept in vector lanes (FP32 without padded rows: 533
    // vector instructions, 198 of them such moves, and 91 VGPRs, now 334, 30
    // and 53; FP64 528 and 153, now 336 and 91; BF16 423 and 84, now 313 and
    // 49).
    int r = rg.r0 + ty;
    int z = r / ny, y = r - z * ny;
    for (; r < rg.r1; r += BY * CPT) {
        RowAddr ra[CPT];
        bool on[CPT];
        int ryk[CPT], rzk[CPT];
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            on[k] = r + k * BY < rg.r1;
            const int ry = UROW ? __builtin_amdgcn_readfirstlane(y) : y;
            const int rz = UROW ? __builtin_amdgcn_readfirstlane(z) : z;
            ryk[k] = ry;
            rzk[k] = rz;
            ra[k] = row_addr(ry, rz, ny, nz, sx, zper, EB);
            y += BY;
            while (y >= ny) {
                y -= ny;
                ++z;
            }
        }
        // PADW: some row group's x range reaches into its row's padding
        // (x1 > nx: the row table asks for it where the padding is a
        // small part of the row): the lanes x in [nx, sx) redo the row's
        // last cell and store zeros (the padding's value since init) in
        // the same store instructions as their neighbours, so that every
        // line of the row is written whole (a line written in part made
        // rows of 250 cells 10 % slower than rows of 256).  A separate
        // instantiation, so that workloads without it carry none of it.
        for (int x = rg.x0 + tx; x < rg.x1; x += BX) {
            R g[CPT][Q];
            const bool pad = PADW && x >= nx;
            const int xs = pad ? nx - 1 : x;  // the cell computed
            const XOff xo = x_off<EB>(xs, nx);
            const uint32_t xst = PADW ? (uint32_t)x * EB : xo.c;  // the cell stored
            bool mine[CPT];
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                mine[k] = on[k];
                if (skip_box && on[k])
                    mine[k] = stamp[((int64_t)(rzk[k] >> TZS) * tny + (ryk[k] >> TYS)) * tnx + (xs >> TXS)] != epoch;
            }
            if (CPT == 1 && !mine[0]) {
                if constexpr (UROW) break;
                else continue;
            }
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                if (CPT > 1 && !mine[k]) continue;
                if constexpr (BUF)
                    pull_buf<ST>(rs, (uint32_t)pb, ra[k], xo, g[k]);
                else
                    pull_raw<ST>(src, pb, ra[k], xo, g[k]);
            }
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                if (CPT > 1 && !mine[k]) continue;
                R out[Q], u[3], rho;
                const uint32_t row = UROW ? __builtin_amdgcn_readfirstlane(ra[k].ro[1][1]) : ra[k].ro[1][1];
                R om = omega, gu = guo;
                if (EXT && moving && (ra[k].wlo || ra[k].whi)) {
                    R kw[4];
#pragma unroll
                    for (int a = 0; a < 4; ++a) kw[a] = (R)(6.0 * B->rho0 * (double)scale * B->uw[a]);
                    wall_shift<R>(g[k], ra[k].wlo, ra[k].whi, kw);
                }
                if (EXT && contrast) {
                    // this step's inside bits (computed by the mesh
                    // chain, which this kernel follows)
                    const uint64_t w = mask[((int64_t)(rzk[k] >> 6) * ny + ryk[k]) * nx + xs];
                    if ((w >> (rzk[k] & 63)) & 1ull) {
                        om = omega_in;
                        gu = guo_in;
                    }
                }
                collide<ST>(g[k], gx, gy, gz, rho0, om, gu, scale, inv, out, u, rho);
                if constexpr (PADW) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) out[i] = pad ? R(0) : out[i];
                }
                if (NTM == 1 || (NTM == 2 && nt)) {
                    if constexpr (BUF)
                        store_buf<ST, true>(rd, (uint32_t)pb, row, xst, out);
                    else
                        store_ptr<ST, true>(dst, pb, row, xst, out);
                } else {
                    if constexpr (BUF)
                        store_buf<ST, false>(rd, (uint32_t)pb, row, xst, out);
                    else
                        store_ptr<ST, false>(dst, pb, row, xst, out);
                }
                if (PADW && pad) continue;
                if (full_u) {
                    const uint64_t e = (row + xst) / EB;
                    uf[e] = u[0];
                    uf[plane + e] = u[1];
                    uf[2 * plane + e] = u[2];
                }
                if (!(rho > R(0) && rho < R(FLT_MAX))) atomicOr(P.status, BIT_RHO);
                if (u[0] * u[0] + u[1] * u[1] + u[2] * u[2] > R(1) / R(3)) {
                    if constexpr (EARLY) {
                        uint64_t bp = (uint64_t)B;
                        asm volatile("" : "+s"(bp));  // keeps the loads in this branch
                        const IBLB_CONST BoxDev *M = (const IBLB_CONST BoxDev *)bp;
                        const int next = *M->ctr + 1;
                        M->fast_tile[band_tile(xs, ryk[k], rzk[k], M->tnx, M->tny)] = next;
                        M->ctr[1] = next;
                    } else {
                        atomicOr(P.status, BIT_MACH);
                    }
                }
            }
            if constexpr (UROW) break;
        }
        if constexpr (UROW) break;
    }
}

// Most waves of the bulk kernel per SIMD: where more would fit, their rows
// come from more places of the population planes at a time and the memory
// delivers less, and they leave no room for the mesh kernels beside them; with
// fewer, too little is in flight.  us per step with 3, 4, 5, 6 and 8:
// 256x256x128 FP64 482, 489, 548, 555, 551; 250x250x150 FP32 314, 294, 291,
// 324, 355 and 64 boxes of 128x128x64 1,112, 997, 962, 964, 1,076; 256x256x128
// BF16 211, 184, 173, 157, 174.  (Before the loops above went, FP64 had 3, FP32
// and BF16 5, at 484, 297, 1,020 and 183 us.)
constexpr int bulk_waves(int st) { return st == 0 ? 3 : st == 1 ? 5 : 6; }

template <int ST, bool UROW, bool NT, int CPT, bool EXT, bool SKIP, bool PADW>
__global__ void __launch_bounds__(K1_MAX_THREADS) __attribute__((amdgpu_waves_per_eu(1, bulk_waves(ST))))
    k_bulk(DevPtrs P, int parity, int full_u, float scale, float inv) {
    const IBLB_CONST RowGroup *rows = (const IBLB_CONST RowGroup *)P.rows;
    // epoch of this step's stamps (written by the mesh chain, which this
    // kernel follows); -2 never matches a stamp
    const int epoch = SKIP ? ((const IBLB_GLOBAL int32_t *)P.step_epoch)[parity] : -2;
    for (int gi = blockIdx.x; gi < P.n_rowgroups; gi += gridDim.x)
        bulk_rows<ST, UROW, NT ? 1 : 0, CPT, EXT, SKIP, PADW>(P, rows[gi], threadIdx.x, threadIdx.y, blockDim.x,
                                                              blockDim.y, parity, epoch, full_u, scale, inv, 0);
}

// ------------------------------------------------------------ spread gather
// Spread force density (Eq. 8) at cell (cx,cy,cz) of band tile gt ([x0..x1]
// x [y0..y1] x [z0..z1]) of box `box`, for the calling lane.  The node
// blocks whose stencil box covers the tile contribute in ascending block
// order; a block's own contribution is the partial sum its node pass
// accumulated over its nodes (read from the block's partial region), or,
// for a block whose region did not fit, the nodes summed here one by one in
// ascending order.  No atomics: the sum order per cell is fixed.
//
// The candidate blocks are the ones the move pass recorded for the tile
// (sorted here); when the records are incomplete the stencil boxes of all
// blocks of the box are tested, in passes of SCAN_GROUP.  Either way one
// lane holds one block's region descriptor, loaded together and handed out
// by lane reads, and the partial values of GATHER_BATCH blocks load side by
// side.  Where a block of the pass has no region, the pass's blocks are taken
// from a list (the scan's in LDS) with their descriptors read one by one, in
// batches of GATHER_BATCH: a batch's blocks with a region, then those without.
// The batches are those of the pass, so every launch adds in the same order.
//
// GROUP: groups of 64 blocks tested together.  Beside the bulk kernel one,
// because the band kernel's waves share the compute units with the bulk
// kernel's and have to fit where one of those has ended.  Four at a time took 103 VGPRs instead of
// 82 (84 now) and the steps became longer: 256x256x128 BF16 179 against 160 us,
// 250x250x150 312 against 293, 64 boxes of 128x128x64 973 against 967.
// Against tests that loaded each bound behind the one before it, the band
// kernel of 160 blocks alone went from 14.2 to 11.8 us.
constexpr int SCAN_GROUPS = SCAN_GROUP / 64;
constexpr int GATHER_BATCH = 4;

template <typename R, int GROUP>
__device__ __forceinline__ void gather_F(const DevPtrs &P, const IBLB_CONST BoxDev *B, int box, int gt,
                                         int slot, int x0, int x1, int y0, int y1, int z0, int z1, int cx,
                                         int cy, int cz, int *hits, R &F0, R &F1, R &F2) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const int N = P.Ntot;
    const bool zper = B->zbc == 1;
    const int nx = B->nx, ny = B->ny, nz = B->nz;
    const int b0 = B->blk_begin, b1 = B->blk_end;
    const IBLB_GLOBAL R *part = (const IBLB_GLOBAL R *)P.part;
    const IBLB_CONST int32_t *breg = (const IBLB_CONST int32_t *)P.breg;

    // add the contributions of blocks id(0..n) (ascending) to F: the blocks
    // with a partial region in order, then those without one (their nodes
    // one by one), also in order
    auto add_blocks = [&](auto id, int n) {
        R v[GATHER_BATCH][3];
        bool ovf[GATHER_BATCH];
        bool any_ovf = false;
#pragma unroll
        for (int k = 0; k < GATHER_BATCH; ++k) {
            v[k][0] = v[k][1] = v[k][2] = R(0);
            ovf[k] = false;
            if (k < n) {
                const int blk = id(k);
                const IBLB_CONST int32_t *br = breg + (int64_t)blk * BREG;
                ovf[k] = br[6] != 0;
                any_ovf |= ovf[k];
                if (!ovf[k]) {
                    int dx = cx - br[0], dy = cy - br[1], dz = cz - br[2];
                    if (dx < 0) dx += nx;
                    if (dy < 0) dy += ny;
                    if (zper && dz < 0) dz += nz;
                    const int ex = br[3], ey = br[4], ez = br[5];
                    if (dx < ex && dy < ey && dz >= 0 && dz < ez) {
                        const int64_t c = (int64_t)blk * 3 * P.reg_cells + 3 * ((dz * ey + dy) * ex + dx);
                        v[k][0] = part[c];
                        v[k][1] = part[c + 1];
                        v[k][2] = part[c + 2];
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < GATHER_BATCH; ++k) {
            if (k < n && !ovf[k]) {
                F0 += v[k][0];
                F1 += v[k][1];
                F2 += v[k][2];
            }
        }
        if (!any_ovf) return;
#pragma unroll 1
        for (int k = 0; k < n; ++k) {
            const int blk = id(k);
            if (breg[(int64_t)blk * BREG + 6] == 0) continue;
            const DropDev &D = P.drops[P.blk_drop[2 * blk]];
            const int j = blk * NB + lane;
            bool nh = false;
            int s0[3] = {0, 0, 0};
            R t[3] = {0, 0, 0};
            if (j - D.node_off < D.n_nodes) {
                const R *qh = (const R *)P.qh, *ql = (const R *)P.ql;
                int b[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) axis_base(qh[a * N + j], ql[a * N + j], b[a], t[a]);
                nh = meets(b[0] - 1, b[0] + 2, x0, x1, nx, true) && meets(b[1] - 1, b[1] + 2, y0, y1, ny, true) &&
                     meets(b[2] - 1, b[2] + 2, z0, z1, nz, zper);
                s0[0] = wrapn(b[0] - 1, nx);
                s0[1] = wrapn(b[1] - 1, ny);
                s0[2] = zper ? wrapn(b[2] - 1, nz) : b[2] - 1;
            }
            uint64_t nmask = __ballot(nh);
            if (!nmask) continue;
            R wx[4], wy[4], wz[4], f[3] = {0, 0, 0};
            axis_weights(t[0], wx);
            axis_weights(t[1], wy);
            axis_weights(t[2], wz);
            if (nh) {
                const R *phi = (const R *)P.phi;
#pragma unroll
                for (int q = 0; q < 3; ++q) f[q] = phi[q * N + j];
            }
            while (nmask) {
                const int nl = __builtin_ctzll(nmask);
                nmask &= nmask - 1;
                int ox = cx - bcast_i(s0[0], nl), oy = cy - bcast_i(s0[1], nl), oz = cz - bcast_i(s0[2], nl);
                if (ox < 0) ox += nx;
                if (oy < 0) oy += ny;
                if (zper && oz < 0) oz += nz;
                const R ax = pick4(ox, bcast(wx[0], nl), bcast(wx[1], nl), bcast(wx[2], nl), bcast(wx[3], nl));
                const R ay = pick4(oy, bcast(wy[0], nl), bcast(wy[1], nl), bcast(wy[2], nl), bcast(wy[3], nl));
                const R az = pick4(oz, bcast(wz[0], nl), bcast(wz[1], nl), bcast(wz[2], nl), bcast(wz[3], nl));
                const R wv = ax * ay * az;
                F0 += bcast(f[0], nl) * wv;
                F1 += bcast(f[1], nl) * wv;
                F2 += bcast(f[2], nl) * wv;
            }
        }
    };

    // the same for blocks that all have a partial region, whose descriptors
    // sit in the lanes: block id(lane) with descriptor ra, rb.  Takes the
    // lanes ln[0 .. n) in this order.
    auto add_lanes = [&](const int (&ln)[GATHER_BATCH], int n, int4 ra, int4 rb, int blk_of) {
        R v[GATHER_BATCH][3];
#pragma unroll
        for (int k = 0; k < GATHER_BATCH; ++k) {
            v[k][0] = v[k][1] = v[k][2] = R(0);
            if (k < n) {
                const int l = ln[k];
                int dx = cx - bcast_i(ra.x, l), dy = cy - bcast_i(ra.y, l), dz = cz - bcast_i(ra.z, l);
                if (dx < 0) dx += nx;
                if (dy < 0) dy += ny;
                if (zper && dz < 0) dz += nz;
                const int ex = bcast_i(ra.w, l), ey = bcast_i(rb.x, l), ez = bcast_i(rb.y, l);
                if (dx < ex && dy < ey && dz >= 0 && dz < ez) {
                    const int64_t c = (int64_t)bcast_i(blk_of, l) * 3 * P.reg_cells + 3 * ((dz * ey + dy) * ex + dx);
                    v[k][0] = part[c];
                    v[k][1] = part[c + 1];
                    v[k][2] = part[c + 2];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < GATHER_BATCH; ++k) {
            if (k < n) {
                F0 += v[k][0];
                F1 += v[k][1];
                F2 += v[k][2];
            }
        }
    };
    const int4 *regs = (const int4 *)P.breg;  // two per block
    // whether the stencil box of descriptor ra, rb meets the tile
    auto meets_block = [&](int4 ra, int4 rb) {
        const bool mx = meets_wrapped(ra.x, ra.w, x0, x1, nx, true);
        const bool my = meets_wrapped(ra.y, rb.x, y0, y1, ny, true);
        const bool mz = meets_wrapped(ra.z, rb.y, z0, z1, nz, zper);
        return mx && my && mz;
    };

    // the recorded candidates: count, flag and the MAXC slots (lane k holds
    // slot k) in one round trip
    const int ncand = ((const IBLB_CONST int32_t *)P.tncand)[(int64_t)slot * P.total_tiles + gt];
    const bool scan = !box_records(b0, b1) ||
                      ((const IBLB_CONST int32_t *)P.scan_all)[slot * P.n_boxes + box] != 0;
    int mine = lane < MAXC ? P.tcand[(int64_t)gt * MAXC + lane] : INT_MAX;
    if (!scan && ncand <= MAXC) {
        mine = lane < ncand ? mine : INT_MAX;
        // every candidate's descriptor in one more
        const int bid = lane < ncand ? mine : b0;
        const int4 ra = regs[2 * (int64_t)bid], rb = regs[2 * (int64_t)bid + 1];
        // rank of each lane's block among the candidates (the ids are distinct)
        int rank = 0;
        for (int k = 0; k < ncand; ++k) rank += __builtin_amdgcn_readlane(mine, k) < mine ? 1 : 0;
        auto lane_of = [&](int r) {
            const uint64_t m = __ballot(lane < ncand && rank == r);
            return m ? (int)__builtin_ctzll(m) : 0;
        };
        const bool any_ovf = __ballot(lane < ncand && rb.z != 0) != 0;
        for (int r0 = 0; r0 < ncand; r0 += GATHER_BATCH) {
            const int n = min(GATHER_BATCH, ncand - r0);
            if (any_ovf) {
                add_blocks([&](int k) { return __builtin_amdgcn_readlane(mine, lane_of(r0 + k)); }, n);
                continue;
            }
            int ln[GATHER_BATCH];
#pragma unroll
            for (int k = 0; k < GATHER_BATCH; ++k) ln[k] = k < n ? lane_of(r0 + k) : 0;
            add_lanes(ln, n, ra, rb, bid);
        }
        return;
    }
    for (int kp = b0; kp < b1; kp += SCAN_GROUP) {
        const int ke = min(kp + SCAN_GROUP, b1);
        const R G0 = F0, G1 = F1, G2 = F2;
        bool any_ovf = false;
        for (int kb = kp; kb < ke; kb += 64 * GROUP) {
            // every block's descriptor first, then the tests (a test that
            // loads only where the one before it passed waits once per test)
            int4 ra[GROUP], rb[GROUP];
#pragma unroll
            for (int g = 0; g < GROUP; ++g) {
                if (g > 0 && kb + 64 * g >= ke) continue;
                const int mb = min(kb + 64 * g + lane, ke - 1);
                ra[g] = regs[2 * (int64_t)mb];
                rb[g] = regs[2 * (int64_t)mb + 1];
            }
            uint64_t hit[GROUP], ovf = 0;
#pragma unroll
            for (int g = 0; g < GROUP; ++g) {
                hit[g] = 0;
                if (g > 0 && kb + 64 * g >= ke) continue;
                hit[g] = __ballot(kb + 64 * g + lane < ke && meets_block(ra[g], rb[g]));
                ovf |= hit[g] & __ballot(rb[g].z != 0);
            }
            any_ovf = ovf != 0;
            if (any_ovf) break;
#pragma unroll
            for (int g = 0; g < GROUP; ++g) {
                uint64_t m = hit[g];
                while (m) {
                    const int n = min(GATHER_BATCH, (int)__popcll(m));
                    int ln[GATHER_BATCH];
#pragma unroll
                    for (int k = 0; k < GATHER_BATCH; ++k) {
                        ln[k] = k < n ? (int)__builtin_ctzll(m) : 0;
                        m &= m - (k < n ? 1 : 0);
                    }
                    add_lanes(ln, n, ra[g], rb[g], kb + 64 * g + lane);
                }
            }
            if constexpr (GROUP == SCAN_GROUPS) break;  // the whole pass
        }
        if (!any_ovf) continue;
        // a hit without a region: the whole pass again, its batches counted
        // over all of its hits whatever GROUP is
        if constexpr (GROUP < SCAN_GROUPS) {
            F0 = G0;
            F1 = G1;
            F2 = G2;
        }
        int total = 0;
        for (int kb = kp; kb < ke; kb += 64) {
            const int mb = min(kb + lane, ke - 1);
            const uint64_t m = __ballot(kb + lane < ke && meets_block(regs[2 * (int64_t)mb], regs[2 * (int64_t)mb + 1]));
            if ((m >> lane) & 1) hits[total + __popcll(m & below)] = kb + lane;
            total += __popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int k0 = 0; k0 < total; k0 += GATHER_BATCH) {
            auto id = [&](int k) { return __builtin_amdgcn_readfirstlane(hits[k0 + k]); };
            add_blocks(id, min(GATHER_BATCH, total - k0));
        }
        __builtin_amdgcn_wave_barrier();  // the list is rewritten by the next pass
    }
}

// ------------------------------------------------------------------- band
// Largest band grid (workgroups of four waves, one wave per listed tile);
// a multiple of eight.
constexpr int BAND_GRID = 8192;
// One wavefront per stamped tile of this epoch, one lane per cell: gather
// the spread force, then (COLLIDE) pull, collide with F = body force +
// spread force, store the populations (the bulk kernel leaves these cells
// alone) and write u to the band; or (!COLLIDE, inspection) store F in the
// band.
// ONE_BOX: a single box, whose descriptor is read beside the list entry
// rather than after it.  xcd: the grid (BAND_GRID workgroups) takes the
// list in one contiguous eighth per XCD instead of interleaved.
template <int ST, bool COLLIDE, bool ONE_BOX, int GROUP>
__device__ __forceinline__ void band_role(const DevPtrs &P, int wg, int nwg, int parity, int full_u, float scale,
                                          float inv, int xcd, int nt, int (*hits)[SCAN_GROUP]) {
    using S = Stor<ST>;
    using R = typename S::R;
    constexpr uint32_t EB = sizeof(typename S::T);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(wg * 4 + (threadIdx.x >> 6));
    const int nwaves = nwg * 4;
    const IBLB_CONST int32_t *tl = (const IBLB_CONST int32_t *)P.tile_list;
    // this step's epoch, both list lengths and the wave's first list entry
    // in one round trip (the entry lies in the list whatever the count; the
    // count decides whether it is used)
    const int ctr = ((const IBLB_CONST int32_t *)P.step_epoch)[parity];
    const int n0 = P.tile_count[0], n1 = P.tile_count[1];
    // this step's epoch becomes the current one (nothing else reads the
    // counter in this launch)
    if (wg == 0 && threadIdx.x == 0) *P.ctr = ctr;
    const int first = min(wave, P.total_tiles - 1);
    const int first_gt = tl[2 * first], first_box = ONE_BOX ? 0 : tl[2 * first + 1];
    // the descriptor fields the tile's addressing needs (box 0's when there
    // is one box: then they load beside the entry)
    struct Geo {
        int tile_base, tnx, tny, nx, ny, nz, sx, zbc;
        uint64_t plane;
        const void *src;
    };
    auto geo = [&](const IBLB_CONST BoxDev *B) {
        return Geo{B->tile_base, B->tnx, B->tny, B->nx, B->ny, B->nz, B->sx, B->zbc, (uint64_t)B->plane,
                   B->f[parity]};
    };
    Geo g0{};
    if constexpr (ONE_BOX) g0 = geo((const IBLB_CONST BoxDev *)P.boxes);
    // keep these loads beside the counter's (not after the count test)
    asm volatile("" ::"s"(ctr), "s"(n0), "s"(n1), "s"(first_gt), "s"(first_box), "s"(g0.tile_base),
                 "s"(g0.tnx), "s"(g0.tny), "s"(g0.nx), "s"(g0.ny), "s"(g0.nz), "s"(g0.sx), "s"(g0.zbc),
                 "s"(g0.plane), "s"(g0.src));
    const int count = min((ctr & 1) ? n1 : n0, P.total_tiles);
    // list positions of this wave: every nwaves-th from its index, or (xcd,
    // a grid of whole groups of eight workgroups) a contiguous eighth of the
    // list per XCD, so that neighbouring tiles, which read the same partial
    // regions and share population lines, are taken on one L2 at about the
    // same time
    int i0 = wave, i1 = count, di = nwaves;
    if (xcd) {
        const ListRange lr = xcd_list_range(wg, threadIdx.x >> 6, nwg, count);
        i0 = __builtin_amdgcn_readfirstlane(lr.first);
        i1 = lr.end;
        di = lr.stride;
    }
    for (int i = i0; i < i1; i += di) {
        // global tile id and its box
        const int gt = (!xcd && i == wave) ? first_gt : tl[2 * i];
        const int box = ONE_BOX ? 0 : ((!xcd && i == wave) ? first_box : tl[2 * i + 1]);
        const IBLB_CONST BoxDev *B = (const IBLB_CONST BoxDev *)P.boxes + box;
        const Geo G = ONE_BOX ? g0 : geo(B);
        const int lt = gt - G.tile_base;
        const int tx = lt % G.tnx, ty = (lt / G.tnx) % G.tny, tz = lt / (G.tnx * G.tny);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
        const int x1 = min(x0 + TX - 1, G.nx - 1), y1 = min(y0 + TY - 1, G.ny - 1),
                  z1 = min(z0 + TZ - 1, G.nz - 1);
        const int cx = x0 + (lane & (TX - 1)), cy = y0 + ((lane >> TXS) & (TY - 1)),
                  cz = z0 + (lane >> (TXS + TYS));
        const bool inside = cx < G.nx && cy < G.ny && cz < G.nz;
        // the populations are pulled first so that their loads are in flight
        // during the force gather
        const uint64_t pb = G.plane * EB;
        const PopRes rs = pop_res(G.src, pb);
        RowAddr ra{};
        XOff xo{};
        R g[Q];
        if (COLLIDE && inside) {
            ra = row_addr(cy, cz, G.ny, G.nz, G.sx, G.zbc == 1, EB);
            xo = x_off<EB>(cx, G.nx);
            pull_buf<ST, true>(rs, (uint32_t)pb, ra, xo, g);
        }
        R F0 = 0, F1 = 0, F2 = 0;
        gather_F<R, GROUP>(P, B, box, gt, ctr & 1, x0, x1, y0, y1, z0, z1, cx, cy, cz, hits[threadIdx.x >> 6], F0,
                    F1, F2);
        if (!COLLIDE) {
            IBLB_GLOBAL R *Fb = (IBLB_GLOBAL R *)B->Fband + (int64_t)lt * 3 * TILE_CELLS;
            Fb[lane] = F0;
            Fb[TILE_CELLS + lane] = F1;
            Fb[2 * TILE_CELLS + lane] = F2;
            continue;
        }
        if (!inside) continue;
        R out[Q], u[3], rho;
        const uint32_t own = ra.ro[1][1] + xo.c;
        if (B->moving && (ra.wlo || ra.whi)) {
            R kw[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) kw[a] = (R)(6.0 * B->rho0 * (double)scale * B->uw[a]);
            wall_shift<R>(g, ra.wlo, ra.whi, kw);
        }
        R om = (R)B->omega, gu = (R)B->guo;
        if (B->contrast) {  // this step's inside bits
            const uint64_t w = ((const IBLB_GLOBAL uint64_t *)B->mask[parity])[((int64_t)(cz >> 6) * B->ny + cy) * B->nx + cx];
            if ((w >> (cz & 63)) & 1ull) {
                om = (R)B->omega_in;
                gu = (R)B->guo_in;
            }
        }
        collide<ST>(g, (R)B->g[0] + F0, (R)B->g[1] + F1, (R)B->g[2] + F2, (R)B->rho0, om, gu, scale, inv,
                    out, u, rho);
        // streaming stores where the bulk kernel uses them (the populations
        // exceed the last-level cache)
        if (nt)
            store_buf<ST, true, true>(pop_res(B->f[parity ^ 1], pb), (uint32_t)pb, ra.ro[1][1], xo.c, out);
        else
            store_buf<ST, false, true>(pop_res(B->f[parity ^ 1], pb), (uint32_t)pb, ra.ro[1][1], xo.c, out);
        IBLB_GLOBAL R *ub = (IBLB_GLOBAL R *)B->uband + (int64_t)lt * 3 * TILE_CELLS;
        ub[lane] = u[0];
        ub[TILE_CELLS + lane] = u[1];
        ub[2 * TILE_CELLS + lane] = u[2];
        if (full_u) {
            IBLB_GLOBAL R *uf = (IBLB_GLOBAL R *)B->ufull;
            const uint64_t e = own / EB, plane = (uint64_t)B->plane;
            uf[e] = u[0];
            uf[plane + e] = u[1];
            uf[2 * plane + e] = u[2];
        }
        if (!(rho > R(0) && rho < R(FLT_MAX))) atomicOr(P.status, BIT_RHO);
        if (u[0] * u[0] + u[1] * u[1] + u[2] * u[2] > R(1) / R(3)) atomicOr(P.status, BIT_MACH);
    }
}

template <int ST, bool COLLIDE, bool ONE_BOX>
__global__ void __launch_bounds__(256)
    k_band(DevPtrs P, int parity, int full_u, float scale, float inv, int xcd, int nt) {
    __shared__ int hits[4][SCAN_GROUP];
    band_role<ST, COLLIDE, ONE_BOX, 1>(P, blockIdx.x, gridDim.x, parity, full_u, scale, inv, xcd, nt, hits);
}

// ------------------------------------------------------- one-queue step
// A small step is the latency of its chain: move, volumes and tile list, node
// forces, band tiles, each launch waiting for the one before.  On two queues
// the bulk kernel runs beside them, but each dependency between the queues
// costs about 10 us, two of them in a step.  Here a step is a line of launches
// on one queue, and the bulk rows go along in the last workgroups of three:
//   PH_MOVE      advection, stamps, records, cleared inside bits | rows, every cell
//   (the volumes and the list alone: launch_aux)
//   PH_NODE      forces and partial spread                       | rows, without the band tiles
//   PH_BAND      band tiles                                      | rows, without the band tiles
// and, when no droplet has a volume penalty, PH_AUX_NODE (inside bits, list
// and forces) in the place of launch_aux and PH_NODE.  The rows beside
// PH_MOVE are computed before the stamps are known; their band cells are
// overwritten by PH_BAND.  With a viscosity contrast rows can only follow the
// inside bits.
//
// At 128x128x64 in FP32 a step takes 45 us so and 58 us on two queues; from
// about 144x144x64 on two queues are faster: larger boxes fill the chip with
// rows in every launch, and each launch ends with its own tail.  The rule that
// chooses (one_queue_size) has the times on both sides.
struct FusedGrid {
    int n0, n1, n2;  // workgroups of the phase's three kinds of mesh work; PH_BAND: n1 rows, then the fast tiles
                     // (last: one workgroup before the rows made the launch 1 us longer at 128x128x64 FP32)
    int r0, bxs;     // first row group; log2 of the threads along x (64 to 256)
};

// LDS of a phase's mesh work, sized at launch (static LDS would claim VGPRs).
template <typename R, int PHASE>
constexpr int fused_lds = PHASE == PH_MOVE     ? MOVE_LDS
                                          : PHASE == PH_BAND   ? (int)sizeof(int[4][SCAN_GROUP])
                                               : (int)sizeof(NodeLds<R, true>);
extern __shared__ __align__(16) char lds[];

template <int ST, bool EXT, int PHASE>
__global__ void __launch_bounds__(256, ST == 0 ? 1 : 4)
    k_fused(DevPtrs P, int parity, int adv, int full_u, float scale, float inv, int nt, FusedGrid G) {
    using R = typename Stor<ST>::R;
    int w = blockIdx.x;
    if (w < G.n0) {
        if constexpr (PHASE == PH_MOVE)
            move_role<R, MOVE_STEP>(P, xcd_item(w, G.n0), w == 0, parity, 1, nullptr, lds);
        else if constexpr (PHASE == PH_BAND) {
            auto hits = (int(*)[SCAN_GROUP])lds;
            if (P.n_boxes == 1) band_role<ST, true, true, SCAN_GROUPS>(P, w, G.n0, parity, full_u, scale, inv, 0, nt, hits);
            else band_role<ST, true, false, SCAN_GROUPS>(P, w, G.n0, parity, full_u, scale, inv, 0, nt, hits);
        } else
            node_role<R, true, true>(P, xcd_item(w, G.n0), lds);
        return;
    }
    w -= G.n0;
    if constexpr (PHASE == PH_MOVE) {
        if (w < G.n1) {
            mask_clear_role(P, w, G.n1, parity);
            return;
        }
        w -= G.n1;
    }
    if constexpr (PHASE == PH_AUX_NODE) {
        if constexpr (EXT) {  // n1 is 0 without a contrast
            if (w < G.n1) {
                inside_role<R>(P, w, parity);
                return;
            }
            w -= G.n1;
        }
        if (w < G.n2) {
            compact_role(P, w, parity, *P.ctr + adv);
            return;
        }
        w -= G.n2;
    }
    if constexpr (PHASE == PH_BAND) {
        if (w == G.n1) {
            fast_role(P, parity);
            return;
        }
    }
    constexpr bool SKIP = PHASE != PH_MOVE;
    const int epoch = PHASE == PH_MOVE       ? -2
                      : PHASE == PH_AUX_NODE ? *P.ctr + adv
                                             : P.step_epoch[parity];
    const IBLB_CONST RowGroup *rows = (const IBLB_CONST RowGroup *)P.rows;
    const int BX = 1 << G.bxs;
    bulk_rows<ST, true, 2, 1, EXT, SKIP, true, !SKIP>(P, rows[G.r0 + w], threadIdx.x & (BX - 1), threadIdx.x >> G.bxs, BX,
                                               256 >> G.bxs, parity, epoch, full_u, scale, inv, nt);
}

// ---------------------------------------------------------------- launchers
template <int ST, bool UROW, bool NT, bool SKIP, bool PADW>
static void launch_bulk_p(const DevPtrs &P, int parity, int full_u, float scale, float inv, const Launch &L,
                          dim3 grid, dim3 block, hipStream_t s) {
    if (P.contrast || P.moving) {
        if (UROW && L.cpt == 2)
            hipLaunchKernelGGL((k_bulk<ST, UROW, NT, 2, true, SKIP, PADW>), grid, block, 0, s, P, parity, full_u,
                               scale, inv);
        else
            hipLaunchKernelGGL((k_bulk<ST, UROW, NT, 1, true, SKIP, PADW>), grid, block, 0, s, P, parity, full_u,
                               scale, inv);
    } else if (UROW && L.cpt == 2) {
        hipLaunchKernelGGL((k_bulk<ST, UROW, NT, 2, false, SKIP, PADW>), grid, block, 0, s, P, parity, full_u, scale,
                           inv);
    } else {
        hipLaunchKernelGGL((k_bulk<ST, UROW, NT, 1, false, SKIP, PADW>), grid, block, 0, s, P, parity, full_u, scale,
                           inv);
    }
}

template <int ST, bool UROW, bool NT, bool SKIP>
static void launch_bulk_c(const DevPtrs &P, int parity, int full_u, float scale, float inv, const Launch &L,
                          dim3 grid, dim3 block, hipStream_t s) {
    if (P.pad_rows)
        launch_bulk_p<ST, UROW, NT, SKIP, true>(P, parity, full_u, scale, inv, L, grid, block, s);
    else
        launch_bulk_p<ST, UROW, NT, SKIP, false>(P, parity, full_u, scale, inv, L, grid, block, s);
}

template <int ST, bool SKIP>
static hipError_t launch_bulk_t(const DevPtrs &P, int parity, int full_u, float scale, const Launch &L,
                                hipStream_t s) {
    // never launch a shape the kernel was not compiled for
    if (L.bx < 1 || L.by < 1 || L.bx * L.by > K1_MAX_THREADS || L.grid < 1 || L.cpt < 1 || L.cpt > 2)
        return hipErrorInvalidValue;
    const dim3 block(L.bx, L.by), grid(L.grid);
    const float inv = 1.0f / scale;
    if (L.bx % 64 == 0) {
        if (L.nt)
            launch_bulk_c<ST, true, true, SKIP>(P, parity, full_u, scale, inv, L, grid, block, s);
        else
            launch_bulk_c<ST, true, false, SKIP>(P, parity, full_u, scale, inv, L, grid, block, s);
    } else {
        if (L.nt)
            launch_bulk_c<ST, false, true, SKIP>(P, parity, full_u, scale, inv, L, grid, block, s);
        else
            launch_bulk_c<ST, false, false, SKIP>(P, parity, full_u, scale, inv, L, grid, block, s);
    }
    return hipGetLastError();
}

template <int ST>
static hipError_t launch_bulk_s(const DevPtrs &P, int parity, int full_u, float scale, const Launch &L,
                                bool skip_band, hipStream_t s) {
    return skip_band ? launch_bulk_t<ST, true>(P, parity, full_u, scale, L, s)
                     : launch_bulk_t<ST, false>(P, parity, full_u, scale, L, s);
}

hipError_t launch_bulk(const DevPtrs &P, int storage, int parity, int full_u, float scale,
                       const Launch &L, bool skip_band, hipStream_t s) {
    switch (storage) {
    case 0: return launch_bulk_s<0>(P, parity, full_u, scale, L, skip_band, s);
    case 1: return launch_bulk_s<1>(P, parity, full_u, scale, L, skip_band, s);
    case 2: return launch_bulk_s<2>(P, parity, full_u, scale, L, skip_band, s);
    default: return launch_bulk_s<3>(P, parity, full_u, scale, L, skip_band, s);
    }
}

// Workgroups of the band kernel (four waves, one tile each at a time; a
// wave loops over what is left of the list) when it has the chip to itself:
// the list's length is not known here, so one wave for each tile there can
// be, up to 32,768 waves; most find nothing and end.
static int band_groups(const DevPtrs &P) { return std::min((P.total_tiles + 3) / 4, BAND_GRID); }
// The same beside the bulk kernel (per = 1) or in the one-queue step (per =
// 4), where empty workgroups take dispatch and room from the bulk rows: `per`
// for each node block, as a block of 64 nodes about one cell apart covers 13
// to 16 tiles, and more where few coarse blocks cover more (45x37x41 with 11
// blocks: 44 workgroups 36 us per step, 176 33 us).  In one queue the band's
// tiles start first and nothing follows them, so each wave gets about one
// (128x128x64 with 160 node blocks: 176 workgroups 56 us per step, 640 46, 4,096
// 50).  Beside the bulk kernel, which takes longer, a wave takes about four
// one after another; us per step with eight workgroups per node block, with
// four and with one: 256x256x128 BF16 176, 170 and 160, 64 boxes of 128x128x64
// FP32 985, 984 and 964, 250x250x150 291, 290 and 290, 256x256x128 FP64 481,
// 481 and 478, 512x512x256 with 16 droplets 1,866, 1,867 and 1,862.
static int shared_band_groups(const DevPtrs &P, int per) {
    return std::max(1, std::min((P.total_tiles + 3) / 4, std::min(std::max(per * P.nblk, std::min(16 * P.nblk, 256)), BAND_GRID)));
}

template <int ST, bool C>
static void launch_band_t(const DevPtrs &P, int parity, int full_u, float scale, int nt, bool shared, hipStream_t s) {
    const int grid = shared ? shared_band_groups(P, 1) : band_groups(P);
    // a full grid (a multiple of eight workgroups) takes the list in XCD
    // ranges; a small one keeps the interleaved order, whose first entry
    // loads beside the list count (latency decides there)
    const int xcd = grid == BAND_GRID ? 1 : 0;
    if (P.n_boxes == 1)
        hipLaunchKernelGGL((k_band<ST, C, true>), dim3(grid), dim3(256), 0, s, P, parity, full_u, scale,
                           1.0f / scale, xcd, nt);
    else
        hipLaunchKernelGGL((k_band<ST, C, false>), dim3(grid), dim3(256), 0, s, P, parity, full_u, scale,
                           1.0f / scale, xcd, nt);
}

hipError_t launch_band(const DevPtrs &P, int storage, int parity, int full_u, float scale, bool collide,
                       int nt, bool shared, hipStream_t s) {
    if (P.nblk == 0 || P.total_tiles == 0) return hipSuccess;
    if (collide) {
        switch (storage) {
        case 0: launch_band_t<0, true>(P, parity, full_u, scale, nt, shared, s); break;
        case 1: launch_band_t<1, true>(P, parity, full_u, scale, nt, shared, s); break;
        case 2: launch_band_t<2, true>(P, parity, full_u, scale, nt, shared, s); break;
        default: launch_band_t<3, true>(P, parity, full_u, scale, nt, shared, s); break;
        }
    } else if (storage == 0) {
        launch_band_t<0, false>(P, parity, full_u, scale, 0, shared, s);
    } else {
        launch_band_t<1, false>(P, parity, full_u, scale, 0, shared, s);
    }
    return hipGetLastError();
}

template <int ST, int PHASE>
static hipError_t launch_fused_p(const DevPtrs &P, int parity, int adv, int full_u, float scale, const Launch &L, int r0,
                                 int nrows, hipStream_t s) {
    FusedGrid G{0, 0, 0, r0, 0};
    while ((1 << G.bxs) < L.bx) ++G.bxs;
    // never launch a shape the kernel was not written for
    if ((1 << G.bxs) != L.bx || L.bx < 64 || L.bx * L.by != 256 || L.cpt != 1 || r0 < 0 || nrows < 0 ||
        r0 + nrows > P.n_rowgroups || !few_blocks(P) || (P.contrast && nrows > 0 && PHASE != PH_NODE && PHASE != PH_BAND))
        return hipErrorInvalidValue;
    if (PHASE == PH_MOVE) {
        G.n0 = P.nblk;
        G.n1 = mask_clear_groups(P);
    } else if (PHASE == PH_AUX_NODE) {
        G.n0 = P.nblk;
        G.n1 = P.contrast ? P.n_chunks : 0;
        G.n2 = compact_groups(P);
    } else {
        G.n0 = PHASE == PH_NODE ? P.nblk : shared_band_groups(P, 4);
    }
    int groups = G.n0 + G.n1 + G.n2 + nrows;
    if (PHASE == PH_BAND) {
        G.n1 = nrows;
        ++groups;
    }
    const dim3 grid(groups), block(256);
    const float inv = 1.0f / scale;
    const size_t bytes = fused_lds<typename Stor<ST>::R, PHASE>;
    if (P.contrast || P.moving)
        hipLaunchKernelGGL((k_fused<ST, true, PHASE>), grid, block, bytes, s, P, parity, adv, full_u, scale, inv, L.nt, G);
    else
        hipLaunchKernelGGL((k_fused<ST, false, PHASE>), grid, block, bytes, s, P, parity, adv, full_u, scale, inv, L.nt, G);
    return hipGetLastError();
}

template <int ST>
static hipError_t launch_fused_s(const DevPtrs &P, int phase, int parity, int adv, int full_u, float scale,
                                 const Launch &L, int r0, int nrows, hipStream_t s) {
    switch (phase) {
    case PH_MOVE: return launch_fused_p<ST, PH_MOVE>(P, parity, adv, full_u, scale, L, r0, nrows, s);
    case PH_NODE: return launch_fused_p<ST, PH_NODE>(P, parity, adv, full_u, scale, L, r0, nrows, s);
    case PH_BAND: return launch_fused_p<ST, PH_BAND>(P, parity, adv, full_u, scale, L, r0, nrows, s);
    case PH_AUX_NODE: return launch_fused_p<ST, PH_AUX_NODE>(P, parity, adv, full_u, scale, L, r0, nrows, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fused(const DevPtrs &P, int storage, int phase, int parity, int adv, int full_u, float scale,
                        const Launch &L, int r0, int nrows, hipStream_t s) {
    switch (storage) {
    case 0: return launch_fused_s<0>(P, phase, parity, adv, full_u, scale, L, r0, nrows, s);
    case 1: return launch_fused_s<1>(P, phase, parity, adv, full_u, scale, L, r0, nrows, s);
    case 2: return launch_fused_s<2>(P, phase, parity, adv, full_u, scale, L, r0, nrows, s);
    default: return launch_fused_s<3>(P, phase, parity, adv, full_u, scale, L, r0, nrows, s);
    }
}

}  // namespace iblb
