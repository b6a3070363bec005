// Device code of the mesh part of a step (gfx950), each piece the work of one
// workgroup of 256 threads, so that a launch can hold several kinds of work:
//   move_role     interpolation and advection of a block of 64 nodes, then
//                 what follows from the new positions alone: tile stamps,
//                 stencil box, tile records
//   volume_role   FP64 volume of a chunk of 256 triangles
//   compact_role  the list of stamped tiles
//   node_role     interface forces and block-partial spread of a node block
//   inside_role, mask_clear_role  the inside bits of the viscosity contrast
// The order within a step is move -> {volume, compact, inside} -> node -> the
// band tiles; without a volume penalty node needs no volume and runs beside
// compact.
#pragma once
#include "iblb_device.h"

namespace iblb {

// ------------------------------------------------------- node and stencil
// Base cell floor(q - 1/2) along one axis, decided exactly from the hi/lo
// pair, and t = q - b - 1/2 in [0, 1].  A coordinate that is not finite or
// absurd (false is returned) is taken as 1/2, which keeps the indices sane.
template <typename R> __device__ __forceinline__ bool axis_base(R qa, R la, int &b, R &t) {
    const bool sane = fabs(qa) < R(1.0e7);
    if (!sane) {
        qa = R(0.5);
        la = R(0);
    }
    const R fl = floor(qa);
    const R rf = (qa - fl - R(0.5)) + la;
    const bool neg = rf < R(0);
    b = (int)fl - (neg ? 1 : 0);
    t = neg ? rf + R(1) : rf;
    return sane;
}
// Peskin 4-point weights: all four share s = sqrt(1 + 4t(1-t)):
//   b-1: (3 - 2t - s)/8, b: (3 - 2t + s)/8, b+1: (1 + 2t + s)/8,
//   b+2: (1 + 2t - s)/8.
template <typename R> __device__ __forceinline__ void axis_weights(R t, R (&w)[4]) {
    const R s = sqrt(R(1) + R(4) * t * (R(1) - t));
    w[0] = (R(3) - R(2) * t - s) * R(0.125);
    w[1] = (R(3) - R(2) * t + s) * R(0.125);
    w[2] = (R(1) + R(2) * t + s) * R(0.125);
    w[3] = (R(1) + R(2) * t - s) * R(0.125);
}

// Node position as the triangle work reads it: one record of two
// four-vectors (hi, lo) per node instead of six separate arrays.
template <typename R> struct NodeRec {
    typename Vec4<R>::T h, l;
};
template <typename R> __device__ __forceinline__ Node3<R> load_rec(const NodeRec<R> *q4, int j) {
    const NodeRec<R> r = q4[j];
    return Node3<R>{{r.h.x, r.h.y, r.h.z}, {r.l.x, r.l.y, r.l.z}};
}

// z range of a block's stencil box inside the fluid.
__device__ __forceinline__ void clip_z(bool zper, int nz, int &zl, int &zh) {
    if (!zper) {
        zl = max(zl, 0);
        zh = min(zh, nz - 1);
    }
}

// ------------------------------------------------------------------- move
// The velocity over the block's stencil box is staged in LDS when it fits;
// wavefront w sums the z-slab w of every node's 4x4x4 stencil, the four slab
// sums are added in slab order, and wavefront 0 advects.  The stencil
// weights are formed again from the positions in each wave (three square
// roots) rather than stored by the node work and read back: 130 B per node
// and step less.  The stamps and records are made here, not beside the
// forces, because they need the new positions only: the list of stamped
// tiles is then built beside the volumes instead of in a launch of its own
// after the forces.
constexpr int MOVE_LDS = 36864;

template <typename R, int MODE>
__device__ __forceinline__ void move_role(const DevPtrs &P, int blk, bool first_block, int parity, int adv,
                                          double *Uout, char *lds) {
    constexpr int MAXR = MOVE_LDS / (3 * (int)sizeof(R));
    R *su = (R *)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const DropDev &D = P.drops[P.blk_drop[2 * blk]];
    const int bi = P.blk_drop[2 * blk + 1];
    const BoxDev &B = P.boxes[bi];
    const int N = P.Ntot, nb = P.nblk;
    const int nx = B.nx, ny = B.ny, nz = B.nz, tnx = B.tnx, tny = B.tny;
    const bool zper = B.zbc == 1;
    const int dims[3] = {nx, ny, nz};
    R *qh = (R *)P.qh, *ql = (R *)P.ql;
    const int j = blk * NB + lane;  // j < Ntot: nodes are padded to whole blocks
    const bool valid = j - D.node_off < D.n_nodes;
    const int epoch = (MODE & MV_STAMP) ? *P.ctr + adv : 0;
    IBLB_GLOBAL int32_t *const stamp = (IBLB_GLOBAL int32_t *)B.stamp[parity];
    const int tile_base = B.tile_base;
    const bool records = box_records(B.blk_begin, B.blk_end);
    R h[3], l[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        h[a] = qh[a * N + j];
        l[a] = ql[a * N + j];
    }
    if constexpr ((MODE & MV_INTERP) != 0) {
        const IBLB_GLOBAL R *ub = (const IBLB_GLOBAL R *)B.uband;
        const int bx0 = P.bbox[0 * nb + blk], bx1 = P.bbox[1 * nb + blk];
        const int by0 = P.bbox[2 * nb + blk], by1 = P.bbox[3 * nb + blk];
        int bz0 = P.bbox[4 * nb + blk], bz1 = P.bbox[5 * nb + blk];
        clip_z(zper, nz, bz0, bz1);
        const int ex = bx1 - bx0 + 1, ey = by1 - by0 + 1, ez = bz1 - bz0 + 1;
        const bool staged = ex > 0 && ey > 0 && ez > 0 && (int64_t)ex * ey * ez <= MAXR && ex <= nx && ey <= ny &&
                            (!zper || ez <= nz);
        auto gidx = [&](int x, int y, int z) -> int64_t {
            return band_tile(x, y, z, tnx, tny) * 3 * TILE_CELLS + band_loc(x, y, z);
        };
        if (staged) {
            // the region's cells in order, four per thread and pass with all
            // their loads issued before the first LDS store
            const int x0w = wrapn(bx0, nx), y0w = wrapn(by0, ny), z0w = zper ? wrapn(bz0, nz) : bz0;
            const int ncell = ex * ey * ez;
            for (int c0 = 0; c0 < ncell; c0 += 4 * 256) {
                R v[4][3];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int c = min(c0 + k * 256 + tid, ncell - 1);
                    const int r = c / ex, ix = c - r * ex;
                    const int iz = r / ey, iy = r - iz * ey;
                    int x = x0w + ix, y = y0w + iy, z = z0w + iz;  // wraps once at most: the region fits the box
                    x = x >= nx ? x - nx : x;
                    y = y >= ny ? y - ny : y;
                    z = zper && z >= nz ? z - nz : z;
                    const int64_t g = gidx(x, y, z);
                    v[k][0] = ub[g];
                    v[k][1] = ub[g + TILE_CELLS];
                    v[k][2] = ub[g + 2 * TILE_CELLS];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int c = c0 + k * 256 + tid;
                    if (c < ncell) {
                        su[c] = v[k][0];
                        su[MAXR + c] = v[k][1];
                        su[2 * MAXR + c] = v[k][2];
                    }
                }
            }
        }
        int b[3];
        R wx[4], wy[4], wz4[4], t;
        axis_base(h[0], l[0], b[0], t);
        axis_weights(t, wx);
        axis_base(h[1], l[1], b[1], t);
        axis_weights(t, wy);
        axis_base(h[2], l[2], b[2], t);
        axis_weights(t, wz4);
        const R wz = wave == 0 ? wz4[0] : (wave == 1 ? wz4[1] : (wave == 2 ? wz4[2] : wz4[3]));
        const int bx = b[0], by = b[1], bz = b[2];
        __syncthreads();
        R U0 = 0, U1 = 0, U2 = 0;
        if (valid) {
            const int z = bz - 1 + wave;
            if (zper || (z >= 0 && z < nz)) {
                if (staged) {
#pragma unroll
                    for (int oy = 0; oy < 4; ++oy) {
                        const int c0 = ((z - bz0) * ey + (by - 1 + oy - by0)) * ex + (bx - 1 - bx0);
#pragma unroll
                        for (int ox = 0; ox < 4; ++ox) {
                            const R w = wx[ox] * wy[oy] * wz;
                            U0 += su[c0 + ox] * w;
                            U1 += su[MAXR + c0 + ox] * w;
                            U2 += su[2 * MAXR + c0 + ox] * w;
                        }
                    }
                } else {
                    const int zw = zper ? wrapn(z, nz) : z;
                    for (int oy = 0; oy < 4; ++oy) {
                        const int y = wrapn(by - 1 + oy, ny);
                        for (int ox = 0; ox < 4; ++ox) {
                            const R w = wx[ox] * wy[oy] * wz;
                            const int64_t g = gidx(wrapn(bx - 1 + ox, nx), y, zw);
                            U0 += ub[g] * w;
                            U1 += ub[g + TILE_CELLS] * w;
                            U2 += ub[g + 2 * TILE_CELLS] * w;
                        }
                    }
                }
            }
        }
        // the slab sums and the new positions take the stage's place
        __syncthreads();
        R(*red)[3][64] = (R(*)[3][64])su;
        R(*qn)[64] = (R(*)[64])(su + 9 * 64);
        if (wave > 0) {
            red[wave - 1][0][lane] = U0;
            red[wave - 1][1][lane] = U1;
            red[wave - 1][2][lane] = U2;
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                U0 += red[k][0][lane];
                U1 += red[k][1][lane];
                U2 += red[k][2][lane];
            }
            if constexpr ((MODE & MV_OUT) != 0) {
                if (valid) {
                    Uout[3 * j + 0] = U0;
                    Uout[3 * j + 1] = U1;
                    Uout[3 * j + 2] = U2;
                }
            }
            if constexpr ((MODE & MV_ADVECT) != 0) {
                const R U[3] = {U0, U1, U2};
                if (valid) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        // two-sum h + U, fold the error into the low part, renormalise
                        const R s = h[a] + U[a];
                        const R bb = s - h[a];
                        const R err = (h[a] - (s - bb)) + (U[a] - bb);
                        const R l2 = l[a] + err;
                        const R h2 = s + l2;
                        h[a] = h2;
                        l[a] = l2 - (h2 - s);
                        qh[a * N + j] = h[a];
                        ql[a * N + j] = l[a];
                    }
                    if (fabs(U0) > R(1) || fabs(U1) > R(1) || fabs(U2) > R(1)) atomicOr(P.status, BIT_JUMP);
                }
                if constexpr ((MODE & MV_GEOM) != 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        qn[a][lane] = h[a];
                        qn[3 + a][lane] = l[a];
                    }
                }
            }
        }
        if constexpr ((MODE & MV_ADVECT) != 0 && (MODE & MV_GEOM) != 0) {
            __syncthreads();
            if (wave > 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    h[a] = qn[a][lane];
                    l[a] = qn[3 + a][lane];
                }
            }
        }
        if ((MODE & MV_EPOCH) != 0 && first_block && tid == 0) *P.ctr = *P.ctr + 1;
    }
    if constexpr ((MODE & MV_GEOM) != 0) {
        int b[3], lo[3], hi[3];
        bool sane = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            R t;
            const bool ok = axis_base(h[a], l[a], b[a], t);
            sane = sane && ok;
            lo[a] = valid ? b[a] - 1 : INT_MAX;
            hi[a] = valid ? b[a] + 2 : INT_MIN;
        }
        if (wave == 0 && valid && !sane) atomicOr(P.status, BIT_JUMP);
        // stencil bounding box of the block (unwrapped cell indices), in
        // every wave
        int bl[3], bh[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            bl[a] = wave_min(lo[a]);
            bh[a] = wave_max(hi[a]);
        }
        if (wave == 1 && valid) {
            NodeRec<R> *rec = (NodeRec<R> *)P.q4 + j;
            rec->h = typename Vec4<R>::T{h[0], h[1], h[2], R(0)};
            rec->l = typename Vec4<R>::T{l[0], l[1], l[2], R(0)};
        }
        if ((MODE & MV_BASE) != 0 && wave == 2 && valid) {
#pragma unroll
            for (int a = 0; a < 3; ++a) P.base[a * N + j] = b[a];
        }
        int zl = bl[2], zh = bh[2];
        clip_z(zper, nz, zl, zh);
        if (wave == 0 && lane == 0) {
            const int ex = bh[0] - bl[0] + 1, ey = bh[1] - bl[1] + 1, ez = zh - zl + 1;
            const bool ovf = ex > nx || ey > ny || (zper && ez > nz) || ez < 1 || (int64_t)ex * ey * ez > P.reg_cells;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                P.bbox[(2 * a) * nb + blk] = bl[a];
                P.bbox[(2 * a + 1) * nb + blk] = bh[a];
            }
            int32_t *br = P.breg + (int64_t)blk * BREG;
            br[0] = wrapn(bl[0], nx);
            br[1] = wrapn(bl[1], ny);
            br[2] = zper ? wrapn(zl, nz) : zl;
            br[3] = ex;
            br[4] = ey;
            br[5] = ez;
            br[6] = ovf ? 1 : 0;
            br[7] = 0;
        }
        if constexpr ((MODE & MV_STAMP) != 0) {
            // epoch stamp of every tile holding a stencil cell (same value
            // from every writer, so plain stores).  Per axis the four
            // stencil cells from b - 1 (wrapped on a periodic axis; cells in
            // a wall are left out) and the tile of each, kept where it
            // differs from the tiles of the cells before it; wave w stamps
            // for the z-slab w of the stencil
            int t3[3][4];
            bool u3[3][4];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int sh = a == 0 ? TXS : (a == 1 ? TYS : TZS);
                const bool per = a < 2 || zper;
                const int s0 = per ? wrapn(b[a] - 1, dims[a]) : b[a] - 1;
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    int c = s0 + o;
                    if (per && c >= dims[a]) c -= dims[a];
                    const bool v = valid && c >= 0 && c < dims[a];
                    t3[a][o] = c >> sh;
                    bool fresh = v;
#pragma unroll
                    for (int k = 0; k < o; ++k) fresh = fresh && !(u3[a][k] && t3[a][k] == t3[a][o]);
                    u3[a][o] = fresh;
                }
            }
            const int tz = wave == 0 ? t3[2][0] : (wave == 1 ? t3[2][1] : (wave == 2 ? t3[2][2] : t3[2][3]));
            const bool uz = wave == 0 ? u3[2][0] : (wave == 1 ? u3[2][1] : (wave == 2 ? u3[2][2] : u3[2][3]));
#pragma unroll
            for (int iy = 0; iy < 4; ++iy)
#pragma unroll
                for (int ix = 0; ix < 4; ++ix)
                    if (uz && u3[1][iy] && u3[0][ix]) stamp[((int64_t)tz * tny + t3[1][iy]) * tnx + t3[0][ix]] = epoch;
            // every band tile that the stencil box covers records the block
            // (slot from an integer counter; the gather sorts the ids, so the
            // order of the records does not matter, but each tile must list a
            // block once); a box covering more than 64 tiles on an axis, or
            // none (all stencil cells in a wall), makes its box's gather scan
            if (records) {
                const int slot = epoch & 1;
                const int lo3[3] = {bl[0], bl[1], zl}, hi3[3] = {bh[0], bh[1], zh};
                TileRun run[3];
                int nta[3];
                bool ok = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const bool per = a < 2 || zper;
                    const int sh = a == 0 ? TXS : (a == 1 ? TYS : TZS);
                    nta[a] = (dims[a] + (1 << sh) - 1) >> sh;
                    run[a] = tile_run(per ? wrapn(lo3[a], dims[a]) : lo3[a], hi3[a] - lo3[a] + 1, dims[a], sh, per);
                    ok = ok && run[a].count >= 1 && run[a].count <= 64;
                }
                if (ok) {
                    const int nt = run[0].count * run[1].count * run[2].count;
                    for (int k = tid; k < nt; k += 256) {
                        const int r = k / run[0].count, ix = k - r * run[0].count;
                        const int iz = r / run[1].count, iy = r - iz * run[1].count;
                        auto at = [&](int a, int i) {
                            const int t = run[a].first + i;
                            return t >= nta[a] ? t - nta[a] : t;
                        };
                        const int gt = tile_base + (at(2, iz) * tny + at(1, iy)) * tnx + at(0, ix);
                        const int pos = atomicAdd(P.tncand + (int64_t)slot * P.total_tiles + gt, 1);
                        if (pos < MAXC) P.tcand[(int64_t)gt * MAXC + pos] = blk;
                    }
                } else if (tid == 0) {
                    P.scan_all[slot * P.n_boxes + bi] = 1;
                }
            }
        }
    }
}

// ----------------------------------------------------------------- volume
// FP64 volume sum_t (a-r).((b-r)x(c-r))/6 of a chunk of 256 triangles
// (positions relative to the droplet's reference point r), fixed tree.
template <typename R>
__device__ __forceinline__ void volume_role(const DevPtrs &P, int ci, double *sv) {
    const TriChunk ch = P.chunks[ci];
    const DropDev &D = P.drops[ch.drop];
    const int t = ch.t0 + threadIdx.x;
    double v = 0.0;
    if (t < ch.t1) {
        const NodeRec<R> *q4 = (const NodeRec<R> *)P.q4;
        const Node3<R> abc[3] = {load_rec(q4, P.tri[3 * t]), load_rec(q4, P.tri[3 * t + 1]),
                                 load_rec(q4, P.tri[3 * t + 2])};
        double p[3][3];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc)
#pragma unroll
            for (int k = 0; k < 3; ++k) p[cc][k] = ((double)abc[cc].h[k] + (double)abc[cc].l[k]) - D.ref[k];
        const double bc0 = p[1][1] * p[2][2] - p[1][2] * p[2][1];
        const double bc1 = p[1][2] * p[2][0] - p[1][0] * p[2][2];
        const double bc2 = p[1][0] * p[2][1] - p[1][1] * p[2][0];
        v = (p[0][0] * bc0 + p[0][1] * bc1 + p[0][2] * bc2) / 6.0;
    }
    sv[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int i = threadIdx.x;
        v = (sv[i] + sv[i + 128]) + (sv[i + 64] + sv[i + 192]);
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) v += __shfl_down(v, k, 64);
        if (i == 0) P.tri_part[ci] = v;
    }
}

// ----------------------------------------------------- stamped-tile list
// One wavefront per chunk of 64 tiles appends the chunk's stamped tiles to
// the list of this epoch (one integer atomic per chunk; the order of the
// list does not affect any result).  Item 0 also clears the other epoch's
// count and names the epoch of this step's stamps.
__device__ __forceinline__ void compact_role(const DevPtrs &P, int item, int parity, int epoch) {
    const int lane = threadIdx.x & 63;
    const int c = __builtin_amdgcn_readfirstlane(item * 4 + (threadIdx.x >> 6));
    const int slot = epoch & 1;
    if (item == 0 && threadIdx.x == 0) {
        P.step_epoch[parity] = epoch;
        P.tile_count[slot ^ 1] = 0;
        for (int b = 0; b < P.n_boxes; ++b) P.scan_all[(slot ^ 1) * P.n_boxes + b] = 0;
    }
    if (c >= P.total_tiles / TILE_CELLS) return;
    // the next epoch's tile records start empty
    P.tncand[(int64_t)(slot ^ 1) * P.total_tiles + c * TILE_CELLS + lane] = 0;
    const int box = P.tchunk_box[c];
    const BoxDev &B = P.boxes[box];
    const int lt = c * TILE_CELLS + lane - B.tile_base;
    const bool st = lt < B.n_tiles && ((const IBLB_GLOBAL int32_t *)B.stamp[parity])[lt] == epoch;
    const uint64_t m = __ballot(st);
    if (m == 0) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(P.tile_count + slot, __popcll(m));
    base = __shfl(base, 0, 64);
    const int k = base + __popcll(m & ((1ull << lane) - 1ull));
    if (st && k < P.total_tiles) {  // one entry per tile and epoch: k < total_tiles always
        P.tile_list[2 * k] = c * TILE_CELLS + lane;
        P.tile_list[2 * k + 1] = box;
    }
}

// ------------------------------------------------------------- fast tiles
// One workgroup beside the band tiles of the one-queue step: if rows computed
// before the stamps met a bare speed above the sound speed, the tiles they
// marked raise the status unless they are stamped; a stamped one is for the
// band to judge.  (In a workgroup of its own because it is on no path there:
// beside the tile list the check cost 128x128x64 in FP32 0.4 us per step.)
__device__ __forceinline__ void fast_role(const DevPtrs &P, int parity) {
    const int epoch = ((const IBLB_CONST int32_t *)P.step_epoch)[parity];
    if (P.ctr[1] != epoch) return;
    for (int b = 0; b < P.n_boxes; ++b) {
        const BoxDev &B = P.boxes[b];
        const IBLB_GLOBAL int32_t *stamp = (const IBLB_GLOBAL int32_t *)B.stamp[parity];
        for (int t = threadIdx.x; t < B.n_tiles; t += 256)
            if (B.fast_tile[t] == epoch && stamp[t] != epoch) atomicOr(P.status, BIT_MACH);
    }
}

// ------------------------------------------------------------------- node
// A block of 64 nodes.  Wave 0, one lane per node, sums over the node's
// incident triangles (ascending triangle id) the corner surface-tension
// forces -sigma dA_t/dq = (sigma/2)(q_prev - q_next) x n_t, the 1-ring area
// chi, the unit face normals and the volume gradient; then the wetting force
// -chi Pi(d) n/3 with Pi from integer powers (Eq. 10) and the optional
// volume penalty.  Waves 1 to 3 meanwhile form the Peskin weights of one axis
// each and clear the LDS.  Then (spread) the nodes go into LDS copies of the
// block's stencil box in ascending order, each lane one of a node's 64
// stencil cells, so that no two lanes of a wave touch the same cell.  With
// at most one block per compute unit (latency decides) they go in as four
// sets (two in FP64) of 16 consecutive nodes, each summed by itself, by as
// many waves at a time as copies of the box fit in the LDS; with more blocks
// as one set.  The sets' sums are added in order when the region is written
// out for the tile gather.
//
// What bounds the spread is the chain of reads, adds and writes through the
// LDS, one after another per node of a wave: hence the sets, and the weights
// of eight nodes formed in registers before their chain.  Tried in its
// place: adds without return on one copy (LDS float atomics; node pass of 160
// blocks 33 us against 9), and sums per cell over the nodes that reach it
// (28 us: a cell in the middle meets over twenty).
//
// The triangles' terms are formed here from the positions, three times per
// triangle over all nodes, instead of once in a pass that writes a record of
// five four-vectors per triangle (160 B per node written, 290 B read back).
// Cells of the LDS copies together.  FEW (at most one block per compute unit):
// 80 KB, which holds all four sets of a box of up to 1,600 cells (two at a
// time of one up to REG_MAX) and leaves
// room for two workgroups per CU; else a largest region once (29 KB in FP32).
template <typename R, bool FEW> constexpr int REG_CELLS = FEW ? (sizeof(R) == 4 ? 6400 : 2944) : MAXP;
template <typename R, bool FEW> struct NodeLds {
    R reg[3 * REG_CELLS<R, FEW> + 4];  // [copy][cell][component]; the end takes what falls in a wall
    R w[12][NB], f[3][NB];
    int first[3][NB];      // the stencil's first cell in the region
    double V;              // the droplet's volume
};
inline bool few_blocks(const DevPtrs &P) { return P.nblk <= P.n_cus; }

// on ? a : b by bit masks (a conditional over several values becomes
// branches, which a wave whose lanes differ walks one after another).
__device__ __forceinline__ float take(bool on, float a, float b) {
    const uint32_t m = on ? ~0u : 0u;
    return __uint_as_float((__float_as_uint(a) & m) | (__float_as_uint(b) & ~m));
}
__device__ __forceinline__ double take(bool on, double a, double b) {
    const uint64_t m = on ? ~0ull : 0ull;
    return __longlong_as_double((int64_t)((((uint64_t)__double_as_longlong(a)) & m) |
                                          (((uint64_t)__double_as_longlong(b)) & ~m)));
}

// x / 6, correctly rounded (in FP32 for every x with a quotient above 1e-36): a
// product with the rounded reciprocal and one exact-remainder correction.
__device__ __forceinline__ float sixth(float x) {
    const float r = 1.0f / 6.0f, q = x * r;
    return __builtin_fmaf(__builtin_fmaf(-6.0f, q, x), r, q);
}
__device__ __forceinline__ double sixth(double x) {
    const double r = 1.0 / 6.0, q = x * r;
    return __builtin_fma(__builtin_fma(-6.0, q, x), r, q);
}

// The block's nodes from S, `sets` sets of them, COPIES at a time into as
// many cleared LDS copies, and the sets' sum in order to `out`.  A single
// copy is shared by three waves, one component each.
template <typename R, bool FEW, int COPIES>
__device__ __forceinline__ void spread_block(NodeLds<R, FEW> &S, int ex, int ey, int ez, int nv, int sets, int wave, int lane,
                                             IBLB_GLOBAL R *out) {
    const int ncell = ex * ey * ez, tid = threadIdx.x;
    const int ox = lane & 3, oy = (lane >> 2) & 3, oz = lane >> 4;
    const int per = NB / sets;
    constexpr int SB = 8;
    constexpr bool SPLIT = COPIES == 1;
    for (int s0 = 0; s0 < sets; s0 += COPIES) {
        if (wave < (SPLIT ? 3 : COPIES)) {
            const int set = SPLIT ? s0 : s0 + wave, r0 = SPLIT ? wave : 3 * wave * ncell;
            const int n1 = min((set + 1) * per, nv);
            for (int n = set * per; n < n1; n += SB) {
                R wv[SB], fv[SB][3];
                int c[SB];
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int nl = n + i;  // past the last node: its slot's data, not added
                    const int rz = S.first[2][nl] + oz;  // region coordinates of this lane's stencil cell
                    const int ry = S.first[1][nl] + oy;
                    const int rx = S.first[0][nl] + ox;
                    wv[i] = S.w[ox][nl] * S.w[4 + oy][nl] * S.w[8 + oz][nl];
                    if constexpr (SPLIT) {
                        fv[i][0] = S.f[wave][nl];
                    } else {
#pragma unroll
                        for (int k = 0; k < 3; ++k) fv[i][k] = S.f[k][nl];
                    }
                    // outside only for wall layers (dropped)
                    const bool on = (nl < n1) & (rz >= 0) & (rz < ez);
                    int cell = r0 + 3 * ((rz * ey + ry) * ex + rx);
                    asm volatile("" : "+v"(cell));  // in every lane: no branch between the batch's loads
                    c[i] = on ? cell : 3 * REG_CELLS<R, FEW>;
                }
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    R *p = S.reg + c[i];
                    if constexpr (SPLIT) {
                        p[0] += fv[i][0] * wv[i];
                    } else {
                        const R v0 = p[0], v1 = p[1], v2 = p[2];
                        p[0] = v0 + fv[i][0] * wv[i];
                        p[1] = v1 + fv[i][1] * wv[i];
                        p[2] = v2 + fv[i][2] * wv[i];
                    }
                }
            }
        }
        __syncthreads();
        // the three components of a cell side by side: the band gather reads
        // a run of a region row as one contiguous stretch of lines
#pragma unroll 2
        for (int c = tid; c < 3 * ncell; c += 256) {
            R v[COPIES];
#pragma unroll
            for (int r = 0; r < COPIES; ++r) v[r] = S.reg[3 * r * ncell + c];
            if (s0 > 0) v[0] += out[c];  // what this thread wrote for the sets before
#pragma unroll
            for (int r = 1; r < COPIES; ++r) v[0] += v[r];
            out[c] = v[0];
        }
        if (s0 + COPIES < sets) {
            __syncthreads();
            for (int c = tid; c < 3 * COPIES * ncell; c += 256) S.reg[c] = R(0);
            __syncthreads();
        }
    }
}

template <typename R, bool FEW, bool SPREAD>
__device__ __forceinline__ void node_role(const DevPtrs &P, int blk, char *lds) {
    NodeLds<R, FEW> &S = *(NodeLds<R, FEW> *)lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // droplet and box in one load, so their records load side by side
    const int d = P.blk_drop[2 * blk], bi = P.blk_drop[2 * blk + 1];
    const DropDev &D = P.drops[d];
    const int N = P.Ntot;
    const int node_off = D.node_off, n_nodes = D.n_nodes;
    const int j = blk * NB + lane;
    const int32_t *br = P.breg + (int64_t)blk * BREG;
    const int ex = SPREAD ? br[3] : 0, ey = SPREAD ? br[4] : 0, ez = SPREAD ? br[5] : 0;
    const bool ovf = SPREAD && br[6] != 0;
    const int ncell = ovf ? 0 : ex * ey * ez;
    constexpr int sets = !FEW ? 1 : (sizeof(R) == 4 ? 4 : 2), cells = REG_CELLS<R, FEW>;
    static_assert(cells >= (FEW ? (sets >= 4 ? 2 : 1) * REG_MAX<R> : MAXP), "one copy fits; two with four sets");
    const int copies = sets >= 4 && 4 * ncell <= cells ? 4 : (sets >= 2 && 2 * ncell <= cells ? 2 : 1);
    if (wave == 0) {
        const int n_exp = D.n_exp, m_exp = D.m_exp;
        const double kvol = D.kvol, V0 = D.V0, Aw = D.A, xi = D.xi;
        const R hs = R(0.5) * (R)D.sigma;
        const NodeRec<R> *q4 = (const NodeRec<R> *)P.q4;
        const int2 *nbr = (const int2 *)P.csr_nb;
        const bool pen = kvol > 0.0;
        R st[3] = {0, 0, 0}, ns[3] = {0, 0, 0}, gv[3] = {0, 0, 0};
        R kw = 0;
        const bool valid = j - node_off < n_nodes;
        if (valid) {
            const Node3<R> self = load_rec(q4, j);
            R chi = 0;
            // batches of incident triangles: every load of a batch is issued
            // (entries past the degree read the last one and are not added)
            // before the first is used
            constexpr int GB = (FEW ? 6 : 4) / (sizeof(R) == 4 ? 1 : 2);
            const int e0 = P.csr_off[j], e1 = P.csr_off[j + 1];
            for (int e = e0; e < e1; e += GB) {
                int2 nb[GB];
#pragma unroll
                for (int k = 0; k < GB; ++k) nb[k] = nbr[min(e + k, e1 - 1)];
                Node3<R> n1[GB], n2[GB];
#pragma unroll
                for (int k = 0; k < GB; ++k) {
                    n1[k] = load_rec(q4, nb[k].x & NODE_MASK);
                    n2[k] = load_rec(q4, nb[k].y);
                }
#pragma unroll
                for (int k = 0; k < GB; ++k) {
                    if (e + k >= e1) continue;
                    R d1[3], d2[3], d3[3], Nt[3], fc[3];
                    // corner 0, 1, 2 of the triangle (a, b, c): the node is
                    // a, b, c and (n1, n2) are (b, c), (c, a), (a, b).  N is
                    // (b - a) x (c - a) in every corner, so that the three
                    // nodes of a triangle round it alike
                    const int corner = (unsigned)nb[k].x >> NODE_BITS;
                    diff(n1[k], self, d1);
                    diff(n2[k], self, d2);
                    diff(n2[k], n1[k], d3);
                    R u[3], v[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        u[a] = take(corner == 0, d1[a], take(corner == 1, -d2[a], d3[a]));
                        v[a] = take(corner == 0, d2[a], take(corner == 1, -d3[a], -d1[a]));
                    }
                    cross3(u, v, Nt);
                    const R len = sqrt(Nt[0] * Nt[0] + Nt[1] * Nt[1] + Nt[2] * Nt[2]);
                    const R il = R(1) / len;
                    const R nt[3] = {Nt[0] * il, Nt[1] * il, Nt[2] * il};
                    cross3(d3, nt, fc);
                    chi += len;
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        const R s = hs * fc[a], g = sixth(Nt[a]);
                        st[a] += s;
                        ns[a] += nt[a];
                        gv[a] += g;
                    }
                }
            }
            chi *= R(0.5);
            const R nl = R(1) / sqrt(ns[0] * ns[0] + ns[1] * ns[1] + ns[2] * ns[2]);
            const R dist = self.h[2] + self.l[2];
            if (!(dist > R(0))) atomicOr(P.status, BIT_WALL);
            const R rr = (R)xi / dist;
            R pn = 1, pm = 1;
            for (int k = 0; k < n_exp; ++k) pn *= rr;
            for (int k = 0; k < m_exp; ++k) pm *= rr;
            const R Pi = (R)Aw * (pn - pm);
            kw = chi * Pi / R(3) * nl;
        }
        // the droplet's volume, summed by another wave meanwhile
        __syncthreads();
        const R kv = pen ? (R)(-kvol * ((S.V - V0) / V0)) : R(0);
        R f[3] = {0, 0, 0};
        if (valid) {
            R *phi = (R *)P.phi;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                f[k] = st[k] - kw * ns[k] + kv * gv[k];
                phi[k * N + j] = f[k];
            }
        }
        if constexpr (SPREAD) {
#pragma unroll
            for (int k = 0; k < 3; ++k) S.f[k][lane] = f[k];
        }
    } else {
        if (wave == 1 && D.kvol > 0.0) {
            const double V = droplet_partial_sum(P.tri_part, D.chunk_off, D.n_chunks, lane);
            if (lane == 0) S.V = V;
        }
        if constexpr (SPREAD) {
            const BoxDev &B = P.boxes[bi];
            const bool zper = B.zbc == 1;
            const int a = wave - 1;
            int lo = P.bbox[(2 * a) * P.nblk + blk], hi = 0;
            if (a == 2) clip_z(zper, B.nz, lo, hi);
            int b;
            R t, w[4];
            axis_base(((const R *)P.qh)[a * N + j], ((const R *)P.ql)[a * N + j], b, t);
            axis_weights(t, w);
#pragma unroll
            for (int k = 0; k < 4; ++k) S.w[4 * a + k][lane] = w[k];
            S.first[a][lane] = b - 1 - lo;  // below 0 along z for cells in the wall
            for (int c = tid - 64; c < 3 * copies * ncell; c += 192) S.reg[c] = R(0);
        }
        __syncthreads();  // the volume
    }
    if constexpr (SPREAD) {
        __syncthreads();
        if (ovf) return;
        const int nv = min(NB, n_nodes - (blk * NB - node_off));
        IBLB_GLOBAL R *out = (IBLB_GLOBAL R *)P.part + (int64_t)blk * 3 * P.reg_cells;
        if constexpr (sets >= 4) {
            if (copies == 4) spread_block<R, FEW, 4>(S, ex, ey, ez, nv, sets, wave, lane, out);
            else spread_block<R, FEW, 2>(S, ex, ey, ez, nv, sets, wave, lane, out);
        } else {
            if (sets == 2 && copies == 2) spread_block<R, FEW, 2>(S, ex, ey, ez, nv, sets, wave, lane, out);
            else spread_block<R, FEW, 1>(S, ex, ey, ez, nv, sets, wave, lane, out);
        }
    }
}

// ------------------------------------------------------------ inside bits
// Cells inside the droplets of boxes with tau_in (Sec. 2, below Eq. 13).  A
// cell is inside when the vertical ray below its centre crosses the closed
// meshes an odd number of times.  Every triangle toggles, in each column
// whose vertical line crosses it, the bits of the cells whose centre lies at
// or above the crossing; XOR does not depend on the order of the toggles,
// so the result is exact and the same in every run.
//   - Coordinates are rounded to the grid of 2^-18 lattice units (half away
//     from zero); the cell centre (i + 1/2) is i 2^18 + 2^17 on that grid.
//   - The line through column point p crosses the triangle when the signs
//     of the three edge functions e_uv(p) = (v_x - u_x)(p_y - u_y) -
//     (v_y - u_y)(p_x - u_x) agree; a zero takes the sign it would have with
//     p moved by (+e, +e^2): that of -(v_y - u_y), else of (v_x - u_x).
//   - With D = e_ab + e_bc + e_ca and N = e_bc a_z + e_ca b_z + e_ab c_z the
//     crossing lies at or below the centre z_c when sign(D) (z_c D - N) >= 0.
// Edge functions and their products are exact in 128-bit integers.
constexpr int64_t QS = 1 << 18, QH = 1 << 17;

__device__ __forceinline__ int64_t floor_div(int64_t a, int64_t b) {  // b > 0
    return a >= 0 ? a / b : -((-a + b - 1) / b);
}
__device__ __forceinline__ int sos_sign(__int128 e, int64_t dx, int64_t dy) {
    if (e > 0) return 1;
    if (e < 0) return -1;
    if (dy != 0) return dy > 0 ? -1 : 1;
    if (dx != 0) return dx > 0 ? 1 : -1;
    return 0;
}
__device__ __forceinline__ __int128 edge_fn(int64_t ux, int64_t uy, int64_t vx, int64_t vy, int64_t px,
                                            int64_t py) {
    return (__int128)(vx - ux) * (py - uy) - (__int128)(vy - uy) * (px - ux);
}

template <typename R>
__device__ __forceinline__ void inside_role(const DevPtrs &P, int ci, int slot) {
    const TriChunk ch = P.chunks[ci];
    const DropDev &D = P.drops[ch.drop];
    const BoxDev &B = P.boxes[D.box];
    if (!B.contrast) return;
    const int t = ch.t0 + threadIdx.x;
    if (t >= ch.t1) return;
    const R *qh = (const R *)P.qh, *ql = (const R *)P.ql;
    const int N = P.Ntot, nx = B.nx, ny = B.ny, nz = B.nz, nzw = B.nzw;
    uint64_t *mask = B.mask[slot];
    int64_t X[3], Y[3], Z[3];
    bool sane = true;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int j = P.tri[3 * t + c];
        const double x = (double)qh[j] + (double)ql[j];
        const double y = (double)qh[N + j] + (double)ql[N + j];
        const double z = (double)qh[2 * N + j] + (double)ql[2 * N + j];
        // |coordinate| < 2^20 keeps every product below in 128 bits (NaN fails too)
        sane = sane && fabs(x) < 0x1p20 && fabs(y) < 0x1p20 && fabs(z) < 0x1p20;
        X[c] = sane ? llround(x * (double)QS) : 0;
        Y[c] = sane ? llround(y * (double)QS) : 0;
        Z[c] = sane ? llround(z * (double)QS) : 0;
    }
    // columns whose point lies in the triangle's xy bounding box
    const int64_t xmin = min(X[0], min(X[1], X[2])), xmax = max(X[0], max(X[1], X[2]));
    const int64_t ymin = min(Y[0], min(Y[1], Y[2])), ymax = max(Y[0], max(Y[1], Y[2]));
    const int64_t iu0 = -floor_div(-(xmin - QH), QS), iu1 = floor_div(xmax - QH, QS);
    const int64_t ju0 = -floor_div(-(ymin - QH), QS), ju1 = floor_div(ymax - QH, QS);
    // a triangle wider than the box (a blown-up mesh; the step reports the
    // instability) is left out rather than looped over
    if (!sane || iu1 - iu0 >= nx || ju1 - ju0 >= ny) return;
    for (int64_t ju = ju0; ju <= ju1; ++ju)
        for (int64_t iu = iu0; iu <= iu1; ++iu) {
            const int64_t px = iu * QS + QH, py = ju * QS + QH;
            const __int128 eab = edge_fn(X[0], Y[0], X[1], Y[1], px, py);
            const __int128 ebc = edge_fn(X[1], Y[1], X[2], Y[2], px, py);
            const __int128 eca = edge_fn(X[2], Y[2], X[0], Y[0], px, py);
            const int s1 = sos_sign(eab, X[1] - X[0], Y[1] - Y[0]);
            const int s2 = sos_sign(ebc, X[2] - X[1], Y[2] - Y[1]);
            const int s3 = sos_sign(eca, X[0] - X[2], Y[0] - Y[2]);
            if (s1 == 0 || s1 != s2 || s2 != s3) continue;
            const __int128 Dt = eab + ebc + eca;
            if (Dt == 0) continue;
            const __int128 Nt = ebc * Z[0] + eca * Z[1] + eab * Z[2];
            auto below = [&](int k) {  // crossing at or below the centre of cell k
                const __int128 d = ((__int128)k * QS + QH) * Dt - Nt;
                return Dt > 0 ? d >= 0 : d <= 0;
            };
            // first cell above the crossing: an estimate in FP64, then exact steps
            const double ea = (double)(X[1] - X[0]) * (double)(py - Y[0]) - (double)(Y[1] - Y[0]) * (double)(px - X[0]);
            const double eb = (double)(X[2] - X[1]) * (double)(py - Y[1]) - (double)(Y[2] - Y[1]) * (double)(px - X[1]);
            const double ec = (double)(X[0] - X[2]) * (double)(py - Y[2]) - (double)(Y[0] - Y[2]) * (double)(px - X[2]);
            const double zs = (eb * (double)Z[0] + ec * (double)Z[1] + ea * (double)Z[2]) / (ea + eb + ec);
            int k0 = (int)fmin(fmax(ceil(zs / (double)QS - 0.5), 0.0), (double)nz);
            while (k0 > 0 && below(k0 - 1)) --k0;
            while (k0 < nz && !below(k0)) ++k0;
            if (k0 >= nz) continue;
            const int i = (int)(iu % nx + (iu % nx < 0 ? nx : 0));
            const int j = (int)(ju % ny + (ju % ny < 0 ? ny : 0));
            for (int w = k0 >> 6; w < nzw; ++w) {
                const uint64_t bits = w == (k0 >> 6) ? (~0ull << (k0 & 63)) : ~0ull;
                atomicXor((unsigned long long *)&mask[((int64_t)w * ny + j) * nx + i], (unsigned long long)bits);
            }
        }
}

// Workgroups that clear the inside bits (0 without a contrast) and that look
// through the tiles for stamps.
inline int mask_clear_groups(const DevPtrs &P) {
    if (!P.contrast) return 0;
    const int64_t g = ((int64_t)P.mask_words + 255) / 256;
    return (int)(g < 1024 ? (g > 0 ? g : 1) : 1024);
}
inline int compact_groups(const DevPtrs &P) { return (P.total_tiles / TILE_CELLS + 3) / 4; }

// Workgroup `item` of `items`: its share of the mask words of every box with
// a contrast, cleared.
__device__ __forceinline__ void mask_clear_role(const DevPtrs &P, int item, int items, int slot) {
    for (int b = 0; b < P.n_boxes; ++b) {
        const BoxDev &B = P.boxes[b];
        if (!B.contrast) continue;
        const int64_t n = (int64_t)B.nzw * B.ny * B.nx;
        uint64_t *m = B.mask[slot];
        for (int64_t i = (int64_t)item * 256 + threadIdx.x; i < n; i += (int64_t)items * 256) m[i] = 0;
    }
}

}  // namespace iblb
