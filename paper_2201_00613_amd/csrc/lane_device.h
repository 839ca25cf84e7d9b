// Diffusion with a block of cells in the registers of each lane, several
// steps per launch (temporal blocking; the blocks of Section "Moving from
// Thread-level to Block-level").
//
//   tile  = a level-M subtree, one workgroup; block = a level-J subtree (the
//           carpet's 64 cells, 9 of the triangle, 25 of the Vicsek cross; 8, 3
//           and 5 where the fractal does not fill the chip), one lane.
//           In-block neighbours are registers; the cells of adjacent blocks a
//           block touches are values those lanes publish in LDS each step.
//           Where every cell read eight neighbours from LDS (nine reads
//           a cell and step), a carpet block reads 40 values and publishes 32
//           per 64 cells.
//   ring  = the blocks of adjacent tiles that hold every cell within K steps
//           of the tile, on lanes of their own.  Their outermost cells become
//           invalid one cell further in per step; K steps never reach the tile.
//
// The arithmetic is that of the one-step kernels: the neighbours' values in
// raster order (a hole's zero added to a partial sum changes nothing in the
// result, so holes are left out), u' = fma(a, fma(-deg, u, S), u), and with
// bfloat16 storage every step rounded as a one-step launch stores it.  Results
// are equal bit for bit.
//
// Measured against one launch per step (level-9 carpet, 100 steps and their mass; 6 launches
// of 16 or 17): binary32 23.19 -> 4.98 ms, bfloat16 with stochastic rounding
// 20.88 -> 9.38 ms, and 61 steps on the level-12 triangle 413 -> 46 us.  What
// bounds the carpet now: a launch moves its 1.2 GB (frames included) in about
// 245 us with nothing to overlap it (one workgroup of eleven waves per CU, 160
// registers a lane), and a step takes 35 us in binary32 (530 vector
// instructions a wave, the LDS busy half of the time) and 83 us with the
// rounding hash (1080 instructions).  A frame of one block (9 steps, ten waves)
// has the same time per step, since one SIMD has three waves either way, and
// twice the launches: 6.64 ms.
#pragma once

#include <algorithm>
#include <utility>

#include "bitbox_device.h"
#include "common.h"
#include "tile_device.h"
#include "xtile_device.h"

namespace sqz {

// ---------------------------------------------------------------------------
// Compile-time plan of a level-J block.
// ---------------------------------------------------------------------------
constexpr int kLaneCells = 64, kLaneHalo = 40;

struct LanePlan {
    int nc, box;
    int lx[kLaneCells], ly[kLaneCells];
    int deg[kLaneCells];            // neighbours, raster order
    int nb[kLaneCells][8];          // < nc: cell of the block; nc + h: halo slot h
    int nh, h_grp[kLaneHalo], h_cell[kLaneHalo], h_exp[kLaneHalo];  // slot: cell of the adjacent block of a group
    int ng, g_dx[8], g_dy[8];       // adjacent blocks
    int ne, e_cell[kLaneCells];     // published cells
    int nd, d_inner[40], d_cnt[40][8];  // distinct neighbour counts: inside the block, in each adjacent block
    int d_of[kLaneCells];
    int order[kLaneCells];          // inner cells (no halo) of the upper rows, cells with a halo, other inner cells
    int n0, n1;                     // of the first two kinds
    bool ok;
};

template <class P, int J>
constexpr LanePlan derive_lane_plan()
{
    LanePlan p{};
    p.ok = true;
    p.nc = cpow(P::K, J);
    p.box = cpow(P::S, J);
    int nu[32 * 32] = {};
    for (int i = 0; i < p.box * p.box; ++i) nu[i] = -1;
    for (int i = 0; i < p.nc; ++i) {
        int v = i, x = 0, y = 0, sp = 1;
        for (int mu = 0; mu < J; ++mu) {
            const int b = v % P::K;
            v /= P::K;
            x += P::OX[b] * sp;
            y += P::OY[b] * sp;
            sp *= P::S;
        }
        p.lx[i] = x;
        p.ly[i] = y;
        nu[y * p.box + x] = i;
    }
    for (int i = 0; i < p.nc; ++i) {
        int inner = 0, cnt[8] = {};
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                if (!dx && !dy) continue;
                const int qx = p.lx[i] + dx, qy = p.ly[i] + dy;
                const int bx = qx < 0 ? -1 : (qx >= p.box ? 1 : 0), by = qy < 0 ? -1 : (qy >= p.box ? 1 : 0);
                const int j = nu[(qy - by * p.box) * p.box + qx - bx * p.box];
                if (j < 0) continue;
                if (bx == 0 && by == 0) {
                    ++inner;
                    p.nb[i][p.deg[i]++] = j;
                    continue;
                }
                int g = -1, h = -1;
                for (int q = 0; q < p.ng; ++q)
                    if (p.g_dx[q] == bx && p.g_dy[q] == by) g = q;
                if (g < 0) {
                    g = p.ng++;
                    p.g_dx[g] = bx;
                    p.g_dy[g] = by;
                }
                for (int q = 0; q < p.nh; ++q)
                    if (p.h_grp[q] == g && p.h_cell[q] == j) h = q;
                if (h < 0) {
                    if (p.nh == kLaneHalo) {
                        p.ok = false;
                        return p;
                    }
                    h = p.nh++;
                    p.h_grp[h] = g;
                    p.h_cell[h] = j;
                }
                ++cnt[g];
                p.nb[i][p.deg[i]++] = p.nc + h;
            }
        int d = -1;
        for (int q = 0; q < p.nd; ++q) {
            bool same = p.d_inner[q] == inner;
            for (int g = 0; g < 8; ++g) same = same && p.d_cnt[q][g] == cnt[g];
            if (same) d = q;
        }
        if (d < 0) {
            if (p.nd == 40) {
                p.ok = false;
                return p;
            }
            d = p.nd++;
            p.d_inner[d] = inner;
            for (int g = 0; g < 8; ++g) p.d_cnt[d][g] = cnt[g];
        }
        p.d_of[i] = d;
    }
    int inner = 0, k = 0;
    for (int i = 0; i < p.nc; ++i) inner += p.d_inner[p.d_of[i]] == p.deg[i];
    for (int part = 0; part < 3; ++part)
        for (int i = 0, seen = 0; i < p.box * p.box; ++i) {  // row by row
            const int c = nu[i];
            if (c < 0) continue;
            const bool in = p.d_inner[p.d_of[c]] == p.deg[c];
            if (in) ++seen;
            const int mine = !in ? 1 : (seen <= inner / 2 ? 0 : 2);
            if (mine != part) continue;
            p.order[k++] = c;
            ++(part == 0 ? p.n0 : (part == 1 ? p.n1 : inner));
        }
    // published cells in the order of the groups that read them, so that one
    // base address per group reaches them all
    for (int h = 0; h < p.nh; ++h) p.h_exp[h] = -1;
    for (int g = 0; g < p.ng; ++g)
        for (int h = 0; h < p.nh; ++h) {
            if (p.h_grp[h] != g) continue;
            for (int e = 0; e < p.ne; ++e)
                if (p.e_cell[e] == p.h_cell[h]) p.h_exp[h] = e;
            if (p.h_exp[h] < 0) {
                p.h_exp[h] = p.ne;
                p.e_cell[p.ne++] = p.h_cell[h];
            }
        }
    return p;
}

template <class P, int J>
struct LanePlanOf {
    static constexpr LanePlan value = derive_lane_plan<P, J>();
    static_assert(value.ok, "block does not fit the lane kernel");
};

// Patterns: block level J, lanes (a multiple of 64,
// more than tile and ring need: the last lane's LDS column stays zero).
// FRAME blocks: the ring is the frame of that many blocks around the tile
// (dense patterns: STEPS is the frame's width in cells); 0: the level-RL
// subtrees that hold the cells next to the tile, which cover STEPS steps
// (their side, one less for the triangles).  LARGE: fractals of more than 2^32
// cells run on it too.
struct LaneTriangle : PatTriangle {
    static constexpr int J = 2, LANES = 832, RL = 4, STEPS = 15, FRAME = 0;
    static constexpr bool LARGE = true;
};
struct LaneTrianglePaper : PatTrianglePaper {
    static constexpr int J = 2, LANES = 832, RL = 4, STEPS = 15, FRAME = 0;
    static constexpr bool LARGE = true;
};
struct LaneVicsek : PatVicsek {
    static constexpr int J = 2, LANES = 704, RL = 3, STEPS = 27, FRAME = 0;
    static constexpr bool LARGE = true;
};
struct LaneCarpet : PatCarpet {
    static constexpr int J = 2, LANES = 768, RL = 0, STEPS = 18, FRAME = 2;
    static constexpr bool LARGE = true;
};
struct LaneCarpetSmall : PatCarpet {
    static constexpr int J = 2, LANES = 192, RL = 0, STEPS = 18, FRAME = 2;
    static constexpr bool LARGE = false;
};
// Fractals that do not fill the chip, where a step's own latency counts: fewer
// cells per lane.
struct LaneTriangleFine : PatTriangle {
    static constexpr int J = 1, LANES = 960, RL = 4, STEPS = 15, FRAME = 0;
    static constexpr bool LARGE = false;
};
struct LaneTrianglePaperFine : PatTrianglePaper {
    static constexpr int J = 1, LANES = 960, RL = 4, STEPS = 15, FRAME = 0;
    static constexpr bool LARGE = false;
};
struct LaneVicsekFine : PatVicsek {
    static constexpr int J = 1, LANES = 768, RL = 3, STEPS = 27, FRAME = 0;
    static constexpr bool LARGE = false;
};
struct LaneCarpetFine : PatCarpet {
    static constexpr int J = 1, LANES = 576, RL = 0, STEPS = 15, FRAME = 5;
    static constexpr bool LARGE = false;
};

// Storage types: G in memory, binary32 in registers.
struct LaneF32 {
    using G = float;
    static constexpr int RND = -1;
};
template <int R, bool WIDE = false>  // sqz_rounding; WIDE: cell indices of more than 32 bits
struct LaneBF16 {
    using G = uint16_t;
    static constexpr int RND = R;
    static constexpr bool WIDX = WIDE;
};

// Memory layout of a workgroup.  Published values: column = lane, row =
// published slot, so that consecutive lanes hit consecutive banks and a
// group's values lie at fixed offsets from one address.  Two copies where they
// fit 64 KB (one barrier per step), else one (two barriers).  At the load and
// the store every wave moves its own 64 blocks through a staging area: V
// elements (16 bytes) per chunk, eight chunks a lane and phase, swizzled so
// that neither side conflicts; V = 1 where a block is not whole chunks.
template <class P, class Op>
struct LaneCfg {
    using PO = LanePlanOf<P, P::J>;
    using G = typename Op::G;
    static constexpr int NC = PO::value.nc, NE = PO::value.ne, NH = PO::value.nh, NG = PO::value.ng;
    static constexpr int V = (NC * sizeof(G)) % 128 == 0 ? 16 / (int)sizeof(G) : 1;
    static constexpr int CH = V > 1 ? 8 : NC, PH = NC / (V * CH);
    static constexpr uint32_t EXW = NE * P::LANES;
    static constexpr int DB = EXW * 8 <= 65536 ? 2 : 1;
    static constexpr uint32_t STW = 64 * (V > 1 ? 32 : NC);  // staging words per wave
    static constexpr uint32_t LDSW = DB * EXW > STW * (P::LANES / 64) ? DB * EXW : STW * (P::LANES / 64);
    static_assert(LDSW * 4 <= 163840, "LDS");
};

struct LaneArgs {
    uint32_t ntiles;
    uint32_t nblk, lanes;        // blocks of a tile; lanes in use
    const uint32_t *lane_src;    // [lanes - nblk] ring block: adjacent tile (0..7) << 28 | block in it
    const uint32_t *lane_nb;     // [lanes][NG] lane of the adjacent block | its tile (8: this one) << 16; ~0: none
    const uint32_t *nbtile;      // [ntiles][8] adjacent tiles, kNuHole32 if none
};

typedef uint32_t lane_u32x4 __attribute__((ext_vector_type(4), aligned(2)));

// rand16 of a cell (x: the cell's low 32 bits xor the term of its high bits,
// plus sx, the terms of the seed and the step).  The finaliser's last x ^= x >> 16
// leaves the upper 16 bits, all that is used, as they are.
__device__ __forceinline__ uint32_t lane_rand16(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    return x >> 16;
}

// base: lo + sx, of which cell I's argument is base + I where no cell index has
// high bits (30 steps: level-12 triangle 22.3 -> 20.7 us, level 9 13.6 -> 12.9;
// level-9 carpet, 100 steps 9.23 -> 9.17 ms); with high bits two to five
// operations a cell take its place.
struct LaneRand {
    uint32_t lo, hx, hx1, sx, base;  // hx1: the term once lo + i has carried
};

template <class P, class Op, int I, int NC, int NH, int ND>
__device__ __forceinline__ float lane_cell(const float (&x)[NC], const float (&h)[NH], const float (&nd)[ND],
                                           float coef, const LaneRand &R)
{
    using PO = LanePlanOf<P, P::J>;
    constexpr int D = PO::value.deg[I];
    float S = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int q = PO::value.nb[I][d];
        const float v = q < NC ? x[q < NC ? q : 0] : h[q < NC ? 0 : q - NC];
        S = d ? S + v : v;
    }
    const float u = fmaf(coef, fmaf(nd[PO::value.d_of[I]], x[I], S), x[I]);
    if constexpr (Op::RND < 0) {
        return u;
    } else {
        uint32_t b = __float_as_uint(u);
        if constexpr (Op::RND == SQZ_ROUND_STOCHASTIC) {
            if constexpr (!Op::WIDX) {
                b += lane_rand16(R.base + (uint32_t)I);
            } else if constexpr ((NC & (NC - 1)) == 0) {  // lo is a multiple of NC: lo + I = lo ^ I
                b += lane_rand16(((R.lo ^ R.hx) ^ (uint32_t)I) + R.sx);
            } else {
                const uint32_t lo = R.lo + I;
                b += lane_rand16((lo ^ (lo < (uint32_t)I ? R.hx1 : R.hx)) + R.sx);
            }
        } else {
            b += 0x7FFFu + ((b >> 16) & 1u);
        }
        return __uint_as_float(b & 0xFFFF0000u);
    }
}

// New values y of cells order[FROM], ...
template <class P, class Op, int FROM, int NC, int NH, int ND, size_t... I>
__device__ __forceinline__ void lane_cells(const float (&x)[NC], const float (&h)[NH], const float (&nd)[ND],
                                           float coef, const LaneRand &R, float (&y)[NC], std::index_sequence<I...>)
{
    using PO = LanePlanOf<P, P::J>;
    auto cell = [&](auto i) {
        constexpr int k = FROM + decltype(i)::value, c = PO::value.order[k];
        y[c] = lane_cell<P, Op, c>(x, h, nd, coef, R);
    };
    (cell(std::integral_constant<int, (int)I>{}), ...);
}

// Tile t, `steps` <= the ring's steps (any number when the fractal is one
// tile).  Every lane of the workgroup calls it.
template <class P, class Op>
__device__ __forceinline__ void lane_tile(const LaneArgs &A, const typename Op::G *__restrict__ in,
                                          typename Op::G *__restrict__ out, uint32_t t, const XOp &op, int32_t steps,
                                          uint32_t *sm)
{
    using C = LaneCfg<P, Op>;
    using PO = LanePlanOf<P, P::J>;
    using G = typename Op::G;
    constexpr int NC = C::NC, NG = C::NG, V = C::V, CH = C::CH, PH = C::PH;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave0 = __builtin_amdgcn_readfirstlane(tid);  // the wave's first lane
    const uint32_t *nbt = A.nbtile + (uint64_t)t * 8;
    uint32_t there = 1u << 8;  // tiles that exist (the same for every lane)
#pragma unroll
    for (int d = 0; d < 8; ++d) there |= (nbt[d] != kNuHole32 ? 1u : 0u) << d;
    // this lane's block: number in the whole fractal, ~0 if it does not exist
    uint32_t bn = ~0u;
    if (tid < A.nblk) {
        bn = t * A.nblk + tid;
    } else if (tid < A.lanes) {
        const uint32_t e = A.lane_src[tid - A.nblk];
        if ((there >> (e >> 28)) & 1u) bn = nbt[e >> 28] * A.nblk + (e & 0xFFFFFFFu);
    }
    uint32_t gb[NG];
    float ex[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const uint32_t e = tid < A.lanes ? A.lane_nb[tid * NG + g] : ~0u;
        const bool ok = e != ~0u && ((there >> ((e >> 16) & 15u)) & 1u);
        gb[g] = ok ? e & 0xFFFFu : P::LANES - 1;
        ex[g] = ok ? 1.0f : 0.0f;
    }
    float nd[PO::value.nd];
#pragma unroll
    for (int q = 0; q < PO::value.nd; ++q) {
        float d = (float)PO::value.d_inner[q];
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (PO::value.d_cnt[q][g]) d += (float)PO::value.d_cnt[q][g] * ex[g];
        nd[q] = -d;
    }
    // load: the wave's 64 blocks, coalesced, through its staging area
    float x[NC];
    uint32_t *const st = sm + (tid >> 6) * C::STW;
    if constexpr (V > 1) {
        uint4 v[PH][CH];
#pragma unroll
        for (int p = 0; p < PH; ++p)
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const uint32_t b = __shfl(bn, i * 8 + (int)(lane >> 3));
                v[p][i] = make_uint4(0u, 0u, 0u, 0u);
                if (b != ~0u) {
                    const lane_u32x4 z = *reinterpret_cast<const lane_u32x4 *>(in + (uint64_t)b * NC + (p * CH + (lane & 7u)) * V);
                    v[p][i] = make_uint4(z.x, z.y, z.z, z.w);
                }
            }
        uint4 *s4 = reinterpret_cast<uint4 *>(st);
#pragma unroll
        for (int p = 0; p < PH; ++p) {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const uint32_t bl = i * 8 + (lane >> 3);
                s4[bl * 8 + ((lane ^ bl) & 7u)] = v[p][i];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const uint4 z = s4[lane * 8 + ((c ^ lane) & 7u)];
                const uint32_t w[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if constexpr (sizeof(G) == 4) {
                        x[(p * CH + c) * V + k] = __uint_as_float(w[k]);
                    } else {
                        x[(p * CH + c) * V + 2 * k] = __uint_as_float(w[k] << 16);
                        x[(p * CH + c) * V + 2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    } else {
        // a wave of the tile's own blocks: one contiguous range in 16-byte loads;
        // with ring blocks: element by element
        float *sf = reinterpret_cast<float *>(st);
        constexpr uint32_t Q = 16 / sizeof(G), NQ = 64 * NC / Q;
        if (wave0 + 64 <= A.nblk) {
            const G *src = in + ((uint64_t)t * A.nblk + wave0) * NC;
#pragma unroll
            for (uint32_t i = 0; i < (NQ + 63) / 64; ++i) {
                const uint32_t k = i * 64 + lane;
                if (k < NQ) {
                    const lane_u32x4 z = *reinterpret_cast<const lane_u32x4 *>(src + k * Q);
                    const uint32_t w[4] = {z.x, z.y, z.z, z.w};
                    uint4 *d = reinterpret_cast<uint4 *>(sf + k * Q);
                    if constexpr (sizeof(G) == 4) {
                        d[0] = make_uint4(w[0], w[1], w[2], w[3]);
                    } else {
                        d[0] = make_uint4(w[0] << 16, w[0] & 0xFFFF0000u, w[1] << 16, w[1] & 0xFFFF0000u);
                        d[1] = make_uint4(w[2] << 16, w[2] & 0xFFFF0000u, w[3] << 16, w[3] & 0xFFFF0000u);
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const uint32_t e = i * 64 + lane, bl = e / NC, c = e - bl * NC;
                const uint32_t b = __shfl(bn, (int)bl);
                sf[e] = b != ~0u ? to_lds(in[(uint64_t)b * NC + c]) : 0.0f;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int c = 0; c < NC; ++c) x[c] = sf[lane * NC + c];
    }
    LaneRand R{};
    if constexpr (Op::RND == SQZ_ROUND_STOCHASTIC) {
        const uint64_t c0 = (uint64_t)bn * NC;
        R.lo = (uint32_t)c0;
        R.hx = (uint32_t)(c0 >> 32) * 0x85EBCA6Bu;
        R.hx1 = R.hx + 0x85EBCA6Bu;
    }
    __syncthreads();  // the staging areas become the published values

    float *const lds = reinterpret_cast<float *>(sm);
    const uint32_t used = blockDim.x;
    for (uint32_t e = tid; e < (uint32_t)(C::DB * C::NE); e += used) lds[e * P::LANES + P::LANES - 1] = 0.0f;
    uint32_t o = 0;  // the copy in use (word offset)
    if (tid < A.lanes) {
#pragma unroll
        for (int e = 0; e < C::NE; ++e) lds[o + e * P::LANES + tid] = x[PO::value.e_cell[e]];
    }
    __syncthreads();
    // A step: half of the inner cells while the halo values arrive, the cells
    // that need them, their publication, and the other inner cells while it
    // completes.
    constexpr int N0 = PO::value.n0, N1 = PO::value.n1;
    for (int32_t s = 0;;) {
        float h[C::NH], y[NC];
#pragma unroll
        for (int q = 0; q < C::NH; ++q) h[q] = lds[o + PO::value.h_exp[q] * P::LANES + gb[PO::value.h_grp[q]]];
        if constexpr (Op::RND == SQZ_ROUND_STOCHASTIC) {
            asm volatile("" : "+v"(R.lo));  // or the per-cell terms are hoisted into a register each
            R.sx = (uint32_t)op.seed * 0x9E3779B9u + (uint32_t)(op.seed >> 32) + (uint32_t)(op.step + s) * 0x7FEB352Du;
            R.base = R.lo + R.sx;
        }
        lane_cells<P, Op, 0>(x, h, nd, op.coef, R, y, std::make_index_sequence<N0>{});
        if constexpr (C::DB == 1) __syncthreads();  // every lane has read this step's halo
        lane_cells<P, Op, N0>(x, h, nd, op.coef, R, y, std::make_index_sequence<N1>{});
        const bool last = ++s == steps;
        if (!last) {
            if constexpr (C::DB == 2) o = C::EXW - o;
            if (tid < A.lanes) {
#pragma unroll
                for (int e = 0; e < C::NE; ++e) lds[o + e * P::LANES + tid] = y[PO::value.e_cell[e]];
            }
        }
        lane_cells<P, Op, N0 + N1>(x, h, nd, op.coef, R, y, std::make_index_sequence<NC - N0 - N1>{});
#pragma unroll
        for (int c = 0; c < NC; ++c) x[c] = y[c];
        if (last) break;
        __syncthreads();
    }
    if constexpr (C::DB == 2) __syncthreads();  // the last halo has been read: staging again
    if constexpr (V > 1) {
        uint4 *s4 = reinterpret_cast<uint4 *>(st);
#pragma unroll
        for (int p = 0; p < PH; ++p) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                uint32_t w[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if constexpr (sizeof(G) == 4)
                        w[k] = __float_as_uint(x[(p * CH + c) * V + k]);
                    else
                        w[k] = __float_as_uint(x[(p * CH + c) * V + 2 * k]) >> 16 |
                               (__float_as_uint(x[(p * CH + c) * V + 2 * k + 1]) & 0xFFFF0000u);
                }
                s4[lane * 8 + ((c ^ lane) & 7u)] = make_uint4(w[0], w[1], w[2], w[3]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const uint32_t bl = i * 8 + (lane >> 3);
                if (wave0 + bl < A.nblk) {
                    const uint4 z = s4[bl * 8 + ((lane ^ bl) & 7u)];
                    const lane_u32x4 y = {z.x, z.y, z.z, z.w};
                    const uint64_t b = t * A.nblk + wave0 + bl;
                    *reinterpret_cast<lane_u32x4 *>(out + b * NC + (p * CH + (lane & 7u)) * V) = y;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    } else {
        float *sf = reinterpret_cast<float *>(st);
#pragma unroll
        for (int c = 0; c < NC; ++c) sf[lane * NC + c] = x[c];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        constexpr uint32_t Q = 16 / sizeof(G), NQ = 64 * NC / Q;
        if (wave0 + 64 <= A.nblk) {
            G *dst = out + ((uint64_t)t * A.nblk + wave0) * NC;
#pragma unroll
            for (uint32_t i = 0; i < (NQ + 63) / 64; ++i) {
                const uint32_t k = i * 64 + lane;
                if (k < NQ) {
                    const uint4 *d = reinterpret_cast<const uint4 *>(sf + k * Q);
                    const uint4 u = d[0];
                    lane_u32x4 z = {u.x, u.y, u.z, u.w};
                    if constexpr (sizeof(G) == 2) {
                        const uint4 v = d[1];
                        z.x = u.x >> 16 | u.y;
                        z.y = u.z >> 16 | u.w;
                        z.z = v.x >> 16 | v.y;
                        z.w = v.z >> 16 | v.w;
                    }
                    *reinterpret_cast<lane_u32x4 *>(dst + k * Q) = z;
                }
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const uint32_t e = i * 64 + lane;
            if (wave0 + e / NC < A.nblk) {
                const uint64_t b = t * A.nblk + wave0;
                if constexpr (sizeof(G) == 4)
                    out[b * NC + e] = sf[e];
                else
                    out[b * NC + e] = (uint16_t)(__float_as_uint(sf[e]) >> 16);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Host side: kernel, tile level and table layout of a fractal.
// ---------------------------------------------------------------------------
template <class F>
auto lane_dispatch(int kind, F &&f)
{
    switch (kind) {
    case 1: return f(LaneTriangle{});
    case 2: return f(LaneTrianglePaper{});
    case 3: return f(LaneVicsek{});
    case 4: return f(LaneCarpet{});
    case 5: return f(LaneCarpetSmall{});
    case 6: return f(LaneTriangleFine{});
    case 7: return f(LaneTrianglePaperFine{});
    case 8: return f(LaneVicsekFine{});
    default: return f(LaneCarpetFine{});
    }
}

template <class P>
bool lane_matches(const FractalHost &F)
{
    if (F.s != P::S || F.k != P::K || F.r < P::J) return false;
    for (int j = 0; j < P::K; ++j)
        if (F.ox[j] != P::OX[j] || F.oy[j] != P::OY[j]) return false;
    return true;
}

// Kernel.  Level-1 blocks where a fractal does not fill the chip and a step
// takes the latency of one lane's work (30 steps, binary32 / bfloat16 with
// stochastic rounding: level-9 triangle 16.8 / 21.5 -> 12.1 / 13.6 us, level 12
// 18.9 / 28.0 -> 18.5 / 22.3; Vicsek level 6 22.6 / 39.0 -> 14.5 / 16.5; carpet
// level 6 50 / 75 -> 27 / 40), level-2 blocks above, where the wider frames and
// the halo reads per cell cost more (triangle level 13 24.4 against 36.1, Vicsek
// level 9 36 against 40, carpet level 7 58 against 127).
inline int lane_kind(const FractalHost &F)
{
    if (lane_matches<LaneTriangleFine>(F)) return F.r >= 13 ? 1 : 6;
    if (lane_matches<LaneTrianglePaperFine>(F)) return F.r >= 13 ? 2 : 7;
    if (lane_matches<LaneVicsekFine>(F)) return F.r >= 9 ? 3 : 8;
    if (lane_matches<LaneCarpetFine>(F)) return F.r >= 8 ? 4 : (F.r == 7 ? 5 : 9);
    return 0;
}

// Tile level.  A fractal of at most one full workgroup is one tile (no ring,
// any number of steps per launch), except where several small ones have the
// shorter step (triangle level 7: 13.9 us as one tile of 729 lanes, 11.6 as
// nine; level 6: 10.0 and 10.5).  Above, the largest tiles that still leave
// tens to hundreds of them: until the chip is full a step takes as long as one
// tile of any size.
inline int lane_level(int kind, int r)
{
    switch (kind) {
    case 1:
    case 2: return r <= 13 ? 7 : 8;
    case 3: return 6;
    case 4: return 5;
    case 5: return 4;
    case 6:
    case 7: return r <= 6 ? r : (r <= 9 ? 5 : (r <= 11 ? 6 : 7));
    case 8: return std::min(r, 4);
    default: return r <= 4 ? r : 3;
    }
}

// What the table builder needs; most: lanes a tile can have.
inline LaneSpec lane_spec(int kind, int r, uint32_t &most)
{
    LaneSpec S{};
    S.M = lane_level(kind, r);
    lane_dispatch(kind, [&](auto p) {
        using P = decltype(p);
        using PO = LanePlanOf<P, P::J>;
        S.J = P::J;
        S.ng = PO::value.ng;
        for (int g = 0; g < S.ng; ++g) {
            S.g_dx[g] = PO::value.g_dx[g];
            S.g_dy[g] = PO::value.g_dy[g];
        }
        S.steps = P::STEPS;
        S.RL = P::RL;
        S.frame = P::FRAME;
        most = P::LANES - 1;
        return 0;
    });
    return S;
}

}  // namespace sqz
