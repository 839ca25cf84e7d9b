// Block-level Squeeze (Section "Moving from Thread-level to Block-level") for
// Life on any replica pattern without a kernel of its own: the level-M subtree
// of a tile expanded on chip as bit rows, several steps per launch.
//
// One workgroup per tile.  The box is the tile's s^M x s^M region with a border of
// D cells from the eight adjacent tiles, rows of W 32-bit words.  Cells and
// border cells are scattered into it bit by bit through tile-invariant tables,
// K <= D rounds run on whole words (a lane slides a window down a strip of one
// word column, full adders as in bitbox_device.h), new states are masked by
// the tile-invariant membership and by which adjacent tiles exist, and the
// tile's cells are read back.  Each round makes one more cell along the box
// edge invalid; the leftmost and rightmost columns, whose neighbours wrap into
// the adjacent rows, are among the first.
//
// The expanded-tile kernel that ran these patterns before (xtile_device.h)
// holds a byte per position and takes at most three steps per launch.
// Measured (s = 4, k = 10): 21 steps of 1e6 cells 79.8 -> 19.6 us (one launch,
// bound by the latency of its steps), of 1e8 cells 3.50 -> 0.89 ms.  Rows that
// the remaining steps no longer reach are computed all the same: leaving them
// out costs an index division a step (16 steps of 1e6 cells 18.3 -> 19.2 us).
#include <algorithm>
#include <vector>

#include "bitbox_device.h"
#include "xtile_device.h"

namespace sqz {

constexpr int kGbBorder = 16, kGbMaxBorder = 32;
constexpr uint64_t kGbFewTiles = 2048;  // at most two tiles per SIMD: a tile's own time counts
constexpr int kGbFewNT = 256, kGbFewStrip = 2;

struct GboxArgs {
    uint32_t ntiles, KM;       // tiles, cells per tile
    uint32_t B, D, W, rows;    // side, border, words per row, rows (B + 2 D)
    uint32_t ring[kGbMaxBorder + 1];  // border cells within d cells of the box: ring[d]
    const uint16_t *pos;       // [KM] box position (row * 32 W + column) of each cell
    const uint32_t *slot;      // [ring[D]] box position | adjacent tile << 16 | cell in it << 19, by distance
    const uint32_t *member;    // [rows * W] membership, adjacent tiles present
    MapParams Pc;              // maps at the coarse level r - M
};

struct GboxConfig {
    int K;          // steps per launch (0: one tile, any number)
    int K2;         // of the tables with the wider border (0: none)
    GboxArgs A, A2;
    void *d_tab, *d_coarse;
};

typedef uint32_t gb_u32 __attribute__((aligned(1)));

// Rows in whole strips, words of a row buffer (a zero word and a zero guard
// row on each side), LDS words (two buffers, membership, eight tile bases).
__host__ __device__ constexpr uint32_t gb_rows(uint32_t rows, int strip) { return (rows + strip - 1) / strip * strip; }
__host__ __device__ constexpr uint32_t gb_buf(uint32_t W, uint32_t nrow) { return 2 + (nrow + 2) * W; }
__host__ __device__ constexpr uint32_t gb_lds(uint32_t W, uint32_t nrow)
{
    return (2 * gb_buf(W, nrow) + nrow * W + 1) / 2 * 2 + 16;
}

// STRIP rows per lane and turn, NT lanes.  One wave and strips of five rows
// where the tiles fill the chip; four waves and strips of two where they do
// not and a tile's own time counts (see launch_life_gbox).
template <int STRIP, int NT>
__global__ void __launch_bounds__(NT) k_life_gbox(GboxArgs A, const uint8_t *__restrict__ in,
                                                  uint8_t *__restrict__ out, int32_t steps)
{
    extern __shared__ __align__(16) uint32_t sm[];
    const uint32_t tid = threadIdx.x, W = A.W, nrow = gb_rows(A.rows, STRIP), NB = gb_buf(W, nrow);
    uint32_t *const mem = sm + 2 * NB;
    uint64_t *const nbase = reinterpret_cast<uint64_t *>(sm + (2 * NB + nrow * W + 1) / 2 * 2);
    const uint64_t t = xcd_remap(blockIdx.x, gridDim.x);
    // the adjacent tiles (eight coarse nu)
    uint32_t *const s_ex = sm + gb_lds(W, nrow);
    if (tid < 64) {
    bool here = false;
    if (tid < 8) {
        const int d = tid < 4 ? (int)tid : (int)tid + 1;
        uint32_t X, Y;
        lam_map32(A.Pc, (uint32_t)t, X, Y);
        const uint64_t nt = nu_map(A.Pc, (int32_t)X + d % 3 - 1, (int32_t)Y + d / 3 - 1);
        here = nt != kHole64;
        nbase[tid] = here ? nt * A.KM : kHole64;
    }
    const uint32_t m8 = (uint32_t)__ballot(here);
    if (tid == 0) *s_ex = (m8 & 15u) | 16u | (m8 & 0xF0u) << 1;  // 3 x 3 tiles, row by row
    }
    for (uint32_t i = tid; i < 2 * NB; i += NT) sm[i] = 0;
    __syncthreads();
    const uint32_t ex = *s_ex;
    uint32_t *const b0 = sm + 1 + W;  // row 0, word 0 of the first buffer
    auto set = [&](uint32_t p) { atomicOr(b0 + (p >> 5), 1u << (p & 31u)); };
    // the tile's cells
    const uint8_t *src = in + t * A.KM;
    if (A.KM % 4 == 0) {
#pragma unroll 4
        for (uint32_t l = 4 * tid; l < A.KM; l += 4 * NT) {
            const uint32_t v = *reinterpret_cast<const gb_u32 *>(src + l);
            const uint2 p = *reinterpret_cast<const uint2 *>(A.pos + l);
            if (v & 1u) set(p.x & 0xFFFFu);
            if (v & 0x100u) set(p.x >> 16);
            if (v & 0x10000u) set(p.y & 0xFFFFu);
            if (v & 0x1000000u) set(p.y >> 16);
        }
    } else {
#pragma unroll 4
        for (uint32_t l = tid; l < A.KM; l += NT)
            if (src[l] & 1u) set(A.pos[l]);
    }
    // border cells within `steps` of the box
    const uint32_t nring = A.ring[steps < (int32_t)A.D ? steps : (int32_t)A.D];
#pragma unroll 4
    for (uint32_t i = tid; i < nring; i += NT) {
        const uint32_t e = A.slot[i];
        const uint64_t nb = nbase[(e >> 16) & 7u];
        if (nb != kHole64 && (in[nb + (e >> 19)] & 1u)) set(e & 0xFFFFu);
    }
    // this tile's membership
    for (uint32_t i = tid; i < nrow * W; i += NT) {
        const uint32_t y = i / W, w = i - y * W;
        uint32_t v = 0;
        if (y < A.rows) {
            const uint32_t e3 = ex >> (y < A.D ? 0 : (y < A.D + A.B ? 3 : 6));
            const int D = (int)A.D, B = (int)A.B;
            v = A.member[i] & (((e3 & 1u) ? col_mask(0, D, (int)w) : 0u) | ((e3 & 2u) ? col_mask(D, D + B, (int)w) : 0u) |
                               ((e3 & 4u) ? col_mask(D + B, 2 * D + B, (int)w) : 0u));
        }
        mem[i] = v;
    }
    __syncthreads();
    uint32_t *s = b0, *d = b0 + NB;
    for (int32_t j = 0; j < steps; ++j) {
        for (uint32_t u = tid; u < W * (nrow / STRIP); u += NT) {
            const uint32_t strip = u / W, o = strip * STRIP * W + (u - strip * W);
            const uint32_t *p = s + o;
            BxRow up = bx_row(p - W), mid = bx_row(p);
#pragma unroll
            for (int r = 0; r < STRIP; ++r) {
                const BxRow dn = bx_row(p + (r + 1) * W);
                d[o + r * W] = bx_life(up, mid, dn) & mem[o + r * W];
                up = mid;
                mid = dn;
            }
        }
        __syncthreads();
        uint32_t *const x = s;
        s = d;
        d = x;
    }
    uint8_t *dst = out + t * A.KM;
    auto get = [&](uint32_t p) { return (s[p >> 5] >> (p & 31u)) & 1u; };
    if (A.KM % 4 == 0) {
        for (uint32_t l = 4 * tid; l < A.KM; l += 4 * NT) {
            const uint2 p = *reinterpret_cast<const uint2 *>(A.pos + l);
            *reinterpret_cast<gb_u32 *>(dst + l) =
                get(p.x & 0xFFFFu) | get(p.x >> 16) << 8 | get(p.y & 0xFFFFu) << 16 | get(p.y >> 16) << 24;
        }
    } else {
        for (uint32_t l = tid; l < A.KM; l += NT) dst[l] = (uint8_t)get(A.pos[l]);
    }
}

void gbox_release(FractalHost &F)
{
    if (!F.gbox) return;
    (void)hipFree(F.gbox->d_tab);
    (void)hipFree(F.gbox->d_coarse);
    delete F.gbox;
    F.gbox = nullptr;
}

// For the patterns that run on expanded tiles, at their tile level.
sqz_status gbox_prepare(FractalHost &F)
{
    F.gbox = nullptr;
    const int M = xtile_level_of(F);
    if (F.tile_kind || F.bitbox || M < 1) return SQZ_OK;
    uint64_t B = 1, KM = 1, nt = 1;
    for (int i = 0; i < M; ++i) B *= F.s, KM *= F.k;
    for (int i = M; i < F.r; ++i) nt *= F.k;
    // a launch holds fewer than 2^32 lanes, and there are at least 64 a tile: more
    // tiles (17 GB of sparse cells) are left to the expanded-tile kernel, whose grid
    // does not grow with them
    if (KM > 8192 || B > 128 || nt * 64 > 0xFFFFFFFFull) return SQZ_OK;
    // Border: up to 16 cells, at most a quarter of the box (a wider one would
    // cost more in border cells than it saves in launches); around a single
    // tile one cell, always empty (a column between the row's ends).
    const bool one = F.r == M;
    const int D = one ? 1 : std::min<int>({kGbBorder, (int)B, std::max(4, (int)B / 4)});
    GboxConfig *C = new GboxConfig();
    C->K = one ? 0 : D;
    // Few tiles: a second set of tables with the widest border (of more than
    // D cells) whose box the lanes still update in one turn.
    if (!one && nt <= kGbFewTiles)
        for (int d = D + 1; d <= std::min<int>(kGbMaxBorder, (int)B); ++d)
            if (((int)B + 2 * d + 31) / 32 * gb_rows((uint32_t)B + 2 * d, kGbFewStrip) / kGbFewStrip <= kGbFewNT) C->K2 = d;
    std::vector<uint8_t> blob;
    size_t at[2][3];  // offsets of pos, slot, member
    auto build = [&](GboxArgs &A, int border, size_t (&o)[3]) {
        A.ntiles = (uint32_t)nt;
        A.KM = (uint32_t)KM;
        A.B = (uint32_t)B;
        A.D = (uint32_t)border;
        A.W = (A.B + 2 * A.D + 31) / 32;
        A.rows = A.B + 2 * A.D;
        std::vector<XRingSlot> ring;
        std::vector<uint32_t> start;
        std::vector<uint16_t> lam;
        std::vector<uint8_t> own;
        const uint32_t P = 32 * A.W;
        xtile_layer_tables(F, M, border, P, A.rows, ring, start, lam, own);
        for (int d = 0; d <= border; ++d) A.ring[d] = start[d];
        std::vector<uint32_t> slot(ring.size()), member((size_t)A.rows * A.W, 0);
        for (size_t i = 0; i < own.size(); ++i)
            if (own[i]) member[i / 32] |= 1u << (i % 32);
        for (size_t i = 0; i < ring.size(); ++i) {
            slot[i] = ring[i].pos | (ring[i].info >> 16) << 16 | (ring[i].info & 0xFFFFu) << 19;
            member[ring[i].pos / 32] |= 1u << (ring[i].pos % 32);
        }
        lam.resize((lam.size() + 7) / 8 * 8, 0);  // read four at a time
        o[0] = (blob.size() + 15) / 16 * 16;
        o[1] = o[0] + lam.size() * 2;
        o[2] = o[1] + slot.size() * 4;
        blob.resize(o[2] + member.size() * 4);
        std::copy(lam.begin(), lam.end(), reinterpret_cast<uint16_t *>(blob.data() + o[0]));
        std::copy(slot.begin(), slot.end(), reinterpret_cast<uint32_t *>(blob.data() + o[1]));
        std::copy(member.begin(), member.end(), reinterpret_cast<uint32_t *>(blob.data() + o[2]));
    };
    build(C->A, D, at[0]);
    if (C->K2) build(C->A2, C->K2, at[1]);
    sqz_status st = build_map_params(F, F.r - M, C->A.Pc, &C->d_coarse);
    if (st != SQZ_OK) {
        delete C;
        return st;
    }
    hipError_t e = hipMalloc(&C->d_tab, blob.size());
    if (e == hipSuccess) e = hipMemcpy(C->d_tab, blob.data(), blob.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (C->d_tab) (void)hipFree(C->d_tab);
        (void)hipFree(C->d_coarse);
        delete C;
        return hip_error(e, "bit box tables");
    }
    C->A2.Pc = C->A.Pc;
    for (int i = 0; i < (C->K2 ? 2 : 1); ++i) {
        GboxArgs &A = i ? C->A2 : C->A;
        const uint8_t *t = (const uint8_t *)C->d_tab;
        A.pos = (const uint16_t *)(t + at[i][0]);
        A.slot = (const uint32_t *)(t + at[i][1]);
        A.member = (const uint32_t *)(t + at[i][2]);
    }
    F.gbox = C;
    return SQZ_OK;
}

// Launches of a single step: ahead of the expanded-tile kernel where cells are
// sparse in their box (s = 4, k = 10, 1e8 cells: 136 against 414 us; s = 3,
// k = 6: 7.2 against 9.4), behind it on the full square (1.7e7 cells: 22.7
// against 20.2), whose bytes it needs no scatter for.
bool gbox_one_step(const FractalHost &F)
{
    return F.gbox && 2ull * F.gbox->A.KM <= (uint64_t)F.gbox->A.B * F.gbox->A.B;
}

// Most steps per launch of a run: those of the wider border where that takes
// fewer launches. A step on its larger box is slower, a launch costs more than
// that (s = 4, k = 10, 1e6 cells, the usual border and the wider one throughout:
// 16 steps, two launches with either, 18.3 and 21.7 us; 21 steps, three and one,
// 25.5 and 19.6; 50 steps, four and two, 46.6 and 45.8).
int gbox_steps_per_launch(const FractalHost &F, int32_t steps)
{
    if (!F.gbox) return -1;
    const GboxConfig &C = *F.gbox;
    return C.K2 && plan_launches(steps, C.K2).size() < plan_launches(steps, C.K).size() ? C.K2 : C.K;
}

sqz_status launch_life_gbox(const FractalHost &F, const uint8_t *in, uint8_t *out, int steps, hipStream_t st)
{
    const GboxConfig &C = *F.gbox;
    if (steps < 1 || (C.K && steps > std::max(C.K, C.K2)))
        return set_error(SQZ_ERR_UNSUPPORTED, "%d steps per launch exceed the border of %d cells", steps,
                         std::max(C.K, C.K2));
    const GboxArgs &A = C.K && steps > C.K ? C.A2 : C.A;
    if (A.ntiles <= kGbFewTiles) {
        const size_t lds = (gb_lds(A.W, gb_rows(A.rows, kGbFewStrip)) + 1) * sizeof(uint32_t);
        hipLaunchKernelGGL((k_life_gbox<kGbFewStrip, kGbFewNT>), dim3(A.ntiles), dim3(kGbFewNT), lds, st, A, in, out,
                           steps);
    } else {
        const size_t lds = (gb_lds(A.W, gb_rows(A.rows, 5)) + 1) * sizeof(uint32_t);
        hipLaunchKernelGGL((k_life_gbox<5, 64>), dim3(A.ntiles), dim3(64), lds, st, A, in, out, steps);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SQZ_OK : hip_error(e, "compact run (bit box) launch");
}

}  // namespace sqz
