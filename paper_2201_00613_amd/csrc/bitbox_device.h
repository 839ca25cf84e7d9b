// Block-level Squeeze (Section "Moving from Thread-level to Block-level")
// for Life on dense patterns of side s = 3 with at most 8 replicas (the
// Sierpinski carpet): the level-M subtree of a tile is expanded on chip into
// a box of bit rows, one bit per position, and Life runs on whole 32-bit row
// words.
//
// Tile  = a level-M subtree (M <= 5): compact cells [t k^M, (t+1) k^M), a
//         3^M x 3^M region of the expanded plane.
// Block = a level-1 subtree: k <= 8 consecutive compact cells in one 3 x 3
//         box, held as one byte of bits (bit j = replica j).
// Box   = the tile's blocks plus a border five blocks (fifteen cells) wide
//         from the eight adjacent tiles, as bit rows: row y, word w = columns
//         32w .. 32w+31.  Each step invalidates one more cell along the box
//         edge, so a launch takes up to fifteen steps (any number where the
//         fractal is one tile).
//
// Per tile: (A) each block's eight bytes are packed to one byte of bits and
// placed in a block grid (one byte per block position, tile-invariant
// positions); the border blocks within reach of the steps come from the
// adjacent tiles, whose bases are eight coarse nu per tile.  (B) Each 32-bit
// row word is assembled from the grid: the row's three bits of each block are cut
// out of four bytes at a time and packed together.
// (C) Life rounds in registers: a lane holds one word column of ten
// consecutive rows.  The words beside its own are in the lanes beside it
// (seven strips of nine words a wave, wave shifts), the rows above and below
// come from LDS, where every lane publishes its first and last row each round:
// two words written and two read per ten.  Bit-sliced full adders in
// three-input operations; new states are masked by the tile-invariant
// membership of each position and by whether the adjacent tile it lies in
// exists.  (D) The rows go back to the grid the same way, and each block's byte
// is unpacked to eight.
//
// Measured (level-9 carpet, 134 million cells): with the rows in LDS (36 words
// read and 10 written per lane and round) and a border of twelve cells, ten
// steps took 112 us and 30 steps, four launches, 400; now 61 us for one step,
// 107 for fifteen and 218 for 30.  A launch moves 2 B per cell and a quarter
// more for borders, 58 us at the rate of a large copy; a round is bound by
// vector issue (168 instructions a wave, 3.3 us), most of which comes on top:
// the tiles fill the chip twice, and the workgroups beside each other load and
// compute at about the same time.  Raised priority outside the rounds keeps
// loads and stores ahead of them (30 steps: 233 -> 218).  Loads held in
// registers over the table look-up cost more than they hide (63 -> 76 us for
// one step), as do fewer workgroups per CU (30 steps: five 9 % more, four 18 %).
#pragma once

#include "common.h"
#include "tile_device.h"

namespace sqz {

struct PatCarpet {  // Sierpinski carpet, replicas row by row
    static constexpr int S = 3, K = 8;
    static constexpr int OX[8] = {0, 1, 2, 0, 2, 0, 1, 2};
    static constexpr int OY[8] = {0, 0, 0, 1, 1, 2, 2, 2};
};

constexpr int kBxBorder = 5;                 // border blocks on each side
constexpr int kBxBC = 3 * kBxBorder;         // border cells on each side
constexpr int kBxMMax = 5;                   // tile level: 3^5 + 30 = 273 columns
// Rows are kBxW words; columns 273 .. 287 are always zero (outside every box,
// masked by membership), so word 8's right neighbour (word 0 of the next strip)
// and word 0's left neighbour (word 8 of the strip before) only ever shift
// zeros or masked columns into the box.
constexpr int kBxW = 9;                      // row words (288 columns)
constexpr int kBxSR = 10;                    // rows of one lane's strip
constexpr int kBxThreads = 256;
constexpr int kBxWaveStrips = 64 / kBxW;     // strips of a wave (63 lanes)
constexpr int kBxStrips = kBxThreads / 64 * kBxWaveStrips;  // 28
constexpr int kBxRows = kBxStrips * kBxSR;   // box rows (280); rows past the box stay zero
constexpr int kBxGR = 81 + 2 * kBxBorder;    // block-grid rows (and columns): 3^4 + 2 * 5
constexpr int kBxGP = 100;                   // bytes per block-grid row (a row of words reads 96)
// LDS words: the rows (and a word read past the last), then the block grid,
// whose place the published rows take: [parity][first, last][strip + 1][word].
constexpr int kBxEx = (kBxRows * kBxW + 1 + 3) / 4 * 4;
constexpr int kBxExW = 2 * 2 * (kBxStrips + 2) * kBxW;
constexpr int kBxNb = kBxEx + (kBxGR * kBxGP + 15) / 16 * 4;  // nine u64 bases, one flag word
constexpr int kBxLds = kBxNb + 20;
constexpr int kBxMaxSteps = kBxBC;           // Life steps per launch (fractals of more than one tile)
static_assert(kBxExW <= kBxNb - kBxEx, "the published rows take the place of the grid");
static_assert(kBxRows >= 3 * kBxGR && 32 * kBxW > 3 * kBxGR, "box fits the lanes");
static_assert(kBxLds * 4 <= 20 * 1024, "eight workgroups per CU");
static_assert(kBxGR * kBxGP < (1 << 14) && kBxGP >= 96, "ring slots; 24 words of a grid row");

struct BitboxConfig {
    int M;
    uint32_t tile;    // k^M cells
    uint32_t nblk;    // k^(M-1) blocks
    uint32_t side;    // 3^M
    uint32_t ring[kBxBorder + 1];  // border blocks within d blocks of the tile: ring[d]
    uint64_t ntiles;  // k^(r-M)
    uint16_t *d_gpos;    // [nblk] grid byte of each block
    uint32_t *d_ring;    // by distance: grid byte | direction << 14 | block index in that tile << 18
    uint32_t *d_member;  // [kBxRows][kBxW] membership of every box position, adjacent tiles present
    MapParams Pc;        // maps at the coarse level r-M
    void *d_coarse;
};

struct BitboxArgs {
    uint64_t ntiles;
    uint32_t tile, nblk, side;
    uint32_t nring[kBxBorder + 1];
    const uint16_t *gpos;
    const uint32_t *ring;
    const uint32_t *member;
    MapParams Pc;
};

inline BitboxArgs bitbox_args(const FractalHost &F)
{
    const BitboxConfig *C = F.bitbox;
    BitboxArgs A;
    A.ntiles = C->ntiles;
    A.tile = C->tile;
    A.nblk = C->nblk;
    A.side = C->side;
    for (int d = 0; d <= kBxBorder; ++d) A.nring[d] = C->ring[d];
    A.gpos = C->d_gpos;
    A.ring = C->d_ring;
    A.member = C->d_member;
    A.Pc = C->Pc;
    return A;
}

template <class Pat>
__host__ __device__ constexpr int replica_at(int x, int y)
{
    for (int j = 0; j < Pat::K; ++j)
        if (Pat::OX[j] == x && Pat::OY[j] == y) return j;
    return -1;
}

// Row Q of four blocks (one byte each): bit x of byte i = position (x, Q) of block i.
template <class Pat, int Q, int X = 0>
__device__ __forceinline__ uint32_t row_field(uint32_t d)
{
    if constexpr (X == 3) {
        return 0u;
    } else {
        constexpr int j = replica_at<Pat>(X, Q);
        uint32_t v = 0;
        if constexpr (j >= X)
            v = (d >> (j - X)) & (0x01010101u << X);
        else if constexpr (j >= 0)
            v = (d << (X - j)) & (0x01010101u << X);
        return v | row_field<Pat, Q, X + 1>(d);
    }
}

// Four 3-bit fields, one per byte -> twelve consecutive bits, and back.
__device__ __forceinline__ uint32_t compact12(uint32_t f)
{
    return __builtin_amdgcn_udot4(f, 0x00400801u, (f >> 15) & 0xE00u, false);
}
__device__ __forceinline__ uint32_t expand12(uint32_t v)
{
    v = (v & 0x3Fu) | ((v << 10) & 0x003F0000u);
    return (v | (v << 5)) & 0x07070707u;
}

// The bytes of four blocks from their rows (f[y]: bit x of byte i = position (x, y) of block i).
template <class Pat, int J = 0>
__device__ __forceinline__ uint32_t block_bytes(const uint32_t (&f)[3])
{
    if constexpr (J == Pat::K) {
        return 0u;
    } else {
        constexpr int x = Pat::OX[J], y = Pat::OY[J];
        return ((f[y] & (0x01010101u << x)) << (J - x)) | block_bytes<Pat, J + 1>(f);
    }
}

// Row 3R + Q of the box, words 3 w .. 3 w + 2, from the 32 blocks g of block row R there.
template <class Pat, int Q>
__device__ __forceinline__ void bx_rowwords(const uint32_t (&g)[8], uint32_t *row)
{
    uint32_t c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = compact12(row_field<Pat, Q>(g[i]));
    row[0] = c[0] | c[1] << 12 | c[2] << 24;
    row[1] = c[2] >> 8 | c[3] << 4 | c[4] << 16 | c[5] << 28;
    row[2] = c[5] >> 4 | c[6] << 8 | c[7] << 20;
}

// Columns [lo, hi) of the box that fall in word w, as a bit mask.
__device__ __forceinline__ uint32_t col_mask(int lo, int hi, int w)
{
    const int a = max(lo - 32 * w, 0), b = min(hi - 32 * w, 32);
    if (b <= a) return 0u;
    const uint32_t top = b == 32 ? 0xFFFFFFFFu : ((1u << b) - 1u);
    return top & ~((1u << a) - 1u);
}

// Life on one row word from three rows (each: the word and its two neighbours
// in the row).  Sums by full adders: the row above and below contribute
// three cells each (sum s3 + 2 c3), the row itself two (s2 + 2 c2).
struct BxRow {
    uint32_t s3, c3, s2, c2, c;
};

__device__ __forceinline__ BxRow bx_row(uint32_t L, uint32_t C, uint32_t R)
{
    const uint32_t W = __builtin_amdgcn_alignbit(C, L, 31), E = __builtin_amdgcn_alignbit(R, C, 1);
    BxRow v;
    v.s3 = __builtin_amdgcn_bitop3_b32(W, C, E, 0x96);  // sum
    v.c3 = __builtin_amdgcn_bitop3_b32(W, C, E, 0xE8);  // carry
    v.s2 = W ^ E;
    v.c2 = W & E;
    v.c = C;
    return v;
}

__device__ __forceinline__ BxRow bx_row(const uint32_t *p) { return bx_row(p[-1], p[0], p[1]); }

__device__ __forceinline__ uint32_t bx_life(const BxRow &u, const BxRow &m, const BxRow &d)
{
    const uint32_t x1 = __builtin_amdgcn_bitop3_b32(u.s3, m.s2, d.s3, 0x96),
                   k1 = __builtin_amdgcn_bitop3_b32(u.s3, m.s2, d.s3, 0xE8);
    // count = x1 + 2 (c3 above + c2 + c3 below + k1): 2 or 3 iff exactly one of the four carries
    const uint32_t none = __builtin_amdgcn_bitop3_b32(u.c3, m.c2, d.c3, 0x01),
                   one = __builtin_amdgcn_bitop3_b32(u.c3, m.c2, d.c3, 0x16);
    const uint32_t two = __builtin_amdgcn_bitop3_b32(k1, none, one, 0xCA);  // k1 ? none : one
    return __builtin_amdgcn_bitop3_b32(two, x1, m.c, 0xE0);                 // two & (x1 | c)
}

// The row word and its neighbours, which the lanes beside hold.
__device__ __forceinline__ BxRow bx_wave_row(uint32_t C)
{
    const uint32_t L = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)C, 0x138, 0xF, 0xF, true),  // from lane - 1
        R = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)C, 0x130, 0xF, 0xF, true);             // from lane + 1
    return bx_row(L, C, R);
}

// One tile, `steps` steps (phases A to D); sm: kBxLds words.  Called by every
// lane of a workgroup of kBxThreads lanes.  Prio: loads and stores before the
// rounds of other workgroups (not beside other kinds of tiles, which wait then).
template <class Pat, bool Prio = true>
__device__ __forceinline__ void bitbox_tile(const BitboxArgs &A, const uint8_t *__restrict__ in,
                                            uint8_t *__restrict__ out, uint64_t t, int32_t steps, uint32_t *sm)
{
    uint32_t *const ex = sm + kBxEx;
    uint8_t *const G = reinterpret_cast<uint8_t *>(ex);
    uint64_t *const s_nb = reinterpret_cast<uint64_t *>(sm + kBxNb);
    uint32_t *const s_there = sm + kBxNb + 18;
    const uint32_t tid = threadIdx.x, wl = tid & 63u;
    // word column and strip of rows kBxSR ls .. kBxSR ls + kBxSR - 1 (a wave's last lane idles in phase C)
    const bool act = wl < (uint32_t)(kBxW * kBxWaveStrips);
    const int lw = act ? (int)(wl % kBxW) : 0, ls = act ? (int)((tid >> 6) * kBxWaveStrips + wl / kBxW) : 0;
    const int side = (int)A.side;
    const uint64_t base = t * A.tile;
    const uint32_t grow = A.side / 3 + 2 * kBxBorder;  // block-grid rows in use
    if constexpr (Prio) __builtin_amdgcn_s_setprio(3);
    // membership of this lane's words with the adjacent tiles present (tile-invariant table)
    uint32_t eff[kBxSR];
#pragma unroll
    for (int r = 0; r < kBxSR; ++r) eff[r] = act ? A.member[(kBxSR * ls + r) * kBxW + lw] : 0u;
    if (tid < 64) {
        bool here = false;
        if (tid < 9) {
            uint32_t X, Y;
            if (A.Pc.N <= 0x100000000ull)
                lam_map32(A.Pc, (uint32_t)t, X, Y);
            else
                lam_map64(A.Pc, t, X, Y);
            const uint64_t nt =
                nu_map(A.Pc, (int32_t)X + (int32_t)(tid % 3) - 1, (int32_t)Y + (int32_t)(tid / 3) - 1);
            s_nb[tid] = nt == kHole64 ? kHole64 : nt * A.tile;
            here = nt != kHole64;
        }
        const uint64_t m = __ballot(here);
        if (tid == 0) *s_there = (uint32_t)m;
    }
    for (uint32_t i = tid; i < (uint32_t)(kBxNb - kBxEx); i += kBxThreads) ex[i] = 0;
    __syncthreads();

    // (A) the tile's blocks and the border blocks into the grid
#pragma unroll 4
    for (uint32_t b = tid; b < A.nblk; b += kBxThreads) {
        const uint2 d = *reinterpret_cast<const uint2 *>(in + base + 8ull * b);
        G[A.gpos[b]] = (uint8_t)pack8(d.x, d.y);
    }
    const uint32_t nring = A.nring[steps < kBxBC ? (steps + 2) / 3 : kBxBorder];
    for (uint32_t i = tid; i < nring; i += kBxThreads) {
        const uint32_t slot = A.ring[i];
        const uint64_t nb = s_nb[(slot >> 14) & 15u];
        if (nb != kHole64) {
            const uint2 d = *reinterpret_cast<const uint2 *>(in + nb + 8ull * (slot >> 18));
            G[slot & 0x3FFFu] = (uint8_t)pack8(d.x, d.y);
        }
    }
    const uint32_t there = *s_there;
    __syncthreads();

    // (B) row words from the grid: unit (block row R, three words) from 32 blocks
    for (uint32_t u = tid; u < grow * (kBxW / 3); u += kBxThreads) {
        const uint32_t R = u / 3, w = u - 3 * R;
        uint32_t g[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) g[i] = ex[R * (kBxGP / 4) + 8 * w + i];
        uint32_t *const row = sm + 3 * R * kBxW + 3 * w;
        bx_rowwords<Pat, 0>(g, row);
        bx_rowwords<Pat, 1>(g, row + kBxW);
        bx_rowwords<Pat, 2>(g, row + 2 * kBxW);
    }
    {
        const uint32_t mL = col_mask(0, kBxBC, lw), mC = col_mask(kBxBC, kBxBC + side, lw),
                       mR = col_mask(kBxBC + side, 2 * kBxBC + side, lw);
#pragma unroll
        for (int r = 0; r < kBxSR; ++r) {
            const int y = kBxSR * ls + r, ry = y < kBxBC ? 0 : (y < kBxBC + side ? 1 : 2);
            const uint32_t e3 = there >> (3 * ry);
            eff[r] &= ((e3 & 1u) ? mL : 0u) | ((e3 & 2u) ? mC : 0u) | ((e3 & 4u) ? mR : 0u);
        }
    }
    __syncthreads();

    // (C) the rounds, behind the loads and stores of the workgroups beside
    if constexpr (Prio) __builtin_amdgcn_s_setprio(0);
    uint32_t x[kBxSR];
    uint32_t *const mine = sm + kBxSR * ls * kBxW + lw;
#pragma unroll
    for (int r = 0; r < kBxSR; ++r) x[r] = act && kBxSR * ls + r < (int)(3 * grow) ? mine[r * kBxW] : 0u;
    constexpr int kRow = (kBxStrips + 2) * kBxW, kPar = 2 * kRow;
    if (tid < 4 * kBxW) {  // above the first strip and below the last
        const uint32_t q = tid / kBxW;
        ex[(q >> 1) * kPar + ((q & 1u) ? (kBxStrips + 1) * kBxW : kRow) + tid % kBxW] = 0;
    }
    uint32_t *e = ex + (ls + 1) * kBxW + lw;  // this lane's first row; kRow further its last
    int par = kPar;
#pragma unroll 1
    for (int32_t j = 0; j < steps; ++j) {
        if (act) {
            e[0] = x[0];
            e[kRow] = x[kBxSR - 1];
        }
        __syncthreads();
        const uint32_t above = e[kRow - kBxW], below = e[kBxW];
        BxRow up = bx_wave_row(above), mid = bx_wave_row(x[0]);
#pragma unroll
        for (int r = 0; r < kBxSR; ++r) {
            const BxRow dn = bx_wave_row(r + 1 < kBxSR ? x[r + 1 < kBxSR ? r + 1 : 0] : below);
            x[r] = bx_life(up, mid, dn) & eff[r];
            up = mid;
            mid = dn;
        }
        e += par;
        par = -par;
    }

    // (D) rows -> block grid (unit: block row R of the tile, four columns) -> bytes
    if constexpr (Prio) __builtin_amdgcn_s_setprio(3);
    if (act) {
#pragma unroll
        for (int r = 0; r < kBxSR; ++r) mine[r * kBxW] = x[r];
    }
    __syncthreads();
    const uint32_t nb = A.side / 3;
    constexpr uint32_t NC4 = (kBxBorder + 81 + 3) / 4 - kBxBorder / 4;  // grid words with columns of a tile
    for (uint32_t u = tid; u < nb * NC4; u += kBxThreads) {
        const uint32_t R = u / NC4 + kBxBorder, i = u % NC4 + kBxBorder / 4;
        const uint32_t *rp = sm + 3 * R * kBxW + (3 * i >> 3);
        uint32_t f[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
            f[q] = expand12(__builtin_amdgcn_alignbit(rp[q * kBxW + 1], rp[q * kBxW], 4 * (3 * i & 7u)));
        ex[R * (kBxGP / 4) + i] = block_bytes<Pat>(f);
    }
    __syncthreads();
#pragma unroll 4
    for (uint32_t b = tid; b < A.nblk; b += kBxThreads) {
        const uint32_t v = G[A.gpos[b]];
        uint2 o2;
        o2.x = spread4(v & 15u);
        o2.y = spread4(v >> 4);
        *reinterpret_cast<uint2 *>(out + base + 8ull * b) = o2;
    }
}

}  // namespace sqz
