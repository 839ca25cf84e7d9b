// Block-level Squeeze (Section "Moving from Thread-level to Block-level") for
// Life on compact storage, bit-sliced across subtrees.
//
// Work decomposition
//   tile    = a level-M subtree, one workgroup.
//   subtile = one of the tile's k^B level-L subtrees (L = M - B, k^B <= 32).
//   word    = one cell position of the subtile for all k^B subtiles at once:
//             bit j of word i is cell i of subtile j.  Subtiles share one
//             geometry, so inside a subtile the neighbours of word i are whole
//             words: no shift, mask or single-bit move is needed, and the rule
//             is full adders on words (one v_bitop3_b32 per sum or carry).
//   block   = a level-J subtree of words (k^J of them), held in the registers
//             of one lane for all steps.  In-block neighbours are registers;
//             the few cells of adjacent blocks it touches (its halo) are words
//             those lanes publish in LDS each step.
// Where a block's halo leaves the subtile, the neighbour lies in another
// subtile: the same cell position with the bits permuted.  Those few words
// ("subtile halo", one per cell adjacent to a subtile) are rebuilt each step
// by the first wave: one lane per (word, bit) reads its source bit and a
// ballot packs 64 of them.
// Cells outside the tile: the few level-RL subtrees of adjacent tiles that
// hold the cells within K steps of the tile (triangle: six subtrees, K = 31)
// form a second, small set of words (bit s = ring subtree s), advanced by
// lanes of their own with the same code.  Each step the outermost cells of
// these subtrees become invalid one cell further in; K steps never reach the
// tile.
//
// Why: the bit-sliced blocks of tile_device.h hold 27 cells of one block in a
// word and pay 62 vector instructions per 27 cells and step, nearly all of
// them moving bits.  Here the triangle needs 45 per 9 words (J = 2) or 121 per
// 27 words (J = 3), each word 27 cells: 0.17-0.19 instructions per cell.
// Measured against those blocks: level-16 triangle, 100 steps, all tiles
// resident: 333 -> 62 us; level 20, 20 steps: two launches of ten (4.68 ms,
// bound by vector issue) -> one in place (1.51 ms, 4.6 TB/s of loads and
// stores, the rate of a large copy); level 13, 25 steps: 23.5 -> 12.0 us;
// level-9 Vicsek cross, 37 steps: 43.4 -> 16.5 us.
#pragma once

#include <algorithm>
#include <utility>

#include "common.h"
#include "tile_device.h"

namespace sqz {

// Bit level B (k^B subtiles per tile), ring level RL, block level J and largest
// subtile level LMAX of a kernel.  STEPS: steps the ring subtrees cover, that
// is, the distance (along member cells outside the tile) up to which every cell
// lies in the level-RL subtrees that hold the cells next to the tile: one step
// less than their side for the triangles, whose next subtrees touch at a
// corner, their side for the Vicsek cross.  *Small: subtiles of at most 243 (625) words,
// always loaded four cells a lane (fewer registers and less LDS, so more
// workgroups per CU: batches).  PARTS: see publish() in slice_tile.
struct SliceTri : PatTriangle {
    static constexpr int B = 3, RL = 5, STEPS = 31, J = 2, LMAX = 8;
    static constexpr bool SMALL = false, PARTS = true;
};
struct SliceTriSmall : SliceTri {
    static constexpr int LMAX = 5;
    static constexpr bool SMALL = true;
};
struct SliceTriWide : SliceTri {
    static constexpr int J = 3;
    static constexpr bool PARTS = false;
};
struct SlicePaper : PatTrianglePaper {
    static constexpr int B = 3, RL = 5, STEPS = 31, J = 2, LMAX = 8;
    static constexpr bool SMALL = false, PARTS = true;
};
struct SlicePaperSmall : SlicePaper {
    static constexpr int LMAX = 5;
    static constexpr bool SMALL = true;
};
struct SlicePaperWide : SlicePaper {
    static constexpr int J = 3;
    static constexpr bool PARTS = false;
};
struct SliceVicsek : PatVicsek {
    static constexpr int B = 2, RL = 3, STEPS = 27, J = 1, LMAX = 5;
    static constexpr bool SMALL = false, PARTS = false;
};
struct SliceVicsekSmall : SliceVicsek {
    static constexpr int LMAX = 4;
    static constexpr bool SMALL = true, PARTS = true;
};
struct SliceVicsekWide : SliceVicsek {
    static constexpr int J = 2;
};

// ---------------------------------------------------------------------------
// Compile-time neighbour lists of a level-J block.
// ---------------------------------------------------------------------------
struct SlicePlan {
    int nc, box;
    int lx[32], ly[32];
    int deg[32];
    int nb[32][8];  // < nc: cell of the block; nc + h: halo slot h
    int nh;         // halo slots: cell h_idx of the adjacent block in direction (h_dx, h_dy)
    int h_dx[kMaxHalo], h_dy[kMaxHalo], h_idx[kMaxHalo];
    int ne;         // published cells of a block: those some adjacent block reads
    int e_cell[32];
    int h_exp[kMaxHalo];  // published slot of the halo cell in its own block
    bool ok;
};

template <class P, int J>
constexpr int slice_local_nu(int x, int y)
{
    int c = 0;
    for (int mu = J; mu >= 1; --mu) {
        const int sc = cpow(P::S, mu - 1);
        const int qx = (x / sc) % P::S, qy = (y / sc) % P::S;
        int j = -1;
        for (int i = 0; i < P::K; ++i)
            if (P::OX[i] == qx && P::OY[i] == qy) j = i;
        if (j < 0) return -1;
        c += j * cpow(P::K, mu - 1);
    }
    return c;
}

template <class P, int J>
constexpr SlicePlan derive_slice_plan()
{
    SlicePlan p{};
    p.ok = true;
    p.nc = cpow(P::K, J);
    p.box = cpow(P::S, J);
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
    }
    for (int pass = 0; pass < 2; ++pass)  // in-block neighbours first, then halo words (they arrive last)
        for (int i = 0; i < p.nc; ++i)
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    if (!dx && !dy) continue;
                    const int qx = p.lx[i] + dx, qy = p.ly[i] + dy;
                    const int bx = qx < 0 ? -1 : (qx >= p.box ? 1 : 0), by = qy < 0 ? -1 : (qy >= p.box ? 1 : 0);
                    const int j = slice_local_nu<P, J>(qx - bx * p.box, qy - by * p.box);
                    if (j < 0 || (pass == 0) != (bx == 0 && by == 0)) continue;
                    if (pass == 0) {
                        p.nb[i][p.deg[i]++] = j;
                        continue;
                    }
                    int h = -1;
                    for (int q = 0; q < p.nh; ++q)
                        if (p.h_dx[q] == bx && p.h_dy[q] == by && p.h_idx[q] == j) h = q;
                    if (h < 0) {
                        if (p.nh == kMaxHalo) {
                            p.ok = false;
                            return p;
                        }
                        h = p.nh++;
                        p.h_dx[h] = bx;
                        p.h_dy[h] = by;
                        p.h_idx[h] = j;
                    }
                    p.nb[i][p.deg[i]++] = p.nc + h;
                }
    for (int i = 0; i < p.nc; ++i)
        for (int h = 0; h < p.nh; ++h)
            if (p.h_idx[h] == i) {
                if (p.ne == 0 || p.e_cell[p.ne - 1] != i) p.e_cell[p.ne++] = i;
                p.h_exp[h] = p.ne - 1;
            }
    return p;
}

template <class P, int J>
struct SlicePlanOf {
    static constexpr SlicePlan value = derive_slice_plan<P, J>();
    static_assert(value.ok, "block halo too large");
};

constexpr int kSliceMaxRing = 8;  // ring subtrees per tile

// LDS of one workgroup: two buffers of published words, or (at the load and
// the store) the words of the tile and its ring.  Byte offsets in a buffer:
// a zero word, the published words of every block (odd pitch, so that lanes
// of consecutive blocks hit different banks), the subtile halo, the ring
// subtrees' halo.
template <class P>
struct SliceCfg {
    static constexpr int J = P::J;
    static constexpr const SlicePlan &PL = SlicePlanOf<P, J>::value;
    static constexpr int KB = cpow(P::K, P::B);
    static constexpr int NG = (KB + 7) / 8;  // byte groups of a word
    static constexpr int PE = PL.ne | 1;
    static constexpr int MAXBLK = cpow(P::K, P::LMAX - J), MAXRBLK = cpow(P::K, P::RL - J);
    static constexpr int LANES = (MAXBLK + MAXRBLK + 63) / 64 * 64;
    static constexpr uint32_t ZERO = 0, EX0 = 16, PITCH = PE * 4;
    static constexpr uint32_t HALO = (EX0 + (MAXBLK + MAXRBLK) * PITCH + 15) / 16 * 16;
    static constexpr uint32_t RHALO = HALO + 4 * PL.nh;
    static constexpr uint32_t BUF = (RHALO + 4 * PL.nh + 255) / 256 * 256;
    static constexpr uint32_t STAGE = 4 * (MAXBLK + MAXRBLK) * PL.nc;
    static constexpr uint32_t LDS = 2 * BUF > STAGE ? 2 * BUF : STAGE;
    static constexpr int NPT = (PL.nh * 32 + 63) / 64;  // ballots of the subtile halo; one more for the ring's
    static_assert(KB <= 32 && PL.nh * kSliceMaxRing <= 64 && PL.nh <= 8, "one ballot holds the ring halo");
    static_assert(MAXRBLK + 8 <= 64, "ring lanes and corner lanes share the first wave");
};

struct SliceArgs {
    uint64_t ntiles;
    uint32_t cells;   // per tile
    uint32_t words;   // per subtile
    uint32_t nblk, lanes;  // blocks of a subtile; lanes in use (with the ring's)
    uint32_t rwords, nring, ncorner;
    uint32_t ring_corner[kSliceMaxRing];  // ring subtree s is this corner subtree of its tile
    uint32_t ring_off[kSliceMaxRing];     // and begins at this cell of it
    uint32_t corner_off[kSliceMaxRing];   // first cell of each corner subtree
    const uint32_t *lane_block;  // [lanes] block of each lane (nblk and up: ring blocks)
    const uint32_t *lane_halo;   // [lanes][nh] LDS offsets of its halo words in a buffer
    const uint32_t *perm;        // [NPT + 1][64] source of each halo bit: offset | bit << 16 | ring subtree << 24
    const uint32_t *nbtile;      // [ntiles][kSliceMaxRing] adjacent tile of each ring subtree, kNuHole32 if none
};

// ---------------------------------------------------------------------------
// Rule
// ---------------------------------------------------------------------------
template <int LUT>
__device__ __forceinline__ uint32_t bop3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, LUT);
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return bop3<0x96>(a, b, c); }
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) { return bop3<0xE8>(a, b, c); }

// Sums of a cell's first neighbour words, which lie in its block.
struct SlicePart {
    uint32_t a, b, c;
};

// Of D neighbours the first IN in the block: how many the part covers (all of
// them: the part is the new state).
constexpr int slice_known(int D, int IN) { return IN == D ? D : (IN >= 5 ? 5 : (IN >= 3 ? 3 : 0)); }

// B3/S23 of a word x with D neighbour words n: alive' = (count == 3) | (x & count == 2), that is exactly
// one weight-2 carry and (odd rest or alive).  KNOWN = 3 or 5: the sums of that many neighbours are in `part`.
template <int D, int KNOWN = 0>
__device__ __forceinline__ uint32_t slice_rule(uint32_t x, const uint32_t *n, const SlicePart &part = SlicePart{})
{
    if constexpr (D < 2) {
        return 0u;
    } else if constexpr (D == 2) {
        return bop3<0x80>(n[0], n[1], x);
    } else {
        const uint32_t s1 = KNOWN >= 3 ? part.a : xor3(n[0], n[1], n[2]), c1 = KNOWN >= 3 ? part.b : maj3(n[0], n[1], n[2]);
        if constexpr (D == 3) {
            return bop3<0xE0>(c1, s1, x);  // c1 & (s1 | x)
        } else if constexpr (D == 4) {
            return bop3<0x78>(c1, s1, n[3]) & bop3<0xBE>(s1, n[3], x);  // (c1 ^ s1 n3) & ((s1 ^ n3) | x)
        } else {
            const uint32_t s2 = KNOWN == 5 ? part.a : xor3(s1, n[3], n[4]), c2 = KNOWN == 5 ? part.c : maj3(s1, n[3], n[4]);
            if constexpr (D == 5) {
                return bop3<0x28>(c1, c2, s2 | x);  // (c1 ^ c2) & (s2 | x)
            } else if constexpr (D == 6) {
                return bop3<0x16>(c1, c2, s2 & n[5]) & bop3<0xBE>(s2, n[5], x);
            } else {
                const uint32_t s3 = xor3(s2, n[5], n[6]), c3 = maj3(s2, n[5], n[6]);
                static_assert(D == 7, "no pattern here has a cell with eight neighbours");
                return bop3<0xE0>(bop3<0x16>(c1, c2, c3), s3, x);
            }
        }
    }
}

template <class P, int J, int I>
constexpr int slice_in_block()
{
    using PO = SlicePlanOf<P, J>;
    int in = 0;
    for (int d = 0; d < PO::value.deg[I]; ++d) in += PO::value.nb[I][d] < PO::value.nc;
    return in;
}

// The part of cell I from its own block's words.
template <class P, int J, int I, int NC>
__device__ __forceinline__ SlicePart slice_part(const uint32_t (&x)[NC])
{
    using PO = SlicePlanOf<P, J>;
    constexpr int D = PO::value.deg[I], KNOWN = slice_known(D, slice_in_block<P, J, I>());
    uint32_t n[8];
#pragma unroll
    for (int d = 0; d < KNOWN; ++d) n[d] = x[PO::value.nb[I][d]];
    SlicePart p{};
    if constexpr (KNOWN == D) {
        p.a = slice_rule<D>(x[I], n);
    } else if constexpr (KNOWN >= 3) {
        p.a = xor3(n[0], n[1], n[2]);
        p.b = maj3(n[0], n[1], n[2]);
        if constexpr (KNOWN == 5) {
            p.c = maj3(p.a, n[3], n[4]);
            p.a = xor3(p.a, n[3], n[4]);
        }
    }
    // computed here, not where it is used
    if constexpr (KNOWN > 0) asm volatile("" : "+v"(p.a));
    if constexpr (KNOWN > 0 && KNOWN != D) asm volatile("" : "+v"(p.b));
    if constexpr (KNOWN == 5 && KNOWN != D) asm volatile("" : "+v"(p.c));
    return p;
}

template <class P, int J, int I, bool PARTS, int NC, int NH>
__device__ __forceinline__ uint32_t slice_cell(const uint32_t (&x)[NC], const uint32_t (&h)[NH], const SlicePart &part)
{
    using PO = SlicePlanOf<P, J>;
    constexpr int D = PO::value.deg[I], KNOWN = PARTS ? slice_known(D, slice_in_block<P, J, I>()) : 0;
    if constexpr (PARTS && KNOWN == D) {
        return part.a;
    } else {
        uint32_t n[8];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int q = PO::value.nb[I][d];
            n[d] = q < NC ? x[q < NC ? q : 0] : h[q < NC ? 0 : q - NC];
        }
        return slice_rule<D, KNOWN>(x[I], n, part);
    }
}

template <class P, int J, int NC, size_t... I>
__device__ __forceinline__ void slice_parts(const uint32_t (&x)[NC], SlicePart (&part)[NC], std::index_sequence<I...>)
{
    ((part[I] = slice_part<P, J, (int)I>(x)), ...);
}

template <class P, int J, bool PARTS, int NC, int NH, size_t... I>
__device__ __forceinline__ void slice_step(uint32_t (&x)[NC], const uint32_t (&h)[NH], const SlicePart (&part)[NC],
                                           std::index_sequence<I...>)
{
    const uint32_t y[] = {slice_cell<P, J, (int)I, PARTS>(x, h, part[I])...};
    ((x[I] = y[I]), ...);
}

// ---------------------------------------------------------------------------
// Load and store: bytes <-> words.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32_u __attribute__((aligned(1)));

// Four dwords whose byte k belongs to cell k and byte group g -> four words
// (and back: the 4 x 4 byte transpose is its own inverse).
__device__ __forceinline__ void transpose4(const uint32_t (&a)[4], uint32_t (&w)[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), t1 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
    const uint32_t u0 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u), u1 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(u0, t0, 0x05040100u);
    w[1] = __builtin_amdgcn_perm(u0, t0, 0x07060302u);
    w[2] = __builtin_amdgcn_perm(u1, t1, 0x05040100u);
    w[3] = __builtin_amdgcn_perm(u1, t1, 0x07060302u);
}

// Q * 4 consecutive cells of every subtile from word i0 on.  The subtiles'
// bytes start at odd addresses: the loads are unaligned, contiguous over the
// lanes.
template <class C, int Q>
__device__ __forceinline__ void slice_load_words(const uint8_t *__restrict__ src, uint32_t words, uint32_t i0,
                                                 uint32_t *stage)
{
    uint32_t acc[C::NG][Q];
#pragma unroll
    for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[g][q] = 0;
#pragma unroll
    for (int j = 0; j < C::KB; ++j) {
        const uint8_t *p = src + (size_t)(j * words) + i0;
        uint32_t v[Q];
        if constexpr (Q == 4) {
            const u32x4_u z = *reinterpret_cast<const u32x4_u *>(p);
            v[0] = z.x, v[1] = z.y, v[2] = z.z, v[3] = z.w;
        } else {
            v[0] = *reinterpret_cast<const u32_u *>(p);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[j >> 3][q] |= v[q] << (j & 7);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t a[4] = {0u, 0u, 0u, 0u}, w[4];
#pragma unroll
        for (int g = 0; g < C::NG; ++g) a[g] = acc[g][q];
        transpose4(a, w);
#pragma unroll
        for (int k = 0; k < 4; ++k) stage[i0 + 4 * q + k] = w[k];
    }
}

// NTS: nontemporal stores.
template <class C, int Q, bool NTS>
__device__ __forceinline__ void slice_store_words(uint8_t *__restrict__ dst, uint32_t words, uint32_t i0,
                                                  const uint32_t *stage)
{
    uint32_t acc[4][Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        uint32_t w[4], a[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = stage[i0 + 4 * q + k];
        transpose4(w, a);
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g][q] = a[g];
    }
#pragma unroll
    for (int j = 0; j < C::KB; ++j) {
        uint8_t *p = dst + (size_t)(j * words) + i0;
        uint32_t v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = (acc[j >> 3][q] >> (j & 7)) & 0x01010101u;
        if constexpr (Q == 4) {
            const u32x4_u z = {v[0], v[1], v[2], v[3]};
            if constexpr (NTS)
                __builtin_nontemporal_store(z, reinterpret_cast<u32x4_u *>(p));
            else
                *reinterpret_cast<u32x4_u *>(p) = z;
        } else {
            *reinterpret_cast<u32_u *>(p) = v[0];
        }
    }
}

// Where the ring subtrees are read: in the compact array itself, or (updates in
// place) in a copy of every tile's corner subtrees, kSliceCornerPitch bytes each.
struct SliceRing {
    const uint8_t *base;
    bool copied;
};
constexpr uint32_t kSliceCornerPitch = 256;

// Four cells of every ring subtree from word i0 on.
__device__ __forceinline__ void slice_load_ring(const SliceArgs &A, const SliceRing &G, const uint32_t *nbt,
                                                uint32_t i0, uint32_t *stage)
{
    const uint64_t stride = G.copied ? (uint64_t)A.ncorner * kSliceCornerPitch : A.cells;
    uint32_t a[4] = {0u, 0u, 0u, 0u}, w[4];
#pragma unroll
    for (uint32_t s = 0; s < (uint32_t)kSliceMaxRing; ++s)
        if (s < A.nring && nbt[s] != kNuHole32)
            a[0] |= *reinterpret_cast<const u32_u *>(G.base + nbt[s] * stride +
                                                     (G.copied ? A.ring_corner[s] * kSliceCornerPitch : A.ring_off[s]) + i0)
                    << s;
    transpose4(a, w);
#pragma unroll
    for (int k = 0; k < 4; ++k) stage[i0 + k] = w[k];
}

// ---------------------------------------------------------------------------
// Resident form: all tiles on the chip at once, ring subtrees exchanged every
// K steps.  A tile's corner subtrees (those other tiles hold as ring
// subtrees) go out as one word per lane and corner: the block's bits and, in
// the bits above them, the exchange's epoch.  A reader polls the word itself
// until it carries the epoch it expects, so an exchange is one store and one
// load of device-scope latency, with no counter, flag or fence, and a tile
// waits for its own neighbours only.  Two copies alternate: a tile writes
// exchange n + 2 only after it has read exchange n + 1 of its neighbours,
// which they wrote after reading its exchange n (adjacency is symmetric).  A
// copy's previous epoch is always two back, so the few bits of it that fit
// above a block's tell it from the one awaited.  Epochs carry over from run to
// run in one word per tile, so no launch has to clear anything and replays of
// a captured run stay in step.
// ---------------------------------------------------------------------------
struct SliceRes {
    uint32_t *xch;    // [2][ntiles][ncorner][rblk]
    uint32_t *epoch;  // [ntiles] exchanges of earlier runs
    uint32_t *loaded; // [ntiles] runs whose start the tile has read
    uint32_t *dead;   // a wait timed out
    uint32_t *flag;   // the same, host-visible
    uint32_t K;       // steps between exchanges
};

// Waits until ready() holds for every active lane, for at most kSpinLimit polls
// and no longer than until another wait of the run has given up (`dead`).  Giving
// up marks the run as timed out and returns, so that every wave ends.
template <class F>
__device__ __forceinline__ void slice_wait(const SliceRes &R, F &&ready)
{
    for (uint32_t spin = 0;; ++spin) {
        if (ready()) break;
        const bool gone =
            (spin & 255u) == 255u && __hip_atomic_load(R.dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        if (gone || spin == kSpinLimit) {
            __hip_atomic_store(R.dead, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(R.flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// One tile, `steps` >= 1 steps (at most K without RES; any number when the
// fractal is one tile).  in, out: the whole compact arrays, the same one for
// an update in place.  tid, NT: this lane and the lanes (whole waves) of the tile;
// several tiles of one launch may share a workgroup, since the barriers depend on
// `steps` alone.  Every lane of the workgroup calls it.
template <class P, bool RES>
__device__ __forceinline__ void slice_tile(const SliceArgs &A, const uint8_t *in, uint8_t *out, uint64_t t,
                                           const SliceRing &G, int32_t steps, const SliceRes &R, uint32_t *sm,
                                           const uint32_t tid, const uint32_t NT)
{
    using C = SliceCfg<P>;
    constexpr int J = C::J;
    using PO = SlicePlanOf<P, J>;
    constexpr int NC = PO::value.nc, NH = PO::value.nh, NE = PO::value.ne, NPT = C::NPT;
    const uint32_t rblk = A.rwords / NC;
    const bool active = tid < A.lanes;
    const uint32_t *nbt = A.nbtile + t * kSliceMaxRing;

    const uint32_t blk = active ? A.lane_block[tid] : 0u;
    uint32_t ha[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) ha[h] = active ? A.lane_halo[tid * NH + h] : C::ZERO;
    // the first wave's halo sources: LDS offset and bit mask (0: no cell there)
    const bool wave0 = __builtin_amdgcn_readfirstlane(tid) == 0;
    uint32_t pa[NPT + 1], pm[NPT + 1];
#pragma unroll
    for (int p = 0; p <= NPT; ++p) pa[p] = C::ZERO, pm[p] = 0;
    if (wave0) {
#pragma unroll
        for (int p = 0; p <= NPT; ++p) {
            const uint32_t e = A.perm[p * 64 + tid], s = e >> 24;
            pa[p] = e & 0xFFFFu;
            pm[p] = 1u << ((e >> 16) & 31u);
            if (pa[p] == C::ZERO || (s < (uint32_t)kSliceMaxRing && nbt[s] == kNuHole32)) pm[p] = 0;
        }
    }
    uint32_t epoch = 0, run = 0;
    if constexpr (RES) {
        epoch = __hip_atomic_load(R.epoch + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        run = 1 + __hip_atomic_load(R.loaded + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // load: words of the tile, then of the ring, into the staging area
    {
        const uint8_t *src = in + t * A.cells;
        const uint32_t rt = A.nring ? (A.rwords + 3) / 4 : 0u;
        // four cells per task where that fills the lanes in one pass, else sixteen
        if (P::SMALL || A.words <= 4 * NT) {
            const uint32_t n = (A.words + 3) / 4;
            for (uint32_t k = tid; k < n; k += NT)
                slice_load_words<C, 1>(src, A.words, 4 * k + 4 <= A.words ? 4 * k : A.words - 4, sm);
        } else if constexpr (!P::SMALL) {
            const uint32_t n = (A.words + 15) / 16;
            for (uint32_t k = tid; k < n; k += NT)
                slice_load_words<C, 4>(src, A.words, 16 * k + 16 <= A.words ? 16 * k : A.words - 16, sm);
        }
        // the ring's tasks go to the last lanes, which have the fewest of the above
        for (uint32_t k = NT - 1 - tid; k < rt; k += NT)
            slice_load_ring(A, G, nbt, 4 * k + 4 <= A.rwords ? 4 * k : A.rwords - 4, sm + A.words);
    }
    __syncthreads();
    if constexpr (RES) {  // this tile's start has been read (every lane holds `run` by now)
        if (tid == 0) __hip_atomic_store(R.loaded + t, run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    uint32_t x[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) x[c] = active ? sm[blk * NC + c] : 0u;
    __syncthreads();

    char *const lds = reinterpret_cast<char *>(sm);
    char *const ex = lds + C::EX0 + blk * C::PITCH;
    SlicePart part[NC];
    // Publish into buffer p: the block's cells that other blocks read, then
    // (first wave, whose lanes hold every source) the subtile and ring halos.
    // The other waves wait for that chain of LDS accesses and ballots: with
    // PARTS they meanwhile add up each cell's neighbours in its own block, and
    // a step's second half is the halo words alone (100 steps: level-16
    // triangle 69.7 -> 66.3 us, level 8 34.8 -> 33.5, level-6 Vicsek 28.6 -> 27.2).
    // Not where the sums cost more registers than they save time (27-cell
    // blocks).  In the first wave they come after
    // the chain: between its reads and ballots they lengthen it (level 8 36.0),
    // and so does raised priority for that wave (level 16 69.8).
    auto publish = [&](auto pp) {
        constexpr uint32_t O = decltype(pp)::value * C::BUF;
        if (active) {
#pragma unroll
            for (int e = 0; e < NE; ++e) *reinterpret_cast<uint32_t *>(ex + O + 4 * e) = x[PO::value.e_cell[e]];
        }
        if (wave0) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint32_t v[NPT + 1];
#pragma unroll
            for (int p = 0; p <= NPT; ++p) v[p] = *reinterpret_cast<const uint32_t *>(lds + O + pa[p]);
            uint64_t b[NPT + 1];
#pragma unroll
            for (int p = 0; p <= NPT; ++p) b[p] = __ballot((v[p] & pm[p]) != 0);
            // lane h < NH: subtile halo word h; lane NH + h: the ring's
            uint32_t w = 0;
#pragma unroll
            for (int h = 0; h < NH; ++h)
                if (tid == (uint32_t)h) w = (uint32_t)(b[h >> 1] >> (32 * (h & 1)));
            if (tid >= (uint32_t)NH) w = (uint32_t)(b[NPT] >> ((tid - NH) * kSliceMaxRing & 63u)) & 0xFFu;
            if (tid < 2u * NH) *reinterpret_cast<uint32_t *>(lds + O + C::HALO + 4 * tid) = w;
        }
        if constexpr (P::PARTS) slice_parts<P, J>(x, part, std::make_index_sequence<NC>{});
    };
    auto advance = [&](auto pp) {
        constexpr uint32_t O = decltype(pp)::value * C::BUF;
        uint32_t h[NH];
#pragma unroll
        for (int q = 0; q < NH; ++q) h[q] = *reinterpret_cast<const uint32_t *>(lds + O + ha[q]);
        slice_step<P, J, P::PARTS>(x, h, part, std::make_index_sequence<NC>{});
    };
    uint32_t nx = 0;  // exchanges done
    auto exchange = [&]() {
        if constexpr (RES) {
            ++nx;
            const uint32_t tag = (epoch + nx) << NC;
            uint32_t *X = R.xch + (size_t)((epoch + nx) & 1u) * A.ntiles * A.ncorner * rblk;
            const bool mine = active && blk < A.nblk;
#pragma unroll 1
            for (uint32_t c = 0; c < A.ncorner; ++c) {
                const uint32_t off = A.corner_off[c];
                const uint32_t j = off / A.words, b0 = (off - j * A.words) / NC;
                if (mine && blk - b0 < rblk) {
                    uint32_t v = tag;
#pragma unroll
                    for (int i = 0; i < NC; ++i) v |= ((x[i] >> j) & 1u) << i;
                    __hip_atomic_store(X + ((size_t)t * A.ncorner + c) * rblk + (blk - b0), v, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (active && blk >= A.nblk) {  // ring lanes: all in the first wave
                const uint32_t rb = blk - A.nblk;
                uint32_t v[kSliceMaxRing];
                slice_wait(R, [&]() {
                    bool ok = true;
#pragma unroll
                    for (uint32_t s = 0; s < (uint32_t)kSliceMaxRing; ++s) {
                        v[s] = 0;
                        if (s < A.nring && nbt[s] != kNuHole32) {
                            v[s] = __hip_atomic_load(X + ((size_t)nbt[s] * A.ncorner + A.ring_corner[s]) * rblk + rb,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            ok &= ((v[s] ^ tag) >> NC) == 0;
                        }
                    }
                    return ok;
                });
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    uint32_t w = 0;
#pragma unroll
                    for (int s = 0; s < kSliceMaxRing; ++s) w |= ((v[s] >> i) & 1u) << s;
                    x[i] = w;
                }
            }
        }
    };

    if (tid < 2) *reinterpret_cast<uint32_t *>(lds + tid * C::BUF + C::ZERO) = 0;
    // Steps between exchanges in a loop of their own: with the exchange inside
    // it, every step was slower (100 steps: level-16 triangle 66.3 -> 61.2 us,
    // level 13 44.3 -> 41.3).
    for (int32_t left = steps;;) {
        const int32_t m = RES && A.nring && left > (int32_t)R.K ? (int32_t)R.K : left;
        publish(std::integral_constant<uint32_t, 0>{});
        __syncthreads();
        for (int32_t c = m;;) {
            advance(std::integral_constant<uint32_t, 0>{});
            if (--c == 0) break;
            publish(std::integral_constant<uint32_t, 1>{});
            __syncthreads();
            advance(std::integral_constant<uint32_t, 1>{});
            if (--c == 0) break;
            publish(std::integral_constant<uint32_t, 0>{});
            __syncthreads();
        }
        left -= m;
        if (!RES || left == 0) break;
        __syncthreads();  // every lane has read its last halo
        exchange();
    }
    if constexpr (RES) {
        // The result of an even step count goes where the start was: the tiles
        // that read ring cells of this one must have done so (an exchange implies it).
        if (out == in && nx == 0 && tid < A.nring && nbt[tid] != kNuHole32) {
            slice_wait(R, [&]() {
                return (int32_t)(__hip_atomic_load(R.loaded + nbt[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - run) >= 0;
            });
        }
    }
    __syncthreads();  // every lane has read its last halo
    if (active && blk < A.nblk) {
#pragma unroll
        for (int c = 0; c < NC; ++c) sm[blk * NC + c] = x[c];
    }
    __syncthreads();
    if constexpr (RES) {
        if (tid == 0) __hip_atomic_store(R.epoch + t, epoch + nx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The wide kernels stream over arrays that outgrow the last-level cache:
    // nontemporal stores (level 20: 1580 -> 1508 us per 20 steps).  The level-16
    // triangle fits it and is read again by the next launch: plain ones (three
    // steps 23.8 -> 20.0 us, 100 steps resident 1.3 us less).
    constexpr bool NTS = !RES && (J == 3 || P::B == 2);
    uint8_t *dst = out + t * A.cells;
    if (P::SMALL || A.words <= 4 * NT) {
        const uint32_t n = (A.words + 3) / 4;
        for (uint32_t k = tid; k < n; k += NT)
            slice_store_words<C, 1, false>(dst, A.words, 4 * k + 4 <= A.words ? 4 * k : A.words - 4, sm);
    } else if constexpr (!P::SMALL) {
        const uint32_t n = (A.words + 15) / 16;
        for (uint32_t k = tid; k < n; k += NT)
            slice_store_words<C, 4, NTS>(dst, A.words, 16 * k + 16 <= A.words ? 16 * k : A.words - 16, sm);
    }
}

// Host side: kernel, tile level and table layout of a fractal.
inline int slice_kind(const FractalHost &F) { return F.tile_kind == 4 ? 1 : F.tile_kind; }

// Tile level and kernel.  Triangles to level 16: at most 243 tiles, one per
// CU, of at least level 8, with level-2 blocks (more waves per SIMD: at level
// 16 three waves of 45 instructions per step rather than one of 121, which
// alone on its SIMD issues at less than half the rate: 70 against 87 us per
// 100 steps).  Above: level-11 tiles with level-3 blocks, several workgroups
// per CU, where the chip is full anyway and the larger block publishes and
// reads a third of the words (level 20, 20 steps: 1.58 against 2.31 ms).
// Vicsek crosses: level-6 tiles with level-1 blocks to level 10 (there 625 of them,
// three per CU: 3 steps 7.4 us and 100 steps 41.7, with 125 level-7 tiles 9.7 and
// 42.5), level-7 tiles with level-2 blocks above.
inline void slice_levels(int kind, int r, int &M, int &var)
{
    if (kind == 3) {
        M = r <= 10 ? std::min(r, 6) : 7;
        var = r <= 10 ? 0 : 2;
    } else {
        M = r >= 17 ? 11 : std::min(r, std::max(8, r - 5));
        var = r >= 17 ? 2 : (M <= 8 ? 0 : 1);
    }
}

// What the table builder needs of a kernel with tiles of level M.
template <class P>
SliceSpec slice_spec(int M)
{
    using C = SliceCfg<P>;
    constexpr int J = P::J;
    constexpr const SlicePlan &PL = C::PL;
    SliceSpec S{};
    S.M = M;
    S.B = P::B;
    S.J = J;
    S.RL = P::RL;
    S.steps = P::STEPS;
    S.nc = PL.nc;
    S.box = PL.box;
    S.nh = PL.nh;
    for (int c = 0; c < 32; ++c) S.cell_exp[c] = -1;
    for (int h = 0; h < PL.nh; ++h) {
        S.h_dx[h] = PL.h_dx[h];
        S.h_dy[h] = PL.h_dy[h];
        S.h_idx[h] = PL.h_idx[h];
        S.h_exp[h] = PL.h_exp[h];
    }
    for (int e = 0; e < PL.ne; ++e) S.cell_exp[PL.e_cell[e]] = e;
    for (int c = 0; c < PL.nc; ++c) {
        S.cell_x[c] = PL.lx[c];
        S.cell_y[c] = PL.ly[c];
    }
    S.max_ring = kSliceMaxRing;
    S.zero = C::ZERO;
    S.ex0 = C::EX0;
    S.pitch = C::PITCH;
    S.halo = C::HALO;
    S.rhalo = C::RHALO;
    S.passes = C::NPT;
    return S;
}

// Calls f with the kernel's pattern type.
template <class F>
auto slice_dispatch(int kind, int var, F &&f)
{
    switch (3 * kind + var) {
    case 3: return f(SliceTriSmall{});
    case 4: return f(SliceTri{});
    case 5: return f(SliceTriWide{});
    case 6: return f(SlicePaperSmall{});
    case 7: return f(SlicePaper{});
    case 8: return f(SlicePaperWide{});
    case 9: return f(SliceVicsekSmall{});
    default: return f(SliceVicsekWide{});  // 11
    }
}

// One tile configuration of a fractal.
struct SliceConfig {
    int kind, var;   // pattern (tile_kind_for), kernel (0 small, 1, 2 wide)
    uint32_t K;      // steps per launch and between exchanges (0: one tile, any number)
    SliceArgs A;
    uint32_t *d_tab; // lane_block, lane_halo, perm, nbtile
    // resident run (null: not available): exchange words, epochs, loaded counts, timed-out word
    uint32_t *d_res;
    uint64_t res_words;
    SliceRes R;
};

// A batch's tiles: small ones (level-8 triangles, level-6 Vicsek crosses at
// most), many per CU.  *own is true where the configuration is the fractal's
// own one, else the caller frees it (slice_free).
sqz_status slice_batch_config(const FractalHost &F, SliceConfig **out, bool *own);
void slice_free(SliceConfig *S);

}  // namespace sqz
