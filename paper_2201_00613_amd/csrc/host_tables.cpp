// Host-only table construction of libsqueeze (declarations and the data
// layouts in host_tables.h).  No HIP: compiled by g++.
#include "host_tables.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <utility>

namespace sqz {

// ---------------------------------------------------------------------------
// Errors
// ---------------------------------------------------------------------------
static thread_local char g_err[512];

sqz_status set_error(sqz_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

const char *last_error_text() { return g_err; }

// ---------------------------------------------------------------------------
// Invariant division
// ---------------------------------------------------------------------------
Div32 make_div32(uint32_t d)
{
    Div32 D;
    D.d = d;
    uint32_t l = 0;
    while (l < 32 && (1ull << l) < d) ++l;
    D.m = (uint32_t)((((unsigned __int128)1 << 32) * (((unsigned __int128)1 << l) - d)) / d + 1);
    D.sh1 = l < 1 ? l : 1;
    D.sh2 = l > 0 ? l - 1 : 0;
    return D;
}

Div64 make_div64(uint64_t d)
{
    Div64 D;
    D.d = d;
    uint32_t l = 0;
    while (l < 64 && ((unsigned __int128)1 << l) < d) ++l;
    D.m = (uint64_t)((((unsigned __int128)1 << 64) * (((unsigned __int128)1 << l) - d)) / d + 1);
    D.sh1 = l < 1 ? l : 1;
    D.sh2 = l > 0 ? l - 1 : 0;
    return D;
}

static uint64_t upow(uint64_t b, int e)
{
    uint64_t p = 1;
    while (e-- > 0) p *= b;
    return p;
}

// ---------------------------------------------------------------------------
// Descriptor
// ---------------------------------------------------------------------------
sqz_status check_descriptor(int32_t s, int32_t k, const int32_t *offs, int32_t r, FractalHost *F)
{
    if (s < 2 || s > kMaxS) return set_error(SQZ_ERR_INVALID, "s=%d outside [2, %d]", s, kMaxS);
    if (k < 1 || k > s * s) return set_error(SQZ_ERR_INVALID, "k=%d outside [1, s*s=%d]", k, s * s);
    if (!offs) return set_error(SQZ_ERR_INVALID, "offsets_xy is NULL");
    if (r < 0) return set_error(SQZ_ERR_INVALID, "r=%d is negative", r);
    int seen[kMaxS * kMaxS];
    for (int i = 0; i < s * s; ++i) seen[i] = -1;
    for (int j = 0; j < k; ++j) {
        const int x = offs[2 * j], y = offs[2 * j + 1];
        if (x < 0 || x >= s || y < 0 || y >= s)
            return set_error(SQZ_ERR_INVALID, "replica %d offset (%d,%d) outside [0,%d)^2", j, x, y, s);
        if (seen[x + s * y] >= 0)
            return set_error(SQZ_ERR_INVALID, "replicas %d and %d share offset (%d,%d)", seen[x + s * y], j, x, y);
        seen[x + s * y] = j;
    }
    // n = s^r < 2^31, N = k^r < 2^62
    uint64_t n = 1, N = 1;
    for (int i = 0; i < r; ++i) {
        n *= (uint64_t)s;
        if (n >= (1ull << 31)) return set_error(SQZ_ERR_RANGE, "n = %d^%d does not fit in 31 bits", s, r);
        N *= (uint64_t)k;
        if (N >= (1ull << 62)) return set_error(SQZ_ERR_RANGE, "N = %d^%d does not fit in 62 bits", k, r);
    }
    if (F) {
        memset(F, 0, sizeof *F);
        F->s = s;
        F->k = k;
        F->r = r;
        F->n = (int64_t)n;
        F->N = N;
        for (int j = 0; j < k; ++j) {
            F->ox[j] = offs[2 * j];
            F->oy[j] = offs[2 * j + 1];
        }
        for (int i = 0; i < s * s; ++i) F->hnu[i] = seen[i];
    }
    return SQZ_OK;
}

// ---------------------------------------------------------------------------
// Map tables
// ---------------------------------------------------------------------------
// Chunk sizes: at most 4096 entries per table, lambda offsets packed in 16
// bits per axis, nu chunk values below 2^31.
static int lam_chunk(int s, int k)
{
    int c = 1;
    while (c < 24 && upow(k, c + 1) <= 4096 && upow(s, c + 1) <= 65536) ++c;
    return c;
}
static int nu_chunk(int s, int k)
{
    int c = 1;
    while (c < 24 && upow(s, 2 * (c + 1)) <= 4096 && upow(k, c + 1) < (1ull << 31)) ++c;
    return c;
}

// Cells of a level's box by position (x + side*y), kNuHole32 for a hole: one
// level at a time, each a copy of the one below per replica.
static std::vector<uint32_t> nu_square(const FractalHost &F, int levels)
{
    const uint64_t s = (uint64_t)F.s, side = upow(s, levels);
    std::vector<uint32_t> t(side * side, kNuHole32);
    t[0] = 0;
    uint64_t sp = 1, kp = 1;  // the sp x sp corner holds the levels done so far
    for (int i = 0; i < levels; ++i) {
        for (int q = (int)(s * s) - 1; q >= 0; --q) {
            const int j = F.hnu[q];
            const uint64_t x0 = (uint64_t)q % s * sp, y0 = (uint64_t)q / s * sp;
            for (uint64_t y = 0; y < sp; ++y)
                for (uint64_t x = 0; x < sp; ++x) {
                    const uint32_t v = t[x + side * y];
                    t[x0 + x + side * (y0 + y)] = j < 0 || v == kNuHole32 ? kNuHole32 : v + (uint32_t)(j * kp);
                }
        }
        sp *= s;
        kp *= (uint64_t)F.k;
    }
    return t;
}

void map_tables(const FractalHost &F, int level, MapParams &P, MapTables &T)
{
    const int s = F.s, k = F.k;
    memset(&P, 0, sizeof P);
    P.s = s;
    P.k = k;
    P.r = level;
    P.n = (int32_t)upow(s, level);
    P.N = upow(k, level);
    const int CL = lam_chunk(s, k), CN = nu_chunk(s, k);
    P.nlam = level == 0 ? 0 : (level + CL - 1) / CL;
    P.nnu = level == 0 ? 0 : (level + CN - 1) / CN;
    const int TL = level == 0 ? 0 : level - CL * (P.nlam - 1);
    const int TN = level == 0 ? 0 : level - CN * (P.nnu - 1);
    P.klam = (uint32_t)upow(k, CL);
    P.slam = (uint32_t)upow(s, CL);
    P.snu = (uint32_t)upow(s, CN);
    P.snu_top = (uint32_t)upow(s, TN);
    P.knu = upow(k, CN);
    P.dklam64 = make_div64(P.klam);
    P.dklam32 = make_div32(P.klam);
    P.dsnu = make_div32(P.snu);

    // lambda tables: digit chunk -> packed (x | y << 16), one level at a time
    auto lam_table = [&](int levels, std::vector<uint32_t> &t) {
        t.assign(upow(k, levels), 0);
        uint64_t cnt = 1, sp = 1;
        for (int i = 0; i < levels; ++i) {
            for (int j = k - 1; j >= 0; --j) {
                const uint32_t o = (uint32_t)(F.ox[j] * sp) + ((uint32_t)(F.oy[j] * sp) << 16);
                for (uint64_t d = 0; d < cnt; ++d) t[j * cnt + d] = t[d] + o;
            }
            cnt *= (uint64_t)k;
            sp *= (uint64_t)s;
        }
    };
    // nu tables: (xc + side*yc) -> base-k replica digits, or hole
    auto nu_table = [&](int levels, std::vector<uint32_t> &t) { t = nu_square(F, levels); };
    std::vector<uint32_t> parts[4];
    if (level > 0) {
        lam_table(CL, parts[0]);
        lam_table(TL, parts[1]);
        nu_table(CN, parts[2]);
        nu_table(TN, parts[3]);
    } else {
        for (auto &p : parts) p.assign(1, 0);
    }
    T.all.clear();
    for (int i = 0; i < 4; ++i) {
        T.off[i] = T.all.size();
        T.all.insert(T.all.end(), parts[i].begin(), parts[i].end());
    }
    P.ntab = (uint32_t)T.all.size();
}

// The side is a compile-time constant in the two patterns' sides: the table
// builders evaluate these maps by the hundred thousand.
template <int SC>
static void lambda_side(const FractalHost &F, int level, uint64_t c, int64_t &x, int64_t &y)
{
    const int64_t s = SC ? SC : F.s;
    const uint32_t k = (uint32_t)F.k;
    int64_t px = 0, py = 0, sp = 1;
    for (int mu = 0; mu < level; ++mu) {
        const uint64_t q = (c >> 32) ? c / k : (uint32_t)c / k;
        const uint32_t b = (uint32_t)(c - q * k);
        c = q;
        px += F.ox[b] * sp;
        py += F.oy[b] * sp;
        sp *= s;
    }
    x = px;
    y = py;
}

template <int SC>
static int64_t nu_side(const FractalHost &F, int level, int64_t x0, int64_t y0)
{
    const uint32_t s = SC ? (uint32_t)SC : (uint32_t)F.s;
    int64_t side = 1;
    for (int i = 0; i < level; ++i) side *= s;
    if (x0 < 0 || y0 < 0 || x0 >= side || y0 >= side) return -1;
    uint32_t x = (uint32_t)x0, y = (uint32_t)y0;  // side < 2^31
    int64_t c = 0, kp = 1;
    for (int mu = 0; mu < level; ++mu) {
        const uint32_t qx = x / s, qy = y / s;
        const int j = F.hnu[x - qx * s + s * (y - qy * s)];
        if (j < 0) return -1;
        c += j * kp;
        kp *= F.k;
        x = qx;
        y = qy;
    }
    return c;
}

void host_lambda(const FractalHost &F, int level, uint64_t c, int64_t &x, int64_t &y)
{
    if (F.s == 2) return lambda_side<2>(F, level, c, x, y);
    if (F.s == 3) return lambda_side<3>(F, level, c, x, y);
    lambda_side<0>(F, level, c, x, y);
}

int64_t host_nu(const FractalHost &F, int level, int64_t x, int64_t y)
{
    if (F.s == 2) return nu_side<2>(F, level, x, y);
    if (F.s == 3) return nu_side<3>(F, level, x, y);
    return nu_side<0>(F, level, x, y);
}

static int64_t floor_div(int64_t a, int64_t b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

typedef std::pair<int64_t, int64_t> Pos;

// Positions outside a level-`level` subtree's box that touch a cell of it and
// are cells themselves if the adjacent subtree they lie in exists.
static std::vector<Pos> subtree_ring(const FractalHost &F, int level)
{
    const int64_t n = (int64_t)upow(F.s, level);
    std::vector<Pos> out;
    auto test = [&](int64_t x, int64_t y) {
        if (host_nu(F, level, x - floor_div(x, n) * n, y - floor_div(y, n) * n) < 0) return;
        for (int d = 0; d < 9; ++d)
            if (host_nu(F, level, x + d % 3 - 1, y + d / 3 - 1) >= 0) {
                out.emplace_back(x, y);
                return;
            }
    };
    for (int64_t x = -1; x <= n; ++x) {
        test(x, -1);
        test(x, n);
    }
    for (int64_t y = 0; y < n; ++y) {
        test(-1, y);
        test(n, y);
    }
    return out;
}

// Positions, in boxes of side rs, of the subtrees that hold the cells next to
// a level-`level` subtree.
static std::vector<Pos> ring_subtrees(const FractalHost &F, int level, int64_t rs)
{
    std::vector<Pos> key;
    for (const Pos &p : subtree_ring(F, level)) {
        const Pos q(floor_div(p.first, rs), floor_div(p.second, rs));
        bool have = false;
        for (const Pos &e : key) have |= e == q;
        if (!have) key.push_back(q);
    }
    return key;
}

// ---------------------------------------------------------------------------
// Launch sizes
// ---------------------------------------------------------------------------
int64_t launch_count(int32_t steps, int K)
{
    return steps < 1 ? 0 : (K < 1 ? 1 : ((int64_t)steps + K - 1) / K);
}

int32_t launch_share(int32_t steps, int64_t n, int64_t i)
{
    return (int32_t)(steps * (i + 1) / n - steps * i / n);
}

std::vector<int> plan_launches(int32_t steps, int K)
{
    int64_t n = launch_count(steps, K);
    if ((n ^ steps) & 1) ++n;
    std::vector<int> plan;
    if (steps < 1) return plan;
    for (int64_t i = 0; i < n; ++i) plan.push_back(launch_share(steps, n, i));
    return plan;
}

std::vector<int> plan_full_launches(int32_t steps, int K)
{
    if (steps < 1) return {};
    std::vector<int> plan((size_t)(steps / K), K);
    if (steps % K) plan.push_back(steps % K);
    if ((plan.size() & 1) != (size_t)(steps & 1))
        for (size_t i = plan.size(); i-- > 0;)
            if (plan[i] >= 2) {
                plan[i] -= 1;
                plan.push_back(1);
                break;
            }
    return plan;
}

std::vector<int> plan_group_launches(int32_t steps, int chosen, int full, bool one_step)
{
    const int K = chosen ? chosen : full;
    std::vector<int> plan = plan_launches(steps, K);
    if (one_step && steps > 1 && K != 1 && (int64_t)plan.size() > launch_count(steps, K)) {
        plan = plan_launches(steps - 1, K);
        plan.push_back(1);
    }
    return plan;
}

std::vector<GroupChoice> group_choices(int most, int full)
{
    std::vector<GroupChoice> v(1, GroupChoice{0, full ? full : 32});  // any number: a long launch
    for (int K : {1, 2, 3, 4, 5, 6, 8, 10})
        if (K <= most && (K > 1 || most == 1)) v.push_back(GroupChoice{K, K});
    return v;
}

// ---------------------------------------------------------------------------
// Bit-sliced tiles
// ---------------------------------------------------------------------------
sqz_status tile_tables(const FractalHost &F, const TileSpec &S, TileTables &T)
{
    const int M = S.M, J = S.J;
    const uint64_t tile = upow(F.k, M), nblocks = upow(F.k, M - J);
    const int64_t side = (int64_t)upow(F.s, M), box = S.box;

    // ring 1: cells of adjacent tiles that touch a cell of this tile
    struct Slot {
        int dx, dy;
        int64_t idx, px, py;  // cell index in the neighbour tile; position relative to this tile
    };
    std::vector<Slot> ring;
    auto find = [&](int64_t qx, int64_t qy) {
        for (size_t i = 0; i < ring.size(); ++i)
            if (ring[i].px == qx && ring[i].py == qy) return (int64_t)i;
        return (int64_t)-1;
    };
    auto outside_member = [&](int64_t qx, int64_t qy, int &tdx, int &tdy) {
        tdx = qx < 0 ? -1 : (qx >= side ? 1 : 0);
        tdy = qy < 0 ? -1 : (qy >= side ? 1 : 0);
        return host_nu(F, M, qx - tdx * side, qy - tdy * side);
    };
    for (const Pos &p : subtree_ring(F, M)) {
        int tdx, tdy;
        const int64_t j = outside_member(p.first, p.second, tdx, tdy);
        ring.push_back(Slot{tdx, tdy, j, p.first, p.second});
    }
    if (ring.size() > (size_t)S.max_tile_halo)
        return set_error(SQZ_ERR_UNSUPPORTED, "tile halo of %zu cells exceeds %d", ring.size(), S.max_tile_halo);
    T.nthalo = (uint32_t)ring.size();

    // rings 2..max_steps (several steps per launch): breadth-first from ring 1
    // over member cells outside the tile (ring d = graph distance d from the
    // tile); all rings must fit max_ring lanes, and ring cells must lie in the
    // adjacent tiles (d < side).
    std::vector<uint32_t> start = {0, (uint32_t)ring.size()};
    uint32_t ksteps = 1;
    for (int d = 2; d <= S.max_steps; ++d) {
        for (uint32_t c = start[d - 2]; c < start[d - 1]; ++c)
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    const int64_t qx = ring[c].px + dx, qy = ring[c].py + dy;
                    if (qx >= 0 && qy >= 0 && qx < side && qy < side) continue;
                    int tdx, tdy;
                    const int64_t j = outside_member(qx, qy, tdx, tdy);
                    if (j >= 0 && find(qx, qy) < 0) ring.push_back(Slot{tdx, tdy, j, qx, qy});
                }
        start.push_back((uint32_t)ring.size());
        if (T.nthalo == 0 || start[d] > (uint32_t)S.max_ring || d >= side) break;
        ksteps = (uint32_t)d;  // rings 1..d fit: d steps per launch
    }
    T.ksteps = ksteps;
    for (int d = 0; d <= S.max_steps && d < 16; ++d) T.ring_start[d] = start[d <= (int)ksteps ? d : ksteps];
    T.tstride = T.ring_start[ksteps];
    T.nsrc = ksteps >= 2 ? T.ring_start[ksteps - 1] : 0;
    ring.resize(T.tstride);

    // adjacent blocks of other tiles that hold ring-1 cells (one LDS word each)
    std::vector<std::pair<int64_t, int64_t>> vblk;
    auto virt_of = [&](int64_t bx, int64_t by) {
        for (size_t g = 0; g < vblk.size(); ++g)
            if (vblk[g].first == bx && vblk[g].second == by) return (int64_t)g;
        return (int64_t)-1;
    };
    for (uint32_t i = 0; i < T.nthalo; ++i) {
        const int64_t bx = floor_div(ring[i].px, box), by = floor_div(ring[i].py, box);
        if (virt_of(bx, by) < 0) vblk.emplace_back(bx, by);
    }
    // LDS entry (byte offset of the word << 16 | bit) of a tile cell and of ring cell i
    auto entry = [](uint32_t word, uint32_t bit) { return (4u * word) << 16 | bit; };
    const uint32_t zero_entry = entry(S.lds_zero, 0);
    auto tile_entry = [&](int64_t j) { return entry((uint32_t)(j / S.nc), (uint32_t)(j % S.nc)); };
    auto ring_entry = [&](size_t i) {
        uint32_t d = 1;
        while ((uint32_t)i >= T.ring_start[d]) ++d;
        if (d == 1) {
            const Slot &s = ring[i];
            const int64_t g = virt_of(floor_div(s.px, box), floor_div(s.py, box));
            return entry(S.lds_virt + (uint32_t)g, (uint32_t)(s.idx % S.nc));
        }
        const uint32_t k = (uint32_t)i - T.nthalo;  // rings 2.. packed in order
        return entry(S.lds_ring2 + k / 32, k % 32);
    };
    T.home.assign(T.tstride ? T.tstride : 1, zero_entry);
    for (uint32_t i = 0; i < T.tstride; ++i) T.home[i] = ring_entry(i);
    // LDS sources of the neighbours of every ring cell that is advanced
    T.rsrc.assign(T.nsrc ? (size_t)T.nsrc * 8 : 1, zero_entry);
    for (uint32_t c = 0; c < T.nsrc; ++c) {
        int n = 0;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                if (!dx && !dy) continue;
                const int64_t qx = ring[c].px + dx, qy = ring[c].py + dy;
                uint32_t e = zero_entry;
                if (qx >= 0 && qy >= 0 && qx < side && qy < side) {
                    const int64_t j = host_nu(F, M, qx, qy);
                    if (j >= 0) e = tile_entry(j);
                } else {
                    int tdx, tdy;
                    if (outside_member(qx, qy, tdx, tdy) >= 0) {
                        const int64_t i = find(qx, qy);  // always a loaded ring cell: ring d-1, d or d+1
                        if (i >= 0 && i < (int64_t)T.tstride) e = ring_entry((size_t)i);
                    }
                }
                T.rsrc[(size_t)c * 8 + n++] = e;
            }
    }

    // adjacent-block words of every block: a block of the tile, the word of
    // an adjacent block of another tile, or a zero word (no such block)
    const int NG = S.ngrp, NP = (NG + 1) / 2;
    T.nbstride = NP > 4 ? (uint32_t)((NP + 3) / 4 * 4) : 4u;
    T.nbt.assign((size_t)nblocks * T.nbstride, 0);
    const int64_t bside = (int64_t)upow(F.s, M - J);
    for (uint64_t b = 0; b < nblocks; ++b) {
        int64_t bx, by;
        host_lambda(F, M - J, b, bx, by);
        for (int g = 0; g < NG; ++g) {
            const int64_t nbx = bx + S.g_dx[g], nby = by + S.g_dy[g];
            uint32_t w = S.lds_zero;
            if (nbx >= 0 && nby >= 0 && nbx < bside && nby < bside) {
                const int64_t nb = host_nu(F, M - J, nbx, nby);
                if (nb >= 0) w = (uint32_t)nb;
            } else {
                const int64_t v = virt_of(nbx, nby);
                if (v >= 0) w = S.lds_virt + (uint32_t)v;
            }
            T.nbt[(size_t)b * T.nbstride + g / 2] |= (4u * w) << (16 * (g & 1));
        }
    }

    // per ring cell: adjacent-tile offset and the cell's index in that tile
    T.slots.assign(T.tstride ? (size_t)T.tstride * 4 : 4, 0);
    for (uint32_t i = 0; i < T.tstride; ++i) {
        T.slots[4 * i] = ring[i].dx;
        T.slots[4 * i + 1] = ring[i].dy;
        T.slots[4 * i + 2] = (int32_t)ring[i].idx;
    }
    // the tile's own cells that any tile loads as ring cells: every index that
    // appears in a ring slot (the slot tables are the same for every tile)
    std::vector<uint8_t> used(tile, 0);
    for (uint32_t i = 0; i < T.tstride; ++i) used[(size_t)ring[i].idx] = 1;
    T.bound.clear();
    for (uint64_t j = 0; j < tile; ++j)
        if (used[j]) T.bound.push_back((uint32_t)j);
    return SQZ_OK;
}

// ---------------------------------------------------------------------------
// Tiles bit-sliced across subtrees
// ---------------------------------------------------------------------------
sqz_status slice_tables(const FractalHost &F, const SliceSpec &S, SliceTables &T)
{
    const int M = S.M, L = M - S.B;
    const int64_t n = (int64_t)upow(F.s, M), sub = (int64_t)upow(F.s, L), rs = (int64_t)upow(F.s, S.RL);
    const uint32_t nsub = (uint32_t)upow(F.k, S.B);
    T.words = (uint32_t)upow(F.k, L);
    T.nblk = (uint32_t)upow(F.k, L - S.J);
    auto find = [](const std::vector<Pos> &v, const Pos &p) {
        for (size_t i = 0; i < v.size(); ++i)
            if (v[i] == p) return (int)i;
        return -1;
    };
    const std::vector<Pos> hs = subtree_ring(F, L);
    if (hs.size() > (size_t)S.nh) return set_error(SQZ_ERR_UNSUPPORTED, "subtile halo of %zu cells", hs.size());

    // Ring subtrees: those holding the cells next to the tile
    std::vector<Pos> key;
    if (M < F.r) {
        key = ring_subtrees(F, M, rs);
        if (key.size() > (size_t)S.max_ring) return set_error(SQZ_ERR_UNSUPPORTED, "%zu ring subtrees", key.size());
        T.K = (uint32_t)S.steps;
        T.rwords = (uint32_t)upow(F.k, S.RL);
    }
    T.nring = (uint32_t)key.size();
    const uint32_t rblk = T.rwords / (uint32_t)S.nc;
    std::vector<Pos> hr;
    if (T.nring) hr = subtree_ring(F, S.RL);
    if (hr.size() > (size_t)S.nh) return set_error(SQZ_ERR_UNSUPPORTED, "ring halo of %zu cells", hr.size());
    for (const Pos &q : key) {
        const int64_t dx = floor_div(q.first * rs, n), dy = floor_div(q.second * rs, n);
        const int64_t c = host_nu(F, M - S.RL, q.first - dx * (n / rs), q.second - dy * (n / rs));
        if (dx < -1 || dx > 1 || dy < -1 || dy > 1 || c < 0) return set_error(SQZ_ERR_UNSUPPORTED, "ring subtree out of reach");
        const uint32_t off = (uint32_t)c * T.rwords;
        size_t e = 0;
        while (e < T.corner.size() && T.corner[e] != off) ++e;
        if (e == T.corner.size()) T.corner.push_back(off);
        T.ring.insert(T.ring.end(), {(int32_t)dx, (int32_t)dy, (int32_t)off, (int32_t)e});
    }

    // LDS source of the cell at (x, y) of the tile's plane: offset | bit << 16 | ring subtree << 24
    const uint32_t none = S.zero | 0xFFu << 24;
    bool ok = true;
    auto source = [&](int64_t x, int64_t y) -> uint32_t {
        uint32_t w, bit, s = 0xFF, b0 = 0;
        if (x >= 0 && y >= 0 && x < n && y < n) {
            const int64_t c = host_nu(F, M, x, y);
            if (c < 0) return none;
            w = (uint32_t)(c % T.words);
            bit = (uint32_t)(c / T.words);
        } else {
            const Pos q(floor_div(x, rs), floor_div(y, rs));
            const int i = find(key, q);
            if (i < 0) return none;
            const int64_t c = host_nu(F, S.RL, x - q.first * rs, y - q.second * rs);
            if (c < 0) return none;
            w = (uint32_t)c;
            bit = s = (uint32_t)i;
            b0 = T.nblk;
        }
        const int e = S.cell_exp[w % (uint32_t)S.nc];
        if (e < 0) {
            ok = false;
            return none;
        }
        return (S.ex0 + (b0 + w / (uint32_t)S.nc) * S.pitch + 4u * (uint32_t)e) | bit << 16 | s << 24;
    };
    T.perm.assign((size_t)(S.passes + 1) * 64, none);
    for (size_t h = 0; h < hs.size(); ++h)
        for (uint32_t j = 0; j < nsub; ++j) {
            int64_t x, y;
            host_lambda(F, S.B, j, x, y);
            T.perm[h * 32 + j] = source(x * sub + hs[h].first, y * sub + hs[h].second);
        }
    for (size_t h = 0; h < hr.size(); ++h)
        for (uint32_t s = 0; s < T.nring; ++s)
            T.perm[(size_t)S.passes * 64 + h * (size_t)S.max_ring + s] =
                source(key[s].first * rs + hr[h].first, key[s].second * rs + hr[h].second);

    // Lanes: the ring's blocks, then the blocks the halo ballots read or whose
    // own halo leaves the subtile (all in the first wave), then the rest.
    std::vector<uint8_t> special(T.nblk, 0);
    for (uint32_t e : T.perm)
        if ((e & 0xFFFFu) >= S.ex0) {
            const uint32_t b = ((e & 0xFFFFu) - S.ex0) / S.pitch;
            if (b < T.nblk) special[b] = 1;
        }
    auto block_halo = [&](int level, uint32_t b, uint32_t first, const std::vector<Pos> &ring, uint32_t ring_off,
                          uint32_t *out) {
        const int64_t side = (int64_t)upow(F.s, level - S.J);
        int64_t bx, by;
        bool leaves = false;
        host_lambda(F, level - S.J, b, bx, by);
        for (int h = 0; h < S.nh; ++h) {
            const int64_t x = bx + S.h_dx[h], y = by + S.h_dy[h];
            out[h] = S.zero;
            if (x >= 0 && y >= 0 && x < side && y < side) {
                const int64_t nb = host_nu(F, level - S.J, x, y);
                if (nb >= 0) out[h] = S.ex0 + (first + (uint32_t)nb) * S.pitch + 4u * (uint32_t)S.h_exp[h];
            } else {
                const int i = find(ring, Pos(x * S.box + S.cell_x[S.h_idx[h]], y * S.box + S.cell_y[S.h_idx[h]]));
                if (i >= 0) out[h] = ring_off + 4u * (uint32_t)i;
                leaves |= i >= 0;
            }
        }
        return leaves;
    };
    std::vector<uint32_t> halo((size_t)(T.nblk + rblk) * (size_t)S.nh);
    for (uint32_t b = 0; b < T.nblk; ++b)
        if (block_halo(L, b, 0, hs, S.halo, &halo[(size_t)b * S.nh])) special[b] = 1;
    for (uint32_t b = 0; b < rblk; ++b) block_halo(S.RL, b, T.nblk, hr, S.rhalo, &halo[(size_t)(T.nblk + b) * S.nh]);
    for (uint32_t b = 0; b < rblk; ++b) T.lane_block.push_back(T.nblk + b);
    for (int pass = 1; pass >= 0; --pass) {
        for (uint32_t b = 0; b < T.nblk; ++b)
            if (special[b] == pass) T.lane_block.push_back(b);
        if (pass && T.lane_block.size() > 64) return set_error(SQZ_ERR_UNSUPPORTED, "%zu lanes in the first wave", T.lane_block.size());
    }
    for (uint32_t b : T.lane_block)
        T.lane_halo.insert(T.lane_halo.end(), halo.begin() + (size_t)b * S.nh, halo.begin() + (size_t)(b + 1) * S.nh);
    return ok ? SQZ_OK : set_error(SQZ_ERR_UNSUPPORTED, "a halo cell is not published");
}

// ---------------------------------------------------------------------------
// Tiles with one block per lane
// ---------------------------------------------------------------------------
void lane_tables(const FractalHost &F, const LaneSpec &S, LaneTables &T)
{
    const int M = S.M;
    const int64_t bs = (int64_t)upow(F.s, M - S.J);
    T.cells = upow(F.k, M);
    T.nblk = (uint32_t)upow(F.k, M - S.J);
    // lane of every block position of the tile's plane within `edge` blocks of
    // the tile: lane | tile << 16 (0..7 adjacent, 8 this one), ~0 if none
    const int64_t rb = S.frame ? S.frame : (int64_t)upow(F.s, S.RL - S.J), edge = M < F.r ? rb : 1, W = bs + 2 * edge;
    std::vector<uint32_t> grid((size_t)(W * W), ~0u);
    std::vector<Pos> pos;
    auto at = [&](int64_t x, int64_t y) -> uint32_t & { return grid[(size_t)((y + edge) * W + x + edge)]; };
    for (uint32_t b = 0; b < T.nblk; ++b) {
        int64_t x, y;
        host_lambda(F, M - S.J, b, x, y);
        at(x, y) = b | 8u << 16;
        pos.emplace_back(x, y);
    }
    auto add_ring = [&](int64_t x, int64_t y) {
        const int64_t tx = floor_div(x, bs), ty = floor_div(y, bs);
        const int64_t b = host_nu(F, M - S.J, x - tx * bs, y - ty * bs);
        if (b < 0) return;
        const int d = (int)((ty + 1) * 3 + (tx + 1));
        const uint32_t d8 = (uint32_t)(d < 4 ? d : d - 1);
        at(x, y) = (uint32_t)pos.size() | d8 << 16;
        pos.emplace_back(x, y);
        T.lane_src.push_back(d8 << 28 | (uint32_t)b);
    };
    if (M < F.r && S.frame) {
        for (int64_t y = -edge; y < bs + edge; ++y)
            for (int64_t x = -edge; x < bs + edge; ++x)
                if (x < 0 || y < 0 || x >= bs || y >= bs) add_ring(x, y);
    } else if (M < F.r) {
        for (const Pos &q : ring_subtrees(F, M, (int64_t)upow(F.s, S.RL)))
            for (uint32_t b = 0; b < upow(F.k, S.RL - S.J); ++b) {
                int64_t x, y;
                host_lambda(F, S.RL - S.J, b, x, y);
                add_ring(q.first * rb + x, q.second * rb + y);
            }
    }
    if (M < F.r) T.K = S.steps;
    T.lanes = (uint32_t)pos.size();
    T.lane_nb.reserve((size_t)T.lanes * S.ng);
    for (const Pos &p : pos)
        for (int g = 0; g < S.ng; ++g) {
            const int64_t x = p.first + S.g_dx[g], y = p.second + S.g_dy[g];
            T.lane_nb.push_back(x < -edge || y < -edge || x >= bs + edge || y >= bs + edge ? ~0u : at(x, y));
        }
}

// ---------------------------------------------------------------------------
// Expanded tiles
// ---------------------------------------------------------------------------
// Adjacent tile (0..8, 4: this one) of a position of the tile's plane, and the
// cell of that tile's box there (kNuHole32: none, or beyond the adjacent tiles).
static int tile_cell(const std::vector<uint32_t> &nu, int64_t side, int64_t x, int64_t y, uint32_t &cell)
{
    const int tdx = x < 0 ? -1 : (x >= side ? 1 : 0), tdy = y < 0 ? -1 : (y >= side ? 1 : 0);
    const int64_t bx = x - tdx * side, by = y - tdy * side;
    cell = bx < 0 || by < 0 || bx >= side || by >= side ? kNuHole32 : nu[(size_t)(bx + side * by)];
    return (tdy + 1) * 3 + (tdx + 1);
}

static uint32_t dir8(int d) { return (uint32_t)(d < 4 ? d : d - 1); }

void xtile_ring_slots(const FractalHost &F, int M, uint32_t P, std::vector<XRingSlot> &out)
{
    const int64_t side = (int64_t)upow(F.s, M);
    const uint64_t KM = upow(F.k, M);
    const std::vector<uint32_t> nu = nu_square(F, M);
    std::vector<uint8_t> seen((size_t)P * P, 0);
    out.clear();
    for (uint64_t c = 0; c < KM; ++c) {
        int64_t x, y;
        host_lambda(F, M, c, x, y);
        if (x > 0 && y > 0 && x < side - 1 && y < side - 1) continue;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                const int64_t qx = x + dx, qy = y + dy;
                uint32_t j;
                const int d = tile_cell(nu, side, qx, qy, j);
                if (d == 4 || j == kNuHole32) continue;
                const uint32_t pos = (uint32_t)((qy + 1) * P + (qx + 1));
                if (seen[pos]) continue;
                seen[pos] = 1;
                out.push_back(XRingSlot{(uint16_t)pos, (dir8(d) << 16) | j});
            }
    }
}

void xtile_cell_entries(const FractalHost &F, int M, uint32_t P, const int field_shift[8],
                        std::vector<uint16_t> &lam, std::vector<uint32_t> &ent)
{
    const int64_t side = (int64_t)upow(F.s, M);
    const uint64_t KM = upow(F.k, M);
    const std::vector<uint32_t> nu = nu_square(F, M);
    lam.assign(KM, 0);
    ent.assign(KM, 0);
    for (int64_t y = 0; y < side; ++y)
        for (int64_t x = 0; x < side; ++x) {
            const uint32_t c = nu[(size_t)(x + side * y)];
            if (c == kNuHole32) continue;
            lam[c] = (uint16_t)((y + 1) * P + (x + 1));
            // member neighbours inside the tile, and per adjacent tile the member
            // cells of that tile (its own copy of the level-M pattern) it touches
            uint32_t cnt[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, q;
            for (int n = 0; n < 9; ++n) {
                if (n == 4) continue;
                const int d = tile_cell(nu, side, x + n % 3 - 1, y + n / 3 - 1, q);
                cnt[d] += q != kNuHole32;
            }
            uint32_t e = lam[c] | cnt[4] << 16;
            for (int d = 0; d < 9; ++d)
                if (d != 4) e |= cnt[d] << field_shift[dir8(d)];  // sides <= 3, corners <= 1
            ent[c] = e;
        }
}

void xtile_layer_tables(const FractalHost &F, int M, int K, uint32_t P, uint32_t rows,
                        std::vector<XRingSlot> &ring, std::vector<uint32_t> &start, std::vector<uint16_t> &lam,
                        std::vector<uint8_t> &mem)
{
    const int64_t B = (int64_t)upow(F.s, M);
    const uint64_t KM = upow(F.k, M);
    const std::vector<uint32_t> nu = nu_square(F, M);
    ring.clear();
    start.assign(1, 0);
    // ring slots by layer: member cells of the adjacent tiles within K of the box
    for (int64_t d = 1; d <= K; ++d) {
        for (int64_t qy = -d; qy < B + d; ++qy) {
            const bool whole = qy == -d || qy == B + d - 1;  // a whole row of the layer, or its two ends
            for (int64_t qx = -d; qx < B + d; qx += whole ? 1 : B + 2 * d - 1) {
                uint32_t j;
                const int dd = tile_cell(nu, B, qx, qy, j);
                if (j == kNuHole32) continue;
                ring.push_back(XRingSlot{(uint16_t)((qy + K) * P + (qx + K)), (dir8(dd) << 16) | j});
            }
        }
        start.push_back((uint32_t)ring.size());
    }
    // box positions of the tile's cells and their membership
    lam.assign(KM, 0);
    mem.assign((size_t)P * rows, 0);
    for (int64_t y = 0; y < B; ++y)
        for (int64_t x = 0; x < B; ++x) {
            const uint32_t c = nu[(size_t)(x + B * y)];
            if (c == kNuHole32) continue;
            lam[c] = (uint16_t)((y + K) * P + (x + K));
            mem[lam[c]] = 1;
        }
}

// ---------------------------------------------------------------------------
// Bit-row tiles
// ---------------------------------------------------------------------------
void bitbox_tables(const FractalHost &F, const BitboxSpec &S, std::vector<uint16_t> &bpos,
                   std::vector<uint32_t> &ring, std::vector<uint32_t> &member)
{
    const int M = S.M, BD = S.border;
    const uint64_t nblk = upow(F.k, M - 1);
    const int64_t sb = (int64_t)upow(3, M - 1), GB = sb + 2 * BD;

    // grid positions of the tile's blocks
    bpos.assign(nblk, 0);
    for (uint64_t b = 0; b < nblk; ++b) {
        int64_t x, y;
        host_lambda(F, M - 1, b, x, y);
        bpos[b] = (uint16_t)((x + BD) | (y + BD) << 7);
    }
    // border blocks: position in an adjacent tile, if a block of the pattern is there
    auto outside_block = [&](int64_t gx, int64_t gy, int &dir) -> int64_t {
        const int64_t bx = gx - BD, by = gy - BD;
        const int64_t tdx = floor_div(bx, sb), tdy = floor_div(by, sb);
        dir = (int)((tdy + 1) * 3 + (tdx + 1));
        return host_nu(F, M - 1, bx - tdx * sb, by - tdy * sb);
    };
    ring.clear();
    for (int64_t gy = 0; gy < GB; ++gy)
        for (int64_t gx = 0; gx < GB; ++gx) {
            const bool inner = gx >= BD && gy >= BD && gx < BD + sb && gy < BD + sb;
            if (inner) continue;
            int dir;
            const int64_t lb = outside_block(gx, gy, dir);
            if (lb >= 0) ring.push_back((uint32_t)(gy * S.grid_pitch + gx) | (uint32_t)dir << 14 | (uint32_t)lb << 18);
        }
    // membership of every box position (adjacent tiles present)
    member.assign((size_t)S.rows * S.words, 0);
    for (int64_t cy = 0; cy < 3 * GB; ++cy)
        for (int64_t cx = 0; cx < 3 * GB; ++cx) {
            if (F.hnu[(int)(cx % 3) + 3 * (int)(cy % 3)] < 0) continue;
            const int64_t gx = cx / 3, gy = cy / 3;
            const bool inner = gx >= BD && gy >= BD && gx < BD + sb && gy < BD + sb;
            int dir;
            const int64_t lb = inner ? host_nu(F, M - 1, gx - BD, gy - BD) : outside_block(gx, gy, dir);
            if (lb >= 0) member[(size_t)cy * S.words + cx / 32] |= 1u << (cx % 32);
        }
}

}  // namespace sqz
