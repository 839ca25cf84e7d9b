// CPU checks of the tables that the multi-step kernels read unchecked: tiles
// bit-sliced across subtrees (slice_device.h), blocks per lane (lane_device.h),
// bit rows of general patterns and of the carpet (gbox.hip, bitbox_device.h).
// The first two are run as the kernels run them, word by word through the same
// memory layout with every offset checked, and compared with brute force over the
// pattern for every step the ring covers.  Host code only; no GPU call.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <utility>
#include <vector>

#include "bitbox_device.h"
#include "lane_device.h"
#include "slice_device.h"

using namespace sqz;

static int g_fail = 0;
#define EXPECT(cond, ...)                                   \
    do {                                                    \
        if (!(cond)) {                                      \
            fprintf(stderr, "FAILED %s:%d: ", __FILE__, __LINE__); \
            fprintf(stderr, __VA_ARGS__);                   \
            fprintf(stderr, "\n");                          \
            if (++g_fail > 20) exit(1);                     \
        }                                                   \
    } while (0)

struct Pattern {
    const char *name;
    int s, k;
    int offs[32];
};
static const Pattern kTri = {"triangle", 2, 3, {0, 0, 1, 0, 0, 1}};
static const Pattern kPaper = {"triangle_paper", 2, 3, {0, 0, 0, 1, 1, 1}};
static const Pattern kVic = {"vicsek", 3, 5, {1, 0, 0, 1, 1, 1, 2, 1, 1, 2}};
static const Pattern kCar = {"carpet", 3, 8, {0, 0, 1, 0, 2, 0, 0, 1, 2, 1, 0, 2, 1, 2, 2, 2}};
static const Pattern kWide = {"wide", 4, 10, {0, 0, 1, 0, 3, 0, 0, 1, 2, 1, 3, 1, 1, 2, 2, 2, 0, 3, 3, 3}};
static const Pattern kSix = {"six", 3, 6, {0, 0, 1, 0, 0, 1, 2, 1, 1, 2, 2, 2}};
static const Pattern kSquare = {"square", 2, 4, {0, 0, 1, 0, 0, 1, 1, 1}};

static int64_t ipow(int64_t b, int e)
{
    int64_t p = 1;
    while (e-- > 0) p *= b;
    return p;
}

static FractalHost make(const Pattern &p, int r)
{
    FractalHost F;
    EXPECT(check_descriptor(p.s, p.k, p.offs, r, &F) == SQZ_OK, "%s r=%d", p.name, r);
    return F;
}

// Compact neighbours of every cell, raster order, -1 where there is none.
static std::vector<int32_t> neighbours(const FractalHost &F)
{
    std::vector<int32_t> nb((size_t)F.N * 8, -1);
    for (uint64_t c = 0; c < F.N; ++c) {
        int64_t x, y;
        host_lambda(F, F.r, c, x, y);
        for (int j = 0, i = 0; j < 9; ++j)
            if (j != 4) nb[c * 8 + i++] = (int32_t)host_nu(F, F.r, x + j % 3 - 1, y + j / 3 - 1);
    }
    return nb;
}

// ---------------------------------------------------------------------------
// Tiles bit-sliced across subtrees
// ---------------------------------------------------------------------------
template <class P>
static void check_slice(const Pattern &pat, int M, int r)
{
    using C = SliceCfg<P>;
    constexpr const SlicePlan &PL = C::PL;
    const FractalHost F = make(pat, r);
    const SliceSpec S = slice_spec<P>(M);
    SliceTables T;
    EXPECT(slice_tables(F, S, T) == SQZ_OK, "%s M=%d: %s", pat.name, M, last_error_text());
    const uint32_t lanes = (uint32_t)T.lane_block.size(), rblk = T.rwords / (uint32_t)PL.nc, nsub = (uint32_t)C::KB;
    EXPECT(lanes == T.nblk + rblk && lanes <= (uint32_t)C::LANES, "%s M=%d: %u lanes of %d", pat.name, M, lanes, C::LANES);
    EXPECT(T.words * nsub == (uint32_t)ipow(F.k, M) && T.words == T.nblk * (uint32_t)PL.nc, "%s M=%d words", pat.name, M);
    EXPECT(T.lane_halo.size() == (size_t)lanes * PL.nh && T.perm.size() == (size_t)(C::NPT + 1) * 64, "%s M=%d sizes", pat.name, M);
    EXPECT(4 * (T.words + T.rwords) <= C::LDS, "%s M=%d staging", pat.name, M);
    EXPECT(T.nring <= (uint32_t)kSliceMaxRing && T.corner.size() <= (size_t)kSliceMaxRing, "%s M=%d ring", pat.name, M);
    std::set<uint32_t> seen(T.lane_block.begin(), T.lane_block.end());
    EXPECT(seen.size() == lanes && *seen.rbegin() == lanes - 1, "%s M=%d: lanes repeat blocks", pat.name, M);
    std::vector<uint32_t> lane_of(lanes);
    for (uint32_t l = 0; l < lanes; ++l) lane_of[T.lane_block[l]] = l;
    // what the first wave reads back it has written itself, and the ring's lanes are in it
    for (uint32_t b = T.nblk; b < lanes; ++b) EXPECT(lane_of[b] < 64, "%s M=%d: ring lane %u", pat.name, M, lane_of[b]);
    for (uint32_t e : T.perm) {
        const uint32_t o = e & 0xFFFFu;
        if (o == C::ZERO) continue;
        EXPECT(o >= C::EX0 && o < C::HALO && (o - C::EX0) % 4 == 0, "%s M=%d: halo source %u", pat.name, M, o);
        const uint32_t b = (o - C::EX0) / C::PITCH;
        EXPECT(b < lanes && lane_of[b] < 64, "%s M=%d: halo source in block %u", pat.name, M, b);
        EXPECT((o - C::EX0) % C::PITCH / 4 < (uint32_t)PL.ne, "%s M=%d: halo source not published", pat.name, M);
    }
    // the exchange takes a corner subtree from one subtile, whole blocks of it
    for (uint32_t off : T.corner)
        EXPECT(off % (uint32_t)PL.nc == 0 && off % T.words + T.rwords <= T.words, "%s M=%d: corner subtree at %u", pat.name, M, off);
    const uint64_t tile = (uint64_t)T.words * nsub;
    FractalHost Fc = F;
    Fc.r = r - M;
    for (uint32_t s = 0; s < T.nring; ++s) {
        const int32_t *e = &T.ring[4 * s];
        EXPECT(T.corner.at((size_t)e[3]) == (uint32_t)e[2] && (uint64_t)e[2] + T.rwords <= tile, "%s M=%d ring %u", pat.name, M, s);
        bool back = false;  // adjacency is symmetric
        for (uint32_t q = 0; q < T.nring; ++q) back |= T.ring[4 * q] == -e[0] && T.ring[4 * q + 1] == -e[1];
        EXPECT(back, "%s M=%d: ring subtree %u has no opposite", pat.name, M, s);
    }

    // the machine
    const std::vector<int32_t> nb = neighbours(F);
    std::mt19937 rng(7 * M + r);
    std::vector<uint8_t> start((size_t)F.N), cur, nxt((size_t)F.N);
    for (uint8_t &v : start) v = rng() % 100 < 45;
    const uint64_t ntiles = F.N / tile;
    std::vector<uint64_t> tiles;
    for (uint64_t t = 0; t < ntiles; t += ntiles <= 12 ? 1 : ntiles / 12) tiles.push_back(t);
    const int K = T.K ? (int)T.K : 9;
    struct State {
        std::vector<uint32_t> w;  // [lanes][nc]
    };
    std::vector<State> st(tiles.size());
    std::vector<std::vector<int64_t>> adj(tiles.size(), std::vector<int64_t>(kSliceMaxRing, -1));
    for (size_t i = 0; i < tiles.size(); ++i) {
        const uint64_t t = tiles[i];
        int64_t X, Y;
        host_lambda(F, r - M, t, X, Y);
        st[i].w.assign((size_t)lanes * PL.nc, 0);
        for (uint32_t s = 0; s < T.nring; ++s) adj[i][s] = host_nu(F, r - M, X + T.ring[4 * s], Y + T.ring[4 * s + 1]);
        for (uint32_t w = 0; w < T.words; ++w)
            for (uint32_t j = 0; j < nsub; ++j) st[i].w[w] |= (uint32_t)start[t * tile + (uint64_t)j * T.words + w] << j;
        for (uint32_t w = 0; w < T.rwords; ++w)
            for (uint32_t s = 0; s < T.nring; ++s)
                if (adj[i][s] >= 0)
                    st[i].w[(size_t)T.nblk * PL.nc + w] |=
                        (uint32_t)start[(uint64_t)adj[i][s] * tile + (uint64_t)T.ring[4 * s + 2] + w] << s;
    }
    cur = start;
    for (int step = 1; step <= K; ++step) {
        for (uint64_t c = 0; c < F.N; ++c) {
            int n = 0;
            for (int j = 0; j < 8; ++j) n += nb[c * 8 + j] >= 0 && cur[nb[c * 8 + j]];
            nxt[c] = n == 3 || (n == 2 && cur[c]);
        }
        cur.swap(nxt);
        for (size_t i = 0; i < tiles.size(); ++i) {
            std::vector<uint32_t> lds(C::BUF / 4, 0);
            std::vector<uint32_t> &x = st[i].w;
            for (uint32_t b = 0; b < lanes; ++b)
                for (int e = 0; e < PL.ne; ++e) lds.at((C::EX0 + b * C::PITCH) / 4 + e) = x[(size_t)b * PL.nc + PL.e_cell[e]];
            uint64_t bal[C::NPT + 1] = {};
            for (int p = 0; p <= C::NPT; ++p)
                for (int l = 0; l < 64; ++l) {
                    const uint32_t e = T.perm[p * 64 + l], o = e & 0xFFFFu, bit = (e >> 16) & 31u, s = e >> 24;
                    bool on = o != C::ZERO && !(s < (uint32_t)kSliceMaxRing && adj[i][s] < 0);
                    if (on) on = (lds.at(o / 4) >> bit) & 1u;
                    bal[p] |= (uint64_t)on << l;
                }
            for (int h = 0; h < PL.nh; ++h) {
                lds.at(C::HALO / 4 + h) = (uint32_t)(bal[h >> 1] >> (32 * (h & 1)));
                lds.at(C::RHALO / 4 + h) = (uint32_t)(bal[C::NPT] >> (h * kSliceMaxRing)) & 0xFFu;
            }
            std::vector<uint32_t> y(x.size());
            for (uint32_t b = 0; b < lanes; ++b)
                for (int c = 0; c < PL.nc; ++c) {
                    uint32_t ones = 0, twos = 0, more = 0;
                    for (int d = 0; d < PL.deg[c]; ++d) {
                        const int q = PL.nb[c][d];
                        const uint32_t o = q < PL.nc ? 0 : T.lane_halo[(size_t)lane_of[b] * PL.nh + (q - PL.nc)];
                        EXPECT(o % 4 == 0, "%s M=%d halo offset %u", pat.name, M, o);
                        const uint32_t v = q < PL.nc ? x[(size_t)b * PL.nc + q] : lds.at(o / 4);
                        const uint32_t c1 = ones & v, c2 = twos & c1;
                        ones ^= v;
                        twos ^= c1;
                        more |= c2;
                    }
                    y[(size_t)b * PL.nc + c] = ~more & twos & (ones | x[(size_t)b * PL.nc + c]);
                }
            x.swap(y);
            uint64_t bad = 0;
            for (uint32_t w = 0; w < T.words; ++w)
                for (uint32_t j = 0; j < nsub; ++j)
                    bad += ((x[w] >> j) & 1u) != cur[tiles[i] * tile + (uint64_t)j * T.words + w];
            EXPECT(bad == 0, "%s M=%d r=%d tile %llu step %d: %llu cells differ", pat.name, M, r,
                   (unsigned long long)tiles[i], step, (unsigned long long)bad);
        }
    }
    printf("%s level %d tiles, level %d: %u lanes, %u ring subtrees, %d steps\n", pat.name, M, r, lanes, T.nring, K);
}

template <class P>
static void check_slices(const Pattern &pat, std::initializer_list<int> levels, int above)
{
    for (int M : levels)
        for (int r = M; r <= M + above; ++r) check_slice<P>(pat, M, r);
}

// The level and kernel every fractal takes are among those checked.
static void check_slice_levels()
{
    for (int kind = 1; kind <= 3; ++kind)
        for (int r = 3; r <= (kind == 3 ? 19 : 30); ++r) {
            int M, var;
            slice_levels(kind, r, M, var);
            if (kind == 3)
                EXPECT(M <= r && (r <= 10 ? var == 0 && M == std::min(r, 6) : var == 2 && M == 7), "vicsek r=%d", r);
            else
                EXPECT(M <= r && (var == 0 ? M <= 8 : (var == 1 ? M >= 9 && M <= 11 : M == 11)), "triangle r=%d", r);
        }
}

// ---------------------------------------------------------------------------
// One block per lane
// ---------------------------------------------------------------------------
// kind, rk: the kernel and the level it is chosen for (r: a smaller one with the same tiles).
template <class P>
static void check_lane(const Pattern &pat, int r, int kind = 0, int rk = 0)
{
    using PO = LanePlanOf<P, P::J>;
    constexpr const LanePlan &PL = PO::value;
    const FractalHost F = make(pat, r);
    uint32_t most = 0;
    const LaneSpec S = lane_spec(kind ? kind : lane_kind(F), rk ? rk : r, most);
    EXPECT(S.J == P::J && most == (uint32_t)P::LANES - 1, "%s r=%d: kernel", pat.name, r);
    LaneTables T;
    lane_tables(F, S, T);
    EXPECT(T.lanes <= most, "%s r=%d: %u lanes of %u", pat.name, r, T.lanes, most);
    EXPECT(T.lane_src.size() == T.lanes - T.nblk && T.lane_nb.size() == (size_t)T.lanes * PL.ng, "%s r=%d sizes", pat.name, r);
    if (T.lanes > most) return;
    for (uint32_t e : T.lane_src) EXPECT((e >> 28) < 8 && (e & 0xFFFFFFFu) < T.nblk, "%s r=%d ring source", pat.name, r);
    for (uint32_t e : T.lane_nb)
        EXPECT(e == ~0u || ((e & 0xFFFFu) < T.lanes && (e >> 16) <= 8), "%s r=%d adjacent lane %x", pat.name, r, e);
    const std::vector<int32_t> nb = neighbours(F);
    std::mt19937_64 rng(r);
    std::vector<uint64_t> cur((size_t)F.N), nxt((size_t)F.N);
    for (uint64_t &v : cur) v = rng();
    const uint64_t ntiles = F.N / T.cells;
    std::vector<uint64_t> tiles;
    for (uint64_t t = 0; t < ntiles; t += ntiles <= 10 ? 1 : ntiles / 10) tiles.push_back(t);
    const int K = T.K ? T.K : 7;
    std::vector<std::vector<uint64_t>> x(tiles.size());
    std::vector<std::vector<int64_t>> adj(tiles.size(), std::vector<int64_t>(9));
    for (size_t i = 0; i < tiles.size(); ++i) {
        int64_t X, Y;
        host_lambda(F, r - S.M, tiles[i], X, Y);
        for (int d = 0; d < 9; ++d) {
            const int64_t t = host_nu(F, r - S.M, X + d % 3 - 1, Y + d / 3 - 1);
            if (d != 4) adj[i][d < 4 ? d : d - 1] = t;
        }
        adj[i][8] = (int64_t)tiles[i];
        x[i].assign((size_t)T.lanes * PL.nc, 0);
        for (uint32_t l = 0; l < T.lanes; ++l) {
            const uint32_t e = l < T.nblk ? 8u << 28 | l : T.lane_src[l - T.nblk];
            const int64_t t = adj[i][l < T.nblk ? 8 : e >> 28];
            const uint64_t b = l < T.nblk ? l : e & 0xFFFFFFFu;
            if (t < 0) continue;
            for (int c = 0; c < PL.nc; ++c) x[i][(size_t)l * PL.nc + c] = cur[((uint64_t)t * T.nblk + b) * PL.nc + c];
        }
    }
    for (int step = 1; step <= K; ++step) {
        for (uint64_t c = 0; c < F.N; ++c) {  // any linear rule with the degree: 3 u + 5 sum + 7 deg, modulo 2^64
            uint64_t s = 0, deg = 0;
            for (int j = 0; j < 8; ++j)
                if (nb[c * 8 + j] >= 0) s += cur[nb[c * 8 + j]], ++deg;
            nxt[c] = 3 * cur[c] + 5 * s + 7 * deg;
        }
        cur.swap(nxt);
        for (size_t i = 0; i < tiles.size(); ++i) {
            // published cells, one row per slot; lanes that do not exist read a zero column
            std::vector<uint64_t> lds((size_t)PL.ne * P::LANES, 0), y(x[i].size());
            for (uint32_t l = 0; l < T.lanes; ++l)
                for (int e = 0; e < PL.ne; ++e) lds.at((size_t)e * P::LANES + l) = x[i][(size_t)l * PL.nc + PL.e_cell[e]];
            for (uint32_t l = 0; l < T.lanes; ++l) {
                uint32_t gb[8];
                int ex[8];
                for (int g = 0; g < PL.ng; ++g) {
                    const uint32_t e = T.lane_nb[(size_t)l * PL.ng + g];
                    ex[g] = e != ~0u && adj[i][e >> 16] >= 0;
                    gb[g] = ex[g] ? e & 0xFFFFu : (uint32_t)P::LANES - 1;
                }
                for (int c = 0; c < PL.nc; ++c) {
                    uint64_t s = 0, deg = (uint64_t)PL.d_inner[PL.d_of[c]];
                    for (int g = 0; g < PL.ng; ++g) deg += (uint64_t)(ex[g] * PL.d_cnt[PL.d_of[c]][g]);
                    for (int d = 0; d < PL.deg[c]; ++d) {
                        const int q = PL.nb[c][d];
                        s += q < PL.nc ? x[i][(size_t)l * PL.nc + q]
                                       : lds.at((size_t)PL.h_exp[q - PL.nc] * P::LANES + gb[PL.h_grp[q - PL.nc]]);
                    }
                    y[(size_t)l * PL.nc + c] = 3 * x[i][(size_t)l * PL.nc + c] + 5 * s + 7 * deg;
                }
            }
            x[i].swap(y);
            uint64_t bad = 0;
            for (uint64_t c = 0; c < T.cells; ++c) bad += x[i][c] != cur[tiles[i] * T.cells + c];
            EXPECT(bad == 0, "%s r=%d tile %llu step %d: %llu cells differ", pat.name, r, (unsigned long long)tiles[i], step,
                   (unsigned long long)bad);
        }
    }
    printf("%s level %d, blocks of level %d: %u lanes of %d, %d steps\n", pat.name, r, P::J, T.lanes, P::LANES, K);
}

// ---------------------------------------------------------------------------
// Bit rows
// ---------------------------------------------------------------------------
// Layer tables with a border of up to 32 cells, packed as gbox.hip packs them.
static void check_layers(const Pattern &pat, int M, int D)
{
    const FractalHost F = make(pat, M + 2);
    const int64_t B = ipow(pat.s, M);
    if (D > B) return;
    const uint32_t W = (uint32_t)(B + 2 * D + 31) / 32, P = 32 * W, rows = (uint32_t)(B + 2 * D);
    std::vector<XRingSlot> ring;
    std::vector<uint32_t> start;
    std::vector<uint16_t> lam;
    std::vector<uint8_t> mem;
    xtile_layer_tables(F, M, D, P, rows, ring, start, lam, mem);
    EXPECT((int)start.size() == D + 1 && start[0] == 0 && start.back() == ring.size(), "%s M=%d D=%d starts", pat.name, M, D);
    EXPECT((uint64_t)P * rows <= 65536 && ipow(pat.k, M) <= 8192, "%s M=%d D=%d: positions and cells fit their fields", pat.name, M, D);
    std::set<uint32_t> pos;
    size_t want = 0;
    for (int64_t y = -D; y < B + D; ++y)
        for (int64_t x = -D; x < B + D; ++x) {
            const int64_t tx = x < 0 ? -1 : (x >= B ? 1 : 0), ty = y < 0 ? -1 : (y >= B ? 1 : 0);
            want += (tx || ty) && host_nu(F, M, x - tx * B, y - ty * B) >= 0;
        }
    EXPECT(ring.size() == want, "%s M=%d D=%d: %zu border cells, want %zu", pat.name, M, D, ring.size(), want);
    for (int d = 1; d <= D; ++d)
        for (uint32_t i = start[d - 1]; i < start[d]; ++i) {
            const uint32_t p = ring[i].pos, dir = ring[i].info >> 16, cell = ring[i].info & 0xFFFFu;
            EXPECT(p < P * rows && dir < 8 && cell < ipow(pat.k, M) && pos.insert(p).second, "%s M=%d D=%d slot %u", pat.name, M, D, i);
            const int64_t x = (int64_t)(p % P) - D, y = (int64_t)(p / P) - D;
            const int64_t ex = x < 0 ? -x : (x >= B ? x - B + 1 : 0), ey = y < 0 ? -y : (y >= B ? y - B + 1 : 0);
            const int d9 = (int)(dir < 4 ? dir : dir + 1), tx = d9 % 3 - 1, ty = d9 / 3 - 1;
            EXPECT((ex > ey ? ex : ey) == d, "%s M=%d D=%d slot %u: layer", pat.name, M, D, i);
            EXPECT(host_nu(F, M, x - tx * B, y - ty * B) == (int64_t)cell, "%s M=%d D=%d slot %u: cell", pat.name, M, D, i);
        }
    for (size_t c = 0; c < lam.size(); ++c) {
        int64_t x, y;
        host_lambda(F, M, c, x, y);
        EXPECT(lam[c] == (uint32_t)(y + D) * P + (uint32_t)(x + D) && mem[lam[c]], "%s M=%d D=%d cell %zu", pat.name, M, D, c);
    }
}

// The carpet's bit rows with the kernel's own border and box.
static void check_bitbox(int M)
{
    const FractalHost F = make(kCar, M + 2);
    BitboxSpec S;
    S.M = M;
    S.border = kBxBorder;
    S.grid_pitch = kBxGP;
    S.rows = kBxRows;
    S.words = kBxW;
    std::vector<uint16_t> bpos;
    std::vector<uint32_t> ring, member;
    bitbox_tables(F, S, bpos, ring, member);
    const int64_t sb = ipow(3, M - 1), G = sb + 2 * kBxBorder, side = 3 * sb;
    EXPECT(bpos.size() == (size_t)ipow(8, M - 1) && member.size() == (size_t)kBxRows * kBxW, "bit rows M=%d sizes", M);
    std::set<uint32_t> pos;
    for (size_t b = 0; b < bpos.size(); ++b) {
        int64_t x, y;
        host_lambda(F, M - 1, b, x, y);
        EXPECT((bpos[b] & 127u) == (uint32_t)(x + kBxBorder) && (bpos[b] >> 7) == (uint32_t)(y + kBxBorder), "bit rows M=%d block %zu", M, b);
    }
    size_t want = 0;
    for (int64_t y = -kBxBorder; y < sb + kBxBorder; ++y)
        for (int64_t x = -kBxBorder; x < sb + kBxBorder; ++x) {
            const int64_t tx = x < 0 ? -1 : (x >= sb ? 1 : 0), ty = y < 0 ? -1 : (y >= sb ? 1 : 0);
            want += (tx || ty) && host_nu(F, M - 1, x - tx * sb, y - ty * sb) >= 0;
        }
    EXPECT(ring.size() == want, "bit rows M=%d: %zu border blocks, want %zu", M, ring.size(), want);
    for (uint32_t e : ring) {
        const uint32_t g = e & 0x3FFFu, dir = (e >> 14) & 15u, lb = e >> 18;
        const int64_t x = (int64_t)(g % kBxGP) - kBxBorder, y = (int64_t)(g / kBxGP) - kBxBorder;
        EXPECT(g < (uint32_t)(kBxGR * kBxGP) && x < G && y < G && dir < 9 && dir != 4 && pos.insert(g).second, "bit rows M=%d slot %x", M, e);
        EXPECT(host_nu(F, M - 1, x - ((int)(dir % 3) - 1) * sb, y - ((int)(dir / 3) - 1) * sb) == (int64_t)lb, "bit rows M=%d slot %x: block", M, e);
    }
    for (int64_t cy = 0; cy < kBxRows; ++cy)
        for (int64_t cx = 0; cx < 32 * kBxW; ++cx) {
            const int64_t x = cx - kBxBC, y = cy - kBxBC;
            const int64_t tx = x < 0 ? -1 : (x >= side ? 1 : 0), ty = y < 0 ? -1 : (y >= side ? 1 : 0);
            const bool in = cx < 3 * G && cy < 3 * G && host_nu(F, M, x - tx * side, y - ty * side) >= 0;
            EXPECT(((member[(size_t)cy * kBxW + cx / 32] >> (cx % 32)) & 1u) == in, "bit rows M=%d membership (%d, %d)", M, (int)cx, (int)cy);
        }
}

int main()
{
    check_slice_levels();
    check_slices<SliceTriSmall>(kTri, {5, 6, 7}, 0);
    check_slices<SliceTriSmall>(kTri, {8}, 3);
    check_slices<SliceTri>(kTri, {9, 10}, 2);
    check_slices<SliceTri>(kTri, {11}, 1);
    check_slices<SliceTriWide>(kTri, {11}, 1);
    check_slices<SlicePaperSmall>(kPaper, {5, 7}, 0);
    check_slices<SlicePaperSmall>(kPaper, {8}, 3);
    check_slices<SlicePaper>(kPaper, {9, 10}, 2);
    check_slices<SlicePaper>(kPaper, {11}, 1);
    check_slices<SlicePaperWide>(kPaper, {11}, 1);
    check_slices<SliceVicsekSmall>(kVic, {3, 4, 5}, 0);
    check_slices<SliceVicsekSmall>(kVic, {6}, 2);
    check_slices<SliceVicsekWide>(kVic, {7}, 2);
    for (int r : {1, 4, 6, 7, 9, 11, 12}) check_lane<LaneTriangleFine>(kTri, r);
    for (int r : {13}) check_lane<LaneTriangle>(kTri, r);
    for (int r : {6, 8, 10, 12}) check_lane<LaneTrianglePaperFine>(kPaper, r);
    for (int r : {13}) check_lane<LaneTrianglePaper>(kPaper, r);
    for (int r : {1, 3, 4, 5, 7, 8}) check_lane<LaneVicsekFine>(kVic, r);
    for (int r : {9}) check_lane<LaneVicsek>(kVic, r);
    for (int r : {1, 3, 4, 5, 6}) check_lane<LaneCarpetFine>(kCar, r);
    check_lane<LaneCarpetSmall>(kCar, 7);
    check_lane<LaneCarpet>(kCar, 6, 4, 8);
    check_lane<LaneTriangle>(kTri, 10, 1, 14);
    check_lane<LaneTrianglePaper>(kPaper, 10, 2, 14);
    for (int D : {4, 5, 8, 13, 16, 25, 32}) {
        for (int M = 1; M <= 3; ++M) check_layers(kWide, M, D);
        for (int M = 2; M <= 4; ++M) check_layers(kSix, M, D);
        for (int M = 3; M <= 6; ++M) check_layers(kSquare, M, D);
    }
    for (int M = 3; M <= 5; ++M) check_bitbox(M);
    if (g_fail) {
        fprintf(stderr, "%d check(s) failed\n", g_fail);
        return 1;
    }
    printf("all checks passed\n");
    return 0;
}
