// Thread-level kernels: the two space maps, the seeded starts and the
// thread-level Squeeze Life step (one lambda and eight nu per cell,
// Section "Exploring Compact Fractal Space").
#include <algorithm>

#include "common.h"

namespace sqz {

namespace {

constexpr int kBlock = 256;

// Grid for a grid-stride loop over `count` items: enough workgroups to fill
// the device several times over, capped so 64-bit counters stay cheap.
inline unsigned grid_for(uint64_t count)
{
    uint64_t g = (count + kBlock - 1) / kBlock;
    if (g > 16384) g = 16384;
    if (g == 0) g = 1;
    return (unsigned)g;
}

__device__ __forceinline__ void lam_any(const MapParams &P, uint64_t c, uint32_t &x, uint32_t &y)
{
    if (P.N <= 0x100000000ull)
        lam_map32(P, (uint32_t)c, x, y);
    else
        lam_map64(P, c, x, y);
}

// The standalone maps stream their inputs from HBM: each lane takes kMapUnroll
// elements (kBlock apart, so every load instruction stays coalesced) per pass
// and issues all their loads before the first map, so the memory latency is
// paid once per kMapUnroll elements instead of once per element.
#ifndef SQZ_MAP_UNROLL
#define SQZ_MAP_UNROLL 8
#endif
constexpr int kMapUnroll = SQZ_MAP_UNROLL;

// Elements are taken in pairs (16-byte loads and stores, at any alignment of
// the buffers).  From kMapLarge elements on (LARGE) the loads and stores are
// nontemporal, since nothing is read twice, and lambda too reads its tables
// from LDS: its random reads were bound by the vector cache.  43 million
// elements, level-16 triangle: lambda 180 -> 120 us, nu 140 -> 130 (5.7 and 5.3
// TB/s).  Below, copying the tables costs lambda what it saves (1e6 elements:
// 6.8 us without, 6.0 with; 7-digit carpet 5.6 and 6.0; 3e4: 5.7 and 6.0).
template <class G, int N>
struct MapVec {  // N elements at any element address
    typedef G T __attribute__((ext_vector_type(N), aligned(sizeof(G))));
};
using map_u64x2 = MapVec<uint64_t, 2>::T;
using map_i32x4 = MapVec<int32_t, 4>::T;
using map_i32x2 = MapVec<int32_t, 2>::T;
static_assert(kMapUnroll % 2 == 0, "pairs");
constexpr int64_t kMapLarge = 1 << 20;

template <bool LARGE, int N, class G>
__device__ __forceinline__ typename MapVec<G, N>::T map_load(const G *p)
{
    const auto *q = reinterpret_cast<const typename MapVec<G, N>::T *>(p);
    if constexpr (LARGE)
        return __builtin_nontemporal_load(q);
    else
        return *q;
}

template <bool LARGE, int N, class G>
__device__ __forceinline__ void map_store(const typename MapVec<G, N>::T &v, G *p)
{
    auto *q = reinterpret_cast<typename MapVec<G, N>::T *>(p);
    if constexpr (LARGE)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

template <bool LARGE>
__global__ void __launch_bounds__(kBlock) k_lambda(MapParams P, const uint64_t *__restrict__ idx, int64_t count,
                                                   int32_t *__restrict__ xy)
{
    extern __shared__ uint32_t s_lam[];
    MapParams L = P;
    if constexpr (LARGE) {
        const uint32_t nwords = (uint32_t)(P.nu_lo - P.lam_lo);
        for (uint32_t i = threadIdx.x; i < nwords; i += kBlock) s_lam[i] = P.lam_lo[i];
        __syncthreads();
        L.lam_lo = s_lam;
        L.lam_top = s_lam + (P.lam_top - P.lam_lo);
    }
    auto map = [&](uint64_t c) {
        uint32_t x = ~0u, y = ~0u;
        if (c < P.N) lam_any(L, c, x, y);
        return make_int2((int)x, (int)y);
    };
    const int64_t stride = (int64_t)gridDim.x * kBlock * kMapUnroll;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock * kMapUnroll + 2 * threadIdx.x; i0 < count; i0 += stride) {
        if (i0 - 2 * threadIdx.x + kMapUnroll * kBlock <= count) {  // a whole pass (the same for every lane)
            map_u64x2 c[kMapUnroll / 2];
#pragma unroll
            for (int u = 0; u < kMapUnroll / 2; ++u)
                c[u] = map_load<LARGE, 2>(idx + i0 + 2 * u * kBlock);
#pragma unroll
            for (int u = 0; u < kMapUnroll / 2; ++u) {
                const int2 p = map(c[u].x), q = map(c[u].y);
                const map_i32x4 o = {p.x, p.y, q.x, q.y};
                map_store<LARGE, 4>(o, xy + 2 * (i0 + 2 * u * kBlock));
            }
        } else {
            uint64_t c[kMapUnroll];
#pragma unroll
            for (int u = 0; u < kMapUnroll; ++u) {
                const int64_t i = i0 + (u / 2) * 2 * kBlock + (u & 1);
                c[u] = i < count ? idx[i] : ~0ull;
            }
#pragma unroll
            for (int u = 0; u < kMapUnroll; ++u) {
                const int64_t i = i0 + (u / 2) * 2 * kBlock + (u & 1);
                if (i < count) {
                    const int2 p = map(c[u]);
                    const map_i32x2 o = {p.x, p.y};
                    *reinterpret_cast<map_i32x2 *>(xy + 2 * i) = o;
                }
            }
        }
    }
}

// nu reads three table entries per point; each workgroup first copies the two
// nu tables into LDS (at most 2 x 4096 words) and then strides over the points.
template <bool LARGE>
__global__ void __launch_bounds__(kBlock) k_nu(MapParams P, const int32_t *__restrict__ xy, int64_t count,
                                               uint64_t *__restrict__ idx)
{
    extern __shared__ uint32_t s_nu[];
    const uint32_t nwords = P.ntab - (uint32_t)(P.nu_lo - P.lam_lo);
    for (uint32_t i = threadIdx.x; i < nwords; i += kBlock) s_nu[i] = P.nu_lo[i];
    __syncthreads();
    MapParams L = P;
    L.nu_lo = s_nu;
    L.nu_top = s_nu + (P.nu_top - P.nu_lo);
    const int64_t stride = (int64_t)gridDim.x * kBlock * kMapUnroll;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock * kMapUnroll + 2 * threadIdx.x; i0 < count; i0 += stride) {
        if (i0 - 2 * threadIdx.x + kMapUnroll * kBlock <= count) {  // a whole pass (the same for every lane)
            map_i32x4 p[kMapUnroll / 2];
#pragma unroll
            for (int u = 0; u < kMapUnroll / 2; ++u)
                p[u] = map_load<LARGE, 4>(xy + 2 * (i0 + 2 * u * kBlock));
#pragma unroll
            for (int u = 0; u < kMapUnroll / 2; ++u) {
                const map_u64x2 o = {nu_map(L, p[u].x, p[u].y), nu_map(L, p[u].z, p[u].w)};
                map_store<LARGE, 2>(o, idx + i0 + 2 * u * kBlock);
            }
        } else {
            map_i32x2 p[kMapUnroll];
#pragma unroll
            for (int u = 0; u < kMapUnroll; ++u) {
                const int64_t i = i0 + (u / 2) * 2 * kBlock + (u & 1);
                p[u] = (map_i32x2)0;
                if (i < count) p[u] = *reinterpret_cast<const map_i32x2 *>(xy + 2 * i);
            }
#pragma unroll
            for (int u = 0; u < kMapUnroll; ++u) {
                const int64_t i = i0 + (u / 2) * 2 * kBlock + (u & 1);
                if (i < count) idx[i] = nu_map(L, p[u].x, p[u].y);
            }
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_fill_compact(MapParams P, uint64_t seed, uint32_t thresh,
                                                         uint8_t *__restrict__ out)
{
    for (uint64_t c = (uint64_t)blockIdx.x * kBlock + threadIdx.x; c < P.N; c += (uint64_t)gridDim.x * kBlock) {
        uint32_t x, y;
        lam_any(P, c, x, y);
        uint64_t h = splitmix64_at(seed, (uint64_t)y * (uint64_t)P.n + x);
        out[c] = (uint8_t)((uint32_t)(h >> 40) < thresh);
    }
}

__global__ void __launch_bounds__(kBlock) k_fill_expanded(MapParams P, uint64_t seed, uint32_t thresh,
                                                          uint8_t *__restrict__ out)
{
    const uint64_t total = (uint64_t)P.n * (uint64_t)P.n;
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (uint64_t)gridDim.x * kBlock) {
        uint32_t y = (uint32_t)(i / (uint32_t)P.n), x = (uint32_t)(i - (uint64_t)y * P.n);
        uint8_t v = 0;
        if (nu_map(P, (int32_t)x, (int32_t)y) != kHole64) v = (uint8_t)((uint32_t)(splitmix64_at(seed, i) >> 40) < thresh);
        out[i] = v;
    }
}

__global__ void __launch_bounds__(kBlock) k_fill_uniform(MapParams P, uint64_t seed, float *__restrict__ out)
{
    for (uint64_t c = (uint64_t)blockIdx.x * kBlock + threadIdx.x; c < P.N; c += (uint64_t)gridDim.x * kBlock) {
        uint32_t x, y;
        lam_any(P, c, x, y);
        uint64_t h = splitmix64_at(seed, (uint64_t)y * (uint64_t)P.n + x);
        out[c] = (float)(uint32_t)(h >> 40) * (1.0f / 16777216.0f);
    }
}

// B3/S23 on the fractal: a member neighbour counts its state; a hole or a
// point outside the box counts nothing.
// One lambda and eight nu per cell make about 27 map-table reads per cell,
// scattered over tables of at most 4 x 4096 words.  Each workgroup copies
// the tables into LDS once and then strides over the cells, so those reads
// are LDS reads rather than divergent vector-memory gathers; only the nine
// state bytes per cell come through the vector-memory path.
constexpr int kCellBlock = 512;

__global__ void __launch_bounds__(kCellBlock) k_life_cell(MapParams P, const uint8_t *__restrict__ in,
                                                          uint8_t *__restrict__ out)
{
    extern __shared__ uint32_t s_tab[];
    for (uint32_t i = threadIdx.x; i < P.ntab; i += kCellBlock) s_tab[i] = P.lam_lo[i];
    __syncthreads();
    MapParams L = P;
    L.lam_lo = s_tab;
    L.lam_top = s_tab + (P.lam_top - P.lam_lo);
    L.nu_lo = s_tab + (P.nu_lo - P.lam_lo);
    L.nu_top = s_tab + (P.nu_top - P.lam_lo);
    for (uint64_t c = (uint64_t)blockIdx.x * kCellBlock + threadIdx.x; c < P.N;
         c += (uint64_t)gridDim.x * kCellBlock) {
        uint32_t x, y;
        lam_any(L, c, x, y);
        uint32_t cnt = 0;
        if (P.nnu >= 2) {
            // A neighbour inside the centre's lowest nu chunk shares every
            // higher chunk with it, so its index is the centre's with the
            // lowest chunk's digits replaced (nu(lambda(c)) = c): one table
            // read instead of a full nu.  Neighbours across the chunk edge
            // take the full map.
            const uint32_t hx = divq(x, P.dsnu), hy = divq(y, P.dsnu);
            const uint32_t lx = x - hx * P.snu, ly = y - hy * P.snu;
            const uint64_t chi = c - L.nu_lo[lx + P.snu * ly];
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                if (j == 4) continue;
                const int dx = j % 3 - 1, dy = j / 3 - 1;
                const uint32_t nx = lx + (uint32_t)dx, ny = ly + (uint32_t)dy;
                uint64_t q;
                if (nx < P.snu && ny < P.snu) {
                    const uint32_t e = L.nu_lo[nx + P.snu * ny];
                    q = e == kNuHole32 ? kHole64 : chi + e;
                } else {
                    q = nu_map(L, (int32_t)x + dx, (int32_t)y + dy);
                }
                if (q != kHole64) cnt += in[q];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                if (j == 4) continue;
                int dx = j % 3 - 1, dy = j / 3 - 1;
                uint64_t q = nu_map(L, (int32_t)x + dx, (int32_t)y + dy);
                if (q != kHole64) cnt += in[q];
            }
        }
        uint32_t self = in[c];
        out[c] = (uint8_t)(cnt == 3 || (self && cnt == 2));
    }
}

// A whole run of a fractal of at most kSmallCells cells: one workgroup, a lane
// per cell, the neighbours found once through the maps and the states in LDS.
// Bound by the latency of a step (eight LDS bytes, a barrier); the kernels for
// larger fractals spend more than that on a step, and a launch per few steps
// (50 steps, byte tiles before: triangle 729 cells 34.7 -> 15.7 us, carpet 512
// cells 68.4 -> 13.5, ten-of-sixteen 1000 cells 145 -> 18.4).
__global__ void __launch_bounds__(kSmallCells) k_life_small(MapParams P, const uint8_t *in, uint8_t *out, int32_t steps)
{
    __shared__ uint8_t s_v[2][kSmallCells + 64];
    const uint32_t c = threadIdx.x, N = (uint32_t)P.N;
    uint32_t q[8], v = 0;
    if (c < N) {
        uint32_t x, y;
        lam_map32(P, c, x, y);
#pragma unroll
        for (int j = 0, i = 0; j < 9; ++j) {
            if (j == 4) continue;
            const uint64_t n = nu_map(P, (int32_t)x + j % 3 - 1, (int32_t)y + j / 3 - 1);
            q[i++] = n == kHole64 ? N : (uint32_t)n;  // byte N stays 0
        }
        v = in[c] & 1u;
        s_v[0][c] = (uint8_t)v;
    }
    if (c < 2) s_v[c][N] = 0;
    __syncthreads();
    for (int32_t s = 0; s < steps; ++s) {
        const uint8_t *src = s_v[s & 1];
        if (c < N) {
            uint32_t cnt = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) cnt += src[q[i]];
            v = cnt == 3 || (v && cnt == 2);
            s_v[~s & 1][c] = (uint8_t)v;
        }
        __syncthreads();
    }
    if (c < N) out[c] = (uint8_t)v;
}

sqz_status after_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SQZ_OK : hip_error(e, what);
}

}  // namespace

// Grid of a map kernel that copies `lds` bytes of tables per workgroup: as many
// workgroups as are resident at once, and no more than the points need.
template <class K>
static sqz_status map_grid(K kernel, size_t lds, int64_t count, unsigned &grid)
{
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, lds);
    if (e != hipSuccess) return hip_error(e, "map occupancy");
    if (per_cu < 1) return set_error(SQZ_ERR_UNSUPPORTED, "map tables (%zu B) do not fit in LDS", lds);
    const uint64_t need = ((uint64_t)count + (uint64_t)kBlock * kMapUnroll - 1) / ((uint64_t)kBlock * kMapUnroll);
    grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(need, (uint64_t)cus * per_cu));
    return SQZ_OK;
}

sqz_status launch_lambda(const MapParams &P, const uint64_t *idx, int64_t count, int32_t *xy, hipStream_t st)
{
    const size_t lds = (size_t)(P.nu_lo - P.lam_lo) * sizeof(uint32_t);
    unsigned grid = 0;
    if (count >= kMapLarge) {
        const sqz_status s = map_grid(k_lambda<true>, lds, count, grid);
        if (s != SQZ_OK) return s;
        hipLaunchKernelGGL(k_lambda<true>, dim3(grid), dim3(kBlock), lds, st, P, idx, count, xy);
    } else {
        grid = grid_for(((uint64_t)count + kMapUnroll - 1) / kMapUnroll);
        hipLaunchKernelGGL(k_lambda<false>, dim3(grid), dim3(kBlock), 0, st, P, idx, count, xy);
    }
    return after_launch("lambda_map launch");
}

sqz_status launch_nu(const MapParams &P, const int32_t *xy, int64_t count, uint64_t *idx, hipStream_t st)
{
    const size_t lds = (size_t)(P.ntab - (uint32_t)(P.nu_lo - P.lam_lo)) * sizeof(uint32_t);
    const auto kernel = count >= kMapLarge ? k_nu<true> : k_nu<false>;
    unsigned grid = 0;
    const sqz_status s = map_grid(kernel, lds, count, grid);
    if (s != SQZ_OK) return s;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), lds, st, P, xy, count, idx);
    return after_launch("nu_map launch");
}

sqz_status launch_fill_bernoulli(const MapParams &P, uint64_t seed, uint32_t thresh24, int expanded, uint8_t *out,
                                 hipStream_t st)
{
    if (expanded) {
        uint64_t total = (uint64_t)P.n * (uint64_t)P.n;
        hipLaunchKernelGGL(k_fill_expanded, dim3(grid_for(total)), dim3(kBlock), 0, st, P, seed, thresh24, out);
    } else {
        hipLaunchKernelGGL(k_fill_compact, dim3(grid_for(P.N)), dim3(kBlock), 0, st, P, seed, thresh24, out);
    }
    return after_launch("fill_bernoulli launch");
}

sqz_status launch_fill_uniform(const MapParams &P, uint64_t seed, float *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_uniform, dim3(grid_for(P.N)), dim3(kBlock), 0, st, P, seed, out);
    return after_launch("fill_uniform launch");
}

sqz_status launch_life_cell(const MapParams &P, const uint8_t *in, uint8_t *out, hipStream_t st)
{
    // as many workgroups as are resident at once: each copies the tables once
    const size_t lds = (size_t)P.ntab * sizeof(uint32_t);
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_life_cell, kCellBlock, lds);
    if (e != hipSuccess) return hip_error(e, "compact_step (cell) occupancy");
    if (per_cu < 1) return set_error(SQZ_ERR_UNSUPPORTED, "map tables (%zu B) do not fit in LDS", lds);
    uint64_t grid = (P.N + kCellBlock - 1) / kCellBlock;
    if (grid > (uint64_t)cus * per_cu) grid = (uint64_t)cus * per_cu;
    if (grid == 0) grid = 1;
    hipLaunchKernelGGL(k_life_cell, dim3((unsigned)grid), dim3(kCellBlock), lds, st, P, in, out);
    return after_launch("compact_step (cell) launch");
}

sqz_status launch_life_small(const MapParams &P, const uint8_t *in, uint8_t *out, int steps, hipStream_t st)
{
    hipLaunchKernelGGL(k_life_small, dim3(1), dim3((unsigned)((P.N + 63) / 64 * 64)), 0, st, P, in, out, steps);
    return after_launch("compact run (small) launch");
}

}  // namespace sqz
