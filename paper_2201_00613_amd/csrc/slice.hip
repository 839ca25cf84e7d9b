// Life on tiles bit-sliced across subtrees (device code in slice_device.h):
// kernels, preparation and launches.
#include <algorithm>
#include <vector>

#include "slice_device.h"

namespace sqz {

template <class P>
__global__ void __launch_bounds__(SliceCfg<P>::LANES)
k_slice(SliceArgs A, const uint8_t *in, uint8_t *out, SliceRing G, int32_t steps)
{
    __shared__ __align__(16) uint32_t sm[SliceCfg<P>::LDS / 4];
    slice_tile<P, false>(A, in, out, xcd_remap(blockIdx.x, gridDim.x), G, steps, SliceRes{}, sm, threadIdx.x,
                         blockDim.x);
}

// Resident run: one workgroup per tile, all on the chip at once.
template <class P>
__global__ void __launch_bounds__(SliceCfg<P>::LANES)
k_slice_run(SliceArgs A, uint8_t *a, uint8_t *b, int32_t steps, SliceRes R)
{
    __shared__ __align__(16) uint32_t sm[SliceCfg<P>::LDS / 4];
    slice_tile<P, true>(A, a, (steps & 1) ? b : a, xcd_remap(blockIdx.x, gridDim.x), SliceRing{a, false}, steps, R, sm,
                        threadIdx.x, blockDim.x);
}

// Every tile's corner subtrees, kSliceCornerPitch bytes each: a wave per subtree.
__global__ void __launch_bounds__(256) k_slice_corners(SliceArgs A, const uint8_t *__restrict__ in,
                                                       uint8_t *__restrict__ out)
{
    const uint64_t i = (uint64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (i >= A.ntiles * A.ncorner) return;
    const uint64_t t = i / A.ncorner;
    const uint32_t k = 4 * (threadIdx.x & 63);
    if (k >= A.rwords) return;
    const uint32_t o = k + 4 <= A.rwords ? k : A.rwords - 4;
    *reinterpret_cast<u32_u *>(out + i * kSliceCornerPitch + o) =
        *reinterpret_cast<const u32_u *>(in + t * A.cells + A.corner_off[i - t * A.ncorner] + o);
}

// Adjacent tile of every ring subtree of every tile.
__global__ void __launch_bounds__(256) k_slice_nb(MapParams Pc, uint64_t ntiles, uint32_t nring,
                                                  const int4 *__restrict__ ring, uint32_t *__restrict__ nbt)
{
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < ntiles * kSliceMaxRing; i += (uint64_t)gridDim.x * 256) {
        const uint64_t t = i / kSliceMaxRing;
        const uint32_t s = (uint32_t)(i % kSliceMaxRing);
        uint32_t v = kNuHole32;
        if (s < nring) {
            uint32_t X, Y;
            lam_map32(Pc, (uint32_t)t, X, Y);
            const uint64_t nt = nu_map(Pc, (int32_t)X + ring[s].x, (int32_t)Y + ring[s].y);
            if (nt != kHole64) v = (uint32_t)nt;
        }
        nbt[i] = v;
    }
}

__global__ void __launch_bounds__(256) k_slice_clear(uint32_t *p, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) p[i] = 0;
}

namespace {

unsigned slice_threads(const SliceConfig &S) { return (S.A.lanes + 63) / 64 * 64; }

}  // namespace

void slice_free(SliceConfig *S)
{
    if (!S) return;
    (void)hipFree(S->d_tab);
    if (S->d_res) (void)hipFree(S->d_res);
    if (S->R.flag) (void)hipHostFree(S->R.flag);
    delete S;
}

void slice_release(FractalHost &F)
{
    slice_free(F.slice);
    F.slice = nullptr;
}

// Tables of tiles of level M for kernel `var`; *out stays null where a subtile
// would be smaller than a block.
static sqz_status slice_build(const FractalHost &F, int M, int var, SliceConfig **out)
{
    *out = nullptr;
    const int kind = slice_kind(F);
    SliceTables T;
    bool small = false;
    sqz_status st = slice_dispatch(kind, var, [&](auto p) {
        using P = decltype(p);
        small = M - P::B < P::J;
        return small ? SQZ_OK : slice_tables(F, slice_spec<P>(M), T);
    });
    if (st != SQZ_OK || small) return st;
    SliceConfig *S = new SliceConfig();
    S->kind = kind;
    S->var = var;
    MapParams Pc;
    void *d_coarse = nullptr;
    if (T.nring) st = build_map_params(F, F.r - M, Pc, &d_coarse);
    if (st != SQZ_OK) {
        delete S;
        return st;
    }
    SliceArgs &A = S->A;
    A.cells = 1;
    for (int i = 0; i < M; ++i) A.cells *= (uint32_t)F.k;
    A.ntiles = F.N / A.cells;
    A.words = T.words;
    A.nblk = T.nblk;
    A.lanes = (uint32_t)T.lane_block.size();
    A.rwords = T.rwords;
    A.nring = T.nring;
    A.ncorner = (uint32_t)T.corner.size();
    for (uint32_t s = 0; s < T.nring; ++s) {
        A.ring_off[s] = (uint32_t)T.ring[4 * s + 2];
        A.ring_corner[s] = (uint32_t)T.ring[4 * s + 3];
    }
    for (uint32_t c = 0; c < A.ncorner; ++c) A.corner_off[c] = T.corner[c];
    S->K = T.K;
    // one allocation: the tables, then the adjacent tiles
    std::vector<uint32_t> all(T.lane_block);
    const size_t o_halo = all.size();
    all.insert(all.end(), T.lane_halo.begin(), T.lane_halo.end());
    const size_t o_perm = all.size();
    all.insert(all.end(), T.perm.begin(), T.perm.end());
    const size_t o_ring = (all.size() + 3) / 4 * 4;
    all.resize(o_ring);
    for (int32_t v : T.ring) all.push_back((uint32_t)v);
    const size_t o_nb = all.size();
    hipError_t e = hipMalloc(&S->d_tab, (o_nb + A.ntiles * kSliceMaxRing) * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpy(S->d_tab, all.data(), all.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        A.lane_block = S->d_tab;
        A.lane_halo = S->d_tab + o_halo;
        A.perm = S->d_tab + o_perm;
        A.nbtile = S->d_tab + o_nb;
        if (T.nring) {
            const unsigned g = (unsigned)std::min<uint64_t>((A.ntiles * kSliceMaxRing + 255) / 256, 16384);
            hipLaunchKernelGGL(k_slice_nb, dim3(g), dim3(256), 0, 0, Pc, A.ntiles, A.nring,
                               reinterpret_cast<const int4 *>(S->d_tab + o_ring), S->d_tab + o_nb);
        } else {  // no adjacent tile is looked up
            hipLaunchKernelGGL(k_slice_clear, dim3(1), dim3(256), 0, 0, S->d_tab + o_nb, A.ntiles * kSliceMaxRing);
        }
        e = hipGetLastError();
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    if (d_coarse) (void)hipFree(d_coarse);
    if (e != hipSuccess) {
        if (S->d_tab) (void)hipFree(S->d_tab);
        delete S;
        return hip_error(e, "slice table setup");
    }
    *out = S;
    return SQZ_OK;
}

// Every pattern with a bit-sliced tile from the level at which a subtile
// holds a block.
sqz_status slice_prepare(FractalHost &F)
{
    F.slice = nullptr;
    if (!F.tile_kind || !F.tile) return SQZ_OK;
    int M, var;
    slice_levels(slice_kind(F), F.r, M, var);
    return slice_build(F, M, var, &F.slice);
}

sqz_status slice_batch_config(const FractalHost &F, SliceConfig **out, bool *own)
{
    *own = true;
    *out = F.slice;
    if (!F.slice || F.slice->var == 0) return SQZ_OK;
    *own = false;
    return slice_build(F, slice_kind(F) == 3 ? 6 : 8, 0, out);
}

// State of the resident run, where the fractal offers one and all tiles are
// surely on the chip at once.  Failure to set it up leaves it unavailable.
void slice_prepare_resident(FractalHost &F)
{
    SliceConfig *S = F.slice;
    if (!S || !tile_few(F)) return;
    const unsigned nt = slice_threads(*S);
    int per_cu = 0, cus = 0;
    int nc = 0;
    const hipError_t q = slice_dispatch(S->kind, S->var, [&](auto p) {
        using P = decltype(p);
        nc = SlicePlanOf<P, P::J>::value.nc;
        if constexpr (P::J == (P::B == 2 ? 2 : 3)) {
            return hipErrorNotSupported;  // the wide kernels have no resident form
        } else {
        hipError_t r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_slice_run<P>, (int)nt, 0);
        hipFuncAttributes fa;
        if (r == hipSuccess) r = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(k_slice_run<P>));
        if (r == hipSuccess) {  // a workgroup's waves are dealt to four SIMDs: the fullest one bounds the count
            const int vgprs = fa.numRegs > 0 ? (fa.numRegs + 7) / 8 * 8 : 512;
            per_cu = std::min(per_cu, std::min(8, 512 / vgprs) / (int)((nt / 64 + 3) / 4));
        }
        return r;
        }
    });
    if (q != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, F.device) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (per_cu < 1 || S->A.ntiles > (uint64_t)per_cu * (uint64_t)cus) return;
    const uint64_t nx = 2 * S->A.ntiles * S->A.ncorner * (S->A.rwords / (uint32_t)nc);
    S->res_words = nx + 2 * S->A.ntiles + 1;
    uint32_t *d = nullptr, *h = nullptr;
    hipError_t e = hipMalloc(&d, S->res_words * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemset(d, 0, S->res_words * sizeof(uint32_t));
    if (e == hipSuccess) e = hipHostMalloc(&h, sizeof(uint32_t), hipHostMallocMapped | hipHostMallocCoherent);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (d) (void)hipFree(d);
        return;
    }
    *h = 0;
    S->d_res = d;
    S->R.xch = d;
    S->R.epoch = d + nx;
    S->R.loaded = S->R.epoch + S->A.ntiles;
    S->R.dead = S->R.loaded + S->A.ntiles;
    S->R.flag = h;
    S->R.K = S->K;
}

bool slice_available(const FractalHost &F) { return F.slice != nullptr; }
bool slice_resident(const FractalHost &F) { return F.slice && F.slice->d_res; }

sqz_status slice_run_resident(const FractalHost &F, uint8_t *a, uint8_t *b, int steps, hipStream_t st)
{
    const SliceConfig &S = *F.slice;
    if (__atomic_exchange_n(S.R.flag, 0u, __ATOMIC_ACQ_REL)) {
        // the epochs of the failed run are unknown: clear them for the next run
        hipLaunchKernelGGL(k_slice_clear, dim3(64), dim3(256), 0, st, S.d_res, S.res_words);
        (void)hipGetLastError();
        return set_error(SQZ_ERR_HIP, "a wait of an earlier resident run timed out: its result is invalid");
    }
    if (steps < 1) return SQZ_OK;
    // Without an exchange and with the result in the other buffer the launch
    // needs no state: the plain kernel, whose tiles wait for nothing (25 steps:
    // level-13 triangle 13.2 -> 11.6 us, level-9 Vicsek 11.0 -> 10.2).
    if (!S.K || (steps <= (int)S.K && (steps & 1))) return slice_run_launches(F, a, b, steps, st);
    slice_dispatch(S.kind, S.var, [&](auto p) {
        using P = decltype(p);
        if constexpr (P::J < (P::B == 2 ? 2 : 3))
            hipLaunchKernelGGL(k_slice_run<P>, dim3((unsigned)S.A.ntiles), dim3(slice_threads(S)), 0, st, S.A, a, b,
                               steps, S.R);
        return 0;
    });
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SQZ_OK : hip_error(e, "resident run launch");
}

// `steps` steps from a; the result in a (even) or b (odd).  Launches of nearly
// equal step counts, at most K each, swap the buffers; where their number has
// the other parity the last one updates its buffer in place, reading its ring
// subtrees from a copy of all corner subtrees in the other buffer (768 bytes a
// tile, a small launch before it) instead of costing a launch over all cells.
sqz_status slice_run_launches(const FractalHost &F, uint8_t *a, uint8_t *b, int steps, hipStream_t st)
{
    const SliceConfig &S = *F.slice;
    if (steps < 1) return SQZ_OK;
    const int64_t n = launch_count(steps, (int)S.K);
    uint8_t *cur = a, *other = b;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t k = launch_share(steps, n, i);
        const bool in_place = i == n - 1 && ((n ^ steps) & 1);
        if (in_place && S.A.nring)
            hipLaunchKernelGGL(k_slice_corners, dim3((unsigned)((S.A.ntiles * S.A.ncorner + 3) / 4)), dim3(256), 0, st,
                               S.A, cur, other);
        const SliceRing G{in_place ? other : cur, in_place};
        uint8_t *dst = in_place ? cur : other;
        slice_dispatch(S.kind, S.var, [&](auto p) {
            hipLaunchKernelGGL(k_slice<decltype(p)>, dim3((unsigned)S.A.ntiles), dim3(slice_threads(S)), 0, st, S.A,
                               cur, dst, G, k);
            return 0;
        });
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_error(e, "compact run (slice) launch");
        if (!in_place) std::swap(cur, other);
    }
    return SQZ_OK;
}

}  // namespace sqz
