// Diffusion with a block of cells per lane, several steps per launch (device
// code in lane_device.h): kernels, preparation and launches.
#include <algorithm>
#include <vector>

#include "lane_device.h"

namespace sqz {

template <class P, class Op>
__global__ void __launch_bounds__(P::LANES) __attribute__((amdgpu_waves_per_eu(P::FRAME ? 3 : 1)))
k_lane(LaneArgs A, const typename Op::G *__restrict__ in, typename Op::G *__restrict__ out, XOp op, int32_t steps)
{
    __shared__ __align__(16) uint32_t sm[LaneCfg<P, Op>::LDSW];
    lane_tile<P, Op>(A, in, out, xcd_remap(blockIdx.x, gridDim.x), op, steps, sm);
}

// The eight adjacent tiles of every tile.
__global__ void __launch_bounds__(256) k_lane_nb(MapParams Pc, uint64_t ntiles, uint32_t *__restrict__ nbt)
{
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < ntiles * 8; i += (uint64_t)gridDim.x * 256) {
        const int d8 = (int)(i & 7), d = d8 < 4 ? d8 : d8 + 1;
        uint32_t X, Y;
        lam_map32(Pc, (uint32_t)(i >> 3), X, Y);
        const uint64_t nt = nu_map(Pc, (int32_t)X + d % 3 - 1, (int32_t)Y + d / 3 - 1);
        nbt[i] = nt == kHole64 ? kNuHole32 : (uint32_t)nt;
    }
}

struct LaneConfig {
    int kind;
    int K;  // steps per launch (0: one tile, any number)
    LaneArgs A;
    uint32_t *d_tab;
};

void lane_release(FractalHost &F)
{
    if (!F.lane) return;
    (void)hipFree(F.lane->d_tab);
    delete F.lane;
    F.lane = nullptr;
}

sqz_status lane_prepare(FractalHost &F)
{
    F.lane = nullptr;
    const int kind = lane_kind(F);
    if (!kind) return SQZ_OK;
    uint32_t most = 0;
    const LaneSpec S = lane_spec(kind, F.r, most);
    LaneTables T;
    lane_tables(F, S, T);
    const uint64_t blocks = T.nblk * (F.N / T.cells);
    if (T.lanes > most || blocks >= 0xFFFFFFFFull) return SQZ_OK;  // left to the one-step kernels
    MapParams Pc;
    void *d_coarse = nullptr;
    sqz_status st = build_map_params(F, F.r - S.M, Pc, &d_coarse);
    if (st != SQZ_OK) return st;
    LaneConfig *L = new LaneConfig();
    L->kind = kind;
    L->K = T.K;
    L->A.ntiles = (uint32_t)(F.N / T.cells);
    L->A.nblk = T.nblk;
    L->A.lanes = T.lanes;
    std::vector<uint32_t> all(T.lane_src);
    all.insert(all.end(), T.lane_nb.begin(), T.lane_nb.end());
    hipError_t e = hipMalloc(&L->d_tab, (all.size() + (uint64_t)L->A.ntiles * 8) * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpy(L->d_tab, all.data(), all.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        L->A.lane_src = L->d_tab;
        L->A.lane_nb = L->d_tab + T.lane_src.size();
        L->A.nbtile = L->d_tab + all.size();
        const unsigned g = (unsigned)std::min<uint64_t>(((uint64_t)L->A.ntiles * 8 + 255) / 256, 16384);
        hipLaunchKernelGGL(k_lane_nb, dim3(g), dim3(256), 0, 0, Pc, L->A.ntiles, L->d_tab + all.size());
        e = hipGetLastError();
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    (void)hipFree(d_coarse);
    if (e != hipSuccess) {
        if (L->d_tab) (void)hipFree(L->d_tab);
        delete L;
        return hip_error(e, "lane table setup");
    }
    F.lane = L;
    return SQZ_OK;
}

bool lane_available(const FractalHost &F) { return F.lane != nullptr; }

// Launches of a single step: ahead of the expanded-tile kernel for the
// triangles (level 14: 16 against 27 us, level 16: 150 against 263) and large
// Vicsek crosses (level 10: 28 against 55; level 8: 7.9 against 6.6), behind
// it for the carpet (level 9: 263 against 238), whose box it fills densely.
bool lane_one_step(const FractalHost &F)
{
    const int kind = F.lane ? F.lane->kind : 0;
    return kind == 1 || kind == 2 || kind == 3 || kind == 6 || kind == 7;
}

// `steps` steps ping-ponging from a: launches of nearly equal step counts, at
// most K each, their number of the step count's parity (one more if need be),
// so that the result lands where one-step launches would leave it.
sqz_status lane_diffuse_run(const FractalHost &F, int dtype, float coef, int rounding, uint64_t seed, uint64_t first,
                            int steps, const void *a, void *b, hipStream_t st)
{
    const LaneConfig &L = *F.lane;
    if (steps < 1) return SQZ_OK;
    int64_t n = launch_count(steps, L.K);
    if ((n ^ steps) & 1) ++n;
    XOp op;
    op.coef = coef;
    op.rounding = (uint32_t)rounding;
    op.seed = seed;
    int32_t done = 0;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t k = launch_share(steps, n, i);
        op.step = first + (uint64_t)done;
        const void *in = (i & 1) ? b : a;
        void *out = (i & 1) ? const_cast<void *>(a) : b;
        if (k == 1 && !lane_one_step(F)) {
            const sqz_status s1 = launch_diffuse(F, dtype, coef, rounding, seed, op.step, in, out, 1, st);
            if (s1 != SQZ_OK) return s1;
            done += k;
            continue;
        }
        lane_dispatch(L.kind, [&](auto p) {
            using P = decltype(p);
            const dim3 block((L.A.lanes + 63) / 64 * 64);
            const dim3 grid(L.A.ntiles);
            auto launch = [&](auto o) {
                using Op = decltype(o);
                using G = typename Op::G;
                hipLaunchKernelGGL((k_lane<P, Op>), grid, block, 0, st, L.A, (const G *)in, (G *)out, op, k);
            };
            if (dtype == SQZ_F32)
                launch(LaneF32{});
            else if (rounding != SQZ_ROUND_STOCHASTIC)
                launch(LaneBF16<SQZ_ROUND_NEAREST_EVEN>{});
            else if (F.N <= 0x100000000ull)
                launch(LaneBF16<SQZ_ROUND_STOCHASTIC>{});
            else if constexpr (P::LARGE)
                launch(LaneBF16<SQZ_ROUND_STOCHASTIC, true>{});
            return 0;
        });
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_error(e, "diffusion (lane) launch");
        done += k;
    }
    return SQZ_OK;
}

}  // namespace sqz
