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

namespace {

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
int lane_kind(const FractalHost &F)
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
int lane_level(int kind, int r)
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

}  // namespace

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
    LaneSpec S{};
    S.M = lane_level(kind, F.r);
    int most = 0;
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
    LaneTables T;
    lane_tables(F, S, T);
    const uint64_t blocks = T.nblk * (F.N / T.cells);
    if (T.lanes > (uint32_t)most || blocks >= 0xFFFFFFFFull) return SQZ_OK;  // left to the one-step kernels
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
