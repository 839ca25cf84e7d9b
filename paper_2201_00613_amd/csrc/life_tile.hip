// Bit-sliced block-level Life kernels (device code in tile_device.h) and
// their host-side preparation: tile halo slots, block-halo tables, per-tile
// halo indices.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "tile_device.h"

namespace sqz {

#ifndef SQZ_TILE_NT  // lanes per workgroup of the compact tiled kernels
#define SQZ_TILE_NT 256
#endif
constexpr int kTileNT = SQZ_TILE_NT;

#ifndef SQZ_BIG_NT  // lanes per workgroup of the level-10 triangle tiles
#define SQZ_BIG_NT 512
#endif
// Lanes per workgroup of a pattern's tiled kernels: SQZ_BIG_NT for the
// level-10 tiles of large triangles (2,187 blocks), else kTileNT.
template <class Pat>
constexpr int nt_of()
{
    return std::is_same<Pat, PatTriangleBig>::value ? SQZ_BIG_NT : kTileNT;
}

template <class Pat, int NT>
__global__ void __launch_bounds__(NT) k_life_tile(TileArgs A, const uint8_t *__restrict__ in,
                                                  uint8_t *__restrict__ out)
{
    using LDS = TileLds<Pat>;
    __shared__ uint32_t s_in[LDS::WORDS];
    __shared__ uint32_t s_out[LDS::WORDS];
    const uint32_t G = gridDim.x;
    for (uint64_t round = 0; round * G < A.ntiles; ++round) {
        const uint64_t t = round * G + xcd_remap(blockIdx.x, G);
        if (t >= A.ntiles) break;  // uniform across the workgroup
        tile_body<Pat, NT>(A, in, out, t, s_in, s_out);
    }
}

// Tile-halo cells of every tile: global compact index of each slot's cell.
__global__ void __launch_bounds__(kBlock) k_tile_halo(MapParams Pc, uint64_t ntiles, uint32_t nthalo,
                                                      uint64_t tile_cells, const int4 *__restrict__ slots,
                                                      uint64_t *__restrict__ outp)
{
    for (uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x; t < ntiles; t += (uint64_t)gridDim.x * kBlock) {
        uint32_t X, Y;
        if (Pc.N <= 0x100000000ull)
            lam_map32(Pc, (uint32_t)t, X, Y);
        else
            lam_map64(Pc, t, X, Y);
        for (uint32_t j = 0; j < nthalo; ++j) {
            const int4 sl = slots[j];  // (tile dx, tile dy, cell index in that tile, unused)
            const uint64_t nt = nu_map(Pc, (int32_t)X + sl.x, (int32_t)Y + sl.y);
            outp[t * nthalo + j] = nt == kHole64 ? kHole64 : nt * tile_cells + (uint64_t)sl.z;
        }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
namespace {

template <class Pat>
bool matches(const FractalHost &F)
{
    if (F.s != Pat::S || F.k != Pat::K) return false;
    for (int j = 0; j < Pat::K; ++j)
        if (F.ox[j] != Pat::OX[j] || F.oy[j] != Pat::OY[j]) return false;
    return true;
}

template <class Pat>
sqz_status prepare(FractalHost &F)
{
    constexpr const BlockPlan &PL = PlanOf<Pat>::value;
    using LDS = TileLds<Pat>;
    TileConfig *T = new TileConfig();
    const int mtop = F.r >= Pat::MBIG ? Pat::MMAX : (Pat::MSMALL < Pat::MMAX ? Pat::MSMALL : Pat::MMAX);
    T->M = F.r < mtop ? F.r : mtop;
    const int M = T->M;
    T->tile = (uint32_t)cpow(Pat::K, M);
    T->nblocks = (uint32_t)cpow(Pat::K, M - Pat::J);

    // tables of the tile (the same for every tile): rings, halos, LDS entries
    TileSpec S;
    S.M = M;
    S.J = Pat::J;
    S.nc = PL.nc;
    S.box = PL.box;
    S.ngrp = PL.ngrp;
    for (int g = 0; g < 8; ++g) {
        S.g_dx[g] = g < PL.ngrp ? PL.g_dx[g] : 0;
        S.g_dy[g] = g < PL.ngrp ? PL.g_dy[g] : 0;
    }
    S.lds_zero = LDS::ZERO;
    S.lds_virt = LDS::VIRT;
    S.lds_ring2 = LDS::WORDS;
    S.max_tile_halo = kMaxTileHalo;
    S.max_ring = kMaxTileHalo;
    S.max_steps = 1;
    TileTables TT;
    if (tile_tables(F, S, TT) != SQZ_OK) {
        delete T;
        return SQZ_ERR_UNSUPPORTED;
    }
    T->nthalo = TT.nthalo;
    T->nbstride = TT.nbstride;
    const std::vector<uint32_t> &nbt = TT.nbt, &home = TT.home;

    // coarse maps and per-tile halo indices
    sqz_status st = build_map_params(F, F.r - M, T->Pc, &T->d_coarse_tables);
    if (st != SQZ_OK) {
        delete T;
        return st;
    }
    T->ntiles = T->Pc.N;
    T->d_nbtab = nullptr;
    T->d_tile_halo = nullptr;
    T->d_ringhome = nullptr;
    int4 *d_slots = nullptr;
    std::vector<int4> hs(T->nthalo ? T->nthalo : 1, make_int4(0, 0, 0, 0));
    for (size_t s = 0; s < T->nthalo; ++s)
        hs[s] = make_int4(TT.slots[4 * s], TT.slots[4 * s + 1], TT.slots[4 * s + 2], 0);
    auto upload = [](uint32_t **d, const std::vector<uint32_t> &h) {
        hipError_t e = hipMalloc(d, h.size() * sizeof(uint32_t));
        return e == hipSuccess ? hipMemcpy(*d, h.data(), h.size() * sizeof(uint32_t), hipMemcpyHostToDevice) : e;
    };
    hipError_t e = upload(&T->d_nbtab, nbt);
    if (e == hipSuccess) e = upload(&T->d_ringhome, home);
    if (e == hipSuccess)
        e = hipMalloc(&T->d_tile_halo, (size_t)T->ntiles * (T->nthalo ? T->nthalo : 1) * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc(&d_slots, hs.size() * sizeof(int4));
    if (e == hipSuccess) e = hipMemcpy(d_slots, hs.data(), hs.size() * sizeof(int4), hipMemcpyHostToDevice);
    if (e == hipSuccess && T->nthalo) {
        uint64_t g = (T->ntiles + kBlock - 1) / kBlock;
        if (g > 16384) g = 16384;
        hipLaunchKernelGGL(k_tile_halo, dim3((unsigned)g), dim3(kBlock), 0, 0, T->Pc, T->ntiles, T->nthalo,
                           (uint64_t)T->tile, d_slots, T->d_tile_halo);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    if (d_slots) (void)hipFree(d_slots);
    if (e != hipSuccess) {
        if (T->d_nbtab) (void)hipFree(T->d_nbtab);
        if (T->d_tile_halo) (void)hipFree(T->d_tile_halo);
        if (T->d_ringhome) (void)hipFree(T->d_ringhome);
        (void)hipFree(T->d_coarse_tables);
        delete T;
        return hip_error(e, "tile table setup");
    }
    F.tile = T;
    return SQZ_OK;
}

template <class Pat>
sqz_status launch(const FractalHost &F, const uint8_t *in, uint8_t *out, hipStream_t st)
{
    const TileConfig *T = F.tile;
    if (((uintptr_t)in & 15) || ((uintptr_t)out & 15))
        return set_error(SQZ_ERR_INVALID, "tiled kernel needs 16-byte aligned buffers");
    const uint64_t grid = T->ntiles < (1ull << 20) ? T->ntiles : (1ull << 20);
    constexpr int NT = nt_of<Pat>();
    hipLaunchKernelGGL((k_life_tile<Pat, NT>), dim3((unsigned)grid), dim3(NT), 0, st, tile_args(F), in, out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SQZ_OK : hip_error(e, "compact step (tile) launch");
}

enum { kNone = 0, kTriangle = 1, kTrianglePaper = 2, kVicsek = 3, kTriangleBig = 4 };

}  // namespace

int tile_kind_for(const FractalHost &F)
{
    if (matches<PatTriangle>(F) && F.r >= SQZ_TRI_TILE_BIG_FROM) return kTriangleBig;
    if (matches<PatTriangle>(F) && F.r >= PatTriangle::J) return kTriangle;
    if (matches<PatTrianglePaper>(F) && F.r >= PatTrianglePaper::J) return kTrianglePaper;
    if (matches<PatVicsek>(F) && F.r >= PatVicsek::J) return kVicsek;
    return kNone;
}

sqz_status tile_prepare(FractalHost &F)
{
    switch (F.tile_kind) {
    case kTriangle: return prepare<PatTriangle>(F);
    case kTriangleBig: return prepare<PatTriangleBig>(F);
    case kTrianglePaper: return prepare<PatTrianglePaper>(F);
    case kVicsek: return prepare<PatVicsek>(F);
    }
    return set_error(SQZ_ERR_UNSUPPORTED, "no tiled kernel");
}

void tile_release(FractalHost &F)
{
    if (!F.tile) return;
    (void)hipFree(F.tile->d_nbtab);
    (void)hipFree(F.tile->d_tile_halo);
    (void)hipFree(F.tile->d_ringhome);
    (void)hipFree(F.tile->d_coarse_tables);
    delete F.tile;
    F.tile = nullptr;
}

int32_t tile_level_of(const FractalHost &F) { return F.tile ? F.tile->M : 0; }

sqz_status launch_life_tile(const FractalHost &F, const uint8_t *in, uint8_t *out, hipStream_t st)
{
    switch (F.tile_kind) {
    case kTriangle: return launch<PatTriangle>(F, in, out, st);
    case kTriangleBig: return launch<PatTriangleBig>(F, in, out, st);
    case kTrianglePaper: return launch<PatTrianglePaper>(F, in, out, st);
    case kVicsek: return launch<PatVicsek>(F, in, out, st);
    }
    return set_error(SQZ_ERR_UNSUPPORTED, "no tiled kernel");
}

// Steps a launch of a run takes at least (sqz_info.run_steps_per_launch): ten,
// or as many as a smaller tile's side allows.
int tile_steps_per_launch(const FractalHost &F)
{
    if (!F.tile) return 0;
    int64_t side = 1;
    for (int i = 0; i < F.tile->M && side <= kMaxSteps; ++i) side *= F.s;
    return (int)std::min<int64_t>(kMaxSteps, side - 1);
}

// Fractals whose one-step tiles are at most eight (of the large ones three) per
// CU: those a resident run is offered for, where the tiles of the run fit too.
bool tile_few(const FractalHost &F)
{
    int cus = 0;
    if (!F.tile || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, F.device) != hipSuccess) return false;
    return F.tile->ntiles <= (uint64_t)(F.tile_kind == kTriangleBig ? 3 : 8) * (uint64_t)cus;
}

}  // namespace sqz
