// Bit-row expanded tiles for Life on the Sierpinski carpet: the kernel (one
// tile per workgroup, device code in bitbox_device.h) and its host-side
// tables: grid positions of a tile's blocks, border blocks of the adjacent
// tiles, membership of every box position.
#include <algorithm>
#include <vector>

#include "bitbox_device.h"

namespace sqz {

template <class Pat>
__global__ void __launch_bounds__(kBxThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_life_bitbox(BitboxArgs A, const uint8_t *__restrict__ in, uint8_t *__restrict__ out, int32_t steps)
{
    __shared__ __align__(16) uint32_t sm[kBxLds];
    bitbox_tile<Pat>(A, in, out, blockIdx.x, steps, sm);
}

namespace {

template <class Pat>
bool bx_matches(const FractalHost &F)
{
    if (F.s != Pat::S || F.k != Pat::K) return false;
    for (int j = 0; j < Pat::K; ++j)
        if (F.ox[j] != Pat::OX[j] || F.oy[j] != Pat::OY[j]) return false;
    return true;
}

template <class Pat>
sqz_status bx_prepare(FractalHost &F)
{
    BitboxConfig *C = new BitboxConfig();
    const int M = F.r < kBxMMax ? F.r : kBxMMax;
    C->M = M;
    C->tile = (uint32_t)cpow(Pat::K, M);
    C->nblk = (uint32_t)cpow(Pat::K, M - 1);
    C->side = (uint32_t)cpow(3, M);

    // grid positions of the tile's blocks, border blocks of the adjacent tiles,
    // membership of every box position (adjacent tiles present)
    BitboxSpec S;
    S.M = M;
    S.border = kBxBorder;
    S.grid_pitch = kBxGP;
    S.rows = kBxRows;
    S.words = kBxW;
    std::vector<uint16_t> bpos;
    std::vector<uint32_t> ring, member;
    bitbox_tables(F, S, bpos, ring, member);
    // border blocks by distance from the tile: a launch loads those its steps reach
    const int side = (int)C->side / 3;
    auto distance = [&](uint32_t slot) {
        const int x = (int)(slot & 0x3FFFu) % kBxGP - kBxBorder, y = (int)(slot & 0x3FFFu) / kBxGP - kBxBorder;
        return std::max(std::max(-x, x - side + 1), std::max(-y, y - side + 1));
    };
    std::stable_sort(ring.begin(), ring.end(), [&](uint32_t a, uint32_t b) { return distance(a) < distance(b); });
    for (int d = 0; d <= kBxBorder; ++d)
        C->ring[d] = (uint32_t)std::count_if(ring.begin(), ring.end(), [&](uint32_t a) { return distance(a) <= d; });

    sqz_status st = build_map_params(F, F.r - M, C->Pc, &C->d_coarse);
    if (st != SQZ_OK) {
        delete C;
        return st;
    }
    C->ntiles = C->Pc.N;
    C->d_gpos = nullptr;
    C->d_ring = nullptr;
    C->d_member = nullptr;
    for (uint16_t &p : bpos) p = (uint16_t)((p >> 7) * kBxGP + (p & 127u));  // x | y << 7 -> grid byte
    hipError_t e = hipMalloc(&C->d_gpos, bpos.size() * sizeof(uint16_t));
    if (e == hipSuccess) e = hipMemcpy(C->d_gpos, bpos.data(), bpos.size() * sizeof(uint16_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&C->d_ring, (ring.size() ? ring.size() : 1) * sizeof(uint32_t));
    if (e == hipSuccess && ring.size())
        e = hipMemcpy(C->d_ring, ring.data(), ring.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&C->d_member, member.size() * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemcpy(C->d_member, member.data(), member.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (C->d_gpos) (void)hipFree(C->d_gpos);
        if (C->d_ring) (void)hipFree(C->d_ring);
        if (C->d_member) (void)hipFree(C->d_member);
        (void)hipFree(C->d_coarse);
        delete C;
        return hip_error(e, "bit-row tile table setup");
    }
    F.bitbox = C;
    return SQZ_OK;
}

template <class Pat>
sqz_status bx_launch(const FractalHost &F, const uint8_t *in, uint8_t *out, int steps, hipStream_t st)
{
    const BitboxConfig *C = F.bitbox;
    const BitboxArgs A = bitbox_args(F);
    const dim3 grid((unsigned)C->ntiles), block(kBxThreads);
    hipLaunchKernelGGL(k_life_bitbox<Pat>, grid, block, 0, st, A, in, out, steps);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SQZ_OK : hip_error(e, "compact step (bit rows) launch");
}

}  // namespace

sqz_status bitbox_prepare(FractalHost &F)
{
    F.bitbox = nullptr;
    // tiles of level >= 3: the border (five blocks) must lie in the eight adjacent tiles
    if (F.r >= 3 && bx_matches<PatCarpet>(F)) return bx_prepare<PatCarpet>(F);
    return SQZ_OK;
}

void bitbox_release(FractalHost &F)
{
    if (!F.bitbox) return;
    (void)hipFree(F.bitbox->d_gpos);
    (void)hipFree(F.bitbox->d_ring);
    (void)hipFree(F.bitbox->d_member);
    (void)hipFree(F.bitbox->d_coarse);
    delete F.bitbox;
    F.bitbox = nullptr;
}

int bitbox_steps_per_launch(const FractalHost &F) { return !F.bitbox ? -1 : (F.bitbox->ntiles == 1 ? 0 : kBxMaxSteps); }

int32_t bitbox_level_of(const FractalHost &F) { return F.bitbox ? F.bitbox->M : 0; }

sqz_status launch_life_bitbox(const FractalHost &F, const uint8_t *in, uint8_t *out, int steps, hipStream_t st)
{
    if (!F.bitbox) return set_error(SQZ_ERR_UNSUPPORTED, "no bit-row tile for this replica pattern and level");
    if (((uintptr_t)in & 7) || ((uintptr_t)out & 7))
        return set_error(SQZ_ERR_INVALID, "bit-row tiles need 8-byte aligned buffers");
    const int K = bitbox_steps_per_launch(F);
    if (steps < 1 || (K && steps > K))
        return set_error(SQZ_ERR_UNSUPPORTED, "%d steps per launch exceed the %d bit-row tiles allow", steps, K);
    return bx_launch<PatCarpet>(F, in, out, steps, st);
}

}  // namespace sqz
