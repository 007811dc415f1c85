// k_bitslice.hip -- Triple-DES over one message, bitsliced: ECB, and the CTR and
// CBC-decrypt modes on the same core (plain launches).
//
// The paper maps one 64-bit block to one GPU thread and notes that the cipher
// is almost entirely bit operations on integers (Abstract; Section IV).  Here a
// lane instead holds 32 blocks as bit planes (bitslice_core.h): no lookup
// tables and no LDS, a fixed data-independent cost per block, and the three
// DES stages of EDE fused in one pass over the data.
//
// The kernel takes every whole 2048-block tile (16 KiB of the message, one
// wave each); its code has only that path, so it fits 128 VGPRs and runs four
// waves per SIMD.  Tiles beyond 2^22 per launch loop grid-stride.  A partial
// last tile runs beside the whole ones, one bit of f per lane (short_core.h):
// a wave alone on it would take 31 us.  Buffers that are only 8-byte aligned
// take the same path (3000001 blocks behind an 8-byte header: 43.4 us a call
// with per-block accesses and a wave on the last block, 43.2 with 16-byte
// accesses and the last block behind the others, 40.2 beside them; with the
// present circuits and transposes 36.1).  The key
// is the same for the whole launch, so its masks come from scalar registers.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "short_core.h"

namespace {

using namespace tdes_bs;

constexpr int kDefaultThreads = 256;     // 4 waves per workgroup
constexpr int kWavesPerSimd = 4;         // at most 128 VGPRs per lane
constexpr uint64_t kMaxGrid = 1u << 20;

// Workgroups of kThreads threads (one wave per 64); the main kernel is built for
// four waves per SIMD whatever the workgroup size (launch_bounds' second
// argument is the minimum number of waves per execution unit).
template <TileMode kMode, int kThreads = kDefaultThreads>
__global__ __launch_bounds__(kThreads, kWavesPerSimd) void tdes_bitslice_kernel(const uint32_t *__restrict__ ks,
                                                                                   const uint8_t *in, uint8_t *out,
                                                                                   uint64_t n_tiles, uint64_t iv) {
    constexpr int kWaves = kThreads / kLanes;
    const uint32_t lane = threadIdx.x % kLanes;
    const uint64_t stride = (uint64_t)gridDim.x * kWaves;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    for (uint64_t tile = (uint64_t)blockIdx.x * kWaves + wave; tile < n_tiles; tile += stride) {
        const uint64_t first = tile * kTileBlocks;
        mode_tile<kMode, true>(ks, in + 8 * first, out + 8 * first, kTileBlocks, lane, first, iv);
    }
}

// A message with a partial last tile: the first tail_groups workgroups take its last tail_blocks blocks one bit
// of f per lane, beside the whole tiles of the others.  (An instance of its own, so that the code of the
// kernel above stays what it is.)
template <TileMode kMode>
__global__ __launch_bounds__(kDefaultThreads, kWavesPerSimd) void tdes_bitslice_ragged_kernel(
    const uint32_t *__restrict__ ks, const uint8_t *in, uint8_t *out, uint64_t n_tiles, uint64_t iv, uint32_t tail_blocks,
    uint32_t tail_groups) {
    static_assert(kDefaultThreads == kShortThreads, "one workgroup size for both parts");
    if (blockIdx.x < tail_groups) {
        const uint64_t done = n_tiles * kTileBlocks;
        short_blocks<kMode>(ks, in + 8 * done, out + 8 * done, tail_blocks, blockIdx.x, true,
                            kMode == TileMode::kCtr ? iv + done : iv);
        return;
    }
    constexpr int kWaves = kDefaultThreads / kLanes;
    const uint32_t lane = threadIdx.x % kLanes;
    const uint64_t stride = (uint64_t)(gridDim.x - tail_groups) * kWaves;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    for (uint64_t tile = (uint64_t)(blockIdx.x - tail_groups) * kWaves + wave; tile < n_tiles; tile += stride) {
        const uint64_t first = tile * kTileBlocks;
        mode_tile<kMode, true>(ks, in + 8 * first, out + 8 * first, kTileBlocks, lane, first, iv);
    }
}

// ECB of a message shorter than a tile, by one wave: what TDES_VARIANT_BITSLICE asks for by name (31 us, where
// the automatic choice takes 3).
__global__ __launch_bounds__(kLanes) void tdes_bitslice_tail_kernel(const uint32_t *__restrict__ ks, const uint8_t *in,
                                                                    uint8_t *out, uint32_t n_blocks) {
    mode_tile<TileMode::kEcb, false>(ks, in, out, n_blocks, threadIdx.x, 0, 0);
}

uint32_t grid_for(uint64_t tiles, int waves_per_group) {
    const uint64_t g = (tiles + waves_per_group - 1) / waves_per_group;
    return (uint32_t)(g < kMaxGrid ? g : kMaxGrid);
}

template <TileMode kMode, int kThreads = kDefaultThreads>
hipError_t launch(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                  hipStream_t stream) {
    constexpr int kWaves = kThreads / kLanes;
    const uint64_t whole = n_blocks / kTileBlocks, done = whole * kTileBlocks;
    const uint32_t rest = (uint32_t)(n_blocks - done);
    if (whole && rest && kThreads == kDefaultThreads) {
        const uint32_t tail = short_groups(rest);
        hipLaunchKernelGGL(tdes_bitslice_ragged_kernel<kMode>, dim3(tail + grid_for(whole, kWaves)), dim3(kThreads), 0,
                           stream, ks, in, out, whole, iv, rest, tail);
        return hipGetLastError();
    }
    if (whole) {
        hipLaunchKernelGGL((tdes_bitslice_kernel<kMode, kThreads>), dim3(grid_for(whole, kWaves)), dim3(kThreads), 0,
                           stream, ks, in, out, whole, iv);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (rest == 0) return hipSuccess;
    // ECB with a workgroup size, or shorter than a tile (the modes come here with neither).
    if (whole) return tdes::launch_short_ecb(ks, in + 8 * done, out + 8 * done, rest, stream);
    hipLaunchKernelGGL(tdes_bitslice_tail_kernel, dim3(1), dim3(kLanes), 0, stream, ks, in, out, rest);
    return hipGetLastError();
}

}  // namespace

namespace tdes {

hipError_t launch_bitslice(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks,
                           hipStream_t stream, uint32_t threads) {
    switch (threads) {
        case 0:
        case kDefaultThreads: return launch<TileMode::kEcb>(ks, in, out, n_blocks, 0, stream);
        case 64: return launch<TileMode::kEcb, 64>(ks, in, out, n_blocks, 0, stream);
        case 128: return launch<TileMode::kEcb, 128>(ks, in, out, n_blocks, 0, stream);
        case 512: return launch<TileMode::kEcb, 512>(ks, in, out, n_blocks, 0, stream);
        case 1024: return launch<TileMode::kEcb, 1024>(ks, in, out, n_blocks, 0, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                      hipStream_t stream) {
    if (n_blocks < kShortBelow) return launch_short_ctr(ks, in, out, n_blocks, iv, stream);
    if (n_blocks <= kPairAgainTo) return launch_pair_ctr(ks, in, out, n_blocks, iv, stream);
    if (n_blocks < kModeTeamBelow) return launch_team_ctr(ks, in, out, n_blocks, iv, stream);
    return launch<TileMode::kCtr>(ks, in, out, n_blocks, iv, stream);
}

hipError_t launch_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                              hipStream_t stream) {
    if (n_blocks < kShortBelow) return launch_short_cbc_decrypt(ks, in, out, n_blocks, iv, stream);
    if (n_blocks <= kPairAgainTo) return launch_pair_cbc_decrypt(ks, in, out, n_blocks, iv, stream);
    if (n_blocks < kModeTeamBelow) return launch_team_cbc_decrypt(ks, in, out, n_blocks, iv, stream);
    return launch<TileMode::kCbcDecrypt>(ks, in, out, n_blocks, iv, stream);
}

}  // namespace tdes
