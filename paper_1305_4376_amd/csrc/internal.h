// internal.h -- declarations shared by libtdes's translation units (not part of the ABI).
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include "../../include/tdes.h"

namespace tdes {

// Words of a schedule: the encryption block, then the decryption block, each
// kDirWords long: its kRoundWords round words (round r uses words 2r, the key
// chunks of boxes 1,7,5,3, and 2r+1) followed by the folded key words of the
// bitsliced kernels (bitslice_maps.h).
constexpr int kRounds = 48;
constexpr int kRoundWords = 2 * kRounds;
constexpr int kDirWords = 200;
static_assert(kRoundWords + 104 <= kDirWords && 2 * kDirWords * 4 == TDES_SCHED_BYTES, "schedule layout");

// Per-device properties the launchers need (cached on first use).
struct DeviceInfo {
    int cu_count;
    int device;
};
int device_info(DeviceInfo *info);

// Makes `device` current for the lifetime of the guard and restores the
// caller's device afterwards (no-op when it already is current).
class DeviceGuard {
  public:
    explicit DeviceGuard(int device) {
        ok_ = hipGetDevice(&prev_) == hipSuccess;
        if (ok_ && prev_ != device) {
            ok_ = hipSetDevice(device) == hipSuccess;
            switched_ = ok_;
        }
    }
    ~DeviceGuard() {
        if (switched_) (void)hipSetDevice(prev_);
    }
    bool ok() const { return ok_; }
    DeviceGuard(const DeviceGuard &) = delete;
    DeviceGuard &operator=(const DeviceGuard &) = delete;

  private:
    int prev_ = 0;
    bool ok_ = false, switched_ = false;
};

// Kernel launchers.  Arguments are already validated; n_blocks > 0.
// `ks` points at the words of one direction.  threads: workgroup size, 0 for
// the kernel's own (256; the table kernel's mostly 512 above 2^16 blocks); otherwise
// 64, 128, 256, 512 or 1024 (hipErrorInvalidValue for anything else).
hipError_t launch_table(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks,
                        hipStream_t stream, uint32_t threads = 0);
hipError_t launch_bitslice(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks,
                           hipStream_t stream, uint32_t threads = 0);
// Short messages (k_short.hip): one bit of f per lane.  n_blocks below 2^32.
hipError_t launch_short_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream);
hipError_t launch_short_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                            hipStream_t stream);
hipError_t launch_short_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                    hipStream_t stream);
// Middling messages (k_team.hip): a workgroup per tile of 2048 blocks.  n_blocks below 2^42.
hipError_t launch_team_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream);
hipError_t launch_team_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                           hipStream_t stream);
hipError_t launch_team_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                   hipStream_t stream);
// Shortish messages (k_pair.hip): table lookups, two lanes per block.  n_blocks below 2^31.
hipError_t launch_pair_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream);
hipError_t launch_pair_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                           hipStream_t stream);
hipError_t launch_pair_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                   hipStream_t stream);
// TDES_VARIANT_AUTO by message length, from launches back to back on MI355X:
//   below kShortBelow   one bit of f per lane: 3.0 us to 2048 blocks, 4.4 at 8192, then 0.29 us per 1024;
//   to kPairTo          two lanes per block: 5.3 us at 8192, 5.7 at 65536, 6.8 at 98304;
//   to kTableTo         the table kernel: 6.4 us at 65536, 6.6 at 2^17, 9.8 at 2^18, where each lane has one
//                       block (with a second pass 16.1 from there on);
//   to kPairAgainTo     two lanes per block: 13.2 us at 5 * 2^16, 14.7 at 3 * 2^17;
//   to kTeamTo          a team per tile: 14.6 us at 3 * 2^17, 14.9 at 2^19, 29.4 at 2^21 (one wave per tile
//                       31.6), 36.7 behind it, where one wave per tile takes 34.6;
//   from there on       one wave per tile.
// The modes have no one-lane table kernel: two lanes per block from kShortBelow to kPairAgainTo.  Their extra
// work costs a lone wave more, so teams take them to kModeTeamBelow: CTR 31.2 us at 2^21 (a wave per tile 39.7),
// CBC decryption 31.1 (37.0).
constexpr uint64_t kShortBelow = 12288;
constexpr uint64_t kPairTo = 90112;
constexpr uint64_t kTableTo = 1ull << 18;
constexpr uint64_t kPairAgainTo = 3ull << 17;
constexpr uint64_t kTeamTo = 1ull << 21;
constexpr uint64_t kModeTeamBelow = 9ull << 18;
hipError_t launch_auto(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream);
// Block-parallel modes (bitsliced): ks is the encryption half for CTR and the
// decryption half for CBC decryption; iv is the 8 IV bytes read as a big-endian integer.
hipError_t launch_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                      hipStream_t stream);
hipError_t launch_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                              hipStream_t stream);
hipError_t launch_fill_splitmix64(uint64_t *dev, uint64_t n_words, uint64_t seed, uint64_t first,
                                  hipStream_t stream);

// Batch contexts of the server launch the 120-VGPR variant of the batch kernel, so that the
// payload fills of later steps run beside it.
void ctx_set_capped(tdes_ctx *c, bool capped);

// A run of serving-payload words (chained generator, k_util.hip) written to base + dst_off, one
// workgroup each; first_word is the run's first word in its request, a multiple of 16384.
struct FillTile {
    uint64_t dst_off;
    uint64_t seed;
    uint64_t first_word;
    uint32_t n_words;
    uint32_t pad;
};
constexpr uint32_t kFillTileWords = 1u << 18;
hipError_t launch_fill_tiles(const FillTile *tiles, uint32_t n_tiles, uint8_t *base, hipStream_t stream);

}  // namespace tdes
