// short_core.h -- Triple-DES over a short message (ECB, CTR, CBC decryption): one output bit of f per lane.
//
// A short message leaves the chip nearly empty, so its time is the chain of 48
// dependent rounds, not the work.  The table kernel's round is a chain through
// LDS (about 200 cycles: address permutes, eight reads, the XORs of their
// results), the bitsliced kernel's a wave's 257 instructions.  Here a wave
// holds two blocks, 32 lanes each, and every lane of a half computes one bit
// of f(R, K) alone, without memory: an S-box output bit is a function of six
// bits, so its truth table is one 64-bit word, held by the lane in two
// registers; shifting that word left by the six input bits brings the wanted
// entry to its sign.  A compare of the signs across the wave then yields both
// blocks' 32-bit f words at once in a scalar register pair, already permuted
// by P because every lane was given the table of its own output bit.  A round
// is six dependent vector instructions and one more for the key:
//     R  = L ^ f           two three-input operations, one per half's word of the pair
//     x  = rotate(R) ^ k   the six bits E feeds the lane's box, at the bottom of the word
//     f' = sign of (table << (x & 63)), gathered by the compare
// IP and FP are made the same way: the lane shifts the 64-bit block left by the
// position of the bit it stands for, and the compare gathers the words.
//
// Bit order: words hold the standard's bit 0 in their most significant bit, so
// lane l of a half stands for bit 31 - l of f and box s reads the six bits from
// word bit 27 - 4s on (cyclically), its first input the highest.
//
// Bound: below about 4096 blocks (two waves per SIMD) the chain, then vector
// issue (the two 64-bit shifts take four times a logic operation's slot).
// Measured back to back, against the table kernel (an empty launch: 1.6 us):
// 256 blocks 3.0 vs 5.7 us, 4096 3.3 vs 6.3, 8192 4.4 vs 6.3, 16384 6.7 vs
// 6.4, 65536 20.2 vs 6.4.
#pragma once
#include <hip/hip_runtime.h>

#include "bitslice_core.h"

namespace tdes_bs {

constexpr int kShortThreads = 256;
constexpr int kBlocksPerWave = 2;
constexpr uint32_t short_groups(uint32_t n_blocks) {
    constexpr uint32_t per = kBlocksPerWave * (kShortThreads / kLanes);
    return (n_blocks + per - 1) / per;
}

// What a lane of a half needs: the truth table of its bit of f (entry x at bit 63 - x) and the
// shift amounts, one per byte (a shift reads only its low five or six bits):
//   pos:  rotation of R to the box's inputs, position of the box's key chunk in the round's 64-bit
//         key word pair, left shifts that bring the lane's bits of L0 and R0 (of the block as loaded) to the top;
//   out:  left shifts of the preoutput that bring the lane's bits of the two output words to the top.
struct alignas(16) ShortLane {
    uint64_t table;
    uint32_t pos, out;
};
struct ShortLanes {
    ShortLane v[32];
};

constexpr ShortLanes make_short_lanes() {
    ShortLanes t{};
    for (int l = 0; l < 32; l++) {
        const int q = 31 - l, src = tdes_spec::kP[q], s = src / 4;
        uint64_t table = 0;
        for (uint32_t x = 0; x < 64; x++)
            table |= (uint64_t)((tdes_spec::sbox(s, x) >> (3 - src % 4)) & 1u) << (63 - x);
        t.v[l].table = table;
        const uint32_t rot = (uint32_t)(27 - 4 * s) & 31, key = 32 * (s % 2) + (uint32_t)key_pos(s, 5);
        const uint32_t l0 = 63 - plane_of_bit(tdes_spec::ip(q)), r0 = 63 - plane_of_bit(tdes_spec::ip(32 + q));
        t.v[l].pos = rot | key << 8 | l0 << 16 | r0 << 24;
        t.v[l].out = (uint32_t)kMaps.out_src[l] | (uint32_t)kMaps.out_src[32 + l] << 8;
    }
    return t;
}

__constant__ ShortLanes g_short = make_short_lanes();

// The 64 lanes' top bits of their (v << n), n read modulo 64.  The empty asm statement keeps the
// compare on the shifted pair's high word (a 64-bit compare is slower).
__device__ __forceinline__ uint64_t gather(uint64_t v, uint32_t n) {
    uint32_t top = (uint32_t)((v << (n & 63)) >> 32);
    asm("" : "+v"(top));
    return __builtin_amdgcn_ballot_w64((int32_t)top < 0);
}

// a ^ (the lower half's lanes: low word of f; the upper half's: high word); hi = ~0 in the upper half's lanes.
__device__ __forceinline__ uint32_t xor_half(uint32_t a, uint64_t f, uint32_t hi) {
    const uint32_t t = __builtin_amdgcn_bitop3_b32(a, (uint32_t)f, hi, 0xB4);            // a ^ (f.lo & ~hi)
    return __builtin_amdgcn_bitop3_b32(t, (uint32_t)(f >> 32), hi, 0x78);                // t ^ (f.hi & hi)
}

// The blocks of workgroup `group` (kShortThreads threads) of a message of n_blocks.  continued (CBC decryption):
// in[0] is not the message's first block.
template <TileMode kMode>
__device__ __forceinline__ void short_blocks(const uint32_t *__restrict__ ks, const uint8_t *in, uint8_t *out,
                                             uint32_t n_blocks, uint32_t group, bool continued, uint64_t iv) {
    const uint32_t lane = threadIdx.x % kLanes;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const uint32_t first = (group * (kShortThreads / kLanes) + wave) * kBlocksPerWave;
    if (first >= n_blocks) return;
    const uint32_t hi = lane < 32 ? 0u : ~0u;
    const uint32_t mine = first + lane / 32;                          // the half's block
    const uint32_t at = mine < n_blocks ? mine : n_blocks - 1;        // (a half past the end repeats the last block)
    const uint2 *src = reinterpret_cast<const uint2 *>(in) + at;
    uint2 data = *src;                                                // CTR: met by the keystream at the end
    const uint64_t table = g_short.v[lane % 32].table;
    const uint32_t pos = g_short.v[lane % 32].pos, out_pos = g_short.v[lane % 32].out;
    uint64_t block = (uint64_t)data.y << 32 | data.x;
    if constexpr (kMode == TileMode::kCtr) block = __builtin_bswap64(iv + at);
    uint2 prev;
    if constexpr (kMode == TileMode::kCbcDecrypt) {
        prev = make_uint2(be_hi_word(iv), be_lo_word(iv));
        if (at != 0 || continued) prev = src[-1];
    }

    const uint32_t rot = pos, key = pos >> 8;
    uint32_t x = xor_half(0, gather(block, pos >> 16), hi);  // L0
    uint32_t y = xor_half(0, gather(block, pos >> 24), hi);  // R0
    auto round = [&](uint32_t &l, uint32_t r, int i) {
        const uint64_t k = (uint64_t)ks[2 * i + 1] << 32 | ks[2 * i];
        const uint32_t e = __builtin_amdgcn_alignbit(r, r, rot) ^ (uint32_t)(k >> (key & 63));
        l = xor_half(l, gather(table, e), hi);
    };
    // Between the stages IP^-1 and IP cancel and only the halves swap.
#pragma unroll
    for (int i = 0; i < 16; i += 2) { round(x, y, i); round(y, x, i + 1); }
#pragma unroll
    for (int i = 16; i < 32; i += 2) { round(y, x, i); round(x, y, i + 1); }
#pragma unroll
    for (int i = 32; i < 48; i += 2) { round(x, y, i); round(y, x, i + 1); }

    const uint64_t pre = (uint64_t)y << 32 | x;                       // preoutput R16 || L16
    uint2 o;
    o.x = xor_half(0, gather(pre, out_pos), hi);
    o.y = xor_half(0, gather(pre, out_pos >> 8), hi);
    if constexpr (kMode == TileMode::kCtr) { o.x ^= data.x; o.y ^= data.y; }
    if constexpr (kMode == TileMode::kCbcDecrypt) { o.x ^= prev.x; o.y ^= prev.y; }
    if (lane % 32 == 0 && mine < n_blocks) reinterpret_cast<uint2 *>(out)[mine] = o;
}

}  // namespace tdes_bs
