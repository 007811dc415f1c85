// team_core.h -- the bitsliced rounds on one tile of 2048 blocks, shared by a team of eight waves.
//
// A wave that runs a tile alone (bitslice_core.h) needs all its 11.5 k vector
// instructions one after the other, and a wave alone on its SIMD issues one
// only every 4.9 cycles (two waves: every 2.35): 31 us a tile, however empty
// the chip is.  Here a workgroup of eight waves takes the tile.  Wave s
// computes box s of every round and keeps in registers the four planes of each
// half that the box's outputs go to; all planes lie in LDS too, from where a
// wave reads the six that its box needs and where it writes back the four it
// changed, with one barrier a round.  The key is folded into the planes
// exactly as in bitslice_core.h (bitslice_maps.h), in LDS too; when every lane
// has its own key, the six inputs are XORed with its key masks instead.
//
// Bound: a round of a team alone on its CU is its chain, about 460 cycles: 29
// vector instructions (145), the reads' and the writes' way through LDS (100
// each; LDS takes 2.2 cycles for a plane read and 3.1 for one written), the
// wait for the slowest box at the barrier.  With several teams on a CU it is
// vector issue and LDS together.
//
// Planes.  64 slots of 64 words (16 KiB): slots 0..31 hold L0, slots 32..63
// R0, and at the end R16 and L16; word l of a slot is the plane's 32 bits of
// lane l's blocks.  Bit j of lane l is block 64 j + l of a wave tile, block j of
// lane l's slot of a lane tile.
//
// In and out.  Thread (wave 2g + h, lane l) moves the 4-byte half h of the
// blocks of bits 8g .. 8g + 7.  It transposes the bits of its eight words byte
// by byte and stores each byte into its plane's slot: plane p of half h is IP
// output bit team_slot(p) - 4h (IP reads one bit position of all eight bytes
// per group of eight outputs).  FP is the same map, so the way out reads the
// same slots.
#pragma once
#include "bitslice_core.h"

namespace tdes_bs {

constexpr int kTeamThreads = 8 * kLanes;
constexpr int kTeamWords = 64 * kLanes;                // LDS words of a wave tile
constexpr int kTeamLaneWords = kTeamWords + 96 * kLanes;  // of a lane tile: the lanes' round words behind the planes

// IP output group (of eight bits) that reads bit i (counted from the least significant) of every byte.
constexpr int ip_row(int i) {
    for (int r = 0; r < 8; r++)
        if (tdes_spec::ip(8 * r) % 8 == 7 - i) return r;
    return -1;
}

// Slot of plane p (of half 0's 32; half 1's lie four slots lower).
constexpr int team_slot(int p) { return 8 * ip_row(p % 8) + 7 - p / 8; }

constexpr bool team_maps_ok() {
    for (int h = 0; h < 2; h++)
        for (int p = 0; p < 32; p++) {
            const int k = team_slot(p) - 4 * h;
            if ((k < 32 ? kMaps.l0[k] : kMaps.r0[k - 32]) != 32 * h + p || kMaps.out_src[32 * h + p] != k) return false;
        }
    return true;
}
static_assert(team_maps_ok(), "plane slots");

// One box with folded masks (bitslice_core.h's sbox_round_folded on the four planes o).
template <int S>
__device__ __forceinline__ void team_sbox(const uint32_t (&in)[6], uint32_t (&o)[4], const uint32_t (&m)[4]) {
    if constexpr (S == 0) sbox0_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 1) sbox1_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 2) sbox2_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 3) sbox3_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 4) sbox4_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 5) sbox5_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 6) sbox6_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
    if constexpr (S == 7) sbox7_m(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3], m[0], m[1], m[2], m[3]);
}

// The same with the key already in the inputs.
template <int S>
__device__ __forceinline__ void team_sbox_plain(const uint32_t (&in)[6], uint32_t (&o)[4]) {
    if constexpr (S == 0) sbox0(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 1) sbox1(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 2) sbox2(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 3) sbox3(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 4) sbox4(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 5) sbox5(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 6) sbox6(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
    if constexpr (S == 7) sbox7(in[0], in[1], in[2], in[3], in[4], in[5], o[0], o[1], o[2], o[3]);
}

// The planes of a half that box S's outputs go to, in the wave of that box.  `half`: this lane's column of
// the half's slots.
template <int S, bool kLaneKeys>
struct TeamPlanes {
    uint32_t v[4];

    static constexpr int plane(int i) { return kMaps.p_inv[4 * S + i]; }

    __device__ __forceinline__ void get(const uint32_t *half) {
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = half[kLanes * plane(i)];
    }
    __device__ __forceinline__ void put(uint32_t *half) const {
#pragma unroll
        for (int i = 0; i < 4; i++) half[kLanes * plane(i)] = v[i];
    }
    // v ^= the planes' bits of w.
    __device__ __forceinline__ void fix(uint32_t w_in) {
        const uint32_t w = key_word<false>(w_in);
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] ^= key_mask(w, plane(i));
    }

    // One round: v ^= box S of the other half's planes at `y`.  One key per tile: with the round's folded
    // words (k0: output masks, k1: corrections); a key per lane: with the box's round word k0.
    __device__ __forceinline__ void round(const uint32_t *y, uint32_t k0_in, uint32_t k1_in) {
        uint32_t in[6], m[4], c[6];
#pragma unroll
        for (int j = 0; j < 6; j++) in[j] = y[kLanes * kMaps.e[6 * S + j]];
        const uint32_t k0 = key_word<kLaneKeys>(k0_in), k1 = key_word<kLaneKeys>(k1_in);
        if constexpr (kLaneKeys) {
#pragma unroll
            for (int j = 0; j < 6; j++) c[j] = key_mask(k0, key_pos(S, j));
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++) m[i] = key_mask(k0, plane(i));
#pragma unroll
            for (int j = 0; j < 6; j++) c[j] = kUses.second_of[6 * S + j] < 0 ? 0 : key_mask(k1, kUses.second_of[6 * S + j]);
        }
        __builtin_amdgcn_sched_barrier(0);  // the masks are extracted while the planes are on their way
#pragma unroll
        for (int j = 0; j < 6; j++)
            if (kLaneKeys || kUses.second_of[6 * S + j] >= 0) in[j] ^= c[j];
        if constexpr (kLaneKeys)
            team_sbox_plain<S>(in, v);
        else
            team_sbox<S>(in, v, m);
    }
};

// The three stages by the wave of box S.  lds: this lane's column.  On entry slots 0..31 hold L0 and
// 32..63 R0, written and not yet waited for; on exit 0..31 hold R16 and 32..63 L16, likewise.  ks: one
// direction's schedule words, wave-uniform; with kLaneKeys the lane's column of the round words in LDS.
template <int S, bool kLaneKeys>
__device__ __forceinline__ void team_rounds(uint32_t *lds, const uint32_t *ks) {
    constexpr int kGroup = 4;  // rounds per turn of the loop, and per load of key words
    const uint32_t *fold = ks + kFoldBase;
    auto word0 = [&](int r) { return kLaneKeys ? ks[kLanes * (2 * r + S % 2)] : fold[kFoldOut + r]; };
    auto word1 = [&](int r) { return kLaneKeys ? 0u : fold[kFoldCorr + r]; };
    TeamPlanes<S, kLaneKeys> a, b;
    uint32_t *x = lds, *y = lds + 32 * kLanes;
    uint32_t k0[kGroup], k1[kGroup];
#pragma unroll
    for (int i = 0; i < kGroup; i++) { k0[i] = word0(i); k1[i] = word1(i); }
    __syncthreads();
    a.get(x);
    b.get(y);
    if constexpr (!kLaneKeys) {
        b.fix(fold[kFoldPre]);
        b.put(y);  // only this wave has read these planes since the barrier
        __syncthreads();
    }
#pragma unroll 1
    for (int r = 0; r < 48; r += kGroup) {
        uint32_t u0[kGroup], u1[kGroup];
        const int n = r + kGroup < 48 ? r + kGroup : r;  // the next words (the last turn reloads its own)
#pragma unroll
        for (int i = 0; i < kGroup; i++) {
            u0[i] = key_word<kLaneKeys>(k0[i]);
            u1[i] = key_word<kLaneKeys>(k1[i]);
            k0[i] = word0(n + i);
            k1[i] = word1(n + i);
        }
#pragma unroll
        for (int i = 0; i < kGroup; i += 2) {
            a.round(y, u0[i], u1[i]);
            a.put(x);  // x's planes were last read before the previous barrier
            __syncthreads();
            b.round(x, u0[i + 1], u1[i + 1]);
            b.put(y);
            __syncthreads();
        }
        if (r % 16 == 16 - kGroup) {
            // Between stages only the halves swap.  The half a stage reads last is the one the next stage
            // reads first, under another folded key.
            const int stage = r / 16;
            if constexpr (!kLaneKeys) a.fix(stage < 2 ? fold[kFoldMid + stage] : fold[kFoldPost + 2]);
            if (stage < 2) {
                if constexpr (!kLaneKeys) {
                    a.put(x);
                    __syncthreads();
                }
                uint32_t *t = x;
                x = y;
                y = t;
                const TeamPlanes<S, kLaneKeys> v = a;
                a = b;
                b = v;
            }
        }
    }
    // After three stages x is slots 0..31 again and a holds L16; the preoutput is R16 || L16.  (No wave
    // reads the slots any more: the last round ended at a barrier.)
    b.put(lds);
    a.put(lds + 32 * kLanes);
}

// A tile by a workgroup of kTeamThreads; every thread of it calls this.  lds: kTeamWords words (kTeamLaneWords
// with a key per lane), free at the call for all waves of the workgroup and free again when the last of them
// has returned.
//
// One key (kLaneKeys false): a wave tile (mode_tile): blocks first_block .. of the message at tin / tout,
// the first n_valid of the 2048 present; all arguments but tid the same for every thread.
// A key per lane (ECB): a lane tile (lane_slot): ks, tin, tout and n_valid (up to 32 blocks) are the lane's,
// the same in every wave.  The lanes' round words are brought to LDS once: read from memory by the eight waves
// in every round, 64 lines at a time, they cost as much as the rounds.
// Blocks that are not present are not loaded and not stored.  8-byte alignment suffices.
template <TileMode kMode, bool kLaneKeys>
__device__ __forceinline__ void team_tile(const uint32_t *ks, const uint8_t *tin, uint8_t *tout,
                                          uint32_t n_valid, uint32_t tid, uint64_t first_block, uint64_t iv,
                                          uint32_t *lds) {
    const uint32_t lane = tid % kLanes;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kLanes);
    const uint32_t h = wave & 1, g = wave >> 1;
    constexpr uint32_t kStep = kLaneKeys ? 1 : kLanes;      // the thread's eight blocks are this far apart
    const uint32_t j0 = kLaneKeys ? 8 * g : 512 * g + lane;  // the first of them
    const uint8_t *src = tin + 8 * (uint64_t)j0 + 4 * h;
    uint32_t w[8];
    typedef unsigned int v4w __attribute__((ext_vector_type(4), aligned(4)));
    v4w key[3];
    if constexpr (kLaneKeys) {
#pragma unroll
        for (int i = 0; i < 3; i++) key[i] = reinterpret_cast<const v4w *>(ks + 12 * wave)[i];
    }
    if constexpr (kLaneKeys) {
        // The thread's eight blocks are 64 bytes in a row, in another line for every lane: two blocks a load.
#pragma unroll
        for (int r = 0; r < 8; r += 2) {
            const uint8_t *p = tin + 8 * (uint64_t)(j0 + r);
            v4u v = {0, 0, 0, 0};
            if (j0 + r + 1 < n_valid) {
                v = *reinterpret_cast<const v4u *>(p);
            } else if (j0 + r < n_valid) {
                const uint2 u = *reinterpret_cast<const uint2 *>(p);
                v.x = u.x;
                v.y = u.y;
            }
            w[r] = h ? v.y : v.x;
            w[r + 1] = h ? v.w : v.z;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 8; r++) {
            if constexpr (kMode == TileMode::kCtr) {
                const uint64_t t = iv + first_block + j0 + kStep * r;  // wraps modulo 2^64
                w[r] = h ? be_lo_word(t) : be_hi_word(t);
            } else {
                w[r] = 0;
                if (j0 + kStep * r < n_valid) w[r] = *reinterpret_cast<const uint32_t *>(src + 8 * kStep * r);
            }
        }
    }
    transpose8(w);
    // half h's planes start 4h slots below half 0's; byte g of a plane's word is this thread's
    uint8_t *column = reinterpret_cast<uint8_t *>(lds + lane - 4 * h * kLanes) + g;
#pragma unroll
    for (int p = 0; p < 32; p++) column[team_slot(p) * (4 * kLanes)] = (uint8_t)(w[p % 8] >> (p & 24));

    uint32_t *mine = lds + lane;
    if constexpr (kLaneKeys) {
        uint32_t *keys = lds + kTeamWords + lane;
#pragma unroll
        for (int i = 0; i < 12; i++) keys[kLanes * (12 * wave + i)] = key[i / 4][i % 4];
        __syncthreads();
        ks = keys;
    }
    switch (wave) {
        case 0: team_rounds<0, kLaneKeys>(mine, ks); break;
        case 1: team_rounds<1, kLaneKeys>(mine, ks); break;
        case 2: team_rounds<2, kLaneKeys>(mine, ks); break;
        case 3: team_rounds<3, kLaneKeys>(mine, ks); break;
        case 4: team_rounds<4, kLaneKeys>(mine, ks); break;
        case 5: team_rounds<5, kLaneKeys>(mine, ks); break;
        case 6: team_rounds<6, kLaneKeys>(mine, ks); break;
        default: team_rounds<7, kLaneKeys>(mine, ks); break;
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < 8; i++) {
        uint32_t b[4];
#pragma unroll
        for (int c = 0; c < 4; c++) b[c] = column[team_slot(8 * c + i) * (4 * kLanes)];
        w[i] = (b[0] | b[1] << 8) | (b[2] | b[3] << 8) << 16;
    }
    transpose8(w);
    uint8_t *dst = tout + 8 * (uint64_t)j0 + 4 * h;
#pragma unroll
    for (int r = 0; r < 8; r++) {
        const uint32_t j = j0 + kStep * r;
        if (j >= n_valid) continue;
        uint32_t v = w[r];
        if constexpr (kMode == TileMode::kCtr) v ^= *reinterpret_cast<const uint32_t *>(src + 8 * kStep * r);
        if constexpr (kMode == TileMode::kCbcDecrypt) {
            uint32_t prev = h ? be_lo_word(iv) : be_hi_word(iv);
            if (first_block + j != 0) prev = *reinterpret_cast<const uint32_t *>(src + 8 * kStep * r - 8);
            v ^= prev;
        }
        *reinterpret_cast<uint32_t *>(dst + 8 * kStep * r) = v;
    }
}

}  // namespace tdes_bs
