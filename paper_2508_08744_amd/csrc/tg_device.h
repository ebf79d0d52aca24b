// Device-side building blocks shared by the kernels: the counter-based hash, the
// 64-bit (distance, id) sort key, and wave-level sort / merge networks.
// gfx950 only: wavefronts are 64 lanes wide.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned long long u64;
typedef unsigned int u32;

#define TG_WAVE 64
#define TG_RANGE_NONINT 8        // word of the range buffer: set when a value of X is not a whole number
#define TG_EMPTY_KEY 0xFFFFFFFFFFFFFFFFull
#define TG_GOLDEN 0x9E3779B97F4A7C15ull
#define TG_ID_MASK 0x7FFFFFFFu     // list word: id in bits 0..30, "fresh" mark in bit 31

// tags of the three random decisions (initial lists, reverse priority, candidate slot)
#define TG_TAG_INIT 1ull
#define TG_TAG_REV(round) (2ull + 4ull * (u64)(round))
#define TG_TAG_SLOT(round) (3ull + 4ull * (u64)(round))

// SplitMix64 output function (Steele, Lea, Flood 2014).
__host__ __device__ inline u64 tg_mix64(u64 z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
// hash(seed, tag, x, y) = mix(mix(mix(seed + tag*golden) + x) + y); the first mix is
// done once on the host per round and passed in as `hs`.
__host__ __device__ inline u64 tg_hash_seed(u64 seed, u64 tag) { return tg_mix64(seed + tag * TG_GOLDEN); }
__device__ inline u64 tg_hash_xy(u64 hs, u64 x, u64 y) { return tg_mix64(tg_mix64(hs + x) + y); }

// Order-preserving map fp32 -> u32 (works for negative values; -0 is folded into +0).
__device__ inline u32 tg_ord(float f)
{
    f += 0.0f;
    u32 b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float tg_unord(u32 o)
{
    u32 b = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(b);
}

// 64-bit key: [63:32] ordered distance bits, [31:2] id, [1] came-from-candidate, [0] fresh.
// Ids are distinct inside any one comparison set, so the two low bits never decide.
__device__ inline u64 tg_key(float dist, u32 id, u32 low2) { return ((u64)tg_ord(dist) << 32) | (u64)((id << 2) | low2); }
__device__ inline u32 tg_key_id(u64 key) { return ((u32)key) >> 2; }
__device__ inline float tg_key_dist(u64 key) { return tg_unord((u32)(key >> 32)); }

__device__ inline int tg_lane() { return (int)__lane_id(); }

__device__ inline u64 tg_shfl64(u64 x, int src)
{
    u32 lo = (u32)__shfl((int)(u32)x, src);
    u32 hi = (u32)__shfl((int)(u32)(x >> 32), src);
    return ((u64)hi << 32) | lo;
}
__device__ inline u64 tg_shfl_xor64(u64 x, int mask)
{
    u32 lo = (u32)__shfl_xor((int)(u32)x, mask);
    u32 hi = (u32)__shfl_xor((int)(u32)(x >> 32), mask);
    return ((u64)hi << 32) | lo;
}
__device__ inline u64 tg_min64(u64 a, u64 b) { return a < b ? a : b; }
__device__ inline u64 tg_max64(u64 a, u64 b) { return a < b ? b : a; }

// Value held by lane (lane ^ XOR).  Inside a row of 16 lanes this is one or two DPP moves
// (quad permutations, mirrors of 8 and 16 lanes, rotation by 8); across rows it goes through
// the LDS crossbar.
template <int CTRL>
__device__ inline u64 tg_dpp64(u64 x)
{
    // every lane has a source inside its row for the controls used here, so no fill value is needed
    const u32 lo = (u32)__builtin_amdgcn_mov_dpp((int)(u32)x, CTRL, 0xF, 0xF, true);
    const u32 hi = (u32)__builtin_amdgcn_mov_dpp((int)(u32)(x >> 32), CTRL, 0xF, 0xF, true);
    return ((u64)hi << 32) | lo;
}
template <int XOR>
__device__ inline u64 tg_partner(u64 x)
{
    if (XOR == 1) return tg_dpp64<0xB1>(x);                     // quad_perm 1,0,3,2
    if (XOR == 2) return tg_dpp64<0x4E>(x);                     // quad_perm 2,3,0,1
    if (XOR == 3) return tg_dpp64<0x1B>(x);                     // quad_perm 3,2,1,0
    if (XOR == 4) return tg_dpp64<0x1B>(tg_dpp64<0x141>(x));    // mirror of 8, then of 4: 7 ^ 3
    if (XOR == 7) return tg_dpp64<0x141>(x);                    // row_half_mirror
    if (XOR == 8) return tg_dpp64<0x128>(x);                    // row_ror 8
    if (XOR == 15) return tg_dpp64<0x140>(x);                   // row_mirror
    return tg_shfl_xor64(x, XOR);
}
// one compare-exchange: the lane keeps the smaller of (key, other) if keep_min, else the larger
__device__ inline u64 tg_cmpx(u64 key, u64 other, bool keep_min)
{
    const bool lt = key < other;
    return (lt != keep_min) ? other : key;
}
template <int SIZE>
__device__ inline u64 tg_sort_level(u64 key, int lane)
{
    // blocks of SIZE lanes: fold each block onto itself, then clean its halves
    key = tg_cmpx(key, tg_partner<SIZE - 1>(key), (lane & (SIZE >> 1)) == 0);
    if (SIZE >= 64) key = tg_cmpx(key, tg_partner<16>(key), (lane & 16) == 0);
    if (SIZE >= 32) key = tg_cmpx(key, tg_partner<8>(key), (lane & 8) == 0);
    if (SIZE >= 16) key = tg_cmpx(key, tg_partner<4>(key), (lane & 4) == 0);
    if (SIZE >= 8) key = tg_cmpx(key, tg_partner<2>(key), (lane & 2) == 0);
    if (SIZE >= 4) key = tg_cmpx(key, tg_partner<1>(key), (lane & 1) == 0);
    return key;
}
// The lane's number, worked out where it is asked for: its six masks, kept across the loop around a network, cost phase 2 and the
// two-hop collection the registers that they have least of.
__device__ inline int tg_lane_here()
{
    int lane = tg_lane();
    asm volatile("" : "+v"(lane));
    return lane;
}
// Ascending bitonic sort of one key per lane across the wave (HALVES: across each half of it), every exchange on whole keys.
template <bool HALVES>
__device__ inline u64 tg_wave_sort_whole(u64 key)
{
    const int lane = tg_lane_here();
    key = tg_sort_level<2>(key, lane);
    key = tg_sort_level<4>(key, lane);
    key = tg_sort_level<8>(key, lane);
    key = tg_sort_level<16>(key, lane);
    key = tg_sort_level<32>(key, lane);
    if (!HALVES) key = tg_sort_level<64>(key, lane);
    return key;
}

// ---- networks on 32-bit keys: an exchange is a move (DPP inside a row of 16 lanes, a lane swap across rows) and a median of three, the
// third being 0 in the lane that keeps the smaller key and all ones in the one that keeps the larger.  (A whole key takes two moves, a
// compare, a mask operation and two selects, across rows two trips through the LDS crossbar.)
template <int CTRL>
__device__ inline u32 tg_dpp32(u32 x)
{
    return (u32)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}
template <int XOR>
__device__ inline u32 tg_partner32(u32 x)
{
    static_assert(XOR == 1 || XOR == 2 || XOR == 7 || XOR == 15, "one DPP move");
    if (XOR == 1) return tg_dpp32<0xB1>(x);
    if (XOR == 2) return tg_dpp32<0x4E>(x);
    if (XOR == 7) return tg_dpp32<0x141>(x);
    return tg_dpp32<0x140>(x);
}
__device__ inline u32 tg_median32(u32 a, u32 b, u32 c) { return max(min(a, b), min(max(a, b), c)); }
// all ones where bit J of the lane is set
template <int J>
__device__ inline u32 tg_lane_bit(int lane) { return (lane & J) ? 0xFFFFFFFFu : 0u; }
// lane ^ J for J = 1, 2, 4, 8, 16, 32; lane ^ J mirrored inside its group for J = 3, 7, 15; the lane with the upper half of bits keeps the larger key
template <int J>
__device__ inline u32 tg_exchange32(u32 x, int lane)
{
    if (J == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return tg_median32(r[0], r[1], tg_lane_bit<32>(lane));
    }
    if (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return tg_median32(r[0], r[1], tg_lane_bit<16>(lane));
    }
    if (J == 15) return tg_median32(x, tg_dpp32<0x140>(x), tg_lane_bit<8>(lane));
    if (J == 8) return tg_median32(x, tg_dpp32<0x128>(x), tg_lane_bit<8>(lane));
    if (J == 7) return tg_median32(x, tg_dpp32<0x141>(x), tg_lane_bit<4>(lane));
    if (J == 4) return tg_median32(x, tg_dpp32<0x1B>(tg_dpp32<0x141>(x)), tg_lane_bit<4>(lane));
    if (J == 3) return tg_median32(x, tg_dpp32<0x1B>(x), tg_lane_bit<2>(lane));
    if (J == 2) return tg_median32(x, tg_dpp32<0x4E>(x), tg_lane_bit<2>(lane));
    return tg_median32(x, tg_dpp32<0xB1>(x), tg_lane_bit<1>(lane));
}
// sorts every group of 2 J lanes whose keys are bitonic
template <int J>
__device__ inline u32 tg_clean32(u32 x, int lane)
{
    if (J >= 32) x = tg_exchange32<32>(x, lane);
    if (J >= 16) x = tg_exchange32<16>(x, lane);
    if (J >= 8) x = tg_exchange32<8>(x, lane);
    if (J >= 4) x = tg_exchange32<4>(x, lane);
    if (J >= 2) x = tg_exchange32<2>(x, lane);
    return tg_exchange32<1>(x, lane);
}
// Ascending sort across the wave of the keys of the first `count` lanes (uniform), the others holding all ones or at least nothing smaller.
__device__ inline u32 tg_wave_sort32_first(u32 x, int count)
{
    const int lane = tg_lane_here();
    // (odd rows run backwards, by inverted keys, for the level of 32, the upper half for the level of 64)
    if (count > 16) x ^= tg_lane_bit<16>(lane);
    x = tg_exchange32<1>(x, lane);
    x = tg_exchange32<1>(tg_exchange32<3>(x, lane), lane);
    x = tg_clean32<2>(tg_exchange32<7>(x, lane), lane);
    x = tg_clean32<4>(tg_exchange32<15>(x, lane), lane);
    if (count > 16) {
        x ^= tg_lane_bit<16>(lane);
        if (count > 32) x ^= tg_lane_bit<32>(lane);
        x = tg_clean32<16>(x, lane);
        if (count > 32) x = tg_clean32<32>(x ^ tg_lane_bit<32>(lane), lane);
    }
    return x;
}
__device__ inline u32 tg_wave_sort32(u32 x) { return tg_wave_sort32_first(x, 64); }

// the key of the lane before (the first: 0) and behind (the last: all ones); HALVES: the two halves of the wave are strangers
template <bool HALVES>
__device__ inline u64 tg_lane_before(u64 x)
{
    const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)x, 0x138, 0xF, 0xF, false);
    const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(x >> 32), 0x138, 0xF, 0xF, false);
    const u64 y = ((u64)hi << 32) | lo;
    return HALVES && tg_lane() == 32 ? 0ull : y;
}
template <bool HALVES>
__device__ inline u64 tg_lane_behind(u64 x)
{
    const u32 lo = (u32)__builtin_amdgcn_update_dpp(-1, (int)(u32)x, 0x130, 0xF, 0xF, false);
    const u32 hi = (u32)__builtin_amdgcn_update_dpp(-1, (int)(u32)(x >> 32), 0x130, 0xF, 0xF, false);
    const u64 y = ((u64)hi << 32) | lo;
    return HALVES && tg_lane() == 31 ? ~0ull : y;
}
// Whole keys by a network on 32-bit ones: the upper 26 bits of a key (of a distance: sign, exponent, 17 bits) with its lane below are
// sorted, the keys fetched in that order, and looked over: keys that agree in those bits may still stand the wrong way round.  One or
// two exchanges of neighbours put a pair or three of them right; more (masses of equal distances) go through the network of whole keys.
__device__ inline u32 tg_short_key(u64 key) { return ((u32)(key >> 32) & ~63u) | (u32)tg_lane(); }
template <bool HALVES>
__device__ inline u64 tg_fetch_sorted(u64 key, u32 order)
{
    const int at = (int)(order << 2) & 252;
    const u32 lo = (u32)__builtin_amdgcn_ds_bpermute(at, (int)(u32)key);
    const u32 hi = (u32)__builtin_amdgcn_ds_bpermute(at, (int)(u32)(key >> 32));
    u64 x = ((u64)hi << 32) | lo;
    if (__ballot(x < tg_lane_before<HALVES>(x)) == 0ull) return x;
    const bool odd = (tg_lane() & 1) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        x = odd ? tg_min64(x, tg_lane_behind<HALVES>(x)) : tg_max64(x, tg_lane_before<HALVES>(x));
        x = tg_cmpx(x, tg_partner<1>(x), !odd);
    }
    if (__ballot(x < tg_lane_before<HALVES>(x)) == 0ull) return x;
    return tg_wave_sort_whole<HALVES>(x);
}
// Ascending sort across the wave where only the first `count` lanes (uniform) hold keys and the others the empty key, which stays behind.
__device__ inline u64 tg_wave_sort_first(u64 key, int count) { return tg_fetch_sorted<false>(key, tg_wave_sort32_first(tg_short_key(key), count)); }
__device__ inline u64 tg_wave_sort(u64 key) { return tg_wave_sort_first(key, 64); }

// a and b are ascending across the wave; returns the 64 smallest keys of their union,
// ascending (the wave-level form of the rank merge of section 4.2).
__device__ inline u64 tg_wave_merge_low(u64 a, u64 b)
{
    const u64 x = tg_min64(a, tg_partner<63>(b));
    return tg_fetch_sorted<false>(x, tg_clean32<32>(tg_short_key(x), tg_lane_here()));
}
// the same two for each half of the wave by itself: 32 keys a half
__device__ inline u64 tg_half_sort(u64 key) { return tg_fetch_sorted<true>(key, tg_wave_sort32_first(tg_short_key(key), 32)); }
__device__ inline u64 tg_half_merge_low(u64 a, u64 b)
{
    const u64 x = tg_min64(a, tg_partner<31>(b));
    return tg_fetch_sorted<true>(x, tg_clean32<16>(tg_short_key(x), tg_lane_here()));
}

__device__ inline u64 tg_lanemask_lt() { return (1ull << tg_lane()) - 1ull; }

// Whether X holds bytes in the wider sense: whole numbers within 255 of each other, small enough that every fp32 sum of the norms,
// the inner products and their combination is exact (2 d max|x|^2 <= 2^24).  range: what the kernel of the norms found.
__device__ inline bool tg_whole_exact(const u32* __restrict__ range, int d)
{
    if (range[TG_RANGE_NONINT] != 0u) return false;
    const float m = fmaxf(fabsf(tg_unord(range[0])), fabsf(tg_unord(range[1])));
    return 2.0f * (float)d * m * m <= 16777216.0f;
}
__device__ inline bool tg_whole_bytes(const u32* __restrict__ range, int d)
{
    return tg_whole_exact(range, d) && tg_unord(range[1]) - tg_unord(range[0]) <= 255.0f;
}

// whether the nodes are taken in g.order (not where X holds bytes and phase 1 reads 128 of them a row: the kernels that would make the
// order end at once then; 1M x 128 bytes, four rounds: 0.25 ms for the order, 0.1 gained)
template <class G>
__device__ inline bool tg_use_order(const G& g) { return g.order && !(g.bytes && tg_whole_bytes(g.bytes, g.d)); }

// work record of the join: anchor | |NEW| << 32 | (|NEW|+|OLD|) << 40
__device__ inline u64 tg_pack_rec(u32 v, int nN, int nT) { return (u64)v | ((u64)nN << 32) | ((u64)nT << 40); }
