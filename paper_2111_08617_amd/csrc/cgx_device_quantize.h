// Device code of the quantizer: encoding of chunks, rows, wide buckets, short ends and
// generic tiles, and the pass-through copy (shared by the quantize and the fused kernels).
#pragma once

#include "cgx_device.h"

namespace cgx {
namespace {

// ---------------------------------------------------------------- quantize

// Bytes 2 of a and b (levels above 16 bits of fraction) in bytes 0 and 1, or 2 and 3, of a word of zeros.
__device__ __forceinline__ uint32_t levels_low(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x0c0c0602u); }
__device__ __forceinline__ uint32_t levels_high(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x06020c0cu); }
// The same positions, with all bits set where the sign bit of a, b is.
__device__ __forceinline__ uint32_t signs_low(float a, float b)
{
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a), 0x0c0c0b09u);
}
__device__ __forceinline__ uint32_t signs_high(float a, float b)
{
    return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a), 0x0b090c0cu);
}

// Codes of BITS bits, one per byte, from levels and sign masks, one per byte.  (level ^ sign) + (sign & 1) within
// BITS bits: no carry leaves a byte.  (At 8 bits the low seven are added apart: level 0 under a set sign would carry.)
template <int BITS>
__device__ __forceinline__ uint32_t signed_bytes(uint32_t level, uint32_t sign)
{
    constexpr uint32_t kOnes = 0x01010101u, kMask = kOnes * ((1u << BITS) - 1u);
    if constexpr (BITS == 8) return (((level ^ sign) & (kOnes * 0x7fu)) + (sign & kOnes)) ^ (sign & (kOnes * 0x80u));
    return ((level ^ (sign & kMask)) + (sign & kOnes)) & kMask;
}

// acc + (level << SHIFT), the level (the sum's upper half) picked, shifted and added by one instruction.
template <int SHIFT>
__device__ __forceinline__ uint32_t add_level(uint32_t acc, uint32_t sum)
{
    static_assert(SHIFT < 16, "the factor is a 16-bit operand");
    uint32_t r;
    if constexpr (SHIFT <= 6)
        asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(sum), "n"(1u << SHIFT), "v"(acc));
    else
        asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(sum), "s"(1u << SHIFT), "v"(acc));
    return r;
}

// Four codes of BITS bits from the four bytes of t (which hold nothing else), first code lowest.
template <int BITS>
__device__ __forceinline__ uint32_t join_bytes(uint32_t t)
{
    constexpr uint32_t kOne = 0x00010001u * ((1u << BITS) - 1u), kTwo = (1u << (2 * BITS)) - 1u;
    // (what the first step leaves above its fields is taken from the shifted word by the second)
    const uint32_t pairs = (t & kOne) | ((t >> (8 - BITS)) & ~kOne);
    return (pairs & kTwo) | ((pairs >> (16 - 2 * BITS)) & ~kTwo);
}

// Eight codes of BITS bits (3, 5, 6, 7) from two words of four.
template <int BITS>
__device__ __forceinline__ uint64_t join_halves(uint32_t lo, uint32_t hi)
{
    const uint32_t low = lo | (hi << (4 * BITS));
    if constexpr (BITS == 3) return low;
    return (uint64_t(hi >> (32 - 4 * BITS)) << 32) | low;
}

// How codes are cut.  2 and 4 bits: the levels are gathered byte by byte from the sums of position and draw, two per
// v_perm_b32, and shifted into place for four codes at once: 10 vector instructions fewer per 8 codes than a minimum, a shift
// and a shift-or per code (kNormSign, whose codes are also cut from the signs: 30 fewer).  The minimum falls away: up to 7 bits
// the position of an element of the bucket does not exceed levels * 65536, since x - mn rounds to at most the range and inv16 to at
// most (1 + 2^-24) of its value, so their product is below levels * 65536 + 1/2 before it is rounded, and that whole number is one
// that binary32 holds.  That says nothing of the zeros in the missing elements of a layer's last group, which may lie any way
// above a bucket of negative values: each level is cut to its field (v_bitop3_b32 joins the bytes and cuts them in one
// instruction), or the fold of the 2-bit codes would carry what is above the field down into the codes of elements that are
// there.  (kNormSign: a missing element's level is 0.)
//
// The other widths (3, 5, 6, 7): four levels at a time are summed at their places by v_mad_u32_u16, which picks the upper half of
// the sum, shifts and adds in one instruction of 4.8 cycles where a shift, a minimum and a shift-or took 12; a missing element's
// level can only reach upwards, into codes that are missing too.  8-bit levels take their minimum two at a time (v_pk_min_u16).
// Signed codes of these widths are cut as bytes and the bytes joined.  Builds in turn on one box, us: binary16 quantize of 26 M
// elements, 3 bits 15.7 -> 15.4, 5 bits 16.3 -> 15.8, 8 bits 15.4 -> 15.3 (355 M, 128 to a bucket, both builds on the same buffers: 8 bits
// 168.3 and 168.4, 5 bits 171.5 -> 168.7; buckets of 96, 8 bits, 202.8 -> 196.7); norm-and-sign of 101 M, 3 bits 48.3 -> 45.0, 8 bits
// 51.5 -> 49.9; fused step of 2 peers, 17 M elements, 3 bits 14.0 -> 13.7, 8 bits 14.3 -> 14.2, norm-and-sign 14.6 -> 13.9.
//
// Measured with the draws of kDrawsQuad below, builds in turn on one box, us: binary16 quantize of 355 M elements 155.0 -> 144.0,
// the fused step of a 13.7 M share of 8 peers 19.4 -> 18.5, norm-and-sign reduce and requantize of it 33.8 -> 32.7.  25.6 M and 1.3 G
// binary32 elements are bound by memory and stay at 19.8 and 988.

// Index of the pair (lower 32 bits) that element `at` (a multiple of 8) behind `first` lies in.  first is uniform over the wave, so
// this is one vector addition; (first + at) >> 1 in 64 bits was two instructions per group.
__device__ __forceinline__ uint32_t first_pair(int64_t first, int at) { return uint32_t(uint64_t(first) >> 1) + uint32_t(at >> 1); }

// The 8 codes of one group, packed: element j of the group has buffer index 2 * pair0 + odd + j, key = generator key of
// the tile.  odd (0 or 1, uniform over a tile: groups start 8 elements apart) tells whether the group starts on the upper
// half of a generator word; then its 8 draws are the 16-bit halves 1..8 of words pair0 .. pair0 + 4 instead of halves
// 0..7 of words pair0 .. pair0 + 3.  DRAWS (Draws, cgx_kernels.h; the host picks the instantiation): kDrawsOdd alone has
// the fifth word and the selection, taken by the tiles that do start on odd elements (20 M ragged binary16 elements in buckets of
// 160, fused, 4 peers: 25.0 -> 24.25 us, first_pair's share in it included; where all tiles start odd the branch costs a large
// binary16 quantize up to half a per cent, 355 M elements of 8 bits 241.1 -> 242.3), and kDrawsQuad knows that pair0 is a multiple of 4: no carry leaves its two lowest bits,
// so the words of its four pairs differ in them alone until the first multiplication: 3 instructions fewer of 76 (by itself, us:
// binary16 quantize of 372 M elements 159 -> 155, fused step of 14.7 M elements and 8 peers 20.65 -> 20.4).
template <int SCHEME, int BITS, int DRAWS>
__device__ __forceinline__ uint64_t encode_group(const float (&x)[8], const Scale &s, uint32_t pair0, uint32_t key,
                                                 uint32_t odd_start)
{
    constexpr uint32_t kLevels = top_level<SCHEME>(BITS);
    uint32_t word[4];
    if (DRAWS == kDrawsQuad) {
        const uint32_t mixed = mix32_head(pair0 ^ key);
#pragma unroll
        for (int k = 0; k < 4; k++) word[k] = mix32_tail(mixed ^ uint32_t(k));
    } else {
#pragma unroll
        for (int k = 0; k < 4; k++) word[k] = mix32((pair0 + k) ^ key);
        if (DRAWS == kDrawsOdd && odd_start) {       // (a branch: half of the tiles of a ragged plan start on even elements)
            const uint32_t next = mix32((pair0 + 4) ^ key);
#pragma unroll
            for (int k = 0; k < 4; k++) word[k] = __builtin_amdgcn_alignbit(k < 3 ? word[k + 1] : next, word[k], 16u);
        }
    }
    uint32_t sum[8];                                 // position of the element between the levels, plus its draw
#pragma unroll
    for (int k = 0; k < 4; k++) {
        // the pair's two draws
        const uint32_t w = word[k];
        sum[2 * k] = position_of<SCHEME>(x[2 * k], s) + (w & 0xffffU);
        sum[2 * k + 1] = position_of<SCHEME>(x[2 * k + 1], s) + (w >> 16);
    }
    [[maybe_unused]] constexpr uint32_t kField = 0x01010101u * ((1u << BITS) - 1u);
    if constexpr (BITS == 4) {
        uint32_t even = levels_low(sum[0], sum[2]) | levels_high(sum[4], sum[6]);
        uint32_t odd = levels_low(sum[1], sum[3]) | levels_high(sum[5], sum[7]);
        if (SCHEME == kNormSign) {
            even = signed_bytes<4>(even, signs_low(x[0], x[2]) | signs_high(x[4], x[6]));
            odd = signed_bytes<4>(odd, signs_low(x[1], x[3]) | signs_high(x[5], x[7]));
        } else {
            even &= kField;
            odd = opaque(odd & kField);
        }
        return even | (odd << 4);
    } else if constexpr (BITS == 2) {
        uint32_t low = levels_low(sum[0], sum[4]) | levels_high(sum[1], sum[5]);       // codes 0, 4, 1, 5
        uint32_t high = levels_low(sum[2], sum[6]) | levels_high(sum[3], sum[7]);      // codes 2, 6, 3, 7
        if (SCHEME == kNormSign) {
            low = signed_bytes<2>(low, signs_low(x[0], x[4]) | signs_high(x[1], x[5]));
            high = signed_bytes<2>(high, signs_low(x[2], x[6]) | signs_high(x[3], x[7]));
        } else {
            low &= kField;
            high = opaque(high & kField);
        }
        const uint32_t t = low | (high << 4);
        return (t | (t >> 14)) & 0xffffu;
    } else if constexpr (SCHEME == kNormSign) {
        const uint32_t lo = signed_bytes<BITS>(levels_low(sum[0], sum[1]) | levels_high(sum[2], sum[3]),
                                               signs_low(x[0], x[1]) | signs_high(x[2], x[3]));
        const uint32_t hi = signed_bytes<BITS>(levels_low(sum[4], sum[5]) | levels_high(sum[6], sum[7]),
                                               signs_low(x[4], x[5]) | signs_high(x[6], x[7]));
        if constexpr (BITS == 8)
            return (uint64_t(hi) << 32) | lo;
        else
            return join_halves<BITS>(join_bytes<BITS>(lo), join_bytes<BITS>(hi));
    } else if constexpr (BITS == 8) {
        // the one width whose levels take the minimum: two at a time
        typedef uint16_t half2u __attribute__((ext_vector_type(2)));
        uint32_t pair[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t levels = __builtin_amdgcn_perm(sum[2 * k + 1], sum[2 * k], 0x07060302u);
            pair[k] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(half2u, levels),
                                                                             half2u{uint16_t(kLevels), uint16_t(kLevels)}));
        }
        const uint32_t lo = __builtin_amdgcn_perm(pair[1], pair[0], 0x06040200u);
        const uint32_t hi = __builtin_amdgcn_perm(pair[3], pair[2], 0x06040200u);
        return (uint64_t(hi) << 32) | lo;
    } else if constexpr (BITS == 1) {
        uint32_t acc = add_level<1>(sum[0] >> 16, sum[1]);
        acc = add_level<3>(add_level<2>(acc, sum[2]), sum[3]);
        acc = add_level<5>(add_level<4>(acc, sum[4]), sum[5]);
        return add_level<7>(add_level<6>(acc, sum[6]), sum[7]);
    } else {
        uint32_t half[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            half[k] = add_level<2 * BITS>(add_level<BITS>(sum[4 * k] >> 16, sum[4 * k + 1]), sum[4 * k + 2]);
            if constexpr (3 * BITS < 16)
                half[k] = add_level<3 * BITS>(half[k], sum[4 * k + 3]);
            else
                half[k] |= (sum[4 * k + 3] >> 16) << (3 * BITS);
        }
        return join_halves<BITS>(half[0], half[1]);
    }
}

// Minimum and maximum (kNormSign: +0 and the largest magnitude) of a lane's chunk, folded into mn / mx.
template <int SCHEME, int OWN>
__device__ __forceinline__ void lane_extent(const float (&x)[OWN][8], float &mn, float &mx)
{
#pragma unroll
    for (int r = 0; r < OWN; r++)
#pragma unroll
        for (int j = 0; j < 8; j++) {
            if (SCHEME == kNormSign) {
                mx = __builtin_fmaxf(mx, __builtin_fabsf(x[r][j]));
            } else {
                mn = __builtin_fminf(mn, x[r][j]);
                mx = __builtin_fmaxf(mx, x[r][j]);
            }
        }
}

// Codes of a chunk whose elements all take the scale s: staged, then sent out.
template <int SCHEME, int BITS, int DRAWS>
__device__ __forceinline__ void encode_chunk(const float (&x)[G][8], const Scale &s, const LaneMap &map,
                                             int64_t first, uint32_t key, uint8_t *__restrict__ out,
                                             uint4v *stage, int lane)
{
#pragma unroll
    for (int r = 0; r < G; r++) {
        const uint32_t pair0 = first_pair(first, map.group(r));
        stage_codes<BITS>(reinterpret_cast<uint8_t *>(stage) + (map.group(r) >> 3) * BITS,
                          encode_group<SCHEME, BITS, DRAWS>(x[r], s, pair0, key, uint32_t(first) & 1u));
    }
    // the chunk's codes leave as whole 16-byte vectors, consecutive across lanes
    wave_lds_fence();
    flush_stage(stage, reinterpret_cast<uint4v *>(out), kChunk * BITS / 128, lane);
    wave_lds_fence();
}

// One chunk held in registers (x) -> meta of its buckets and its packed codes.
// first = buffer index of the chunk's first element; key = generator key of the tile.
// meta_chunk points at the meta of the chunk's first bucket.
template <int SCHEME, int BITS, int DRAWS>
__device__ __forceinline__ void quantize_chunk(const float (&x)[G][8], const LaneMap &map, int lane, int64_t first,
                                               uint32_t key, float *__restrict__ meta_chunk,
                                               uint8_t *__restrict__ out, uint4v *stage)
{
    constexpr uint32_t kLevels = top_level<SCHEME>(BITS);
    float mn = SCHEME == kNormSign ? 0.0f : x[0][0], mx = mn;
    lane_extent<SCHEME>(x, mn, mx);
    if (SCHEME == kNormSign)
        group_max(mx, map.lg, lane);
    else
        group_minmax(mn, mx, map.lg, lane);
    const Scale s = bucket_scale(mn, mx, int(kLevels));
    if (map.lp == 0) store_meta<SCHEME>(meta_chunk, map.bi, s);
    encode_chunk<SCHEME, BITS, DRAWS>(x, s, map, first, key, out, stage, lane);
}

// The same for buckets of 32 or 64 elements, with the chunk held row by row: group r of lane l
// is elements [512 r + 8 l, 512 r + 8 l + 8) of the chunk, so every load instruction of the
// caller covers 64 consecutive groups (with the bucket-major mapping a lane's four groups would
// be one or two whole buckets and each load instruction would touch 32 or 64 separate lines,
// 16 to 64 bytes of each: measured 21 % of the HBM peak at 32-element buckets).  A bucket is
// bucket / 8 neighbouring lanes of one row; a lane serves four buckets and pays the two
// divisions four times.
template <int SCHEME, int BITS, int DRAWS>
__device__ __forceinline__ void quantize_chunk_rows(const float (&x)[G][8], int bucket, int lane, int64_t first,
                                                    uint32_t key, float *__restrict__ meta_chunk,
                                                    uint8_t *__restrict__ out, uint4v *stage)
{
    constexpr uint32_t kLevels = top_level<SCHEME>(BITS);
    constexpr int kRow = kWave * 8;                  // elements per row
    const int lg = bucket == 32 ? 2 : 3;             // log2(lanes per bucket)
    const int buckets_per_row = kRow / bucket;
#pragma unroll
    for (int r = 0; r < G; r++) {
        float mn, mx;
        if (SCHEME == kNormSign) {
            mn = 0.0f;
            mx = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; j++) mx = __builtin_fmaxf(mx, __builtin_fabsf(x[r][j]));
            group_max(mx, lg, lane);
        } else {
            mn = x[r][0];
            mx = x[r][0];
#pragma unroll
            for (int j = 1; j < 8; j++) {
                mn = __builtin_fminf(mn, x[r][j]);
                mx = __builtin_fmaxf(mx, x[r][j]);
            }
            group_minmax(mn, mx, lg, lane);
        }
        const Scale s = bucket_scale(mn, mx, int(kLevels));
        if ((lane & ((1 << lg) - 1)) == 0) store_meta<SCHEME>(meta_chunk, r * buckets_per_row + (lane >> lg), s);
        const int e = r * kRow + lane * 8;           // the group's first element within the chunk
        const uint32_t pair0 = first_pair(first, e);
        stage_codes<BITS>(reinterpret_cast<uint8_t *>(stage) + (e >> 3) * BITS,
                          encode_group<SCHEME, BITS, DRAWS>(x[r], s, pair0, key, uint32_t(first) & 1u));
    }
    wave_lds_fence();
    flush_stage(stage, reinterpret_cast<uint4v *>(out), kChunk * BITS / 128, lane);
    wave_lds_fence();
}

// A chunk fetched through the wave's LDS area, so that every load instruction takes 1 KB of consecutive bytes; each lane
// then reads its groups from there.  Read into registers directly, a lane's 32 consecutive bytes come from two
// instructions that each cover every other 16 bytes of 2 KB; a kernel that only moves bytes loses 5 to 9 % of its
// rate with that pattern.  ALIGNED: the chunk starts on a 16-byte boundary and the loads go straight into LDS (no
// registers held while in flight).  Otherwise they pass through registers, at the alignment of an element: for
// binary32 (quantize of 67 M elements in ragged layers, us: 4 bit, buckets of 512, 56.5 read directly and 52.4 this way,
// 52 where the layers are aligned; 2 bit, 128, 64.4 and 51.2; 4 bit, 32, 61.4 and 55.5).  A lane's 8 binary16
// elements are one vector, so that type has no such pattern to avoid.
// The area must hold the chunk as stored (kChunk elements of DT).
template <int DT, bool ALIGNED, typename Map>
__device__ __forceinline__ void chunk_through_lds(const void *__restrict__ grad, int64_t first, const Map &map,
                                                  float (&x)[G][8], uint4v *stage, int lane)
{
    constexpr int S = DT == CGX_F16 ? 2 : 4;
    constexpr int kVecs = kChunk * S / 16;
    static_assert(kVecs % kWave == 0, "whole load instructions");
    const uint8_t *at = reinterpret_cast<const uint8_t *>(grad) + first * S;
    if constexpr (ALIGNED) {
        const uint4v *src = reinterpret_cast<const uint4v *>(at);
#pragma unroll
        for (int k = 0; k < kVecs / kWave; k++) load_to_lds16(src + k * kWave + lane, stage + k * kWave);
        wait_vector_memory();
    } else {
        using Vec = std::conditional_t<DT == CGX_F16, uint4u2, uint4u4>;
        const Vec *src = reinterpret_cast<const Vec *>(at);
        uint4v raw[kVecs / kWave];
#pragma unroll
        for (int k = 0; k < kVecs / kWave; k++) raw[k] = __builtin_nontemporal_load(src + k * kWave + lane);
#pragma unroll
        for (int k = 0; k < kVecs / kWave; k++) stage[k * kWave + lane] = raw[k];
    }
    wave_lds_fence();
#pragma unroll
    for (int r = 0; r < G; r++) {
        if (DT == CGX_F16) {
            const half8v h = *reinterpret_cast<const half8v *>(reinterpret_cast<const _Float16 *>(stage) + map.group(r));
#pragma unroll
            for (int j = 0; j < 8; j++) x[r][j] = float(h[j]);
        } else {
            const float4v *p = reinterpret_cast<const float4v *>(reinterpret_cast<const float *>(stage) + map.group(r));
            const float4v a = p[0], b = p[1];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                x[r][j] = a[j];
                x[r][4 + j] = b[j];
            }
        }
    }
    wave_lds_fence();      // the codes are staged in the same area
}

// VIA_LDS: every vectorised tile of the plan starts on a 16-byte boundary of the buffer (a property
// of the tile table; the host picks the instantiation).
template <int SCHEME, int DT, int BITS, int DRAWS, bool VIA_LDS = false>
__device__ __forceinline__ void quantize_fast(const void *__restrict__ grad, uint8_t *__restrict__ packed,
                                              float *__restrict__ meta, const Tile &tile, int bucket,
                                              uint32_t seed_lo, uint32_t seed_hi, int lane, uint4v *stage)
{
    const LaneMap map(tile, bucket, lane);
    const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
    const int chunks = int(tile.count / kChunk);
    const int buckets_per_chunk = kChunk / bucket;
    for (int c = 0; c < chunks; c++) {
        const int64_t first = tile.elem0 + int64_t(c) * kChunk;
        float x[G][8];
        if constexpr (VIA_LDS || DT == CGX_F32) {
            chunk_through_lds<DT, VIA_LDS>(grad, first, map, x, stage, lane);
        } else {
#pragma unroll
            for (int r = 0; r < G; r++) load8<DT>(grad, first + map.group(r), x[r]);
        }
        quantize_chunk<SCHEME, BITS, DRAWS>(x, map, lane, first, key,
                                     meta + kMetaFloats<SCHEME> * (tile.bucket0 + c * buckets_per_chunk),
                                     packed + tile.packed_off + int64_t(c) * (kChunk * BITS / 8), stage);
    }
}

// Row-by-row mapping: group r of a lane is elements [512 r + 8 lane, + 8) of the chunk.
struct RowMap {
    int lane;
    __device__ __forceinline__ int group(int r) const { return r * (kWave * 8) + lane * 8; }
};

// quantize_fast for buckets of 32 or 64 elements (row-by-row mapping).
template <int SCHEME, int DT, int BITS, int DRAWS>
__device__ __forceinline__ void quantize_fast_rows(const void *__restrict__ grad, uint8_t *__restrict__ packed,
                                                   float *__restrict__ meta, const Tile &tile, int bucket,
                                                   uint32_t seed_lo, uint32_t seed_hi, int lane, uint4v *stage)
{
    const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
    const int chunks = int(tile.count / kChunk);
    const int buckets_per_chunk = kChunk / bucket;
    for (int c = 0; c < chunks; c++) {
        const int64_t first = tile.elem0 + int64_t(c) * kChunk;
        float x[G][8];
        if constexpr (DT == CGX_F32) {
            chunk_through_lds<DT, false>(grad, first, RowMap{lane}, x, stage, lane);
        } else {
#pragma unroll
            for (int r = 0; r < G; r++) load8<DT>(grad, first + RowMap{lane}.group(r), x[r]);
        }
        quantize_chunk_rows<SCHEME, BITS, DRAWS>(x, bucket, lane, first, key,
                                          meta + kMetaFloats<SCHEME> * (tile.bucket0 + c * buckets_per_chunk),
                                          packed + tile.packed_off + int64_t(c) * (kChunk * BITS / 8), stage);
    }
}

// The codes of a lane's groups of a run (8 * BITS bits each, group after group) into LDS, OWN * BITS bytes per lane.
// The area starts on 16 bytes.
template <int BITS, int OWN>
__device__ __forceinline__ void stage_run_codes(uint8_t *area, const uint64_t (&codes)[OWN], int lane)
{
    if constexpr (OWN == 4) {
        // 32 codes are BITS whole dwords
        constexpr int kAlign = BITS % 4 == 0 ? 16 : BITS % 2 == 0 ? 8 : 4;
        uint32_t w[BITS + 2] = {};
#pragma unroll
        for (int r = 0; r < OWN; r++) {
            const int d = r * BITS / 4, shift = r * BITS % 4 * 8;
            w[d] |= uint32_t(codes[r] << shift);
            w[d + 1] |= uint32_t((codes[r] << shift) >> 32);
            if (shift && BITS > 4) w[d + 2] |= uint32_t(codes[r] >> (64 - shift));
        }
        __builtin_memcpy(__builtin_assume_aligned(area + lane * (4 * BITS), kAlign), w, 4 * BITS);
    } else {
#pragma unroll
        for (int r = 0; r < OWN; r++) stage_codes<BITS>(area + (lane * OWN + r) * BITS, codes[r]);
    }
}

// LDS a wave needs to quantize a run of storage type DT: the chunk as stored; later its codes with 16 bytes of
// padding, an extent per lane and a scale per bucket.
template <int DT>
constexpr int kRunStageBytes = kChunk * (DT == CGX_F16 ? 2 : 4) > kChunk + 16 + 2 * kWave * 8 ? kChunk * (DT == CGX_F16 ? 2 : 4)
                                                                                              : kChunk + 16 + 2 * kWave * 8;

// Extent (kNormSign: +0 and the largest magnitude) of the elements of a run that a lane holds; nothing: the neutral one.
template <int SCHEME, int OWN>
__device__ __forceinline__ float2 run_extent(const float (&x)[OWN][8], const Run &run)
{
    // kNormSign: the zeros of the missing elements are neutral for the largest magnitude
    float mn = SCHEME == kNormSign ? 0.0f : __builtin_inff(), mx = SCHEME == kNormSign ? 0.0f : -__builtin_inff();
    if (SCHEME == kNormSign || run.left >= 8 * OWN) {
        lane_extent<SCHEME>(x, mn, mx);
    } else {
#pragma unroll
        for (int r = 0; r < OWN; r++) {
            const int v = run.valid(r);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                mn = __builtin_fminf(mn, j < v ? x[r][j] : __builtin_inff());
                mx = __builtin_fmaxf(mx, j < v ? x[r][j] : -__builtin_inff());
            }
        }
    }
    return make_float2(mn, mx);
}

// The run's codes under a scale per lane: staged, then sent out with `pad` zero bytes behind them.  out is a multiple
// of 4 bytes, and so is the number of bytes written: a run starts a multiple of 32 codes into its segment of the
// stream and either ends one or is padded to the segment's 16 bytes.
template <int SCHEME, int BITS, int DRAWS, int OWN>
__device__ __forceinline__ void encode_run(const float (&x)[OWN][8], const Run &run, Scale s, int lane, int64_t first,
                                           uint32_t key, uint8_t *__restrict__ out, uint32_t pad, uint4v *stage)
{
    // What the widths have in common (draws, positions between the levels) is not computed ahead of the choice of a
    // width: it would take 50 registers.
    asm volatile("" : "+v"(lane), "+v"(s.inv16) : "i"(BITS));
    uint8_t *area = reinterpret_cast<uint8_t *>(stage);
    uint64_t codes[OWN];
#pragma unroll
    for (int r = 0; r < OWN; r++) {
        const uint32_t pair0 = first_pair(first, (lane * OWN + r) * 8);
        codes[r] = encode_group<SCHEME, BITS, DRAWS>(x[r], s, pair0, key, uint32_t(first) & 1u);
        const int v = run.valid(r);
        codes[r] &= v == 8 ? ~uint64_t(0) : (uint64_t(1) << (v * BITS)) - 1u;       // nothing past the end
        // one group after the other: together they cost the kernel registers that every path of it then pays
        __builtin_amdgcn_sched_barrier(0);
    }
    stage_run_codes<BITS>(area, codes, lane);
    if (lane < 4) reinterpret_cast<uint32_t *>(area + kWave * OWN * BITS)[lane] = 0;      // padding behind the last lane's codes
    wave_lds_fence();
    const int bytes = (run.count * BITS + 7) / 8 + int(pad), vecs = bytes / 16;
    for (int v = lane; v < vecs; v += kWave) __builtin_nontemporal_store(stage[v], reinterpret_cast<uint4u4 *>(out) + v);
    if (lane < (bytes & 15) / 4) reinterpret_cast<uint32_t *>(out)[vecs * 4 + lane] = reinterpret_cast<const uint32_t *>(area)[vecs * 4 + lane];
    wave_lds_fence();
}

// x holds a run (zeros where there is no element) -> meta of its buckets and its packed codes.  The scale of a
// bucket comes from an extent per lane parked in LDS: the lanes are split into sets of P (a power of two,
// 64 / P >= buckets > 32 / P, so a lane folds at most two entries), each of which folds the extents of one bucket.
template <int SCHEME, int BITS, int DRAWS, int OWN>
__device__ __forceinline__ void quantize_run_regs(const float (&x)[OWN][8], const Run &run, int lane, int64_t first, uint32_t key,
                                                  float *__restrict__ meta, uint8_t *__restrict__ out, uint32_t pad, uint4v *stage)
{
    constexpr uint32_t kLevels = top_level<SCHEME>(BITS);
    float2 *extents = reinterpret_cast<float2 *>(reinterpret_cast<uint8_t *>(stage) + kChunk + 16), *scales = extents + kWave;
    extents[lane] = run_extent<SCHEME>(x, run);
    wave_lds_fence();
    const int lgP = run.buckets > 1 ? __builtin_clz(uint32_t(run.buckets - 1)) - 26 : 6, P = 1 << lgP;
    const int bucket = lane >> lgP, part = lane & (P - 1), entry = bucket * run.lanes + part;
    float mn = SCHEME == kNormSign ? 0.0f : __builtin_inff(), mx = SCHEME == kNormSign ? 0.0f : -__builtin_inff();
    if (part < run.lanes && entry < kWave) {
        const float2 e = extents[entry];
        mn = e.x, mx = e.y;
    }
    if (part + P < run.lanes && entry + P < kWave) {
        const float2 e = extents[entry + P];
        if (SCHEME != kNormSign) mn = min_plain(mn, e.x);
        mx = max_plain(mx, e.y);
    }
    if (SCHEME == kNormSign)
        group_max(mx, lgP, lane);
    else
        group_minmax(mn, mx, lgP, lane);
    const Scale of_set = bucket_scale(mn, mx, int(kLevels));
    if (part == 0 && bucket < run.buckets) {
        store_meta<SCHEME>(meta, uint32_t(bucket), of_set);
        scales[bucket] = make_float2(of_set.mn, of_set.inv16);
    }
    wave_lds_fence();
    const float2 own = scales[run.bi];
    encode_run<SCHEME, BITS, DRAWS>(x, run, Scale{0.0f, own.x, own.y}, lane, first, key, out, pad, stage);
}

// OWN: groups a lane holds.  A wave pays for them whether or not all its lanes have elements.
template <int SCHEME, int DT, int BITS, int DRAWS, int OWN = G>
__device__ __forceinline__ void quantize_run(const void *__restrict__ grad, uint8_t *__restrict__ packed,
                                             float *__restrict__ meta, const Tile &tile, int bucket,
                                             uint32_t seed_lo, uint32_t seed_hi, int lane, uint4v *stage)
{
    const Run run(int(tile.count), bucket, lane, OWN);
    const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
    RunLoad<DT> load;
    load.issue(grad, tile.elem0, run.count, lane);
    float x[OWN][8];
    load.finish(run.count, lane, stage, x);
    quantize_run_regs<SCHEME, BITS, DRAWS>(x, run, lane, tile.elem0, key, meta + kMetaFloats<SCHEME> * tile.bucket0,
                                         packed + tile.packed_off, tile.pad, stage);
}

// A run that 24 elements per lane hold, none of the lanes across two buckets: its bucket size is a multiple of 24, or it lies
// in one bucket (as every run of buckets of more than 1024 elements does).
__device__ __forceinline__ bool three_groups_hold(const Tile &tile, int bucket)
{
    return tile.count <= uint32_t(kWave * 24) && tile.count > uint32_t(kWave * 16) && (bucket % 24 == 0 || tile.count <= uint32_t(bucket));
}

// What no other path takes (a tile across two key blocks of the generator): one bucket at a time, two passes.
// value(j) gives element j of the tile (called twice per element).  With BATCH the values
// of a pass are fetched 8 at a time so that plain loads overlap; without it (value() is
// itself a reduction over the peers) they are taken one by one.
template <int SCHEME, bool BATCH, typename Value>
__device__ __forceinline__ void quantize_generic(Value value, uint8_t *__restrict__ out,
                                                 float *__restrict__ meta, const Tile &tile, uint32_t pad,
                                                 int bucket, uint32_t seed_lo, uint32_t seed_hi, int lane)
{
    const int b = int(tile_bits(tile));
    const uint32_t levels = top_level<SCHEME>(b);
    // kNormSign: the maximum runs over magnitudes and the minimum stays +0
    const auto seen = [](float x) { return SCHEME == kNormSign ? __builtin_fabsf(x) : x; };
    for (uint32_t k0 = 0; k0 < tile.count; k0 += uint32_t(bucket)) {
        const uint32_t cnt = tile.count - k0 < uint32_t(bucket) ? tile.count - k0 : uint32_t(bucket);
        float mn = SCHEME == kNormSign ? 0.0f : __builtin_inff(), mx = SCHEME == kNormSign ? 0.0f : -__builtin_inff();
        if (BATCH) {
            for (uint32_t j0 = 0; j0 < cnt; j0 += 8 * kWave) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const uint32_t j = j0 + u * kWave + lane;
                    x[u] = value(k0 + (j < cnt ? j : 0));           // clamped: the bucket's first element again
                }
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    if (SCHEME != kNormSign) mn = __builtin_fminf(mn, x[u]);
                    mx = __builtin_fmaxf(mx, seen(x[u]));
                }
            }
        } else {
            for (uint32_t j = lane; j < cnt; j += kWave) {
                const float x = value(k0 + j);
                if (SCHEME != kNormSign) mn = __builtin_fminf(mn, x);
                mx = __builtin_fmaxf(mx, seen(x));
            }
        }
        if (SCHEME == kNormSign)
            group_max(mx, 6, lane);
        else
            group_minmax(mn, mx, 6, lane);
        const Scale s = bucket_scale(mn, mx, int(levels));
        if (lane == 0) store_meta<SCHEME>(meta, tile.bucket0 + k0 / uint32_t(bucket), s);

        const uint32_t groups = (cnt + 7) / 8;
        for (uint32_t g = lane; g < groups; g += kWave) {
            const uint32_t valid = cnt - g * 8 < 8 ? cnt - g * 8 : 8;
            const uint64_t i0 = uint64_t(tile.elem0) + k0 + g * 8;
            uint64_t acc = 0;
            if (BATCH) {
                float x[8];
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) x[j] = value(k0 + g * 8 + (j < valid ? j : 0));
#pragma unroll
                for (uint32_t j = 0; j < 8; j++) {
                    const uint64_t q = code_of<SCHEME>(x[j], s, draw16(seed_lo, seed_hi, i0 + j), levels, b);
                    if (j < valid) acc |= q << (j * b);
                }
            } else {
                for (uint32_t j = 0; j < valid; j++) {
                    const uint64_t q =
                        code_of<SCHEME>(value(k0 + g * 8 + j), s, draw16(seed_lo, seed_hi, i0 + j), levels, b);
                    acc |= q << (j * b);
                }
            }
            const uint32_t nbytes = (valid * b + 7) / 8;
            uint8_t *p = out + uint64_t(k0 / 8 + g) * b;
            for (uint32_t k = 0; k < nbytes; k++) p[k] = uint8_t(acc >> (8 * k));
        }
    }
    if (pad) {
        const uint64_t end = (uint64_t(tile.count) * b + 7) / 8;
        if (uint32_t(lane) < pad) out[end + lane] = 0;
    }
}

// Pass-through tile of the quantize kernels: verbatim copy, then the layer's zero padding.  WIDTH lanes work on it, this
// one is number `lane`.
template <int DT, int WIDTH = kWave>
__device__ __forceinline__ void copy_tile(const void *__restrict__ grad, uint8_t *__restrict__ packed, const Tile &tile, int lane)
{
    constexpr int S = DT == CGX_F16 ? 2 : 4;
    const uint8_t *src = reinterpret_cast<const uint8_t *>(grad) + tile.elem0 * S;
    uint8_t *dst = packed + tile.packed_off;
    const uint32_t bytes = tile.count * S;
    const uint32_t vecs = bytes / 16;
    // all loads of a tile (kCopyPiece elements) in flight together
    constexpr int kLoads = kCopyPiece * S / 16 / WIDTH > 0 ? kCopyPiece * S / 16 / WIDTH : 1;
    for (uint32_t v0 = lane; v0 < vecs; v0 += kLoads * WIDTH) {
        uint4v raw[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; u++)
            if (v0 + u * WIDTH < vecs) raw[u] = reinterpret_cast<const uint4u2 *>(src)[v0 + u * WIDTH];
#pragma unroll
        for (int u = 0; u < kLoads; u++)
            if (v0 + u * WIDTH < vecs) reinterpret_cast<uint4v *>(dst)[v0 + u * WIDTH] = raw[u];
    }
    for (uint32_t k = vecs * 16 + lane; k < bytes + tile.pad; k += WIDTH) dst[k] = k < bytes ? src[k] : uint8_t(0);
}

}  // namespace
}  // namespace cgx
