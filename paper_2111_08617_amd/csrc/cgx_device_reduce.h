// Device code of the dequantize-and-reduce: decoding of staged codes, the peers' loop, sums of
// chunks, short ends, generic and pass-through tiles (shared by the reduce, fused and
// statistics kernels).
#pragma once

#include "cgx_device.h"

namespace cgx {
namespace {

// ---------------------------------------------------------------- dequantize + reduce

// The four bytes of t as floats.  The byte-wise decoders below put one code into every byte of a register and convert
// the bytes with v_cvt_f32_ubyte0..3; seeing through the mask (hence opaque), the compiler would instead extract every
// code with a v_bfe_u32 of its own and convert byte 0 (two instructions of the slow issue class per code instead of one).
__device__ __forceinline__ void bytes_to_float(uint32_t t, float &b0, float &b1, float &b2, float &b3)
{
    b0 = float(t & 0xffu);
    b1 = float((t >> 8) & 0xffu);
    b2 = float((t >> 16) & 0xffu);
    b3 = float(t >> 24);
}

// The same for signed bytes: one conversion each (sub-dword operand, sign-extended).
__device__ __forceinline__ void signed_bytes_to_float(uint32_t t, float &b0, float &b1, float &b2, float &b3)
{
    b0 = float(int32_t(int8_t(t)));
    b1 = float(int32_t(int8_t(t >> 8)));
    b2 = float(int32_t(int8_t(t >> 16)));
    b3 = float(int32_t(t) >> 24);
}

// Two conversions per instruction: v_cvt_scalef32_pk_f32_fp8 / _fp4 turn two bytes, or the two nibbles of a byte, into floats
// and multiply them by a power of two, at 5.4 cycles of a SIMD where one v_cvt_f32_ubyte takes 4.7.  Codes are small whole
// numbers, and the subnormals and the first binade of such a format form one linear grid: an E4M3 byte q <= 15 is q / 512, an E2M1
// nibble q <= 3 is q / 2.  Times 512 (2) that is float(q), exactly.  Builds in turn on one box, us: a 13.7 M share of 8 peers in one
// fused step (2, 3, 4 and 8 bits) 20.1 -> 19.4, 16.8 M elements of 4 bits 22.7 -> 21.7, the 1.3 B share 187.2 -> 185.4; the
// reduce of 34 M at 2 bits 63.1 -> 60.9, at 4 bits 72.2 -> 70.5.  Nibbles against bytes for the 2-bit codes, everything else alike: that
// reduce 60.9 and 63.5, that share 19.4 and 19.7, but fused steps of 2 bits alone 20.9 and 20.5 (16.8 M; 67 M 64.8 and 63.6).
// Not taken where it measured slower: 3-bit
// codes spread to bytes (fused, 8 peers, 23.7 -> 24.8), signed 2-bit codes as nibbles of sign and magnitude (21.8 -> 22.6), 2-bit
// codes of a single peer, bound by what they write (67 M elements in 4 shares 47.5 -> 47.9), and 2-bit codes of runs, whose upper
// bits have to be cleared first (fused, 8 peers, buckets of 992, 24.8 byte by byte, 26.5 as nibbles).
constexpr float kByteScale = 512.0f, kNibbleScale = 2.0f;

__device__ __forceinline__ void small_bytes_to_float(uint32_t t, float &b0, float &b1, float &b2, float &b3)
{
    const auto lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(t, kByteScale, false);
    const auto hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(t, kByteScale, true);
    b0 = lo[0], b1 = lo[1], b2 = hi[0], b3 = hi[1];
}

// Eight nibbles of at most 3, lowest first.
__device__ __forceinline__ void nibbles_to_float(uint32_t t, float (&f)[8])
{
    const auto p0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(t, kNibbleScale, 0), p1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(t, kNibbleScale, 1);
    const auto p2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(t, kNibbleScale, 2), p3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(t, kNibbleScale, 3);
    f[0] = p0[0], f[1] = p0[1], f[2] = p1[0], f[3] = p1[1];
    f[4] = p2[0], f[5] = p2[1], f[6] = p3[0], f[7] = p3[1];
}

// Levels of one group of 8 codes as floats (kNormSign: signed levels).  BYTEWISE: 2-bit codes by v_cvt_f32_ubyte.  Signed 2-bit codes
// are extracted one by one: as bytes that v_perm_b32 selects the fused step of 14.7 M takes 20.6 us for 19.3.
template <int SCHEME, int BITS, bool BYTEWISE>
__device__ __forceinline__ void codes_to_float(uint64_t v, float (&f)[8])
{
    constexpr bool kSigned = SCHEME == kNormSign;
    const uint32_t w = uint32_t(v);
    if (BITS == 8) {
        if (kSigned) {
            signed_bytes_to_float(w, f[0], f[1], f[2], f[3]);
            signed_bytes_to_float(uint32_t(v >> 32), f[4], f[5], f[6], f[7]);
        } else {
            bytes_to_float(w, f[0], f[1], f[2], f[3]);
            bytes_to_float(uint32_t(v >> 32), f[4], f[5], f[6], f[7]);
        }
    } else if (BITS == 4) {
        // one code per byte: even codes in one register, odd ones in another
        if (kSigned) {
            // a nibble with its sign bit flipped is level + 8, and 0x78 more is level + 0x80: no byte carries
            // (a conversion of a signed byte costs what one of an unsigned byte does, and no 8.0 is subtracted per code: fused step of 8
            // peers, 14.7 M elements, 24.4 -> 22.1 us)
            const uint32_t h = w ^ 0x88888888u;
            const uint32_t even = ((h & 0x0f0f0f0fu) + 0x78787878u) ^ 0x80808080u;
            const uint32_t odd = (((h >> 4) & 0x0f0f0f0fu) + 0x78787878u) ^ 0x80808080u;
            signed_bytes_to_float(opaque(even), f[0], f[2], f[4], f[6]);
            signed_bytes_to_float(opaque(odd), f[1], f[3], f[5], f[7]);
        } else {
            small_bytes_to_float(w & 0x0f0f0f0fu, f[0], f[2], f[4], f[6]);
            small_bytes_to_float((w >> 4) & 0x0f0f0f0fu, f[1], f[3], f[5], f[7]);
        }
    } else if (BITS == 2 && !kSigned && BYTEWISE) {
        // four codes per register: the upper half holds the codes that follow those of the lower half
        const uint32_t x = opaque(((w & 0xffffu) << 14) | (w & 0xffffu));
        bytes_to_float(opaque(x & 0x03030303u), f[0], f[4], f[1], f[5]);
        bytes_to_float(opaque((x >> 4) & 0x03030303u), f[2], f[6], f[3], f[7]);
    } else if (BITS == 2 && !kSigned) {
        // a code per nibble: codes 0, 2, 4, 6 in the lower half of the register, the odd ones in the upper half
        const uint32_t codes = (((w & 0xffffu) << 14) | (w & 0xffffu)) & 0x33333333u;
        float n[8];
        nibbles_to_float(codes, n);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            f[2 * k] = n[k];
            f[2 * k + 1] = n[4 + k];
        }
    } else if (kSigned) {
#pragma unroll
        for (int j = 0; j < 8; j++)      // sign-extending field extract
            f[j] = float(int32_t(uint32_t(v >> (j * BITS)) << (32 - BITS)) >> (32 - BITS));
    } else {
        constexpr uint64_t kMask = (1u << BITS) - 1u;
#pragma unroll
        for (int j = 0; j < 8; j++) f[j] = float(uint32_t((v >> (j * BITS)) & kMask));
    }
}

// The codes of a lane's G groups of a run, group r's 8 in the low 8 * BITS bits of v[r] (bits above are unspecified).
// codes: the run's first code in LDS, a multiple of 4 bytes, of 8 at 2 and 6 bits and of 16 at 4 and 8 bits (a run
// starts a multiple of 32 codes into its layer).
template <int BITS>
__device__ __forceinline__ void run_codes(const uint8_t *codes, int lane, uint64_t (&v)[G])
{
    if constexpr (G == 4) {
        // 32 codes are BITS whole dwords
        constexpr int kAlign = BITS % 4 == 0 ? 16 : BITS % 2 == 0 ? 8 : 4;
        uint32_t w[BITS + 2];
        __builtin_memcpy(w, __builtin_assume_aligned(codes + lane * (4 * BITS), kAlign), 4 * BITS);
        w[BITS] = w[BITS + 1] = 0;
#pragma unroll
        for (int r = 0; r < G; r++) {
            const int d = r * BITS / 4, shift = r * BITS % 4 * 8;
            const uint32_t lo = shift ? __builtin_amdgcn_alignbit(w[d + 1], w[d], shift) : w[d];
            const uint32_t hi = BITS <= 4 ? 0u : shift ? __builtin_amdgcn_alignbit(w[d + 2], w[d + 1], shift) : w[d + 1];
            v[r] = (uint64_t(hi) << 32) | lo;
        }
    } else {
#pragma unroll
        for (int r = 0; r < G; r++) v[r] = staged_codes<BITS>(codes, (lane * G + r) * BITS);
    }
}

// Folds peers w0 .. w0+WB-1 into acc.  Each peer's share of the chunk (kChunk*BITS/8 bytes)
// is fetched as whole 16-byte vectors, consecutive across lanes, directly into the wave's
// LDS staging area, and read back by the lanes that own the codes.
// RUN: the chunk is a run (code_off unused).  Its codes start on a multiple of 4 bytes only; the vectors that
// cover them are fetched (nvecs of them from the 16-byte boundary at or before in_off: they stay inside the layer's
// segment, which starts and ends on 16 bytes).  What lies behind the run's end in LDS is stale, and so are the
// sums of elements past the end: the caller drops them.
template <int BITS>
constexpr int kRunLead = BITS % 4 == 0 ? 0 : 16;      // bytes between that boundary and the first code, at most 12

template <int SCHEME, int BITS, int WB, bool RUN, typename Peers>
__device__ __forceinline__ void reduce_peers(Peers &peers, int w0, int64_t in_off, uint32_t g,
                                             const int (&code_off)[G], float (&acc)[G][8], uint4v *stage,
                                             int lane, int nvecs)
{
    constexpr int kBytes = kChunk * BITS / 8 + (RUN ? kRunLead<BITS> : 0);        // per peer
    constexpr int kVecs = kBytes / 16;
    constexpr int kPerLane = (kVecs + kWave - 1) / kWave;
    const int lead = RUN && kRunLead<BITS> ? int(in_off & 15) : 0;
    float2 m[WB];
#pragma unroll
    for (int i = 0; i < WB; i++) {
        const uint4v *in = reinterpret_cast<const uint4v *>(peers.packed[w0 + i] + (in_off - lead));
#pragma unroll
        for (int k = 0; k < kPerLane; k++) {
            const int v = lane + k * kWave;
            if (RUN ? v < nvecs : (kVecs % kWave == 0 || v < kVecs)) {
                // a block of one peer is what a decompression (W = 1) consists of: ordinary loads there
                if (WB == 1)
                    load_to_lds16_cached(in + v, stage + i * kVecs + k * kWave);
                else
                    load_to_lds16(in + v, stage + i * kVecs + k * kWave);
            }
        }
        m[i] = load_meta<SCHEME>(peers.meta[w0 + i], g);
    }
    wait_vector_memory();
    wave_lds_fence();
    const uint8_t *codes = reinterpret_cast<const uint8_t *>(stage) + lead;
#pragma unroll
    for (int i = 0; i < WB; i++) {
        uint64_t run[G];
        if constexpr (RUN) run_codes<BITS>(codes + i * kBytes, lane, run);
#pragma unroll
        for (int r = 0; r < G; r++) {
            float f[8];
            uint64_t v;
            if constexpr (RUN)
                v = run[r];
            else
                v = staged_codes<BITS>(codes + i * kBytes, code_off[r]);
            codes_to_float<SCHEME, BITS, WB == 1 || RUN>(v, f);
#pragma unroll
            for (int j = 0; j < 8; j++) acc[r][j] = __fadd_rn(acc[r][j], decode<SCHEME>(f[j], m[i]));
        }
        // keep the scheduler from hoisting every peer's LDS reads to the top (registers)
        if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    wave_lds_fence();
}

// peers staged together: 8 if their packed bytes fit the staging area (one chunk of sums,
// kChunk * 4 bytes), else 4; the odd widths take 4 (their two or three dwords per group
// and peer are all in flight together: at 8 peers the 3-bit path alone raised the fused
// kernel from 106 to 125 registers, which cost every other width up to 50 % there)
template <int BITS>
constexpr int kPeerBlock = (kStagedOverRead<BITS> != 0 || 8 * (kChunk * BITS / 8) > kChunk * 4) ? 4 : 8;

// Sum over the W peers of one chunk's dequantized values, added to acc in peer order.
template <int SCHEME, int BITS, typename Peers>
__device__ __forceinline__ void reduce_chunk(Peers &peers, int W, int64_t in_off, uint32_t g,
                                             const LaneMap &map, float (&acc)[G][8], uint4v *stage, int lane)
{
    constexpr int kBytes = kChunk * BITS / 8;
    static_assert(kPeerBlock<BITS> * kBytes + kStagedOverRead<BITS> <= kChunk * 4, "staging area too small");
    int code_off[G];
#pragma unroll
    for (int r = 0; r < G; r++) code_off[r] = (map.group(r) >> 3) * BITS;
    for_peer_blocks<kPeerBlock<BITS>>(W, [&](int w0, auto wb) {
        reduce_peers<SCHEME, BITS, decltype(wb)::value, false>(peers, w0, in_off, g, code_off, acc, stage, lane, 0);
    });
}

// The same for a run whose codes start at byte in_off and whose first bucket is bucket0.
template <int SCHEME, int BITS, typename Peers>
__device__ __forceinline__ void reduce_run(Peers &peers, int W, int64_t in_off, uint32_t bucket0, const Run &run,
                                           float (&acc)[G][8], uint4v *stage, int lane)
{
    constexpr int kBytes = kChunk * BITS / 8 + kRunLead<BITS>;
    static_assert(kPeerBlock<BITS> * kBytes + (G == 4 ? 0 : kStagedOverRead<BITS>) <= kChunk * 4, "staging area too small");
    const int nvecs = (int(in_off & 15) + (run.count * BITS + 7) / 8 + 15) / 16;
    const int unused[G] = {};
    for_peer_blocks<kPeerBlock<BITS>>(W, [&](int w0, auto wb) {
        reduce_peers<SCHEME, BITS, decltype(wb)::value, true>(peers, w0, in_off, bucket0 + uint32_t(run.bi), unused, acc, stage, lane,
                                                              nvecs);
    });
}

// -0 is the identity of binary32 addition for every addend, signed zeros included, so
// the first peer's value enters the sum unchanged.
__device__ __forceinline__ void clear_sums(float (&acc)[G][8])
{
#pragma unroll
    for (int r = 0; r < G; r++)
#pragma unroll
        for (int j = 0; j < 8; j++) acc[r][j] = -0.0f;
}

// acc = the sums of a run over the W peers.
template <int SCHEME, int BITS, typename Peers>
__device__ __forceinline__ void sum_run(Peers &peers, int W, int64_t in_off, uint32_t bucket0, const Run &run,
                                        float (&acc)[G][8], uint4v *stage, int lane)
{
    clear_sums(acc);
    reduce_run<SCHEME, BITS>(peers, W, in_off, bucket0, run, acc, stage, lane);
}

// The sums of a run's missing elements (stale LDS bytes decoded to anything) become 0.
__device__ __forceinline__ void clear_missing(float (&acc)[G][8], const Run &run)
{
    if (run.left < 8 * G) {
#pragma unroll
        for (int r = 0; r < G; r++) {
            const int v = run.valid(r);
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (j >= v) acc[r][j] = 0.0f;
        }
    }
}

// The fused kernels' arguments as the kernarg segment lays them out: offset of the peers' table behind the scalars.
struct FusedArguments {
    const Tile *tiles_in, *tiles_out;
    int64_t n_tiles;
    int W, dt;
    uint32_t seed_lo, seed_hi;
    uint8_t *packed_out;
    float *meta_out;
    PeerPtrs peers;
};

// What a reduction starts from and where it goes: element e of the tile's buffer is
// init[e] (binary32 or binary16; init == nullptr: nothing) and is written to out[e]
// (binary32, or binary16 rounded to nearest even).
struct SumIo {
    const void *init;
    int init_dt;
    void *out;
    int out_dt;
    int keep;          // StorePolicy of the result: see flush_stage_to_elements
};

__device__ __forceinline__ void init8(const SumIo &io, int64_t e, float (&acc)[8])
{
    if (!io.init) {
#pragma unroll
        for (int j = 0; j < 8; j++) acc[j] = -0.0f;
    } else if (io.init_dt == CGX_F16) {
        load8<CGX_F16>(io.init, e, acc);
    } else {
        load8<CGX_F32>(io.init, e, acc);
    }
}

__device__ __forceinline__ float init1(const SumIo &io, int64_t e)
{
    if (!io.init) return -0.0f;
    return io.init_dt == CGX_F16 ? load_elem<CGX_F16>(io.init, e) : load_elem<CGX_F32>(io.init, e);
}

// A sum rounded to binary16.  The sum is a binary32 number first: with one peer, whose value is a multiply-add, the
// compiler would otherwise form v_fma_mixlo_f16, which rounds once instead of twice.
__device__ __forceinline__ _Float16 to_half(float v)
{
    asm("" : "+v"(v));
    return _Float16(v);
}

__device__ __forceinline__ void store1(const SumIo &io, int64_t e, float v)
{
    if (io.out_dt == CGX_F16)
        reinterpret_cast<_Float16 *>(io.out)[e] = to_half(v);
    else
        reinterpret_cast<float *>(io.out)[e] = v;
}

// 8 consecutive results to a 16-byte aligned position.
__device__ __forceinline__ void store8(const SumIo &io, int64_t e, const float (&acc)[8])
{
    if (io.out_dt == CGX_F16) {
        half8v h;
#pragma unroll
        for (int j = 0; j < 8; j++) h[j] = to_half(acc[j]);
        *reinterpret_cast<half8u *>(reinterpret_cast<_Float16 *>(io.out) + e) = h;
    } else {
        float4u *p = reinterpret_cast<float4u *>(reinterpret_cast<float *>(io.out) + e);
        p[0] = float4v{acc[0], acc[1], acc[2], acc[3]};
        p[1] = float4v{acc[4], acc[5], acc[6], acc[7]};
    }
}

template <int SCHEME, int BITS, typename Peers>
__device__ __forceinline__ void reduce_fast(Peers &peers, int W, const SumIo &io, const Tile &tile,
                                            int bucket, int lane, uint4v *stage)
{
    const LaneMap map(tile, bucket, lane);
    const int chunks = int(tile.count / kChunk);
    const int buckets_per_chunk = kChunk / bucket;
    for (int c = 0; c < chunks; c++) {
        const int64_t first = tile.elem0 + int64_t(c) * kChunk;
        float acc[G][8];
#pragma unroll
        for (int r = 0; r < G; r++) init8(io, first + map.group(r), acc[r]);
        reduce_chunk<SCHEME, BITS>(peers, W, tile.packed_off + int64_t(c) * (kChunk * BITS / 8),
                                   tile.bucket0 + c * buckets_per_chunk + map.bi, map, acc, stage, lane);
        // the results leave through LDS as well, so that every store instruction writes 1 KB of
        // consecutive addresses
        if (io.out_dt == CGX_F16) {
#pragma unroll
            for (int r = 0; r < G; r++) {
                half8v h;
#pragma unroll
                for (int j = 0; j < 8; j++) h[j] = to_half(acc[r][j]);
                reinterpret_cast<half8v *>(stage)[map.group(r) >> 3] = h;
            }
            wave_lds_fence();
            flush_stage_to_elements(stage, reinterpret_cast<uint4u2 *>(reinterpret_cast<_Float16 *>(io.out) + first),
                                    kChunk / 8, lane, io.keep);
        } else {
#pragma unroll
            for (int r = 0; r < G; r++) {
                float4v *p = reinterpret_cast<float4v *>(stage) + (map.group(r) >> 2);
                p[0] = float4v{acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
                p[1] = float4v{acc[r][4], acc[r][5], acc[r][6], acc[r][7]};
            }
            wave_lds_fence();
            flush_stage_to_elements(stage, reinterpret_cast<uint4u2 *>(reinterpret_cast<float *>(io.out) + first),
                                    kChunk / 4, lane, io.keep);
        }
        wave_lds_fence();
    }
}

// Sums of a run: start values come in and sums go out as whole 16-byte vectors, consecutive across lanes, through the
// staging area; the elements behind the last whole vector one by one.
template <int SCHEME, int BITS, typename Peers>
__device__ __forceinline__ void reduce_run_tile(Peers &peers, int W, const SumIo &io, const Tile &tile,
                                                int bucket, int lane, uint4v *stage)
{
    const Run run(int(tile.count), bucket, lane);
    float acc[G][8];
    if (!io.init) {
        clear_sums(acc);
    } else if (io.init_dt == CGX_F16) {
        RunLoad<CGX_F16> load;
        load.issue(io.init, tile.elem0, run.count, lane);
        load.finish(run.count, lane, stage, acc);
    } else {
        RunLoad<CGX_F32> load;
        load.issue(io.init, tile.elem0, run.count, lane);
        load.finish(run.count, lane, stage, acc);
    }
    reduce_run<SCHEME, BITS>(peers, W, tile.packed_off, tile.bucket0, run, acc, stage, lane);
    if (io.out_dt == CGX_F16) {
#pragma unroll
        for (int r = 0; r < G; r++) {
            half8v h;
#pragma unroll
            for (int j = 0; j < 8; j++) h[j] = to_half(acc[r][j]);
            stage[run_slot<G>(lane * G + r)] = __builtin_bit_cast(uint4v, h);
        }
        wave_lds_fence();
        const int vecs = run.count / 8, e = vecs * 8 + lane;
        _Float16 *out = reinterpret_cast<_Float16 *>(io.out) + tile.elem0;
        flush_stage_to_elements(stage, reinterpret_cast<uint4u2 *>(out), vecs, lane, io.keep, run_slot<G>);
        if (e < run.count) out[e] = reinterpret_cast<const _Float16 *>(stage + run_slot<G>(vecs))[lane];
    } else {
#pragma unroll
        for (int r = 0; r < G; r++) {
            stage[run_slot<2 * G>(lane * 2 * G + 2 * r)] =
                __builtin_bit_cast(uint4v, (float4v{acc[r][0], acc[r][1], acc[r][2], acc[r][3]}));
            stage[run_slot<2 * G>(lane * 2 * G + 2 * r + 1)] =
                __builtin_bit_cast(uint4v, (float4v{acc[r][4], acc[r][5], acc[r][6], acc[r][7]}));
        }
        wave_lds_fence();
        const int vecs = run.count / 4, e = vecs * 4 + lane;
        float *out = reinterpret_cast<float *>(io.out) + tile.elem0;
        flush_stage_to_elements(stage, reinterpret_cast<uint4u2 *>(out), vecs, lane, io.keep, run_slot<2 * G>);
        if (e < run.count) out[e] = reinterpret_cast<const float *>(stage + run_slot<2 * G>(vecs))[lane];
    }
    wave_lds_fence();
}

// Ordered sum over the peers of element j of a generic quantized tile (start = the value
// the sum starts from).
template <int SCHEME, typename Peers>
__device__ __forceinline__ float generic_sum(Peers &peers, int W, const Tile &tile, int bucket,
                                             uint32_t j, float start)
{
    const int b = int(tile_bits(tile));
    const uint32_t mask = (1u << b) - 1u;
    const uint32_t g = tile.bucket0 + j / uint32_t(bucket);
    const uint64_t bit = uint64_t(j) * b;
    const int64_t at = tile.packed_off + int64_t(bit >> 3);
    const uint32_t shift = uint32_t(bit & 7);
    const bool two = shift + b > 8;                  // a code spans at most two bytes
    float acc = start;
    for_peer_blocks<8>(W, [&](int w0, auto wb) {
        constexpr int WB = decltype(wb)::value;
        uint32_t lo[WB], hi[WB];
        float2 m[WB];
#pragma unroll
        for (int i = 0; i < WB; i++) {
            const uint8_t *p = peers.packed[w0 + i] + at;
            lo[i] = p[0];
            hi[i] = two ? p[1] : 0u;
            m[i] = load_meta<SCHEME>(peers.meta[w0 + i], g);
        }
#pragma unroll
        for (int i = 0; i < WB; i++) {
            const uint32_t code = ((lo[i] | (hi[i] << 8)) >> shift) & mask;
            const float level = SCHEME == kNormSign ? float(int32_t(code << (32 - b)) >> (32 - b)) : float(code);
            acc = __fadd_rn(acc, decode<SCHEME>(level, m[i]));
        }
    });
    return acc;
}

// Ordered sum over the peers of 8 consecutive elements of a pass-through tile (16-byte
// aligned) and of a single element.
template <int DT, typename Peers>
__device__ __forceinline__ void copy_sum8(Peers &peers, int W, const Tile &tile, uint32_t g,
                                          float (&acc)[8])
{
    for_peer_blocks<8>(W, [&](int w0, auto wb) {
        constexpr int WB = decltype(wb)::value;
        Raw8<DT> raw[WB];
#pragma unroll
        for (int i = 0; i < WB; i++) raw[i].load(peers.packed[w0 + i] + tile.packed_off, int64_t(g) * 8);
#pragma unroll
        for (int i = 0; i < WB; i++) {
            float x[8];
            raw[i].widen(x);
#pragma unroll
            for (int j = 0; j < 8; j++) acc[j] = __fadd_rn(acc[j], x[j]);
        }
    });
}

template <int DT, typename Peers>
__device__ __forceinline__ float copy_sum1(Peers &peers, int W, const Tile &tile, uint32_t j, float start)
{
    float acc = start;
    for_peer_blocks<8>(W, [&](int w0, auto wb) {
        constexpr int WB = decltype(wb)::value;
        float x[WB];
#pragma unroll
        for (int i = 0; i < WB; i++) x[i] = load_elem<DT>(peers.packed[w0 + i] + tile.packed_off, j);
#pragma unroll
        for (int i = 0; i < WB; i++) acc = __fadd_rn(acc, x[i]);
    });
    return acc;
}

// Pass-through tile of the reduce kernels: plain ordered sum of the stored values; element j
// of the tile starts from / goes to position e0 + j of io.  WIDTH lanes work on it, this one is number `lane`.
template <int DT, int WIDTH = kWave, typename Peers>
__device__ __forceinline__ void reduce_copy(Peers &peers, int W, const SumIo &io, int64_t e0, const Tile &tile, int lane)
{
    const uint32_t groups = tile.count / 8;
    for (uint32_t g = lane; g < groups; g += WIDTH) {
        float acc[8];
        init8(io, e0 + int64_t(g) * 8, acc);
        copy_sum8<DT>(peers, W, tile, g, acc);
        store8(io, e0 + int64_t(g) * 8, acc);
    }
    for (uint32_t j = groups * 8 + lane; j < tile.count; j += WIDTH)
        store1(io, e0 + j, copy_sum1<DT>(peers, W, tile, j, init1(io, e0 + j)));
}

}  // namespace
}  // namespace cgx
