// Buckets longer than a chunk (2080 ... 8192 elements) in cgx_quantize and cgx_dequant_reduce_requantize and their
// relatives: one block per tile, a tile is (at most) one bucket.
//
// Bound by HBM (quantize) and by the vector ALUs (fused), like the kernels of shorter buckets.  A bucket's elements do
// not fit a wave's registers, but they fit a block's: wave w holds chunk w of the bucket, the waves' extents meet
// in LDS behind one barrier, and every wave then cuts the codes of its chunk.  (One wave per bucket needs a second pass
// for the codes -- over the buffer in the quantizer, over all peers' codes in the fused kernel -- and a launch over
// a few buckets leaves the chip to a few waves.)  Against that, us per call: quantize of 67 M binary32 elements, 4 bit,
// buckets of 8192: 82 -> 54, of 6144 (went element by element): 155 -> 59; binary16, 8192: 49 -> 42; fused, 8 peers, 34 M
// elements: 8192: 125 -> 48; quantize of 54 k elements: 18 -> 5.
// WAVES: 4, or 2 where no bucket of the launch is longer than 4096 (with 4, half of the waves of such a launch are idle:
// quantize of 67 M elements in buckets of 4096 72 us with 4, 55 us with 2, 74 us in two passes; fused, 34 M elements, 62, 48
// and 122 us).
#include "cgx_device_quantize.h"
#include "cgx_device_reduce.h"

namespace cgx {
namespace {

// The share of a wave in a tile of one bucket.
struct Share {
    int at, count;                           // first element within the tile, elements (0: none)
    bool last;                               // holds the tile's last element
    __device__ __forceinline__ Share(const Tile &tile, int wave)
    {
        const int left = int(tile.count) - wave * kChunk;
        at = wave * kChunk;
        count = left < 0 ? 0 : left < kChunk ? left : kChunk;
        last = count > 0 && left <= kChunk;
    }
};

// Scale of the bucket whose chunks the block's waves hold (x: zeros where there is no element).
template <int SCHEME, int WAVES>
__device__ __forceinline__ Scale block_scale(const float (&x)[G][8], const Run &run, int bits, uint4v *stage_all, int stage_vecs, int wave,
                                             int lane)
{
    // (at the start of every wave's staging area, which is free at this point)
    const auto extent_of = [&](int w) { return reinterpret_cast<float2 *>(stage_all + w * stage_vecs); };
    float2 own = run_extent<SCHEME>(x, run);
    if (SCHEME == kNormSign)
        group_max(own.y, 6, lane);
    else
        group_minmax(own.x, own.y, 6, lane);
    if (lane == 0) *extent_of(wave) = own;
    __syncthreads();
    float mn = extent_of(0)->x, mx = extent_of(0)->y;
#pragma unroll
    for (int w = 1; w < WAVES; w++) {
        const float2 e = *extent_of(w);
        if (SCHEME != kNormSign) mn = min_plain(mn, e.x);
        mx = max_plain(mx, e.y);
    }
    __syncthreads();                         // the areas are free again
    return bucket_scale(mn, mx, int(top_level<SCHEME>(bits)));
}

template <int SCHEME, int DT, int DRAWS, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void quantize_wide_kernel(const void *__restrict__ grad, const Tile *__restrict__ tiles,
                                                                int64_t n_tiles, uint32_t seed_lo, uint32_t seed_hi,
                                                                uint8_t *__restrict__ packed, float *__restrict__ meta)
{
    __shared__ uint4v stage_all[WAVES][kRunStageBytes<DT> / 16];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = int(threadIdx.x) & 63;
    uint4v *stage = stage_all[wave];
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const Tile tile = tiles[t];
        const int bucket = tile_bucket(tile);
        const bool quantized = is_quantized_kind(tile_kind(tile));
        if (quantized && one_key_block(tile)) {
            const Share share(tile, wave);
            const Run run(share.count, bucket, lane);
            RunLoad<DT> load;
            load.issue(grad, tile.elem0 + share.at, share.count, lane);
            float x[G][8];
            load.finish(share.count, lane, stage, x);
            const Scale s = block_scale<SCHEME, WAVES>(x, run, int(tile_bits(tile)), stage_all[0], int(sizeof(stage_all[0]) / 16), wave, lane);
            if (threadIdx.x == 0) store_meta<SCHEME>(meta, tile.bucket0, s);
            const int64_t first = tile.elem0 + share.at;
            const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
            if (share.count > 0)
                CGX_FOR_BITS(tile_bits(tile), (encode_run<SCHEME, BITS, DRAWS>(x, run, s, lane, first, key,
                                                                             packed + tile.packed_off + share.at * BITS / 8,
                                                                             share.last ? tile.pad : 0u, stage)))
        } else if (quantized) {
            if (wave == 0)
                quantize_generic<SCHEME, true>([&](uint32_t j) { return load_elem<DT>(grad, tile.elem0 + j); },
                                               packed + tile.packed_off, meta, tile, tile.pad, bucket, seed_lo, seed_hi, lane);
        } else {
            copy_tile<DT, WAVES * kWave>(grad, packed, tile, int(threadIdx.x));
        }
    }
}

template <int SCHEME, int DRAWS, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, 4) void fused_wide_kernel(const Tile *__restrict__ tiles_in,
                                                             const Tile *__restrict__ tiles_out, int64_t n_tiles, int W,
                                                             int dt, uint32_t seed_lo, uint32_t seed_hi,
                                                             uint8_t *__restrict__ packed_out,
                                                             float *__restrict__ meta_out, const PeerPtrs peers_argument)
{
    (void)peers_argument;
    KernargPeers &peers = kernel_argument_peers(offsetof(FusedArguments, peers));
    __shared__ uint4v stage_all[WAVES][kChunk / 4];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = int(threadIdx.x) & 63;
    uint4v *stage = stage_all[wave];
    for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        const Tile tile = tiles_in[t];
        const int bucket = tile_bucket(tile);
        const int64_t out_off = tiles_out[t].packed_off;
        const uint32_t out_pad = tiles_out[t].pad;
        const bool quantized = is_quantized_kind(tile_kind(tile));
        if (quantized && one_key_block(tile)) {
            const Share share(tile, wave);
            const Run run(share.count, bucket, lane);
            float acc[G][8];
            if (share.count > 0)
                CGX_FOR_BITS(tile_bits(tile), (sum_run<SCHEME, BITS>(peers, W, tile.packed_off + share.at * BITS / 8, tile.bucket0,
                                                                     run, acc, stage, lane)))
            else
                clear_sums(acc);
            clear_missing(acc, run);
            const Scale s = block_scale<SCHEME, WAVES>(acc, run, int(tile_bits(tile)), stage_all[0], int(sizeof(stage_all[0]) / 16), wave, lane);
            if (threadIdx.x == 0) store_meta<SCHEME>(meta_out, tile.bucket0, s);
            const int64_t first = tile.elem0 + share.at;
            const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
            if (share.count > 0)
                CGX_FOR_BITS(tile_bits(tile), (encode_run<SCHEME, BITS, DRAWS>(acc, run, s, lane, first, key,
                                                                             packed_out + out_off + share.at * BITS / 8,
                                                                             share.last ? out_pad : 0u, stage)))
        } else if (quantized) {
            if (wave == 0)
                quantize_generic<SCHEME, false>(
                    [&](uint32_t j) { return generic_sum<SCHEME>(peers, W, tile, bucket, j, -0.0f); },
                    packed_out + out_off, meta_out, tile, out_pad, bucket, seed_lo, seed_hi, lane);
        } else {
            // pass-through: the sum is written as binary32 into the output stream, then its padding
            const SumIo io{nullptr, CGX_F32, packed_out + out_off, CGX_F32, 0};
            if (dt == CGX_F16)
                reduce_copy<CGX_F16, WAVES * kWave>(peers, W, io, 0, tile, int(threadIdx.x));
            else
                reduce_copy<CGX_F32, WAVES * kWave>(peers, W, io, 0, tile, int(threadIdx.x));
            uint8_t *end = packed_out + out_off + uint64_t(tile.count) * 4;
            if (threadIdx.x < out_pad) end[threadIdx.x] = 0;
        }
    }
}

// One block per tile, unless the configuration caps the grid.
inline unsigned wide_grid(int64_t n_tiles, const LaunchConfig &cfg)
{
    int64_t blocks = n_tiles;
    if (cfg.max_blocks > 0 && blocks > cfg.max_blocks) blocks = cfg.max_blocks;
    if (blocks > 0x7fffffff) blocks = 0x7fffffff;
    return unsigned(blocks);
}

}  // namespace

hipError_t launch_quantize_wide(int scheme, const void *grad, int dt, const Tile *tiles, int64_t n_tiles, int draws,
                                int32_t longest, uint64_t seed, void *packed, void *meta, const LaunchConfig &cfg,
                                hipStream_t stream)
{
    if (n_tiles == 0) return hipSuccess;
    using Kernel = void (*)(const void *, const Tile *, int64_t, uint32_t, uint32_t, uint8_t *, float *);
#define CGX_WIDE(S, D, O) {quantize_wide_kernel<S, D, O, 2>, quantize_wide_kernel<S, D, O, 4>}
#define CGX_WIDE_SCHEMES(O) \
    {{CGX_WIDE(kMinMax, CGX_F32, O), CGX_WIDE(kMinMax, CGX_F16, O)}, {CGX_WIDE(kNormSign, CGX_F32, O), CGX_WIDE(kNormSign, CGX_F16, O)}}
    static const Kernel table[3][2][2][2] = {CGX_WIDE_SCHEMES(kDrawsQuad), CGX_WIDE_SCHEMES(kDrawsEven), CGX_WIDE_SCHEMES(kDrawsOdd)};
#undef CGX_WIDE_SCHEMES
#undef CGX_WIDE
    const int waves = longest <= 2 * kChunk ? 2 : 4;
    const Kernel kernel = table[draws][scheme == kSchemeNormSign][dt == CGX_F16][waves == 4];
    hipLaunchKernelGGL(kernel, dim3(wide_grid(n_tiles, cfg)), dim3(waves * kWave), 0, stream, grad, tiles, n_tiles,
                       uint32_t(seed), uint32_t(seed >> 32), static_cast<uint8_t *>(packed), static_cast<float *>(meta));
    return hipGetLastError();
}

hipError_t launch_dequant_reduce_requantize_wide(int scheme, const PeerPtrs &peers, int W, int dt, const Tile *tiles_in,
                                                 const Tile *tiles_out, int64_t n_tiles, int draws, int32_t longest,
                                                 uint64_t seed, void *packed_out, void *meta_out, const LaunchConfig &cfg,
                                                 hipStream_t stream)
{
    if (n_tiles == 0) return hipSuccess;
    using Kernel = void (*)(const Tile *, const Tile *, int64_t, int, int, uint32_t, uint32_t, uint8_t *, float *,
                            const PeerPtrs);
#define CGX_WIDE(S, O) {fused_wide_kernel<S, O, 2>, fused_wide_kernel<S, O, 4>}
    static const Kernel table[3][2][2] = {{CGX_WIDE(kMinMax, kDrawsQuad), CGX_WIDE(kNormSign, kDrawsQuad)},
                                          {CGX_WIDE(kMinMax, kDrawsEven), CGX_WIDE(kNormSign, kDrawsEven)},
                                          {CGX_WIDE(kMinMax, kDrawsOdd), CGX_WIDE(kNormSign, kDrawsOdd)}};
#undef CGX_WIDE
    const int waves = longest <= 2 * kChunk ? 2 : 4;
    const Kernel kernel = table[draws][scheme == kSchemeNormSign][waves == 4];
    hipLaunchKernelGGL(kernel, dim3(wide_grid(n_tiles, cfg)), dim3(waves * kWave), 0, stream, tiles_in, tiles_out, n_tiles, W,
                       dt, uint32_t(seed), uint32_t(seed >> 32), static_cast<uint8_t *>(packed_out),
                       static_cast<float *>(meta_out), peers);
    return hipGetLastError();
}

}  // namespace cgx
