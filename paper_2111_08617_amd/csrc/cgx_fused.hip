// cgx_dequant_reduce_requantize: the fused kernel and its launcher.
#include "cgx_device_quantize.h"
#include "cgx_device_reduce.h"

namespace cgx {
namespace {

// ---------------------------------------------------------------- fused reduce + requantize

// The sums of a chunk never leave the registers: reduce_chunk feeds quantize_chunk.
template <int SCHEME, int BITS, int DRAWS, typename Peers>
__device__ __forceinline__ void fused_fast(Peers &peers, int W, const Tile &tile, int64_t out_off,
                                           int bucket, uint32_t seed_lo, uint32_t seed_hi,
                                           uint8_t *__restrict__ packed_out, float *__restrict__ meta_out,
                                           int lane, uint4v *stage)
{
    const LaneMap map(tile, bucket, lane);
    const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
    const int chunks = int(tile.count / kChunk);
    const int buckets_per_chunk = kChunk / bucket;
    for (int c = 0; c < chunks; c++) {
        float acc[G][8];
        clear_sums(acc);
        const int64_t in_off = tile.packed_off + int64_t(c) * (kChunk * BITS / 8);
        const uint32_t g = tile.bucket0 + c * buckets_per_chunk + map.bi;
        reduce_chunk<SCHEME, BITS>(peers, W, in_off, g, map, acc, stage, lane);
        quantize_chunk<SCHEME, BITS, DRAWS>(acc, map, lane, tile.elem0 + int64_t(c) * kChunk, key,
                                     meta_out + kMetaFloats<SCHEME> * (tile.bucket0 + c * buckets_per_chunk),
                                     packed_out + out_off + int64_t(c) * (kChunk * BITS / 8), stage);
    }
}

// A run: its sums feed the quantizer in the same lane order.
template <int SCHEME, int BITS, int DRAWS, typename Peers>
__device__ __forceinline__ void fused_run(Peers &peers, int W, const Tile &tile, int64_t out_off, uint32_t out_pad,
                                          int bucket, uint32_t seed_lo, uint32_t seed_hi,
                                          uint8_t *__restrict__ packed_out, float *__restrict__ meta_out, int lane,
                                          uint4v *stage)
{
    const Run run(int(tile.count), bucket, lane);
    const uint32_t key = rng_key(seed_lo, seed_hi, uint32_t((uint64_t(tile.elem0) >> 1) >> 32));
    float acc[G][8];
    sum_run<SCHEME, BITS>(peers, W, tile.packed_off, tile.bucket0, run, acc, stage, lane);
    clear_missing(acc, run);
    quantize_run_regs<SCHEME, BITS, DRAWS>(acc, run, lane, tile.elem0, key, meta_out + kMetaFloats<SCHEME> * tile.bucket0,
                                         packed_out + out_off, out_pad, stage);
}

// tiles_in follows the layout of the chunks (storage type dt), tiles_out that of the
// output (binary32 pass-through layers); the two tables list the same tiles in the same order.
template <int SCHEME, int DRAWS>
__global__ __launch_bounds__(kBlock) void fused_kernel(const Tile *__restrict__ tiles_in,
                                                        const Tile *__restrict__ tiles_out, int64_t n_tiles, int W,
                                                        int dt, uint32_t seed_lo, uint32_t seed_hi,
                                                        uint8_t *__restrict__ packed_out,
                                                        float *__restrict__ meta_out, const PeerPtrs peers_argument)
{
    (void)peers_argument;
    KernargPeers &peers = kernel_argument_peers(offsetof(FusedArguments, peers));
    __shared__ uint4v stage_all[kWavesPerBlock][kChunk / 4];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    int lane_of_wave = int(threadIdx.x) & 63;
    uint4v *stage = stage_all[wave];
    const int64_t stride = int64_t(gridDim.x) * kWavesPerBlock;
    for (int64_t t = int64_t(blockIdx.x) * kWavesPerBlock + wave; t < n_tiles; t += stride) {
        // the lane index is made opaque once per tile: otherwise everything that depends on the
        // lane alone (offsets, masks, of every bit width's path) is hoisted out of this loop and
        // stays in registers across all of it
        asm volatile("" : "+v"(lane_of_wave));
        const int lane = lane_of_wave;
        const Tile tile = tiles_in[t];
        const int bucket = tile_bucket(tile);       // per tile: a launch may mix sizes of one lane mapping
        const int64_t out_off = tiles_out[t].packed_off;
        const uint32_t out_pad = tiles_out[t].pad;
        const uint32_t kind = tile_kind(tile);
        if (kind == kQuantFast) {
            CGX_FOR_BITS(tile_bits(tile), (fused_fast<SCHEME, BITS, DRAWS>(peers, W, tile, out_off, bucket, seed_lo,
                                                                     seed_hi, packed_out, meta_out, lane, stage)))
        } else if (is_quantized_kind(kind) && tile.count <= uint32_t(kChunk) && one_key_block(tile)) {
            CGX_FOR_BITS(tile_bits(tile), (fused_run<SCHEME, BITS, DRAWS>(peers, W, tile, out_off, out_pad, bucket, seed_lo,
                                                                        seed_hi, packed_out, meta_out, lane, stage)))
        } else if (is_quantized_kind(kind)) {
            quantize_generic<SCHEME, false>(
                [&](uint32_t j) { return generic_sum<SCHEME>(peers, W, tile, bucket, j, -0.0f); },
                packed_out + out_off, meta_out, tile, out_pad, bucket, seed_lo, seed_hi, lane);
        } else {
            // pass-through: the sum is written as binary32 into the output stream, then its padding
            const SumIo io{nullptr, CGX_F32, packed_out + out_off, CGX_F32, 0};
            if (dt == CGX_F16)
                reduce_copy<CGX_F16>(peers, W, io, 0, tile, lane);
            else
                reduce_copy<CGX_F32>(peers, W, io, 0, tile, lane);
            uint8_t *end = packed_out + out_off + uint64_t(tile.count) * 4;
            if (uint32_t(lane) < out_pad) end[lane] = 0;
        }
    }
}

}  // namespace

// This file is compiled once per chunk size (CGX_GROUPS = 2 and 4): launch_dequant_reduce_requantize_g2, _g4.
hipError_t CGX_CONCAT(launch_dequant_reduce_requantize_g, CGX_GROUPS)(int scheme, const PeerPtrs &peers, int W, int dt, const Tile *tiles_in,
                                            const Tile *tiles_out, int64_t n_tiles, int draws,
                                            uint64_t seed, void *packed_out, void *meta_out,
                                            const LaunchConfig &cfg, hipStream_t stream)
{
    if (n_tiles == 0) return hipSuccess;
    const dim3 grid(grid_for(n_tiles, cfg)), block(kBlock);
    using Kernel = void (*)(const Tile *, const Tile *, int64_t, int, int, uint32_t, uint32_t, uint8_t *, float *,
                            const PeerPtrs);
    static const Kernel table[3][2] = {{fused_kernel<kMinMax, kDrawsQuad>, fused_kernel<kNormSign, kDrawsQuad>},
                                       {fused_kernel<kMinMax, kDrawsEven>, fused_kernel<kNormSign, kDrawsEven>},
                                       {fused_kernel<kMinMax, kDrawsOdd>, fused_kernel<kNormSign, kDrawsOdd>}};
    const Kernel kernel = table[draws][scheme == kSchemeNormSign];
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, tiles_in, tiles_out, n_tiles, W, dt, uint32_t(seed),
                       uint32_t(seed >> 32), static_cast<uint8_t *>(packed_out), static_cast<float *>(meta_out), peers);
    return hipGetLastError();
}

}  // namespace cgx
