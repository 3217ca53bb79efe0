// cgx_quantize / cgx_requantize / cgx_qsgd_quantize: the quantize kernel and its launcher.
#include "cgx_device_quantize.h"

namespace cgx {
namespace {

// DRAWS: where the plan's quantized tiles start (see encode_group).
// VIA_LDS: every vectorised tile starts on a 16-byte boundary and the bucket-major mapping reads its
// chunks through LDS (see chunk_through_lds); never with kDrawsOdd.
template <int SCHEME, int DT, int MAP, int DRAWS, bool VIA_LDS = false>
__global__ __launch_bounds__(kBlock) void quantize_kernel(const void *__restrict__ grad,
                                                           const Tile *__restrict__ tiles, int64_t n_tiles,
                                                           uint32_t seed_lo, uint32_t seed_hi,
                                                           uint8_t *__restrict__ packed,
                                                           float *__restrict__ meta)
{
    // per-wave staging area: a chunk as stored, then its packed codes (see kRunStageBytes)
    __shared__ uint4v stage_all[kWavesPerBlock][kRunStageBytes<DT> / 16];
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    int lane_of_wave = int(threadIdx.x) & 63;
    uint4v *stage = stage_all[wave];
    const int64_t stride = int64_t(gridDim.x) * kWavesPerBlock;
    int64_t t = int64_t(blockIdx.x) * kWavesPerBlock + wave;
    if (t >= n_tiles) return;
    Tile upcoming = tiles[t];
    for (; t < n_tiles; t += stride) {
        // the lane index is made opaque once per tile: otherwise everything that depends on the
        // lane alone (offsets, masks, of every bit width's path) is hoisted out of this loop and
        // stays in registers across all of it
        asm volatile("" : "+v"(lane_of_wave));
        const int lane = lane_of_wave;
        const Tile tile = upcoming;
        // a wave that takes more than one tile has the next descriptor on its way meanwhile
        if (t + stride < n_tiles) upcoming = tiles[t + stride];
        const int bucket = tile_bucket(tile);       // per tile: a launch may mix sizes of one lane mapping
        const uint32_t kind = tile_kind(tile);
        if (kind == kQuantFast) {
            if constexpr (MAP == kMapRows) {
                CGX_FOR_BITS(tile_bits(tile), (quantize_fast_rows<SCHEME, DT, BITS, DRAWS>(grad, packed, meta, tile, bucket,
                                                                                      seed_lo, seed_hi, lane, stage)))
            } else {
                CGX_FOR_BITS(tile_bits(tile), (quantize_fast<SCHEME, DT, BITS, DRAWS, VIA_LDS>(
                                                  grad, packed, meta, tile, bucket, seed_lo, seed_hi, lane, stage)))
            }
        } else if (is_quantized_kind(kind) && tile.count <= uint32_t(kChunk) && one_key_block(tile)) {
            // (one bucket of 1056 ... 1536 elements per tile: the lanes past its end cost as much as the others.  Quantize of
            // 67 M elements, us with four groups per lane and with three: binary32, buckets of 1056, 79.8 and 71.3, of 1184,
            // 73.8 and 64.8; binary16 70.5 and 59.3, 64.4 and 53.2)
            if (G == 4 && MAP == kMapBuckets && three_groups_hold(tile, bucket)) {
                if constexpr (G == 4 && MAP == kMapBuckets) {
                    CGX_FOR_BITS(tile_bits(tile), (quantize_run<SCHEME, DT, BITS, DRAWS, 3>(grad, packed, meta, tile, bucket, seed_lo,
                                                                                         seed_hi, lane, stage)))
                }
            } else {
                CGX_FOR_BITS(tile_bits(tile), (quantize_run<SCHEME, DT, BITS, DRAWS>(grad, packed, meta, tile, bucket,
                                                                                     seed_lo, seed_hi, lane, stage)))
            }
        } else if (is_quantized_kind(kind)) {
            quantize_generic<SCHEME, true>([&](uint32_t j) { return load_elem<DT>(grad, tile.elem0 + j); },
                                           packed + tile.packed_off, meta, tile, tile.pad, bucket, seed_lo,
                                           seed_hi, lane);
        } else {
            copy_tile<DT>(grad, packed, tile, lane);
        }
    }
}

}  // namespace

// This file is compiled once per chunk size (CGX_GROUPS = 2 and 4): launch_quantize_g2, launch_quantize_g4.
hipError_t CGX_CONCAT(launch_quantize_g, CGX_GROUPS)(int scheme, const void *grad, int dt, const Tile *tiles, int64_t n_tiles, int draws,
                           bool through_lds, int32_t bucket, uint64_t seed, void *packed, void *meta,
                           const LaunchConfig &cfg, hipStream_t stream)
{
    if (n_tiles == 0) return hipSuccess;
    // Four fifths of the waves that one tile each would take: every fourth wave takes a second tile, whose
    // descriptor it fetches while it works on the first.  For the kernel of 1024-element chunks on plans of up to
    // 2^19 tiles.  Measured by kernel trace, the two grids alternating on one box: ResNet-50 plan (25 k tiles)
    // 20.9 -> 20.0 us, the requantize of a 13.7 M-element share 12.6 -> 11.9 us, full BERT-base buffer 77.6 ->
    // 76.3 us, a 44 M-element share 34.6 -> 34.2 us; the 1.3 G-element buffer (1.28 M tiles) 978 -> 988 us and
    // binary16 input (2048-element chunks, two per tile) 25.5 -> 26.7 us on a small buffer, hence the limits.
    // With one and a half tiles per wave the gain is gone from 100 M elements on, with two it is a loss.
    LaunchConfig shaped = cfg;
    if (kGroups == 2 && cfg.max_blocks == 0 && cfg.quantize_tiles_per_wave_x4 > 4 && n_tiles <= (int64_t(1) << 19)) {
        const int64_t blocks = (n_tiles + kWavesPerBlock - 1) / kWavesPerBlock;
        shaped.max_blocks = int((blocks * 4 + cfg.quantize_tiles_per_wave_x4 - 1) / cfg.quantize_tiles_per_wave_x4);
    }
    const dim3 grid(grid_for(n_tiles, shaped)), block(kBlock);
    const uint32_t seed_lo = uint32_t(seed), seed_hi = uint32_t(seed >> 32);
    using Kernel = void (*)(const void *, const Tile *, int64_t, uint32_t, uint32_t, uint8_t *, float *);
#define CGX_QUANTIZE_MAPS(S, D, O) \
    {quantize_kernel<S, D, kMapBuckets, O>, quantize_kernel<S, D, kMapRows, O>}
#define CGX_QUANTIZE_SCHEMES(O) \
    {{CGX_QUANTIZE_MAPS(kMinMax, CGX_F32, O), CGX_QUANTIZE_MAPS(kMinMax, CGX_F16, O)}, \
     {CGX_QUANTIZE_MAPS(kNormSign, CGX_F32, O), CGX_QUANTIZE_MAPS(kNormSign, CGX_F16, O)}}
    static const Kernel table[3][2][2][2] = {CGX_QUANTIZE_SCHEMES(kDrawsQuad), CGX_QUANTIZE_SCHEMES(kDrawsEven),
                                             CGX_QUANTIZE_SCHEMES(kDrawsOdd)};
#undef CGX_QUANTIZE_SCHEMES
#undef CGX_QUANTIZE_MAPS
#define CGX_QUANTIZE_LDS(S, O) {quantize_kernel<S, CGX_F32, kMapBuckets, O, true>, quantize_kernel<S, CGX_F16, kMapBuckets, O, true>}
    // (binary16 with kDrawsEven: whole chunks on 16 bytes, and a layer of less than a chunk that starts on 2, 4 or 6 mod 8.
    // Quantize of 105 M and 26 M elements beside such a layer, 4 bit, buckets of 128, us through LDS and without: 57 and 61,
    // 15.9 and 17.5; 105 M at 2 bits 47.5 and 53.5)
    static const Kernel lds_table[2][2][2] = {{CGX_QUANTIZE_LDS(kMinMax, kDrawsQuad), CGX_QUANTIZE_LDS(kNormSign, kDrawsQuad)},
                                              {CGX_QUANTIZE_LDS(kMinMax, kDrawsEven), CGX_QUANTIZE_LDS(kNormSign, kDrawsEven)}};
#undef CGX_QUANTIZE_LDS
    const Kernel kernel = through_lds && draws != kDrawsOdd && cfg.via_lds
                              ? lds_table[draws][scheme == kSchemeNormSign][dt == CGX_F16]
                              : table[draws][scheme == kSchemeNormSign][dt == CGX_F16][mapping_of(bucket, kChunk)];
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, grad, tiles, n_tiles, seed_lo, seed_hi,
                       static_cast<uint8_t *>(packed), static_cast<float *>(meta));
    return hipGetLastError();
}

}  // namespace cgx
