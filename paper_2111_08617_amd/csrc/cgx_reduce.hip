// cgx_dequant_reduce and its relatives: the reduce kernel and its launcher.
#include "cgx_device_reduce.h"

namespace cgx {
namespace {

// The arguments as the kernarg segment lays them out (each at its natural alignment, in order): gives the
// offset of the peers' table behind the scalars.
struct ReduceArguments {
    const Tile *tiles;
    int64_t n_tiles;
    int W, dt;
    const void *init;
    void *out;
    int init_dt, out_dt, keep;
    uint32_t narrow, pieces, inv_pieces;
    PeerPtrs peers;
};

// SINGLE: a decompression (W = 1, no start values) into storage type SINGLE, bound by the eight bytes it writes per byte
// it reads.  It needs half of the reduction's registers and LDS, and more waves then keep stores in flight (59 instead of 101
// vector registers at 2048-element chunks, eight waves per SIMD instead of four; 36 instead of 86 at 1024, eight instead of
// five): 8 shares of 355 M elements to binary16 187 -> 166 us; to binary32, 4 bits, codes from memory, 268 M elements 224 ->
// 185 us, 67 M 58 -> 49.  (Decompressed again and again from codes that the memory-side cache holds, 162 -> 170 and 43.5 ->
// 44.5.)
constexpr int kAnyOut = -1;

template <int SCHEME, int SINGLE>
__global__ __launch_bounds__(kBlock) void reduce_kernel(const Tile *__restrict__ tiles, int64_t n_tiles, int W_argument, int dt,
                                                         const void *init, void *out, int init_dt, int out_dt,
                                                         int keep, uint32_t narrow, uint32_t pieces, uint32_t inv_pieces,
                                                         const PeerPtrs peers_argument)
{
    // the vectorised tiles index the table with constants (it then sits in scalar registers);
    // the other kinds index it at run time and read it from the kernarg segment
    const PeerPtrs &peers = peers_argument;
    KernargPeers &peers_in_memory = kernel_argument_peers(offsetof(ReduceArguments, peers));
    constexpr bool kSingle = SINGLE != kAnyOut;
    const int W = kSingle ? 1 : W_argument;
    const SumIo io{kSingle ? nullptr : init, init_dt, out, kSingle ? SINGLE : out_dt, kSingle ? int(kStoreThrough) : keep};
    // per-wave staging area: a chunk of results, or the packed bytes of a block of peers (at 8 bits a chunk of a single
    // peer takes kChunk bytes, half of its binary16 results)
    __shared__ uint4v stage_all[kWavesPerBlock][kChunk / (SINGLE == CGX_F16 ? 8 : 4)];
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
        // The tiles behind the first `narrow` hold a bucket longer than a chunk each: `pieces` waves take a chunk of it
        // each (a sum needs no whole bucket).  Per tile of 6144 elements in a wave of its own, reducing 67 M elements of 8
        // peers took 486 us, and takes 97; buckets of 4096, 99 and 92.
        const Piece piece(t, narrow, pieces, inv_pieces);
        Tile tile = tiles[piece.tile];
        if (t >= int64_t(narrow) && !piece.cut(tile, kChunk)) continue;
        const int bucket = tile_bucket(tile);       // per tile: a launch may mix sizes of one lane mapping
        const uint32_t kind = tile_kind(tile);
        if (is_vector_kind(kind)) {      // a wide tile is chunks of one bucket: kChunk / bucket == 0 below
            CGX_FOR_BITS(tile_bits(tile), (reduce_fast<SCHEME, BITS>(peers, W, io, tile, bucket, lane, stage)))
        } else if (is_quantized_kind(kind)) {
            CGX_FOR_BITS(tile_bits(tile), (reduce_run_tile<SCHEME, BITS>(peers_in_memory, W, io, tile, bucket, lane, stage)))
        } else if (dt == CGX_F16) {
            reduce_copy<CGX_F16>(peers_in_memory, W, io, tile.elem0, tile, lane);
        } else {
            reduce_copy<CGX_F32>(peers_in_memory, W, io, tile.elem0, tile, lane);
        }
    }
}

}  // namespace

// This file is compiled once per chunk size (CGX_GROUPS = 2 and 4): launch_dequant_reduce_g2, launch_dequant_reduce_g4.
hipError_t CGX_CONCAT(launch_dequant_reduce_g, CGX_GROUPS)(int scheme, const PeerPtrs &peers, int W, int dt, const ReduceTiles &tiles,
                                 const void *init, int init_dt, void *out, int out_dt,
                                 int store_policy, const LaunchConfig &cfg, hipStream_t stream)
{
    if (tiles.count == 0) return hipSuccess;
    const dim3 grid(grid_for(tiles.count, cfg)), block(kBlock);
    using Kernel = void (*)(const Tile *, int64_t, int, int, const void *, void *, int, int, int, uint32_t, uint32_t, uint32_t,
                            const PeerPtrs);
    const uint32_t narrow = tiles.pieces > 1 ? tiles.narrow : 0xffffffffu;
    // (a decompression to binary32 runs the build for chunks of 1024 elements, one to binary16 that for 2048: 4 KB of
    // results per wave either way)
    constexpr int kSingleOut = kGroups == 2 ? CGX_F32 : CGX_F16;
    const bool single = store_policy == kStoreThrough && out_dt == kSingleOut;
    static const Kernel table[2][2] = {{reduce_kernel<kMinMax, kAnyOut>, reduce_kernel<kNormSign, kAnyOut>},
                                       {reduce_kernel<kMinMax, kSingleOut>, reduce_kernel<kNormSign, kSingleOut>}};
    const bool decompression = single && W == 1 && !init;
    const Kernel kernel = table[decompression][scheme == kSchemeNormSign];
    // Where the waves' stores do not start on 64 bytes of the result, two waves write into the lines between them, and eight
    // waves per SIMD have more such lines open than pays: LDS that nothing uses holds the kernel to seven, or six.  With 8, 7,
    // 6 and 5 waves, us, 4 bits, 268 M elements: to binary32 in layers of odd lengths 268, 234, 232, 242 (codes still in the
    // memory-side cache 284, 274, 261, 247), on 16 bytes 257, 251, 255, 271 (266, 263, 266, 277); to binary16, odd lengths,
    // 139, 128, 124, 124 (122, 117, 121, 128).  On 64 bytes eight are the best: 185, 200, 205, 219, unless the codes are in
    // that cache: 170, 169, 167, 162.
    const auto lds_for = [](unsigned waves) {
        return 160 * 1024 / waves / 128 * 128 - unsigned(sizeof(uint4v)) * kWavesPerBlock * kChunk / (kGroups == 2 ? 4 : 8);
    };
    const unsigned unused_lds = !decompression || !tiles.off_64_bytes[out_dt]               ? 0
                                : out_dt == CGX_F32 && tiles.off_16_bytes[out_dt] ? lds_for(6) : lds_for(7);
    hipLaunchKernelGGL(kernel, grid, block, unused_lds, stream, tiles.tiles, tiles.count, W, dt, init, out, init_dt, out_dt, store_policy,
                       narrow, tiles.pieces, Piece::inverse(tiles.pieces), peers);
    return hipGetLastError();
}

}  // namespace cgx
