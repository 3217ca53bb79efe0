// Host-side plan: validation of the layer table, sizes of the packed stream
// and meta array, and the tile table the kernels walk.
//
// A tile is a contiguous run of elements of ONE layer that one wavefront
// processes: whole buckets of a quantized layer (paper Sec. 4.3: buckets are
// compressed independently; Sec. 4.1: layers are never mixed) or a piece of a
// pass-through layer.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/cgx.h"

#if defined(__HIPCC__)
#define CGX_HOST_DEVICE __host__ __device__
#else
#define CGX_HOST_DEVICE
#endif
#define CGX_ALWAYS_INLINE inline __attribute__((always_inline))      // a call in a kernel would move its tile to scratch

namespace cgx {

// A chunk is what a wavefront handles per pass of the vectorised path: 64 lanes x `groups` groups
// of 8 consecutive elements.  A kernel is compiled for one chunk size (2 groups = 1024 elements or
// 4 groups = 2048 elements) and walks a tile table built for that size: a vectorised tile is a
// whole number of chunks.
constexpr int chunk_of(int groups) { return 64 * 8 * groups; }
// Elements per pass-through tile of the norm statistic (and of the tables of cgx_plan_tiles).
constexpr int kCopyTile = 8192;
// Elements per pass-through tile of the other kernels: a wave moves what its loads can have in flight together.  A
// longer tile is a chain of round trips that outlasts the rest of a short launch (a reduce of 7.6 M elements with 124
// layers, 8 peers, and the requantize of its sums: 36.1 us with pieces of 2048, 33.8 us with 1024).
constexpr int kCopyPiece = 1024;

enum TileKind : uint32_t {
    kQuantSlow = 0,  // none of the others: a ragged end, a longer bucket, or a tile across two of the generator's key blocks
    kQuantFast = 1,  // power-of-two bucket <= chunk, whole chunks
    kCopyFast = 3,   // pass-through, 16-byte vectors
    kQuantWide = 4,  // one whole power-of-two bucket longer than a chunk (4096, 8192)
    kQuantTail = 5,  // power-of-two bucket <= chunk, the last tile of a layer, shorter than a chunk (run as a kQuantAny)
    kQuantAny = 6    // whole buckets of a size that is no power of two (a multiple of 32, at most a chunk in all)
};

// Chunk-shaped quantized tiles (whole chunks of the bucket-major or row-by-row mapping).
CGX_HOST_DEVICE inline bool is_vector_kind(uint32_t kind) { return kind == kQuantFast || kind == kQuantWide; }
CGX_HOST_DEVICE inline bool is_quantized_kind(uint32_t kind) { return kind != kCopyFast; }
// Tiles that make up the bulk of a plan (the others go first in the table).
CGX_HOST_DEVICE inline bool is_streamed_kind(uint32_t kind) { return is_vector_kind(kind) || kind == kQuantAny; }

struct Tile {               // 32 bytes, read by the kernels with scalar loads
    int64_t elem0;          // first element, index in the fused buffer
    int64_t packed_off;     // byte offset of the tile's payload in the packed stream
    uint32_t bucket0;       // index of the tile's first bucket in the meta array
    uint32_t count;         // elements in the tile
    uint32_t info;          // bits [0:3] bit width, [4:7] TileKind, [8:11] log2(lanes per bucket), [12:20] bucket / 32
    uint32_t pad;           // zero bytes to append after the payload (last tile of a layer)
};
static_assert(sizeof(Tile) == 32, "tile layout is shared with the kernels");

CGX_HOST_DEVICE inline uint32_t tile_bits(const Tile &t) { return t.info & 15u; }
CGX_HOST_DEVICE inline uint32_t tile_kind(const Tile &t) { return (t.info >> 4) & 15u; }
CGX_HOST_DEVICE inline uint32_t tile_lpb_log2(const Tile &t) { return (t.info >> 8) & 15u; }
// Bucket size of a quantized tile (0 for pass-through tiles): info bits [12:20] hold bucket / 32.
CGX_HOST_DEVICE inline int tile_bucket(const Tile &t) { return int((t.info >> 12) & 0x1ffu) * 32; }

// How the vectorised tiles of a bucket size are laid over the lanes, which fixes the kernel
// instantiation of a launch: kMapBuckets for 96..chunk (bucket-major), kMapRows for 32 and 64
// (row by row; needs more registers, so a kernel of its own keeps the others' occupancy),
// kMapWide above the chunk size (a tile is one bucket of several chunks).  One launch serves
// every bucket size of one class.
enum LaneMapping { kMapBuckets = 0, kMapRows = 1, kMapWide = 2 };
inline int mapping_of(int bucket, int chunk) { return bucket <= 64 ? kMapRows : bucket > chunk ? kMapWide : kMapBuckets; }

struct PlanShape {
    size_t packed_bytes = 0;
    size_t meta_bytes = 0;
    uint64_t n_buckets = 0;
};

// Returns CGX_OK or the status code of the first violated rule.
int validate_plan(int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int dt);
// The same rule for a bucket size per layer (every entry, also those of pass-through layers).
int validate_layer_buckets(int32_t L, const int32_t *layer_buckets);

// Sizes only (layout rules of cgx.h).  The plan must be valid.  layer_buckets, if not null,
// gives every layer its own bucket size and `bucket` is ignored.
PlanShape plan_shape(int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int dt,
                     const int32_t *layer_buckets = nullptr);

// Tile table for kernels with chunks of `chunk` elements.  `chunks_per_tile` bounds the length of
// fast tiles.
// With `slots` and `layer_first` (both or neither): numbering the tiles layer by layer and,
// inside a layer, by first element, tile t of the table has number slots[t], and layer l owns
// the numbers layer_first[l] .. layer_first[l + 1] - 1 (the per-layer statistics keep one
// partial sum per tile and add them up in that order).
// With layer_buckets (a bucket size per layer) the table holds the tiles of the layers whose
// bucket size has the lane mapping of `bucket` (mapping_of at this chunk size) only, at their places in the whole
// plan's streams, and the pass-through layers' with with_copies.
// copy_tile: elements per pass-through tile (kCopyTile or kCopyPiece).  longer_than: quantized layers with buckets of at
// most this size are left out too.
void build_tiles(int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int dt, int chunk,
                 int chunks_per_tile, std::vector<Tile> &tiles, std::vector<uint32_t> *slots = nullptr,
                 std::vector<int64_t> *layer_first = nullptr, const int32_t *layer_buckets = nullptr,
                 bool with_copies = true, int copy_tile = kCopyTile, int longer_than = 0);

// What one launch of a quantizer, the fused kernel or the error statistic walks: a launch runs one kernel
// instantiation, so a plan whose layers have bucket sizes of several lane mappings takes one per mapping.  The first
// part also holds the pass-through layers, a part of mapping kMapWide is the last one.
struct TablePart {
    int32_t bucket = 0;          // smallest bucket size in use: names the lane mapping
    int32_t longest = 0;         // longest bucket size in use
    int chunk = 0;               // elements per chunk of the kernel that walks it
    int64_t first = 0, count = 0;
    bool odd = false;            // some quantized tile starts on an odd element index
    bool quads = true;           // every quantized tile starts on a multiple of 8 elements
    bool aligned = true;         // every vectorised quantized tile starts on a 16-byte boundary of the buffer

    // The quantizer fetches the part's chunks through LDS, with whole-line loads.  Short tiles that start elsewhere have no say
    // in it, but for an odd start, whose draws take a kernel that is not built for both.
    bool through_lds() const { return aligned && !odd && mapping_of(bucket, chunk) == kMapBuckets; }
};

// The table of a plan, which all calls with the same chunk and tile lengths share: a program that has run one of them
// may capture any of them.
struct PlanTable {
    std::vector<Tile> tiles;
    std::vector<TablePart> parts;
    // Per-layer numbering of the tiles that carry a partial sum (see build_tiles): all of them in a table of kCopyTile
    // pieces; in one of kCopyPiece pieces the quantized ones (a pass-through layer has no error).  Empty unless asked for.
    std::vector<uint32_t> slots;
    std::vector<int64_t> layer_first;
    int64_t stats_tiles = 0;     // tiles in pieces of kCopyTile: partial sums that a workspace of the statistics holds

    // A reduction walks all parts in one launch and needs no whole buckets.  Tiles from `narrow()` on hold one bucket
    // longer than a chunk each and go to pieces() waves, a chunk of the bucket each.
    int64_t narrow() const;
    int pieces() const;
};
constexpr uint32_t kNoSlot = 0xffffffffu;
// long_chunk (0: none): layers with buckets longer than `chunk` go to parts of their own, for the kernels with chunks of
// long_chunk elements.
PlanTable build_table(int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int dt, int chunk,
                      int chunks_per_tile, bool numbered, const int32_t *layer_buckets = nullptr, int copy_tile = kCopyPiece,
                      int long_chunk = 0);

// The tiles of a plan as a reduction walks them: `count` pieces of work, of which the first `narrow` are a tile each and
// the others, `pieces` (at most 8) per tile, a chunk of a tile.  With pieces == 1, narrow == count.
struct ReduceTiles {
    const Tile *tiles = nullptr;
    int64_t count = 0;
    uint32_t narrow = 0, pieces = 1;
    // by storage type of the result: most elements lie in tiles that do not start on 64, on 16 bytes of it
    bool off_64_bytes[2] = {false, false}, off_16_bytes[2] = {false, false};
};
constexpr int64_t kMostPieces = int64_t(1) << 29;     // pieces of the tiles behind the narrow ones: see Piece

// Piece of work number t: tile number `tile`, chunk number `piece` of it.
struct Piece {
    int64_t tile;
    uint32_t piece = 0;
    // ceil(2^32 / pieces): the upper half of its product with a number below kMostPieces is the quotient for up to 8 pieces
    // (the error of the inverse, at most 7 / 8, times the number stays below 2^32 / 8)
    static uint32_t inverse(uint32_t pieces) { return pieces > 1 ? uint32_t(((uint64_t(1) << 32) + pieces - 1) / pieces) : 0u; }
    CGX_HOST_DEVICE CGX_ALWAYS_INLINE Piece(int64_t t, uint32_t narrow, uint32_t pieces, uint32_t inv) : tile(t)
    {
        if (t >= int64_t(narrow)) {
            const uint32_t u = uint32_t(t - int64_t(narrow)), q = uint32_t((uint64_t(u) * inv) >> 32);
            piece = u - q * pieces;
            tile = int64_t(narrow) + q;
        }
    }
    // Leaves the piece's share in the tile (one behind the narrow ones); false: there is none.
    CGX_HOST_DEVICE CGX_ALWAYS_INLINE bool cut(Tile &t, int chunk) const
    {
        if (!is_quantized_kind(tile_kind(t))) return piece == 0;
        const uint32_t at = piece * uint32_t(chunk);
        if (at >= t.count) return false;
        t.elem0 += at;
        t.packed_off += at / 8 * tile_bits(t);
        t.count = t.count - at < uint32_t(chunk) ? t.count - at : uint32_t(chunk);
        return true;
    }
};

}  // namespace cgx
