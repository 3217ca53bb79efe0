// extern "C" entry points of libcgx.so (see include/cgx.h): argument checks,
// the per-plan tile table cache, and kernel launches on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <vector>

#include "../../include/cgx_diag.h"
#include "cgx_kernels.h"
#include "cgx_plan.h"

namespace {

using cgx::Tile;

// How the tiles of a table are cut.
struct TableKind {
    int chunk = 0;              // elements per chunk of the kernels that walk it
    int chunks_per_tile = 0;
    int copy_tile = cgx::kCopyPiece;      // elements per tile of a pass-through layer
    int long_chunk = 0;         // not 0: the chunk of the layers with buckets longer than `chunk`
    bool operator==(const TableKind &o) const
    {
        return chunk == o.chunk && chunks_per_tile == o.chunks_per_tile && copy_tile == o.copy_tile && long_chunk == o.long_chunk;
    }
};

struct CachedPlan {
    // identity
    int device = 0;
    int32_t bucket = 0;
    int dt = 0;
    uint64_t digest = 0;        // hash of (off, bits, layer_buckets): compared before the arrays themselves
    TableKind kind;
    std::vector<int64_t> off;
    std::vector<uint8_t> bits;
    std::vector<int32_t> layer_buckets;   // empty: `bucket` for every layer
    // content
    cgx::PlanShape shape;
    std::vector<cgx::TablePart> parts;
    int64_t n_tiles = 0;
    int64_t stats_tiles = 0;    // partial sums that a workspace of the statistics holds
    cgx::ReduceTiles reduce;    // the tiles as a reduction walks them
    bool one_bit_layers = false;
    Tile *d_tiles = nullptr;
    // per-layer numbering of the tiles (for the statistics): slot of every tile, first slot of every layer
    uint32_t *d_slots = nullptr;
    int64_t *d_layer_first = nullptr;
    uint64_t last_use = 0;      // cache clock at the latest look-up
    bool pinned = false;        // a stream capture has recorded launches that read these tables: never dropped
};

void free_plan(CachedPlan &p)
{
    if (p.d_tiles) (void)hipFree(p.d_tiles);
    if (p.d_slots) (void)hipFree(p.d_slots);
    if (p.d_layer_first) (void)hipFree(p.d_layer_first);
    p.d_tiles = nullptr;
    p.d_slots = nullptr;
    p.d_layer_first = nullptr;
}

template <typename T>
bool upload(T **dst, const std::vector<T> &src)
{
    if (src.empty()) return true;
    const size_t bytes = src.size() * sizeof(T);
    if (hipMalloc(reinterpret_cast<void **>(dst), bytes) != hipSuccess) return false;
    return hipMemcpy(*dst, src.data(), bytes, hipMemcpyHostToDevice) == hipSuccess;
}

std::mutex g_mutex;
// A caller that keeps changing its plan (new bit widths every so often) must not grow the
// cache without bound: beyond kMaxPlans entries (those that captured graphs read are not counted) the least
// recently used one is dropped.  An
// entry handed out stays alive while its call uses it (shared ownership); its device tables
// are released when the last owner lets go, and hipFree waits for launches still reading them.
// The cache object itself is never destroyed, so nothing is freed during process exit, when
// the HIP runtime may already be gone.
constexpr int64_t kMaxPlans = 64;
using PlanRef = std::shared_ptr<const CachedPlan>;
std::vector<std::shared_ptr<CachedPlan>> &g_plans = *new std::vector<std::shared_ptr<CachedPlan>>();
uint64_t g_clock = 0;

int env_int(const char *name, int fallback)
{
    const char *v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : fallback;
}

// Launch-shape overrides for the tests and for measurements (listed in include/cgx_diag.h): read once.
const cgx::LaunchConfig &launch_config()
{
    static const cgx::LaunchConfig cfg = [] {
        cgx::LaunchConfig c;
        c.chunks_per_tile = env_int("CGX_CHUNKS_PER_TILE", 0);
        c.max_blocks = env_int("CGX_MAX_BLOCKS", c.max_blocks);
        c.via_lds = env_int("CGX_VIA_LDS", c.via_lds);
        c.keep_sums_max_bytes = long(env_int("CGX_KEEP_SUMS_MB", int(c.keep_sums_max_bytes >> 20))) << 20;
        c.dequantize_through = env_int("CGX_DEQUANTIZE_THROUGH", c.dequantize_through);
        c.reduce_groups = env_int("CGX_REDUCE_GROUPS", 0) == 2 ? 2 : env_int("CGX_REDUCE_GROUPS", 0) == 4 ? 4 : 0;
        c.quantize_tiles_per_wave_x4 = env_int("CGX_QUANTIZE_TILES_PER_WAVE_X4", c.quantize_tiles_per_wave_x4);
        c.quantize_groups = env_int("CGX_QUANTIZE_GROUPS", 0) == 2 ? 2 : env_int("CGX_QUANTIZE_GROUPS", 0) == 4 ? 4 : 0;
        return c;
    }();
    return cfg;
}

// Chunks per vectorised tile.  One keeps the most loads in flight and wins wherever a wave's
// chunk is 4 KB of input or more.  Two cases differ on buffers that fill the chip many times over
// (measured; shorter buffers lose to the coarser tail of the launch):
//  - cgx_quantize on binary16, which is the heaviest in arithmetic per byte: a wave takes 2 chunks
//    (354 M elements: 155 -> 149 us; 4 chunks: 156 us);
//  - the fused reduce + requantize, which is bound by arithmetic: 2 chunks (3-6 % faster at
//    164-268 M elements for every width).
// Bucket sizes of a call: one for all layers, or one per layer (per_layer != nullptr).
struct Buckets {
    int32_t uniform;
    const int32_t *per_layer;
};

enum CallKind { kQuantizeCall, kFusedCall, kOtherCall };

// Elements per chunk of the kernel a call runs.  The quantizer of binary32 input takes chunks of 1024
// elements (4 KB per wave and pass: measured, a streaming kernel sustains about a tenth more with 4 KB
// per wave than with 8 KB, and the quantizer follows it: 0.74 -> 0.78 of the HBM peak on 1.3 G
// elements); on binary16 a chunk of 2048 elements is 4 KB already.  The reduce, fused and statistics
// kernels take 2048 (a peer's codes of a chunk then fill a whole load instruction at 4 bits), but a decompression to binary32
// (reduce_impl) and the fused call on short binary32 buffers (fused_impl) 1024.
// A call with a bucket of more than 1024 elements takes the quantizer of 2048-element chunks also on binary32: such a
// bucket fits its chunk or a block of its waves (cgx_wide.hip).  The whole call takes it, one launch for all sizes
// up to 2048 instead of two (ResNet-50 with sizes by layer length, 128 / 512 / 2048: 36 us of quantizing in two launches
// of 1024-element chunks, in which a bucket of 2048 is read twice,
// 26 us in one launch of 2048-element chunks).
// A chunk takes whole buckets, and lanes without elements cost as much as the others.  Where chunks of 1024 elements spend
// at least a quarter more lanes than those of 2048 (352, 384, 544 ... 672 and 768 of the multiples of 32), binary32 takes the
// longer ones.  Measured, 1024 against 2048, us: 67 M elements in buckets of 672 72.6 and 51.2, 384 62.8 and 52.3, 768 63.8
// and 50.7; 8.4 M 11.4 and 10.6, 10.3 and 10.6, 10.3 and 9.5.  Where they save less, the longer ones lose on short buffers:
// buckets of 288 (1.17) 60.6 and 53.2 on 67 M elements, 10.0 and 10.6 on 8.4 M; 224 (1.12) 57.8 and 52.7, 9.6 and 10.7.

// Lanes' worth of elements that the quantizer of `chunk` spends per element of buckets of a size (at most the chunk).
double lanes_spent(int32_t bucket, int chunk)
{
    const int32_t held = chunk / bucket * bucket;
    // (runs of up to 1536 elements take three groups per lane, see three_groups_hold)
    const int32_t lanes = chunk == cgx::chunk_of(4) && held <= 1536 && held > 1024 && bucket % 24 == 0 ? 1536 : chunk;
    return double(lanes) / held;
}

// Chunks of a quantize call (see TableKind).  The arrays of the (checked) plan are read only where the layers have sizes
// of their own.
// A binary32 call with buckets of more than 1024 elements in some layers and 100 M elements or more in the others leaves
// the others to the kernel of the shorter chunks, in a launch of their own.  Layers of 512 with 3 % of 2048, one launch and
// two, us: 67 M elements 50.9 and 52.8, 134 M 100.8 and 98.1, 268 M 202 and 195, 537 M 405 and 387; half of 2048: 134 M 99.7
// and 99.9, 268 M 201 and 195.
struct Chunks {
    int chunk, long_chunk;
};
Chunks quantize_chunks(int dt, const Buckets &buckets, int32_t L, const int64_t *off, const uint8_t *bits)
{
    const int shorter = cgx::chunk_of(2), longer = cgx::chunk_of(4);
    double in_shorter = 0.0, in_longer = 0.0;
    int64_t short_elements = 0, long_elements = 0;
    const auto add = [&](int64_t elements, int32_t bucket) {
        (bucket > shorter ? long_elements : short_elements) += elements;
        if (bucket <= 0 || bucket > shorter) return;
        in_shorter += double(elements) * lanes_spent(bucket, shorter);
        in_longer += double(elements) * lanes_spent(bucket, longer);
    };
    if (!buckets.per_layer)
        add(1, buckets.uniform);
    else
        for (int32_t l = 0; l < L; l++)
            if (bits[l] != 0 && off[l + 1] > off[l]) add(off[l + 1] - off[l], buckets.per_layer[l]);
    const int forced = launch_config().quantize_groups;
    const bool fills_longer = in_longer > 0.0 && in_shorter >= 1.24 * in_longer;
    if (long_elements > 0) {
        const bool apart = forced > 0 ? forced == 2 && short_elements > 0 : short_elements >= int64_t(3) << 25 && !fills_longer;
        return dt == CGX_F32 && apart ? Chunks{shorter, longer} : Chunks{longer, 0};
    }
    if (forced > 0) return {cgx::chunk_of(forced), 0};
    return {dt == CGX_F32 && !fills_longer ? shorter : longer, 0};
}

int draws_of(const cgx::TablePart &part) { return part.odd ? cgx::kDrawsOdd : part.quads ? cgx::kDrawsQuad : cgx::kDrawsEven; }

int tile_length(CallKind call, int dt, int64_t n)
{
    const int forced = launch_config().chunks_per_tile;
    if (forced > 0) return forced;
    if (call == kQuantizeCall && dt == CGX_F16 && n >= (int64_t(1) << 24)) return 2;
    if (call == kFusedCall && n >= (int64_t(1) << 27)) return 2;
    return 1;
}

bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Pointers (and chunks) that no check of a call can refuse.  Only such calls take the quick look-up of a table
// (known_plan): it asks the stream whether it captures and pins what it finds for a capture, and a call that is refused
// must leave both alone.
bool plain(const void *p) { return p && !misaligned(p); }
bool plain_chunks(const void *const *packed, const void *const *meta, int32_t W, int32_t most)
{
    if (W < 1 || W > most || !packed || !meta) return false;
    for (int32_t w = 0; w < W; w++)
        if (!plain(packed[w]) || !plain(meta[w])) return false;
    return true;
}

// A 64-bit digest of the plan's arrays, eight bytes at a time (multiply and xor-shift per word): a look-up
// compares this one word per cached plan and the arrays themselves only on a match.
uint64_t plan_digest(int32_t L, const int64_t *off, const uint8_t *bits, const int32_t *layer_buckets)
{
    uint64_t h = 0x9e3779b97f4a7c15ull ^ uint64_t(L);
    const auto mix = [&h](const void *p, size_t bytes) {
        const unsigned char *c = static_cast<const unsigned char *>(p);
        for (size_t i = 0; i < bytes; i += 8) {
            uint64_t w = 0;
            std::memcpy(&w, c + i, bytes - i < 8 ? bytes - i : 8);
            h = (h ^ w) * 0xff51afd7ed558ccdull;
            h ^= h >> 32;
        }
    };
    mix(off, sizeof(int64_t) * (size_t(L) + 1));
    mix(bits, size_t(L));
    if (layer_buckets) mix(layer_buckets, sizeof(int32_t) * size_t(L));
    return h;
}

// What identifies a tile table.
struct PlanKey {
    int32_t L;
    const int64_t *off;
    const uint8_t *bits;
    int32_t bucket;
    int dt;
    TableKind kind;
    const int32_t *layer_buckets;
    uint64_t digest;
};

// The cached table of a key, or nothing (g_mutex is held).  A table found during a stream capture is pinned, see get_plan.
PlanRef cached_plan(const PlanKey &k, int device, bool capturing, bool renew = true)
{
    for (const auto &p : g_plans) {
        if (p->digest == k.digest && p->device == device && p->bucket == k.bucket && p->dt == k.dt && p->kind == k.kind &&
            p->bits.size() == size_t(k.L) && p->layer_buckets.size() == (k.layer_buckets ? size_t(k.L) : 0) &&
            (!k.layer_buckets || k.L == 0 ||
             std::memcmp(p->layer_buckets.data(), k.layer_buckets, sizeof(int32_t) * size_t(k.L)) == 0) &&
            std::memcmp(p->bits.data(), k.bits, size_t(k.L)) == 0 &&
            std::memcmp(p->off.data(), k.off, sizeof(int64_t) * (size_t(k.L) + 1)) == 0) {
            if (renew) p->last_use = ++g_clock;
            if (capturing) p->pinned = true;
            return p;
        }
    }
    return nullptr;
}

bool is_capturing(hipStream_t stream)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool capturing = hipStreamIsCapturing(stream, &capture) == hipSuccess && capture == hipStreamCaptureStatusActive;
    if (!capturing) (void)hipGetLastError();       // a refused query (legacy stream beside a capture) is not this call's error
    return capturing;
}

// The table of a plan with one bucket size that an earlier call has checked and built, found by the arrays' contents;
// such a call needs neither the checks of the layer table nor its sizes again (2 us at 300 layers).  Nothing
// is found for arguments that those checks would refuse: tables exist for checked plans only, and 1-bit layers
// are left to them under the norm-and-sign quantizer.
// instead (may be null): a kind that the call prefers if the plan has both tables (it does not count as used then).
PlanRef known_plan(hipStream_t stream, int scheme, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits,
                   const Buckets &buckets, int dt, const TableKind &kind, const TableKind *instead = nullptr)
{
    // (what the checks find out without reading the arrays keeps them unread)
    if (buckets.per_layer || L <= 0 || n <= 0 || !off || !bits || (dt != CGX_F32 && dt != CGX_F16) || buckets.uniform < 32 ||
        buckets.uniform > 8192 || buckets.uniform % 32 || off[L] != n)
        return nullptr;
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return nullptr;
    PlanKey key{L, off, bits, buckets.uniform, dt, kind, nullptr, plan_digest(L, off, bits, nullptr)};
    const bool capturing = is_capturing(stream);
    std::lock_guard<std::mutex> lock(g_mutex);
    PlanRef plan = cached_plan(key, device, capturing);
    if (plan && scheme == cgx::kSchemeNormSign && plan->one_bit_layers) return nullptr;
    if (plan && instead) {
        key.kind = *instead;
        if (PlanRef other = cached_plan(key, device, capturing, false)) return other;
    }
    return plan;
}

// Finds or builds the device-resident tile table of a (valid) plan for a call on `stream`.
// A graph that is being captured keeps the raw table pointers of the launches recorded into it, so a table
// found during a capture is pinned for the life of the library (never the one dropped for a new plan),
// and a table that does not exist yet is not built during a capture (that would allocate and copy
// synchronously in the middle of it): the call fails with CGX_ERR_CAPTURE and records nothing.
// built (may be null): whether the table is a new one.
// spare: a table the call can do without.  It is built only where the cache has an entry left (else CGX_ERR_CAPACITY), and
// until a call looks it up for itself it is the first to be dropped: it never displaces a table in use.
int get_plan(hipStream_t stream, int32_t L, const int64_t *off, const uint8_t *bits, const Buckets &buckets, int dt,
             const TableKind &kind, PlanRef *out, bool *built = nullptr, bool spare = false)
{
    const int32_t bucket = buckets.uniform;
    const int32_t *layer_buckets = buckets.per_layer;
    const uint64_t digest = plan_digest(L, off, bits, layer_buckets);       // before the lock is taken
    std::lock_guard<std::mutex> lock(g_mutex);
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return CGX_ERR_HIP;
    const bool capturing = is_capturing(stream);
    *out = cached_plan(PlanKey{L, off, bits, bucket, dt, kind, layer_buckets, digest}, device, capturing, !spare);
    if (built) *built = !*out;
    if (*out) return CGX_OK;
    if (capturing) return CGX_ERR_CAPTURE;
    const bool full = std::count_if(g_plans.begin(), g_plans.end(), [](const auto &p) { return !p->pinned; }) >= kMaxPlans;
    if (spare && full) return CGX_ERR_CAPACITY;
    std::shared_ptr<CachedPlan> plan(new CachedPlan, [](CachedPlan *p) {
        free_plan(*p);
        delete p;
    });
    plan->digest = digest;
    plan->device = device;
    plan->bucket = bucket;
    plan->dt = dt;
    plan->kind = kind;
    plan->off.assign(off, off + L + 1);
    plan->bits.assign(bits, bits + L);
    if (layer_buckets) plan->layer_buckets.assign(layer_buckets, layer_buckets + L);
    plan->one_bit_layers = std::find(bits, bits + L, uint8_t(1)) != bits + L;
    plan->shape = cgx::plan_shape(L, off, bits, bucket, dt, layer_buckets);
    // (the statistics walk tables of the default chunk length in tiles of one chunk)
    const bool numbered = kind.chunk == cgx::kDefaultChunk && kind.chunks_per_tile == tile_length(kOtherCall, dt, off[L]);
    cgx::PlanTable table = cgx::build_table(L, off, bits, bucket, dt, kind.chunk, kind.chunks_per_tile, numbered, layer_buckets,
                                            kind.copy_tile, kind.long_chunk);
    if (table.tiles.size() > size_t(0xffffffffu) || table.stats_tiles > int64_t(0xffffffffu)) return CGX_ERR_SIZE;
    plan->n_tiles = int64_t(table.tiles.size());
    plan->stats_tiles = table.stats_tiles;
    const int64_t narrow = table.narrow(), wide = plan->n_tiles - narrow;
    const int pieces = table.pieces();
    if (pieces > 1 && wide * pieces >= cgx::kMostPieces) return CGX_ERR_SIZE;
    if (!upload(&plan->d_tiles, table.tiles) || !upload(&plan->d_slots, table.slots) ||
        !upload(&plan->d_layer_first, numbered ? table.layer_first : std::vector<int64_t>())) {
        free_plan(*plan);
        return CGX_ERR_HIP;
    }
    plan->reduce = cgx::ReduceTiles{plan->d_tiles, narrow + wide * pieces, uint32_t(narrow), uint32_t(pieces)};
    int64_t off_grid[4] = {0, 0, 0, 0};               // elements in tiles that start off 4, 8, 16, 32 elements
    for (const Tile &t : table.tiles)
        for (int k = 0; k < 4; k++) off_grid[k] += (t.elem0 & ((4 << k) - 1)) != 0 ? t.count : 0;
    plan->reduce.off_16_bytes[CGX_F32] = 2 * off_grid[0] > off[L];
    plan->reduce.off_16_bytes[CGX_F16] = 2 * off_grid[1] > off[L];
    plan->reduce.off_64_bytes[CGX_F32] = 2 * off_grid[2] > off[L];
    plan->reduce.off_64_bytes[CGX_F16] = 2 * off_grid[3] > off[L];
    plan->parts = std::move(table.parts);
    plan->last_use = spare ? 0 : ++g_clock;
    if (full) {
        // drop the least recently used table that no captured graph reads
        size_t oldest = g_plans.size();
        for (size_t i = 0; i < g_plans.size(); i++)
            if (!g_plans[i]->pinned && (oldest == g_plans.size() || g_plans[i]->last_use < g_plans[oldest]->last_use))
                oldest = i;
        if (oldest != g_plans.size()) g_plans.erase(g_plans.begin() + long(oldest));
    }
    *out = plan;
    g_plans.push_back(std::move(plan));
    return CGX_OK;
}

// Plan check of an entry point: the common rules, and for the norm-and-sign quantizer no
// 1-bit layers (a sign bit alone carries no level).
int check_plan(int scheme, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, const Buckets &buckets,
               int dt)
{
    int rc = cgx::validate_plan(n, L, off, bits, buckets.per_layer ? 32 : buckets.uniform, dt);
    if (rc != CGX_OK) return rc;
    if (buckets.per_layer) {
        rc = cgx::validate_layer_buckets(L, buckets.per_layer);
        if (rc != CGX_OK) return rc;
    }
    if (scheme == cgx::kSchemeNormSign)
        for (int32_t l = 0; l < L; l++)
            if (bits[l] == 1) return CGX_ERR_BITS;
    return CGX_OK;
}

int quantize_impl(int scheme, const void *grad, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits,
                  const Buckets &buckets, uint64_t seed, int dt, void *packed, void *meta, void *stream)
{
    const hipStream_t queue = static_cast<hipStream_t>(stream);
    const int per_tile = tile_length(kQuantizeCall, dt, n);
    PlanRef plan = !buckets.per_layer && plain(grad) && plain(packed) && plain(meta)
                       ? known_plan(queue, scheme, n, L, off, bits, buckets, dt, {quantize_chunks(dt, buckets, L, off, bits).chunk, per_tile})
                       : nullptr;
    cgx::PlanShape shape;
    if (plan) {
        shape = plan->shape;
    } else {
        const int rc = check_plan(scheme, n, L, off, bits, buckets, dt);
        if (rc != CGX_OK) return rc;
        if (n == 0) return CGX_OK;
        shape = cgx::plan_shape(L, off, bits, buckets.uniform, dt, buckets.per_layer);
    }
    if (!grad || !packed || (shape.meta_bytes && !meta)) return CGX_ERR_NULL;
    if (misaligned(grad) || misaligned(packed) || misaligned(meta)) return CGX_ERR_ALIGN;
    if (!plan) {
        const Chunks chunks = quantize_chunks(dt, buckets, L, off, bits);
        const int rc = get_plan(queue, L, off, bits, buckets, dt, {chunks.chunk, per_tile, cgx::kCopyPiece, chunks.long_chunk}, &plan);
        if (rc != CGX_OK) return rc;
    }
    for (const cgx::TablePart &part : plan->parts) {
        const auto launch_quantize = part.chunk == cgx::chunk_of(2) ? cgx::launch_quantize_g2 : cgx::launch_quantize_g4;
        const Tile *tiles = plan->d_tiles + part.first;
        const hipError_t e =
            cgx::mapping_of(part.bucket, part.chunk) == cgx::kMapWide
                ? cgx::launch_quantize_wide(scheme, grad, dt, tiles, part.count, draws_of(part), part.longest, seed, packed, meta,
                                            launch_config(), queue)
                : launch_quantize(scheme, grad, dt, tiles, part.count, draws_of(part), part.through_lds(), part.bucket, seed, packed, meta,
                                  launch_config(), queue);
        if (e != hipSuccess) return CGX_ERR_HIP;
    }
    return CGX_OK;
}

// Shared body of the dequantize / reduce entry points: out = [local +] deq_0 + ... + deq_{W-1}.
int reduce_impl(int scheme, const void *const *packed, const void *const *meta, int32_t W, int64_t n, int32_t L,
                const int64_t *off, const uint8_t *bits, const Buckets &buckets, int dt, const void *local,
                int local_dt, bool want_local, void *out, int out_dt, void *stream)
{
    // A decompression (one chunk, nothing to add to) writes eight bytes per byte it reads; a kernel that only
    // moves bytes in that mix sustains 0.75 of the HBM peak with 8 KB written per wave and 0.91 with 4 KB, so it
    // takes the kernel of 1024-element chunks (to binary16 2048 elements are 4 KB).
    const bool decompression = W == 1 && !want_local && launch_config().dequantize_through;
    const int forced = launch_config().reduce_groups;
    int chunk = forced > 0 ? cgx::chunk_of(forced)
                : decompression && out_dt == CGX_F32 ? cgx::chunk_of(2) : cgx::kDefaultChunk;
    const int per_tile = tile_length(kOtherCall, dt, n);
    const hipStream_t queue = static_cast<hipStream_t>(stream);
    PlanRef plan = plain_chunks(packed, meta, W, CGX_MAX_PEERS) && plain(out) && (!want_local || plain(local))
                       ? known_plan(queue, scheme, n, L, off, bits, buckets, dt, {chunk, per_tile})
                       : nullptr;
    if (!plan) {
        const int rc = check_plan(scheme, n, L, off, bits, buckets, dt);
        if (rc != CGX_OK) return rc;
    }
    if (W < 1 || W > CGX_MAX_PEERS) return CGX_ERR_PEERS;
    if (n == 0) return CGX_OK;
    const cgx::PlanShape shape =
        plan ? plan->shape : cgx::plan_shape(L, off, bits, buckets.uniform, dt, buckets.per_layer);
    if (!packed || !meta || !out || (want_local && !local)) return CGX_ERR_NULL;
    for (int w = 0; w < W; w++) {
        if (!packed[w] || (shape.meta_bytes && !meta[w])) return CGX_ERR_NULL;
        if (misaligned(packed[w]) || misaligned(meta[w])) return CGX_ERR_ALIGN;
    }
    if (misaligned(out) || misaligned(local)) return CGX_ERR_ALIGN;
    if (!plan) {
        bool built = false;
        int rc = get_plan(queue, L, off, bits, buckets, dt, {chunk, per_tile}, &plan, &built);
        // A decompression in chunks of 1024 elements must not need another table than its plan's other calls where a
        // program captures one of them after having run the other: under a capture it takes their table if its own does
        // not exist, and when it builds its own for a plan that is quantized in chunks of 2048, it builds theirs too.
        if (rc == CGX_ERR_CAPTURE && chunk != cgx::kDefaultChunk) {
            chunk = cgx::kDefaultChunk;
            rc = get_plan(queue, L, off, bits, buckets, dt, {chunk, per_tile}, &plan);
        } else if (rc == CGX_OK && built && chunk != cgx::kDefaultChunk &&
                   (buckets.per_layer || buckets.uniform > chunk ||
                    (dt == CGX_F32 && quantize_chunks(dt, buckets, L, off, bits).chunk != chunk))) {
            PlanRef others;                           // (this call does without it)
            if (get_plan(queue, L, off, bits, buckets, dt, {cgx::kDefaultChunk, per_tile}, &others) != CGX_OK) (void)hipGetLastError();
        }
        if (rc != CGX_OK) return rc;
    }
    const auto launch_reduce = chunk == cgx::kDefaultChunk ? cgx::launch_dequant_reduce_g4 : cgx::launch_dequant_reduce_g2;
    // peers are folded in order, kPeersPerLaunch at a time, so the sum order is local, 0, 1, ..., W-1;
    // a later launch starts from the binary32 result of the one before (W <= kPeersPerLaunch
    // whenever the output is not binary32: only cgx_dequantize asks for that, with W = 1)
    for (int w0 = 0; w0 < W; w0 += cgx::kPeersPerLaunch) {
        const int k = W - w0 < cgx::kPeersPerLaunch ? W - w0 : cgx::kPeersPerLaunch;
        cgx::PeerPtrs peers{};
        for (int i = 0; i < k; i++) {
            peers.packed[i] = static_cast<const uint8_t *>(packed[w0 + i]);
            peers.meta[i] = static_cast<const float *>(meta[w0 + i]);
        }
        const void *init = w0 == 0 ? local : out;
        const int init_dt = w0 == 0 ? local_dt : CGX_F32;
        // a result that fits the 256 MB memory-side cache with room to spare is left there for the
        // call that consumes it (requantize, the optimizer): measured on 102 MB of sums, the reduce
        // runs 7 % and the requantize after it 10 % faster; on 658 MB the reader loses what the
        // writer gains.  A decompression's stores go through at system scope whatever the size.
        const bool small = int64_t(n) * (out_dt == CGX_F16 ? 2 : 4) <= launch_config().keep_sums_max_bytes;
        const int policy = decompression ? cgx::kStoreThrough : small ? cgx::kStoreKeep : cgx::kStoreStream;
        const hipError_t e = launch_reduce(scheme, peers, k, dt, plan->reduce, init, init_dt, out, out_dt, policy,
                                           launch_config(), queue);
        if (e != hipSuccess) return CGX_ERR_HIP;
    }
    return CGX_OK;
}

// Most elements of a fused call in chunks of 1024 elements: what chunks of 2048 would give two waves on each of 1024 SIMDs.
constexpr int64_t kMostShortFused = int64_t(4) << 20;

int fused_impl(int scheme, const void *const *packed, const void *const *meta, int32_t W, int64_t n, int32_t L,
               const int64_t *layer_offsets, const uint8_t *bits_per_layer, const Buckets &buckets, int dt,
               uint64_t seed, void *packed_out, void *meta_out, void *stream)
{
    const hipStream_t queue = static_cast<hipStream_t>(stream);
    // Chunks of 1024 elements (7 waves per SIMD, 71 registers) where chunks of 2048 (4 waves, 121 registers) would leave half of the
    // wave slots empty and keep the others twice as long.  us with chunks of 2048 and of 1024: 8 peers, 4 bits, buckets of 512, 2.1 M
    // elements 8.1 and 7.2, 4.2 M 10.0 and 9.0; 7 peers, 2 bits, buckets of 992, 2.1 M 8.8 and 7.6.  Beyond, it depends on widths and
    // sizes: 5.2 M, 7 peers, 992, 2 and 8 bits 10.8 and 11.1, 12.0 and 12.4, 4 bits 11.7 and 11.4; 8 peers of 6.3 M at 4 bits 12.0 and
    // 11.0, 16 peers of 6.3 M in buckets of 96 23.1 and 18.7, 10 M 14.6 and 15.4, 67 M 75.0 and 81.5 (the scales and meta that a wave pays per chunk).
    // The table is the binary32 quantizer's, and a bucket size
    // that it lays over chunks of 2048 stays with them here (binary16 chunks too: they would need a table of their own).
    // The plan's tables stay those of chunks of 2048: they are looked up, built and renewed whichever this call walks, so that a
    // reduction or a statistic can be captured after it.  The other one is a spare (see get_plan): a program whose plans fill the
    // cache keeps the tables it would have without it, and its fused calls walk those.
    const TableKind usual{cgx::kDefaultChunk, tile_length(kFusedCall, dt, n)}, brief{cgx::chunk_of(2), usual.chunks_per_tile};
    const bool shorter = dt == CGX_F32 && !buckets.per_layer && n <= kMostShortFused &&
                         quantize_chunks(dt, buckets, L, layer_offsets, bits_per_layer).chunk == brief.chunk;
    // tables of the chunks and of the output, which lays out its pass-through layers as binary32
    PlanRef in, out;
    if (plain_chunks(packed, meta, W, CGX_MAX_FUSED_PEERS) && plain(packed_out) && plain(meta_out)) {
        in = known_plan(queue, scheme, n, L, layer_offsets, bits_per_layer, buckets, dt, usual, shorter ? &brief : nullptr);
        out = dt == CGX_F32 || !in ? in
                                   : known_plan(queue, scheme, n, L, layer_offsets, bits_per_layer, buckets, CGX_F32, usual);
    }
    const bool known = in && out;
    if (!known) {
        const int rc = check_plan(scheme, n, L, layer_offsets, bits_per_layer, buckets, dt);
        if (rc != CGX_OK) return rc;
    }
    if (W < 1 || W > CGX_MAX_FUSED_PEERS) return CGX_ERR_PEERS;
    if (n == 0) return CGX_OK;
    const cgx::PlanShape shape =
        known ? in->shape : cgx::plan_shape(L, layer_offsets, bits_per_layer, buckets.uniform, dt, buckets.per_layer);
    if (!packed || !meta || !packed_out || (shape.meta_bytes && !meta_out)) return CGX_ERR_NULL;
    for (int w = 0; w < W; w++) {
        if (!packed[w] || (shape.meta_bytes && !meta[w])) return CGX_ERR_NULL;
        if (misaligned(packed[w]) || misaligned(meta[w])) return CGX_ERR_ALIGN;
    }
    if (misaligned(packed_out) || misaligned(meta_out)) return CGX_ERR_ALIGN;
    cgx::PeerPtrs peers{};
    for (int i = 0; i < W; i++) {
        peers.packed[i] = static_cast<const uint8_t *>(packed[i]);
        peers.meta[i] = static_cast<const float *>(meta[i]);
    }
    if (!known) {
        int rc = get_plan(queue, L, layer_offsets, bits_per_layer, buckets, dt, usual, &in);
        if (shorter) {
            PlanRef other;                            // (a captured call may find the quantizer's table alone)
            const int spare = get_plan(queue, L, layer_offsets, bits_per_layer, buckets, dt, brief, &other, nullptr, true);
            if (rc == CGX_ERR_HIP || spare == CGX_ERR_HIP) (void)hipGetLastError();
            if (spare == CGX_OK) {
                in = other;
                rc = CGX_OK;
            }
        }
        if (rc != CGX_OK) return rc;
        out = in;
        if (dt != CGX_F32) rc = get_plan(queue, L, layer_offsets, bits_per_layer, buckets, CGX_F32, usual, &out);
        if (rc != CGX_OK) return rc;
    }
    if (in->n_tiles != out->n_tiles) return CGX_ERR_SIZE;     // cannot happen: same tiling for both layouts
    const auto launch_fused = in->kind.chunk == cgx::kDefaultChunk ? cgx::launch_dequant_reduce_requantize_g4
                                                                    : cgx::launch_dequant_reduce_requantize_g2;
    for (const cgx::TablePart &part : in->parts) {
        const Tile *tiles_in = in->d_tiles + part.first, *tiles_out = out->d_tiles + part.first;
        const hipError_t e =
            cgx::mapping_of(part.bucket, part.chunk) == cgx::kMapWide
                ? cgx::launch_dequant_reduce_requantize_wide(scheme, peers, W, dt, tiles_in, tiles_out, part.count, draws_of(part),
                                                             part.longest, seed, packed_out, meta_out, launch_config(), queue)
                : launch_fused(scheme, peers, W, dt, tiles_in, tiles_out, part.count, draws_of(part), seed, packed_out, meta_out,
                               launch_config(), queue);
        if (e != hipSuccess) return CGX_ERR_HIP;
    }
    return CGX_OK;
}

// Number of tiles (= doubles of workspace) of the plan the statistics walk; bits == nullptr:
// the all-pass-through plan cgx_layer_sqnorms uses.
int stats_tiles(int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int dt,
                int64_t *n_tiles)
{
    std::vector<uint8_t> zeros;
    if (!bits) {
        zeros.assign(size_t(L > 0 ? L : 0), 0);
        bits = zeros.data();
        bucket = 32;
    }
    const int rc = cgx::validate_plan(n, L, off, bits, bucket, dt);
    if (rc != CGX_OK) return rc;
    std::vector<Tile> tiles;
    cgx::build_tiles(L, off, bits, bucket, dt, cgx::kDefaultChunk, tile_length(kOtherCall, dt, n), tiles);
    *n_tiles = int64_t(tiles.size());
    return CGX_OK;
}

int sqerrors_impl(int scheme, const void *grad, const void *packed, const void *meta, int64_t n, int32_t L,
                  const int64_t *off, const uint8_t *bits, const Buckets &buckets, int dt, double *sqerr,
                  void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_plan(scheme, n, L, off, bits, buckets, dt);
    if (rc != CGX_OK) return rc;
    if (L == 0) return CGX_OK;
    const cgx::PlanShape shape = cgx::plan_shape(L, off, bits, buckets.uniform, dt, buckets.per_layer);
    if (!sqerr || (n > 0 && (!grad || !packed || !workspace)) || (shape.meta_bytes && !meta)) return CGX_ERR_NULL;
    if (misaligned(grad) || misaligned(packed) || misaligned(meta) || misaligned(workspace) ||
        (reinterpret_cast<uintptr_t>(sqerr) & 7u))
        return CGX_ERR_ALIGN;
    // every launch leaves its tiles' partial sums in the workspace; the last one adds them up layer by layer
    PlanRef plan;
    rc = get_plan(static_cast<hipStream_t>(stream), L, off, bits, buckets, dt,
                  {cgx::kDefaultChunk, tile_length(kOtherCall, dt, n)}, &plan);
    if (rc != CGX_OK) return rc;
    if (workspace_bytes < size_t(plan->stats_tiles) * sizeof(double)) return CGX_ERR_SIZE;
    for (const cgx::TablePart &part : plan->parts) {
        const hipError_t e = cgx::launch_layer_sqerrors(
            scheme, grad, dt, packed, meta, plan->d_tiles + part.first, plan->d_slots + part.first, part.count, part.aligned,
            plan->d_layer_first, L, static_cast<double *>(workspace), sqerr, launch_config(), static_cast<hipStream_t>(stream),
            &part == &plan->parts.back());
        if (e != hipSuccess) return CGX_ERR_HIP;
    }
    return CGX_OK;
}

}  // namespace

extern "C" {

int cgx_sizes(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket,
              cgx_dtype dt, size_t *packed_bytes, size_t *meta_bytes)
{
    const int rc = cgx::validate_plan(n, L, layer_offsets, bits_per_layer, bucket, int(dt));
    if (rc != CGX_OK) return rc;
    const cgx::PlanShape s = cgx::plan_shape(L, layer_offsets, bits_per_layer, bucket, int(dt));
    if (packed_bytes) *packed_bytes = s.packed_bytes;
    if (meta_bytes) *meta_bytes = s.meta_bytes;
    return CGX_OK;
}

int cgx_quantize(const void *grad, int64_t n, int32_t L, const int64_t *layer_offsets,
                 const uint8_t *bits_per_layer, int32_t bucket, uint64_t seed, cgx_dtype dt, void *packed,
                 void *meta, void *stream)
{
    return quantize_impl(cgx::kSchemeMinMax, grad, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, seed, int(dt), packed, meta, stream);
}

int cgx_requantize(const float *sum, int64_t n, int32_t L, const int64_t *layer_offsets,
                   const uint8_t *bits_per_layer, int32_t bucket, uint64_t seed, void *packed, void *meta,
                   void *stream)
{
    return quantize_impl(cgx::kSchemeMinMax, sum, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, seed, CGX_F32, packed, meta, stream);
}

int cgx_dequant_reduce(const void *const *packed, const void *const *meta, int32_t W, int64_t n, int32_t L,
                       const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket, cgx_dtype dt,
                       float *sum, void *stream)
{
    return reduce_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt), nullptr, CGX_F32,
                       false, sum, CGX_F32, stream);
}

int cgx_dequant_reduce_add(const void *local, cgx_dtype local_dt, const void *const *packed,
                           const void *const *meta, int32_t W, int64_t n, int32_t L,
                           const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket,
                           cgx_dtype dt, float *sum, void *stream)
{
    if (local_dt != CGX_F32 && local_dt != CGX_F16) return CGX_ERR_DTYPE;
    return reduce_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt), local, int(local_dt),
                       true, sum, CGX_F32, stream);
}

int cgx_dequantize(const void *packed, const void *meta, int64_t n, int32_t L, const int64_t *layer_offsets,
                   const uint8_t *bits_per_layer, int32_t bucket, cgx_dtype dt, cgx_dtype out_dt, void *out,
                   void *stream)
{
    if (out_dt != CGX_F32 && out_dt != CGX_F16) return CGX_ERR_DTYPE;
    const void *const p[1] = {packed}, *const m[1] = {meta};
    return reduce_impl(cgx::kSchemeMinMax, p, m, 1, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt), nullptr, CGX_F32, false, out,
                       int(out_dt), stream);
}

int cgx_dequant_reduce_requantize(const void *const *packed, const void *const *meta, int32_t W, int64_t n,
                                  int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                  int32_t bucket, cgx_dtype dt, uint64_t seed, void *packed_out, void *meta_out,
                                  void *stream)
{
    return fused_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt), seed,
                      packed_out, meta_out, stream);
}

int cgx_layered_sizes(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                      const int32_t *buckets_per_layer, cgx_dtype dt, size_t *packed_bytes, size_t *meta_bytes)
{
    const int rc = check_plan(cgx::kSchemeMinMax, n, L, layer_offsets, bits_per_layer, Buckets{32, buckets_per_layer},
                              int(dt));
    if (rc != CGX_OK) return rc;
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    const cgx::PlanShape s = cgx::plan_shape(L, layer_offsets, bits_per_layer, 32, int(dt), buckets_per_layer);
    if (packed_bytes) *packed_bytes = s.packed_bytes;
    if (meta_bytes) *meta_bytes = s.meta_bytes;
    return CGX_OK;
}

int cgx_layered_quantize(const void *grad, int64_t n, int32_t L, const int64_t *layer_offsets,
                         const uint8_t *bits_per_layer, const int32_t *buckets_per_layer, uint64_t seed,
                         cgx_dtype dt, void *packed, void *meta, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return quantize_impl(cgx::kSchemeMinMax, grad, n, L, layer_offsets, bits_per_layer, Buckets{32, buckets_per_layer},
                         seed, int(dt), packed, meta, stream);
}

int cgx_layered_requantize(const float *sum, int64_t n, int32_t L, const int64_t *layer_offsets,
                           const uint8_t *bits_per_layer, const int32_t *buckets_per_layer, uint64_t seed,
                           void *packed, void *meta, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return quantize_impl(cgx::kSchemeMinMax, sum, n, L, layer_offsets, bits_per_layer, Buckets{32, buckets_per_layer},
                         seed, CGX_F32, packed, meta, stream);
}

int cgx_layered_dequant_reduce(const void *const *packed, const void *const *meta, int32_t W, int64_t n, int32_t L,
                               const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                               const int32_t *buckets_per_layer, cgx_dtype dt, float *sum, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return reduce_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer,
                       Buckets{32, buckets_per_layer}, int(dt), nullptr, CGX_F32, false, sum, CGX_F32, stream);
}

int cgx_layered_dequant_reduce_add(const void *local, cgx_dtype local_dt, const void *const *packed,
                                   const void *const *meta, int32_t W, int64_t n, int32_t L,
                                   const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                   const int32_t *buckets_per_layer, cgx_dtype dt, float *sum, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    if (local_dt != CGX_F32 && local_dt != CGX_F16) return CGX_ERR_DTYPE;
    return reduce_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer,
                       Buckets{32, buckets_per_layer}, int(dt), local, int(local_dt), true, sum, CGX_F32, stream);
}

int cgx_layered_dequantize(const void *packed, const void *meta, int64_t n, int32_t L, const int64_t *layer_offsets,
                           const uint8_t *bits_per_layer, const int32_t *buckets_per_layer, cgx_dtype dt,
                           cgx_dtype out_dt, void *out, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    if (out_dt != CGX_F32 && out_dt != CGX_F16) return CGX_ERR_DTYPE;
    const void *const p[1] = {packed}, *const m[1] = {meta};
    return reduce_impl(cgx::kSchemeMinMax, p, m, 1, n, L, layer_offsets, bits_per_layer, Buckets{32, buckets_per_layer},
                       int(dt), nullptr, CGX_F32, false, out, int(out_dt), stream);
}

int cgx_layered_dequant_reduce_requantize(const void *const *packed, const void *const *meta, int32_t W, int64_t n,
                                          int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                          const int32_t *buckets_per_layer, cgx_dtype dt, uint64_t seed,
                                          void *packed_out, void *meta_out, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return fused_impl(cgx::kSchemeMinMax, packed, meta, W, n, L, layer_offsets, bits_per_layer,
                      Buckets{32, buckets_per_layer}, int(dt), seed, packed_out, meta_out, stream);
}

int cgx_layered_stats_workspace(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                const int32_t *buckets_per_layer, cgx_dtype dt, size_t *bytes)
{
    if (!bytes || (L > 0 && !buckets_per_layer)) return CGX_ERR_NULL;
    const Buckets buckets{32, buckets_per_layer};
    const int rc = check_plan(cgx::kSchemeMinMax, n, L, layer_offsets, bits_per_layer, buckets, int(dt));
    if (rc != CGX_OK) return rc;
    *bytes = size_t(cgx::build_table(L, layer_offsets, bits_per_layer, 32, int(dt), cgx::kDefaultChunk,
                                     tile_length(kOtherCall, int(dt), n), false, buckets_per_layer)
                        .stats_tiles) * sizeof(double);
    return CGX_OK;
}

int cgx_layered_layer_sqerrors(const void *grad, const void *packed, const void *meta, int64_t n, int32_t L,
                               const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                               const int32_t *buckets_per_layer, cgx_dtype dt, double *sqerr, void *workspace,
                               size_t workspace_bytes, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return sqerrors_impl(cgx::kSchemeMinMax, grad, packed, meta, n, L, layer_offsets, bits_per_layer,
                         Buckets{32, buckets_per_layer}, int(dt), sqerr, workspace, workspace_bytes, stream);
}

int cgx_qsgd_sizes(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                   int32_t bucket, cgx_dtype dt, size_t *packed_bytes, size_t *meta_bytes)
{
    const int rc = check_plan(cgx::kSchemeNormSign, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt));
    if (rc != CGX_OK) return rc;
    const cgx::PlanShape s = cgx::plan_shape(L, layer_offsets, bits_per_layer, bucket, int(dt));
    if (packed_bytes) *packed_bytes = s.packed_bytes;
    if (meta_bytes) *meta_bytes = s.meta_bytes / 2;            // one float per bucket
    return CGX_OK;
}

int cgx_qsgd_quantize(const void *grad, int64_t n, int32_t L, const int64_t *layer_offsets,
                      const uint8_t *bits_per_layer, int32_t bucket, uint64_t seed, cgx_dtype dt, void *packed,
                      void *meta, void *stream)
{
    return quantize_impl(cgx::kSchemeNormSign, grad, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, seed, int(dt),
                         packed, meta, stream);
}

int cgx_qsgd_dequant_reduce(const void *const *packed, const void *const *meta, int32_t W, int64_t n, int32_t L,
                            const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket,
                            cgx_dtype dt, float *sum, void *stream)
{
    return reduce_impl(cgx::kSchemeNormSign, packed, meta, W, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt),
                       nullptr, CGX_F32, false, sum, CGX_F32, stream);
}

int cgx_qsgd_dequant_reduce_requantize(const void *const *packed, const void *const *meta, int32_t W, int64_t n,
                                       int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                       int32_t bucket, cgx_dtype dt, uint64_t seed, void *packed_out,
                                       void *meta_out, void *stream)
{
    return fused_impl(cgx::kSchemeNormSign, packed, meta, W, n, L, layer_offsets, bits_per_layer, Buckets{bucket, nullptr}, int(dt),
                      seed, packed_out, meta_out, stream);
}

int cgx_qsgd_layered_sizes(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                           const int32_t *buckets_per_layer, cgx_dtype dt, size_t *packed_bytes, size_t *meta_bytes)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    const int rc = check_plan(cgx::kSchemeNormSign, n, L, layer_offsets, bits_per_layer, Buckets{32, buckets_per_layer},
                              int(dt));
    if (rc != CGX_OK) return rc;
    const cgx::PlanShape s = cgx::plan_shape(L, layer_offsets, bits_per_layer, 32, int(dt), buckets_per_layer);
    if (packed_bytes) *packed_bytes = s.packed_bytes;
    if (meta_bytes) *meta_bytes = s.meta_bytes / 2;
    return CGX_OK;
}

int cgx_qsgd_layered_quantize(const void *grad, int64_t n, int32_t L, const int64_t *layer_offsets,
                              const uint8_t *bits_per_layer, const int32_t *buckets_per_layer, uint64_t seed,
                              cgx_dtype dt, void *packed, void *meta, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return quantize_impl(cgx::kSchemeNormSign, grad, n, L, layer_offsets, bits_per_layer,
                         Buckets{32, buckets_per_layer}, seed, int(dt), packed, meta, stream);
}

int cgx_qsgd_layered_dequant_reduce(const void *const *packed, const void *const *meta, int32_t W, int64_t n,
                                    int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                                    const int32_t *buckets_per_layer, cgx_dtype dt, float *sum, void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return reduce_impl(cgx::kSchemeNormSign, packed, meta, W, n, L, layer_offsets, bits_per_layer,
                       Buckets{32, buckets_per_layer}, int(dt), nullptr, CGX_F32, false, sum, CGX_F32, stream);
}

int cgx_qsgd_layered_dequant_reduce_requantize(const void *const *packed, const void *const *meta, int32_t W,
                                               int64_t n, int32_t L, const int64_t *layer_offsets,
                                               const uint8_t *bits_per_layer, const int32_t *buckets_per_layer,
                                               cgx_dtype dt, uint64_t seed, void *packed_out, void *meta_out,
                                               void *stream)
{
    if (L > 0 && !buckets_per_layer) return CGX_ERR_NULL;
    return fused_impl(cgx::kSchemeNormSign, packed, meta, W, n, L, layer_offsets, bits_per_layer,
                      Buckets{32, buckets_per_layer}, int(dt), seed, packed_out, meta_out, stream);
}

int cgx_layer_stats_workspace(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                              int32_t bucket, cgx_dtype dt, size_t *bytes)
{
    if (!bytes) return CGX_ERR_NULL;
    int64_t n_tiles = 0;
    const int rc = stats_tiles(n, L, layer_offsets, bits_per_layer, bucket, int(dt), &n_tiles);
    if (rc != CGX_OK) return rc;
    *bytes = size_t(n_tiles) * sizeof(double);
    return CGX_OK;
}

int cgx_layer_sqnorms(const void *buf, int64_t n, int32_t L, const int64_t *layer_offsets, cgx_dtype dt,
                      double *sqnorm, void *workspace, size_t workspace_bytes, void *stream)
{
    const std::vector<uint8_t> zeros(size_t(L > 0 ? L : 0), 0);
    int rc = cgx::validate_plan(n, L, layer_offsets, zeros.data(), 32, int(dt));
    if (rc != CGX_OK) return rc;
    if (L == 0) return CGX_OK;
    if (!sqnorm || (n > 0 && (!buf || !workspace))) return CGX_ERR_NULL;
    if (misaligned(buf) || misaligned(workspace) || (reinterpret_cast<uintptr_t>(sqnorm) & 7u)) return CGX_ERR_ALIGN;
    PlanRef plan;
    rc = get_plan(static_cast<hipStream_t>(stream), L, layer_offsets, zeros.data(), Buckets{32, nullptr}, int(dt),
                  {cgx::kDefaultChunk, tile_length(kOtherCall, int(dt), n), cgx::kCopyTile}, &plan);
    if (rc != CGX_OK) return rc;
    if (workspace_bytes < size_t(plan->stats_tiles) * sizeof(double)) return CGX_ERR_SIZE;
    const hipError_t e = cgx::launch_layer_sqnorms(buf, int(dt), plan->d_tiles, plan->d_slots, plan->n_tiles,
                                                   plan->d_layer_first, L, static_cast<double *>(workspace), sqnorm,
                                                   launch_config(), static_cast<hipStream_t>(stream));
    return e == hipSuccess ? CGX_OK : CGX_ERR_HIP;
}

int cgx_layer_sqnorms_noalloc(const void *buf, int64_t n, int32_t L, const int64_t *layer_offsets, cgx_dtype dt,
                              double *sqnorm, void *stream)
{
    // the checks of validate_plan that concern the layer table (this call has no widths), without
    // the heap: nothing here allocates
    if (n < 0 || L < 0) return CGX_ERR_SIZE;
    if (L > 0 && !layer_offsets) return CGX_ERR_NULL;
    if (dt != CGX_F32 && dt != CGX_F16) return CGX_ERR_DTYPE;
    if (L == 0) return n == 0 ? CGX_OK : CGX_ERR_SIZE;
    if (layer_offsets[0] != 0) return CGX_ERR_OFFSETS;
    for (int32_t l = 0; l < L; l++)
        if (layer_offsets[l + 1] < layer_offsets[l]) return CGX_ERR_OFFSETS;
    if (layer_offsets[L] != n || n / 32 > int64_t(0xfffffff0u)) return CGX_ERR_SIZE;
    if (L > CGX_NOALLOC_MAX_LAYERS) return CGX_ERR_CAPACITY;
    // number of each layer's first work item: runs of kCopyTile elements, layer by layer
    static thread_local int64_t first[CGX_NOALLOC_MAX_LAYERS + 1];
    first[0] = 0;
    for (int32_t l = 0; l < L; l++)
        first[l + 1] = first[l] + (layer_offsets[l + 1] - layer_offsets[l] + cgx::kCopyTile - 1) / cgx::kCopyTile;
    if (first[L] > CGX_NOALLOC_MAX_TILES) return CGX_ERR_CAPACITY;
    if (!sqnorm || (n > 0 && !buf)) return CGX_ERR_NULL;
    if (misaligned(buf) || (reinterpret_cast<uintptr_t>(sqnorm) & 7u)) return CGX_ERR_ALIGN;
    const hipError_t e = cgx::launch_layer_sqnorms_noalloc(buf, int(dt), layer_offsets, first, L, sqnorm,
                                                           static_cast<hipStream_t>(stream));
    return e == hipSuccess ? CGX_OK : CGX_ERR_HIP;
}

int cgx_layer_sqerrors(const void *grad, const void *packed, const void *meta, int64_t n, int32_t L,
                       const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket, cgx_dtype dt,
                       double *sqerr, void *workspace, size_t workspace_bytes, void *stream)
{
    return sqerrors_impl(cgx::kSchemeMinMax, grad, packed, meta, n, L, layer_offsets, bits_per_layer,
                         Buckets{bucket, nullptr}, int(dt), sqerr, workspace, workspace_bytes, stream);
}

int cgx_qsgd_layer_sqerrors(const void *grad, const void *packed, const void *meta, int64_t n, int32_t L,
                            const int64_t *layer_offsets, const uint8_t *bits_per_layer, int32_t bucket,
                            cgx_dtype dt, double *sqerr, void *workspace, size_t workspace_bytes, void *stream)
{
    return sqerrors_impl(cgx::kSchemeNormSign, grad, packed, meta, n, L, layer_offsets, bits_per_layer,
                         Buckets{bucket, nullptr}, int(dt), sqerr, workspace, workspace_bytes, stream);
}

int cgx_plan_tiles(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                   int32_t bucket, cgx_dtype dt, void *tiles_out, int64_t capacity, int64_t *n_tiles)
{
    return cgx_plan_tiles_chunk(n, L, layer_offsets, bits_per_layer, bucket, dt, cgx::kDefaultChunk, tiles_out, capacity,
                                n_tiles);
}

int cgx_plan_tiles_chunk(int64_t n, int32_t L, const int64_t *layer_offsets, const uint8_t *bits_per_layer,
                         int32_t bucket, cgx_dtype dt, int32_t chunk_elements, void *tiles_out, int64_t capacity,
                         int64_t *n_tiles)
{
    const int rc = cgx::validate_plan(n, L, layer_offsets, bits_per_layer, bucket, int(dt));
    if (rc != CGX_OK) return rc;
    if (chunk_elements != cgx::chunk_of(2) && chunk_elements != cgx::chunk_of(4)) return CGX_ERR_SIZE;
    if (!n_tiles || (capacity > 0 && !tiles_out)) return CGX_ERR_NULL;
    std::vector<Tile> tiles;
    cgx::build_tiles(L, layer_offsets, bits_per_layer, bucket, int(dt), chunk_elements, 1, tiles);
    *n_tiles = int64_t(tiles.size());
    const int64_t k = capacity < *n_tiles ? capacity : *n_tiles;
    if (k > 0) std::memcpy(tiles_out, tiles.data(), size_t(k) * sizeof(Tile));
    return CGX_OK;
}

int cgx_stream_probe_shaped(const void *src, size_t read_bytes, void *dst, size_t write_bytes,
                            const cgx_probe_shape *shape, void *stream)
{
    if (!shape || (read_bytes && !src) || (write_bytes && !dst)) return CGX_ERR_NULL;
    if (read_bytes % 16 || write_bytes % 16) return CGX_ERR_SIZE;
    if (misaligned(src) || misaligned(dst)) return CGX_ERR_ALIGN;
    const int32_t s = shape->slice_bytes, t = shape->block_threads;
    if (s < 1024 || s > (1 << 20) || (s & (s - 1)) || (t != 64 && t != 128 && t != 256 && t != 512 && t != 1024) ||
        shape->load_policy < 0 || shape->load_policy > 3 || shape->store_policy < 0 || shape->store_policy > 4 ||
        (shape->xcd_contiguous != 0 && shape->xcd_contiguous != 1) || shape->max_blocks < 0 ||
        (shape->paired_loads != 0 && shape->paired_loads != 1) || shape->alu_ops_per_pass < 0 ||
        shape->alu_ops_per_pass > 65536 || shape->lds_bytes_per_block < 0 || shape->lds_bytes_per_block > 65536)
        return CGX_ERR_SIZE;
    cgx::ProbeShape k;
    k.slice_bytes = s;
    k.block_threads = t;
    k.load_policy = shape->load_policy;
    k.store_policy = shape->store_policy;
    k.xcd_contiguous = shape->xcd_contiguous;
    k.max_blocks = shape->max_blocks;
    k.paired_loads = shape->paired_loads;
    k.alu_ops_per_pass = shape->alu_ops_per_pass;
    k.lds_bytes_per_block = shape->lds_bytes_per_block;
    const hipError_t e = cgx::launch_stream_probe(src, read_bytes, dst, write_bytes, k, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? CGX_OK : CGX_ERR_HIP;
}

int cgx_stream_probe(const void *src, size_t read_bytes, void *dst, size_t write_bytes, void *stream)
{
    const cgx_probe_shape shape = {8192, 256, 1, 1, 0, 0, 0, 0, 0};      // the kernels' own style
    return cgx_stream_probe_shaped(src, read_bytes, dst, write_bytes, &shape, stream);
}

const char *cgx_issue_probe_form(int32_t form) { return cgx::issue_probe_form(form); }

int cgx_issue_probe(int32_t form, int32_t blocks, int32_t iterations, void *out, size_t out_bytes, void *stream)
{
    if (!out) return CGX_ERR_NULL;
    if (!cgx::issue_probe_form(form) || blocks < 1 || blocks > 65536 || iterations < 1 || iterations > (1 << 20) ||
        out_bytes < size_t(blocks) * 256 * 4)
        return CGX_ERR_SIZE;
    if (misaligned(out)) return CGX_ERR_ALIGN;
    const hipError_t e = cgx::launch_issue_probe(form, blocks, iterations, out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? CGX_OK : CGX_ERR_HIP;
}

const char *cgx_status_string(int status)
{
    switch (status) {
    case CGX_OK: return "ok";
    case CGX_ERR_NULL: return "a required pointer is NULL";
    case CGX_ERR_SIZE: return "n or L is negative, too large, or n does not match layer_offsets[L]";
    case CGX_ERR_OFFSETS: return "layer_offsets must start at 0 and never decrease";
    case CGX_ERR_BITS: return "bits_per_layer entries must be 0 (pass-through) or 1..8 (2..8 for the cgx_qsgd_ calls)";
    case CGX_ERR_BUCKET: return "bucket must be a multiple of 32 in [32, 8192]";
    case CGX_ERR_PEERS: return "W must be in [1, 64]";
    case CGX_ERR_DTYPE: return "unknown storage type";
    case CGX_ERR_HIP: return "the HIP runtime reported an error";
    case CGX_ERR_ALIGN: return "device pointers must be 16-byte aligned";
    case CGX_ERR_CAPTURE: return "the stream is capturing a graph and this plan's tables do not exist yet: run the call "
                                 "once outside the capture first";
    case CGX_ERR_CAPACITY: return "the plan exceeds the fixed tables of a no-allocation entry point "
                                  "(CGX_NOALLOC_MAX_LAYERS layers, CGX_NOALLOC_MAX_TILES work items)";
    default: return "unknown status";
    }
}

int cgx_shutdown(void)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    int rc = CGX_OK;
    // the tables go away with their last owner; hipFree waits for work that still reads them
    g_plans.clear();
    return rc;
}

}  // extern "C"
