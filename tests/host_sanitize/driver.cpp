// Host-only exerciser for a build with -fsanitize=address,undefined: the plan code of the library
// (validation, sizes, tile tables), its bit-width assigners, and the CPU oracle, on plans with every
// kind of layer.  Any out-of-bounds access, overflow or misaligned access aborts the run; the
// invariants checked here make it fail with a message.  Test infrastructure: links the oracle.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../include/cgx.h"
#include "../../paper_2111_08617_amd/csrc/cgx_plan.h"

extern "C" {
int oracle_sizes(int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int32_t dt,
                 uint64_t *packed_bytes, uint64_t *meta_bytes);
int oracle_quantize(const void *grad, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket,
                    uint64_t seed, int32_t dt, uint8_t *packed, float *meta);
int oracle_dequant_reduce(const uint8_t *const *packed, const float *const *meta, int32_t W, int64_t n, int32_t L,
                          const int64_t *off, const uint8_t *bits, int32_t bucket, int32_t dt, float *sum32,
                          double *sum64, double *abs64);
int oracle_unpack_codes(const uint8_t *packed, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits,
                        int32_t bucket, int32_t dt, uint8_t *codes);
int oracle_qsgd_sizes(int64_t n, int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int32_t dt,
                      uint64_t *packed_bytes, uint64_t *meta_bytes);
int oracle_qsgd_quantize(const void *grad, int64_t n, int32_t L, const int64_t *off, const uint8_t *bits,
                         int32_t bucket, uint64_t seed, int32_t dt, uint8_t *packed, float *meta);
int oracle_qsgd_dequant_reduce(const uint8_t *const *packed, const float *const *meta, int32_t W, int64_t n,
                               int32_t L, const int64_t *off, const uint8_t *bits, int32_t bucket, int32_t dt,
                               float *sum32, double *sum64, double *abs64);
void oracle_float_to_half(const float *in, int64_t count, uint16_t *out);
int oracle_layer_sqnorms(const void *buf, int64_t n, int32_t L, const int64_t *off, int32_t dt, double *out);
}

#define CHECK(cond)                                                                 \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                           \
        }                                                                           \
    } while (0)

struct Plan {
    std::vector<int64_t> off;
    std::vector<uint8_t> bits;
    int64_t n() const { return off.back(); }
    int32_t L() const { return int32_t(bits.size()); }
};

static Plan edge_plan(int bucket, std::mt19937 &rng)
{
    // every width, pass-through layers, empty layers, layers shorter than a bucket, ragged ends, whole
    // chunks, layers that start on odd elements
    const int sizes[] = {5000, 37, 0, 64, 4096 + 13, 1, 8 * bucket, 2 * bucket + 31, 1000, 3, 12345, 777, 2048, 8192 * 2, 1024};
    const int widths[] = {4, 0, 3, 2, 8, 5, 1, 3, 0, 4, 6, 7, 2, 4, 8};
    Plan p;
    p.off.push_back(0);
    for (size_t i = 0; i < sizeof(sizes) / sizeof(sizes[0]); i++) {
        p.off.push_back(p.off.back() + sizes[i] + int(rng() % 3 == 0));
        p.bits.push_back(uint8_t(widths[i]));
    }
    return p;
}

static void check_tiles(const Plan &p, int bucket, int dt, int chunk, int chunks_per_tile, const int32_t *layer_buckets)
{
    using namespace cgx;
    CHECK(validate_plan(p.n(), p.L(), p.off.data(), p.bits.data(), bucket, dt) == CGX_OK);
    const PlanShape shape = plan_shape(p.L(), p.off.data(), p.bits.data(), bucket, dt, layer_buckets);
    std::vector<int> covered(size_t(p.n()), 0);
    // a plan with a bucket size per layer takes one table per lane mapping in use
    const int classes[3] = {32, 128, 8192};
    size_t total_tiles = 0;
    for (int c = 0; c < (layer_buckets ? 3 : 1); c++) {
        const int launch_bucket = layer_buckets ? classes[c] : bucket;
        if (layer_buckets && mapping_of(launch_bucket, chunk) != c + (c == 0 ? 1 : c == 1 ? -1 : 0)) continue;
        std::vector<Tile> tiles;
        std::vector<uint32_t> slots;
        std::vector<int64_t> first;
        build_tiles(p.L(), p.off.data(), p.bits.data(), launch_bucket, dt, chunk, chunks_per_tile, tiles, &slots, &first,
                    layer_buckets, c == 0);
        CHECK(slots.size() == tiles.size() && first.size() == size_t(p.L()) + 1);
        total_tiles += tiles.size();
        std::vector<char> slot_used(tiles.size(), 0);
        for (size_t t = 0; t < tiles.size(); t++) {
            const Tile &tile = tiles[t];
            CHECK(tile.count > 0 && tile.elem0 >= 0 && tile.elem0 + tile.count <= p.n());
            for (uint32_t j = 0; j < tile.count; j++) covered[size_t(tile.elem0 + j)]++;
            const uint32_t b = tile_bits(tile);
            const uint64_t payload = b ? (uint64_t(tile.count) * b + 7) / 8 : uint64_t(tile.count) * (dt == CGX_F16 ? 2 : 4);
            CHECK(tile.packed_off >= 0 && uint64_t(tile.packed_off) + payload + tile.pad <= shape.packed_bytes);
            if (b) {
                const int own = tile_bucket(tile);
                CHECK(own >= 32 && own % 32 == 0);
                CHECK(uint64_t(tile.bucket0) + (tile.count + own - 1) / own <= shape.n_buckets);
                if (is_vector_kind(tile_kind(tile))) CHECK(tile.count % uint32_t(chunk) == 0 || tile_kind(tile) == kQuantWide);
            }
            CHECK(slots[t] < tiles.size() && !slot_used[slots[t]]);
            slot_used[slots[t]] = 1;
        }
    }
    CHECK(total_tiles > 0);
    for (int64_t i = 0; i < p.n(); i++) CHECK(covered[size_t(i)] == 1);    // the tables together: every element once
}

// The table that the entry points build and every call of a plan walks: its parts, the numbering of the statistics, and the
// pieces of a reduction (by the arithmetic that the kernel runs).
static void check_table(const Plan &p, int bucket, int dt, int chunk, int chunks_per_tile, const int32_t *layer_buckets, int copy_tile,
                        int long_chunk = 0)
{
    using namespace cgx;
    const PlanShape shape = plan_shape(p.L(), p.off.data(), p.bits.data(), bucket, dt, layer_buckets);
    const PlanTable table = build_table(p.L(), p.off.data(), p.bits.data(), bucket, dt, chunk, chunks_per_tile, true, layer_buckets,
                                        copy_tile, long_chunk);
    const auto own_bucket = [&](size_t l) { return layer_buckets ? layer_buckets[l] : bucket; };
    // where every layer's segment of the stream and its first bucket lie
    std::vector<uint64_t> segment(size_t(p.L()) + 1), first_bucket(size_t(p.L()) + 1);
    for (size_t l = 0; l < p.bits.size(); l++) {
        const uint64_t len = uint64_t(p.off[l + 1] - p.off[l]), b = p.bits[l];
        segment[l + 1] = segment[l] + ((b ? (len * b + 7) / 8 : len * (dt == CGX_F16 ? 2 : 4)) + 15) / 16 * 16;
        first_bucket[l + 1] = first_bucket[l] + (b ? (len + own_bucket(l) - 1) / own_bucket(l) : 0);
    }
    CHECK(segment.back() == shape.packed_bytes && first_bucket.back() == shape.n_buckets);
    std::vector<int> covered(size_t(p.n()), 0);
    const auto check_tile = [&](const Tile &tile, bool whole) {
        CHECK(tile.count > 0 && tile.elem0 >= 0 && tile.elem0 + tile.count <= p.n());
        for (uint32_t j = 0; j < tile.count; j++) covered[size_t(tile.elem0 + j)]++;
        size_t l = 0;
        while (p.off[l + 1] <= tile.elem0) l++;
        CHECK(tile.elem0 + tile.count <= p.off[l + 1] && tile_bits(tile) == p.bits[l]);
        const uint64_t in_layer = uint64_t(tile.elem0 - p.off[l]), b = p.bits[l];
        const uint64_t at = segment[l] + (b ? in_layer * b / 8 : in_layer * (dt == CGX_F16 ? 2 : 4));
        const uint64_t payload = b ? (uint64_t(tile.count) * b + 7) / 8 : uint64_t(tile.count) * (dt == CGX_F16 ? 2 : 4);
        CHECK(uint64_t(tile.packed_off) == at && (!b || in_layer * b % 8 == 0));
        // zero padding behind the last tile of a layer and nowhere else
        if (whole) CHECK(tile.pad == (tile.elem0 + tile.count == p.off[l + 1] ? segment[l + 1] - at - payload : 0));
        if (b) {
            CHECK(tile_bucket(tile) == own_bucket(l) && tile.bucket0 == first_bucket[l] + in_layer / own_bucket(l));
            CHECK(!whole || in_layer % own_bucket(l) == 0);                 // whole buckets, from the first element of one on
        } else {
            CHECK(int(tile.count) <= copy_tile);
        }
        return l;
    };
    int64_t next = 0;
    for (size_t k = 0; k < table.parts.size(); k++) {
        const TablePart &part = table.parts[k];
        CHECK(part.first == next && (part.chunk == chunk || (part.chunk == long_chunk && part.bucket > chunk)));
        if (k > 0 && part.chunk == table.parts[k - 1].chunk)
            CHECK(mapping_of(part.bucket, part.chunk) > mapping_of(table.parts[k - 1].bucket, part.chunk));
        if (k > 0) CHECK(part.chunk >= table.parts[k - 1].chunk);
        next += part.count;
        bool odd = false, quads = true, aligned = true;
        for (int64_t t = part.first; t < part.first + part.count; t++) {
            const Tile &tile = table.tiles[size_t(t)];
            const size_t l = check_tile(tile, true);
            if (p.bits[l] == 0) {
                CHECK(k == 0);
                continue;
            }
            CHECK(mapping_of(own_bucket(l), part.chunk) == mapping_of(part.bucket, part.chunk));
            CHECK(own_bucket(l) >= part.bucket && own_bucket(l) <= part.longest);
            // a block of waves, or one wave, holds the tile
            if (mapping_of(part.bucket, part.chunk) == kMapWide) CHECK(int(tile.count) <= own_bucket(l));
            else CHECK(int(tile.count) <= (tile_kind(tile) == kQuantFast ? chunks_per_tile : 1) * part.chunk);
            if (long_chunk) CHECK((own_bucket(l) > chunk) == (part.chunk == long_chunk));
            odd |= tile.elem0 & 1;
            quads &= tile.elem0 % 8 == 0;
            if (is_vector_kind(tile_kind(tile))) aligned &= tile.elem0 * (dt == CGX_F16 ? 2 : 4) % 16 == 0;
        }
        CHECK(odd == part.odd && quads == part.quads && aligned == part.aligned);
    }
    CHECK(next == int64_t(table.tiles.size()));
    for (int c : covered) CHECK(c == 1);
    // one number per tile that carries a partial sum, a layer's numbers together and in the order of its elements
    CHECK(table.slots.size() == table.tiles.size() && table.layer_first.size() == size_t(p.L()) + 1 && table.layer_first[0] == 0);
    std::vector<int64_t> element(size_t(table.layer_first.back()), -1);
    int64_t stats = 0;
    for (size_t l = 0; l < p.bits.size(); l++)
        stats += p.bits[l] ? table.layer_first[l + 1] - table.layer_first[l] : (p.off[l + 1] - p.off[l] + kCopyTile - 1) / kCopyTile;
    CHECK(stats == table.stats_tiles && table.layer_first.back() <= stats);
    for (size_t t = 0; t < table.tiles.size(); t++) {
        size_t l = 0;
        while (p.off[l + 1] <= table.tiles[t].elem0) l++;
        if (p.bits[l] == 0 && copy_tile != kCopyTile) {
            CHECK(table.slots[t] == kNoSlot);
            continue;
        }
        CHECK(table.slots[t] >= table.layer_first[l] && table.slots[t] < table.layer_first[l + 1] && element[table.slots[t]] == -1);
        element[table.slots[t]] = table.tiles[t].elem0;
    }
    for (size_t s = 0; s < element.size(); s++) CHECK(element[s] >= 0 && (s == 0 || element[s] > element[s - 1]));
    if (long_chunk) return;                                                 // (no reduction walks such a table)
    // a reduction's pieces
    const int64_t narrow = table.narrow(), wide = int64_t(table.tiles.size()) - narrow;
    const uint32_t pieces = uint32_t(table.pieces()), inv = Piece::inverse(pieces);
    const uint32_t bound = pieces > 1 ? uint32_t(narrow) : 0xffffffffu;
    CHECK(pieces <= 8);
    std::fill(covered.begin(), covered.end(), 0);
    for (int64_t t = 0; t < narrow + wide * pieces; t++) {
        const Piece piece(t, bound, pieces, inv);
        CHECK(piece.tile >= 0 && piece.tile < int64_t(table.tiles.size()));
        Tile tile = table.tiles[size_t(piece.tile)];
        if (t >= int64_t(bound) && !piece.cut(tile, chunk)) continue;
        const size_t l = check_tile(tile, false);
        if (p.bits[l] == 0 || tile_kind(tile) == kQuantFast) continue;
        CHECK(int(tile.count) <= chunk);
        if (tile_kind(tile) == kQuantWide) CHECK(int(tile.count) == chunk);
        if (own_bucket(l) > chunk)                                          // no piece crosses a bucket
            CHECK((tile.elem0 - p.off[l]) / own_bucket(l) == (tile.elem0 + tile.count - 1 - p.off[l]) / own_bucket(l));
    }
    for (int c : covered) CHECK(c == 1);
}

// Which plans' chunks the quantizer fetches through LDS: all whose whole chunks start on 16 bytes, wherever on an even element
// their short tiles start.
static void check_through_lds()
{
    using namespace cgx;
    const struct {
        std::vector<int64_t> sizes;
        int dt;
        bool quads, through_lds;
    } plans[] = {{{204800, 8, 8, 204800}, CGX_F16, true, true},   {{204800, 4, 12, 204800}, CGX_F16, false, true},
                 {{204800, 4, 12, 204800}, CGX_F32, false, true}, {{204800, 3, 13, 204800}, CGX_F16, false, false},
                 {{204800, 4, 204800}, CGX_F16, false, false},    {{204800, 4, 204800}, CGX_F32, false, true}};
    for (const auto &plan : plans) {
        std::vector<int64_t> off(1, 0);
        for (int64_t size : plan.sizes) off.push_back(off.back() + size);
        const std::vector<uint8_t> bits(plan.sizes.size(), 4);
        const PlanTable table = build_table(int32_t(bits.size()), off.data(), bits.data(), 128, plan.dt, plan.dt == CGX_F16 ? 2048 : 1024, 1, false);
        CHECK(table.parts.size() == 1 && table.parts[0].quads == plan.quads && table.parts[0].through_lds() == plan.through_lds);
    }
}

static void check_piece_division(std::mt19937 &rng)
{
    for (uint32_t pieces = 2; pieces <= 8; pieces++)
        for (int k = 0; k < 200000; k++) {
            const int64_t u = k < 1000 ? k : k < 2000 ? cgx::kMostPieces - 1 - (k - 1000) : int64_t(rng() % uint64_t(cgx::kMostPieces));
            const cgx::Piece piece(u + 5, 5, pieces, cgx::Piece::inverse(pieces));
            CHECK(piece.tile == 5 + u / pieces && piece.piece == u % pieces);
        }
}

static void check_oracle(const Plan &p, int bucket, int dt, std::mt19937 &rng)
{
    std::normal_distribution<float> normal(0.0f, 1.0f);
    const int64_t n = p.n();
    std::vector<float> x(size_t(n) + 1);
    for (auto &v : x) v = normal(rng) * 0.01f;
    std::vector<uint16_t> h(size_t(n) + 1);
    oracle_float_to_half(x.data(), n, h.data());
    const void *grad = dt == CGX_F16 ? static_cast<const void *>(h.data()) : static_cast<const void *>(x.data());
    uint64_t pb = 0, mb = 0;
    CHECK(oracle_sizes(n, p.L(), p.off.data(), p.bits.data(), bucket, dt, &pb, &mb) == 0);
    const cgx::PlanShape shape = cgx::plan_shape(p.L(), p.off.data(), p.bits.data(), bucket, dt);
    CHECK(shape.packed_bytes == pb && shape.meta_bytes == mb);           // the library's sizes are the oracle's
    // exactly sized buffers: a write past the end is an error the sanitizer reports
    std::vector<std::vector<uint8_t>> packed(3, std::vector<uint8_t>(pb));
    std::vector<std::vector<float>> meta(3, std::vector<float>(mb / 4));
    const uint8_t *pp[3];
    const float *mp[3];
    for (int w = 0; w < 3; w++) {
        CHECK(oracle_quantize(grad, n, p.L(), p.off.data(), p.bits.data(), bucket, 100 + w, dt, packed[w].data(),
                              meta[w].data()) == 0);
        pp[w] = packed[w].data();
        mp[w] = meta[w].data();
    }
    std::vector<uint8_t> codes(static_cast<size_t>(n));
    CHECK(oracle_unpack_codes(pp[0], n, p.L(), p.off.data(), p.bits.data(), bucket, dt, codes.data()) == 0);
    for (int32_t l = 0; l < p.L(); l++)
        for (int64_t i = p.off[l]; i < p.off[l + 1]; i++)
            CHECK(p.bits[l] ? codes[size_t(i)] < (1u << p.bits[l]) : codes[size_t(i)] == 0xff);
    std::vector<float> s32(static_cast<size_t>(n));
    std::vector<double> s64(static_cast<size_t>(n)), a64(static_cast<size_t>(n));
    CHECK(oracle_dequant_reduce(pp, mp, 3, n, p.L(), p.off.data(), p.bits.data(), bucket, dt, s32.data(), s64.data(),
                                a64.data()) == 0);
    for (int64_t i = 0; i < n; i++) CHECK(std::fabs(double(s32[size_t(i)]) - s64[size_t(i)]) <= 1e-6 * a64[size_t(i)] + 1e-45);
    std::vector<double> sq(size_t(p.L()));
    CHECK(oracle_layer_sqnorms(grad, n, p.L(), p.off.data(), dt, sq.data()) == 0);
    // norm-and-sign form (no 1-bit layers)
    Plan q = p;
    for (auto &b : q.bits) b = b == 1 ? 2 : b;
    uint64_t qpb = 0, qmb = 0;
    CHECK(oracle_qsgd_sizes(n, q.L(), q.off.data(), q.bits.data(), bucket, dt, &qpb, &qmb) == 0);
    std::vector<uint8_t> qp(qpb);
    std::vector<float> qm(qmb / 4);
    CHECK(oracle_qsgd_quantize(grad, n, q.L(), q.off.data(), q.bits.data(), bucket, 7, dt, qp.data(), qm.data()) == 0);
    const uint8_t *qpp[1] = {qp.data()};
    const float *qmp[1] = {qm.data()};
    CHECK(oracle_qsgd_dequant_reduce(qpp, qmp, 1, n, q.L(), q.off.data(), q.bits.data(), bucket, dt, s32.data(),
                                     s64.data(), a64.data()) == 0);
}

static void check_assigners(const Plan &p, std::mt19937 &rng)
{
    std::uniform_real_distribution<double> uni(0.0, 10.0);
    std::vector<double> norms(size_t(p.L()));
    for (auto &v : norms) v = uni(rng);
    const uint8_t cands[4] = {8, 2, 4, 3};
    std::vector<uint8_t> out(size_t(p.L()), 0xee);
    for (int k = 1; k <= 4; k++) {
        CHECK(cgx_assign_bits_kmeans(p.L(), p.off.data(), norms.data(), p.bits.data(), cands, k, 50, out.data()) == CGX_OK);
        for (int32_t l = 0; l < p.L(); l++) {
            const bool takes_part = p.bits[l] != 0 && p.off[l + 1] > p.off[l];
            bool is_cand = false;
            for (int c = 0; c < k; c++) is_cand |= out[size_t(l)] == cands[c];
            CHECK(takes_part ? is_cand : out[size_t(l)] == 0);
        }
        CHECK(cgx_assign_bits_linear(p.L(), p.off.data(), norms.data(), p.bits.data(), cands, k, out.data()) == CGX_OK);
        const int32_t sizes[3] = {128, 1024, 4096};
        std::vector<int32_t> buckets(size_t(p.L()), -1);
        CHECK(cgx_assign_buckets_from_bits(p.L(), out.data(), cands, k, sizes, 3, buckets.data()) == CGX_OK);
        for (int32_t b : buckets) CHECK(b == 128 || b == 1024 || b == 4096);
    }
    CHECK(cgx_assign_bits_kmeans(p.L(), p.off.data(), norms.data(), p.bits.data(), cands, 0, 50, out.data()) == CGX_ERR_SIZE);
}

int main()
{
    std::mt19937 rng(12345);
    check_piece_division(rng);
    check_through_lds();
    const int buckets[] = {32, 64, 96, 128, 512, 1024, 2048, 4096, 8192, 8160};
    int plans = 0;
    for (int bucket : buckets) {
        const Plan p = edge_plan(bucket, rng);
        for (int dt : {int(CGX_F32), int(CGX_F16)}) {
            for (int chunk : {1024, 2048})
                for (int cpt : {1, 3}) {
                    check_tiles(p, bucket, dt, chunk, cpt, nullptr);
                    for (int copy_tile : {cgx::kCopyTile, cgx::kCopyPiece})
                        for (int b : {bucket, bucket + 32 <= 8192 ? bucket + 32 : 8000})
                            check_table(p, b, dt, chunk, cpt, nullptr, copy_tile);
                }
            check_oracle(p, bucket, dt, rng);
            plans++;
        }
        std::vector<int32_t> per_layer(size_t(p.L()));
        for (auto &b : per_layer) b = buckets[rng() % 10];
        CHECK(cgx::validate_layer_buckets(p.L(), per_layer.data()) == CGX_OK);
        for (int chunk : {1024, 2048}) {
            check_tiles(p, 32, CGX_F32, chunk, 1, per_layer.data());
            for (int dt : {int(CGX_F32), int(CGX_F16)}) check_table(p, 32, dt, chunk, 1, per_layer.data(), cgx::kCopyPiece);
        }
        check_table(p, 32, CGX_F32, 1024, 1, per_layer.data(), cgx::kCopyPiece, 2048);
        for (auto &b : per_layer) b = b > 1024 ? 1056 + 32 * int(rng() % 224) : 96 * (1 + int(rng() % 10));
        for (int chunk : {1024, 2048}) check_table(p, 32, CGX_F32, chunk, 1, per_layer.data(), cgx::kCopyPiece);
        check_table(p, 32, CGX_F32, 1024, 1, per_layer.data(), cgx::kCopyPiece, 2048);
        const Plan copies{p.off, std::vector<uint8_t>(p.bits.size(), 0)};
        check_table(copies, 32, CGX_F32, 2048, 1, per_layer.data(), cgx::kCopyPiece);
        check_table(copies, bucket, CGX_F16, 2048, 1, nullptr, cgx::kCopyTile);
        check_assigners(p, rng);
    }
    // rejected plans stay rejected without touching anything
    const int64_t bad_off[3] = {0, 10, 5};
    const uint8_t two_bits[2] = {4, 4};
    CHECK(cgx::validate_plan(5, 2, bad_off, two_bits, 128, CGX_F32) == CGX_ERR_OFFSETS);
    CHECK(cgx::validate_plan(5, 2, nullptr, two_bits, 128, CGX_F32) == CGX_ERR_NULL);
    std::printf("host sanitize driver: %d plans, all checks passed\n", plans);
    return 0;
}
