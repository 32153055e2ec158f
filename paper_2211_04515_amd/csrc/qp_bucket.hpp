// The directed search by value buckets (qp_search_bucket.hip): the plan that its set-up makes on the device, and the
// layout of its part of the workspace.
#pragma once

#include "qp_common.hpp"

namespace qp {

constexpr uint32_t kBkThreads = 1024;        // lanes of a sorting block
constexpr uint32_t kBkCands = 128;           // most candidates of a sweep
#ifndef QP_BUCKET_TILES
#define QP_BUCKET_TILES 256                  // sorting blocks that run side by side: one per compute unit
#endif
#ifndef QP_BUCKET_WIDTH
#define QP_BUCKET_WIDTH 1024                 // most buckets of a sign
#endif
#ifndef QP_BUCKET_SUM_BLOCKS
#define QP_BUCKET_SUM_BLOCKS 1024            // summing blocks: four per compute unit
#endif
// Senders of 9.7 M elements, t = 100, with 2^-8 / 2^-10 / 2^-12: Laplace data at 2 bit 116 / 113 / 226 us (too many binades for 256 buckets, left to the
// streaming kernel), 8 bit 135 / 144 / 145; lognormal data at 2 bit 157 / 144 / 141; after GELU, 4 bit 143 / 143 / 145.
#ifndef QP_BUCKET_DEPTH
#define QP_BUCKET_DEPTH 0x1p-10              // smallest element that has a bucket, as a share of |mean| + s_E
#endif
#ifndef QP_BUCKET_DENSE
#define QP_BUCKET_DENSE 5.0                  // one end of a dense sweep over the other: thresholds as many as at twice the coarser end
#endif
#ifndef QP_BUCKET_SEGMENT
#define QP_BUCKET_SEGMENT (1u << 24)         // elements that are sorted at a time (bounds the workspace: 67 MB)
#endif
constexpr uint32_t kBkTiles = QP_BUCKET_TILES, kBkWidth = QP_BUCKET_WIDTH, kBkSumBlocks = QP_BUCKET_SUM_BLOCKS;
constexpr uint32_t kBkColumns = kBkSumBlocks;                    // partial sums of a candidate per segment
constexpr uint32_t kBkRounds = 10;                               // 16-byte loads of a lane of a sorting block
constexpr uint32_t kBkTileMax = 37u * kBkThreads;                // elements of a tile: 148 KB of LDS
constexpr uint32_t kBkKeys = 2u * kBkWidth;                      // buckets of both signs
constexpr uint32_t kBkRow = kBkKeys + 4u;                        // table entries of a tile
// entries of one bucket's lists, and of those that one block makes
constexpr uint32_t kBkCutCap = 512, kBkOwnCap = 96, kBkPieceCap = 768;
constexpr uint32_t kBkCutAll = (1u << 19) / kBkTiles, kBkClassAll = (1u << 16) / kBkTiles, kBkPieceAll = (1u << 19) / kBkTiles;   // of one sorting block

// Elements of a sample, and most of them outside the buckets.  Those are scored one by one at about the streaming search's rate, so at
// 9.7 M elements, where the buckets save 98 us of 208 (2 bit) or 64 (8 bit), half to a third of a tensor uses that up: a fifth outside 177 / 198
// and 196 / 201 us.
constexpr uint32_t kBkSample = 1024, kBkSampleOut = 384;
struct BucketPlan {
    uint32_t unsuited;    // 1: the set-up leaves this tensor to the streaming kernel ...
    uint32_t fallback;    // ... or the sort does
    uint32_t shift;       // bits of an element's pattern below its bucket
    uint32_t first;       // |pattern| >> shift of bucket 0
    uint32_t width;       // buckets of a sign
    uint32_t centre;      // the bucket of the mean: every candidate has a threshold there, so its elements count as outside
    uint32_t uneven;      // 1: some tile has so many elements outside the buckets that all blocks share them
};
// An element's bucket; 2 width: outside.
__device__ __forceinline__ uint32_t bucket_key(const BucketPlan &p, float x)
{
    const uint32_t w = __float_as_uint(x), u = ((w & 0x7fffffffu) >> p.shift) - p.first;
    const uint32_t key = u + (w >> 31) * p.width;
    return u < p.width && key != p.centre ? key : 2u * p.width;
}
constexpr uint32_t kBkDirect = 12;    // most sums of a bucket that are formed in registers: each takes a share of the bucket 1 us, however small
// How the elements of a bucket are rounded for some candidates: r(x) = x / 2^k - frac to the nearest whole number, ties to the
// even (or to the odd) one.  With f = x - base, a whole multiple of the bucket's last place 2^a, 2^k (r(x) - r(base)) is
// ((f + add) + m) - m in 32 bits: add is what base / 2^k - frac is off r(base), in 2^k; m = 1.5 * 2^23 * 2^k or the next
// multiple of 2^k, so that the sum's last place is 2^k and ties go to r(x)'s parity.  Class 0 of every bucket leaves the elements as
// they are: add = m = 0, k = a.
struct BucketClass { float add, m, unit, pad; };     // unit = 2^-k
// A sum: of a class, over the elements with |f| >= from.
struct BucketSum { float from, add, m, unit; };
struct BucketRec {
    uint32_t cut, cls, piece;         // where the bucket's cuts, classes and further pieces start
    uint32_t ncut, ncls;
    uint32_t nsum;                    // sums that its pieces refer to; 0: summed by interval
    uint32_t pad[2];
    BucketSum sum[kBkDirect];
};
// A candidate's constant piece of a bucket: sum of 4^k (r(x) - r(base) + e)^2, k the bucket's last place + dk, over the elements
// from cut `from` on and before cut `to` (0: the bucket's start; kBkNone: its end; cuts count from 1).  Where the sums are formed in
// registers, from and to are places in BucketRec::sum.
struct BucketPiece { double e; uint8_t cls, dk; uint16_t from, to, next; };
static_assert(sizeof(BucketPiece) == 16 && sizeof(BucketRec) == 224 && sizeof(BucketClass) == 16 && sizeof(BucketSum) == 16, "layout");
constexpr uint32_t kBkNone = 0xffffu;

struct BucketLayout {
    uint32_t segments, tile, tiles;   // of the largest segment
    size_t plan, totals, recs, shapes, cuts, classes, pieces, further, table, partials, sorted, end;
};
inline BucketLayout bucket_layout(uint64_t n, size_t at)
{
    BucketLayout l;
    l.segments = ceil_div_u64(n, QP_BUCKET_SEGMENT);
    const uint64_t m = (n + l.segments - 1) / l.segments;
    const uint32_t rounds = ceil_div_u64(m, (uint64_t)kBkTiles * kBkTileMax);
    l.tile = (ceil_div_u64(m, (uint64_t)kBkTiles * rounds) + 3u) / 4u * 4u;
    l.tiles = ceil_div_u64(m, l.tile);
    auto take = [&](size_t bytes) { const size_t o = at; at += (bytes + 255) / 256 * 256; return o; };
    at = (at + 255) / 256 * 256;
    l.plan = take(sizeof(BucketPlan));
    l.totals = take((size_t)l.segments * kBkKeys * 4 + (size_t)l.segments * 4);   // the last words: zeros of a segment
    l.recs = take(kBkKeys * sizeof(BucketRec));
    l.shapes = take(kBkKeys * 4);
    l.cuts = take((size_t)kBkTiles * kBkCutAll * 4);
    l.classes = take((size_t)kBkTiles * kBkClassAll * sizeof(BucketClass));
    l.pieces = take((size_t)kBkKeys * kBkCands * sizeof(BucketPiece));
    l.further = take((size_t)kBkTiles * kBkPieceAll * sizeof(BucketPiece));
    l.table = take((size_t)l.tiles * kBkRow * 2);
    l.partials = take((size_t)kBkCands * kBkColumns * l.segments * 8);
    l.sorted = take(((size_t)l.tiles * l.tile + 4) * 4);
    l.end = at;
    return l;
}

struct BucketSetup {
    BucketPlan *plan;       // null: no such search follows
    uint32_t *totals;
    uint32_t words;         // of totals
    uint32_t width;         // most buckets of a sign ...
    uint32_t dense_width;   // ... of a dense sweep (see bucket_plan); 0: such a sweep is left to the streaming kernel
    const float *x;
    uint64_t n;
};

// One block, behind setup_candidates: where the buckets lie, and whether this tensor suits them.
// st: the tensor's statistics where they are on the device.
__device__ inline void bucket_plan(const BucketSetup &b, const GridModel &g, const qp_stats_t *st, int safe, const Cand *cands, uint32_t ncand)
{
    __shared__ BucketPlan sh_plan;
    __shared__ uint32_t sh_out[kFinThreads / kWave];
    __shared__ double sh_inv[kFinThreads / kWave];
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < b.words; i += blockDim.x) b.totals[i] = 0u;
    double inv = 0.0;
    if (tid < ncand && cands[tid].scale > 0.0f) inv = 1.0 / (double)cands[tid].scale;   // (the lane's own store, see setup_candidates)
    inv = wave_sum(inv);
    if (tid % kWave == 0) sh_inv[tid / kWave] = inv;
    __syncthreads();
    if (tid == 0) {
        for (uint32_t w = 1; w < (ncand + kWave - 1) / kWave; ++w) inv += sh_inv[w];
        // b_R far below b_E (after ReLU or GELU, by 10 to 20): most candidates' thresholds lie much closer than the first one's
        const bool dense = fmax(g.s_e, g.s_r) > QP_BUCKET_DENSE * fmin(g.s_e, g.s_r);
        const uint32_t width = dense && b.dense_width ? b.dense_width : b.width;
        // up to 16 s_E from the mean: with 8 / 16 / 32 of them Laplace data at 8 bit takes 137 / 144 / 145 us, lognormal data at 2 bit 145 / 144 / 141
        const double am = fabs(g.mean) + g.s_e, reach = 16.0 * g.s_e;
        const double lo = fmax(am * QP_BUCKET_DEPTH, fabs(g.mean) - reach), hi = fabs(g.mean) + reach;
        const uint32_t plo = __float_as_uint((float)lo), phi = __float_as_uint((float)hi);
        const bool ok = g.s_e > 0.0 && hi >= lo && plo >= (27u << 23) && phi <= (227u << 23);
        uint32_t shift = 8u;
        if (ok)
            while ((phi >> shift) - (plo >> shift) + 1u > width) ++shift;
        // thresholds that a typical bucket holds, all candidates together.  The lists have room for 512; nothing measured comes near 250 (190 the
        // most, after a GELU of N(0, 6^2) at 8 bit and t = 127, and that by buckets is faster: 197 / 242 us)
        const double cell = (double)__uint_as_float(__float_as_uint((float)am) & 0x7f800000u) * (double)(1u << shift) * 0x1p-23;
        BucketPlan p{};
        p.unsuited = (!ok || !safe || (dense && b.dense_width == 0u) || shift > 19u || !(inv * cell <= 250.0)) ? 1u : 0u;
        p.fallback = p.unsuited;
        p.shift = shift;
        p.first = plo >> shift;
        p.width = ok ? (phi >> shift) - (plo >> shift) + 1u : 1u;
        const uint32_t mean = __float_as_uint((float)g.mean), u = ((mean & 0x7fffffffu) >> shift) - p.first;
        p.centre = u < p.width ? u + (mean >> 31) * p.width : 0xffffffffu;
        sh_plan = p;
        *b.plan = p;
    }
    // The sort costs its time whatever becomes of it.  Elements outside the buckets (scored one by one) cluster at zero or the mean, in
    // one bin of the histogram; where that holds a quarter of the tensor a sample tells whether they are too many.
    if (st && 4ull * st->peak_count < b.n) return;
    __syncthreads();
    const BucketPlan p = sh_plan;
    uint32_t out = 0u;
    for (uint32_t i = tid; i < kBkSample; i += blockDim.x) {
        const float v = b.x[(uint64_t)(i * 2654435769u) * b.n >> 32];
        out += v != 0.0f && bucket_key(p, v) == 2u * p.width ? 1u : 0u;
    }
    out = wave_sum_u32(out);
    if (tid % kWave == 0) sh_out[tid / kWave] = out;
    __syncthreads();
    if (tid != 0) return;
    for (uint32_t w = 1; w < blockDim.x / kWave; ++w) out += sh_out[w];
    if (out > kBkSampleOut) b.plan->unsuited = b.plan->fallback = 1u;
}

// Whether such a search takes this call, given room in the workspace (the caller's business).
bool bucket_search_eligible(uint64_t n, int dtype, const SearchPlan &plan);
// Whether the search takes some bitwidth's call of these settings: whether a workspace should hold its part.
bool bucket_search_wanted(uint64_t n, uint32_t t_steps, uint32_t stride);
size_t bucket_search_end(uint64_t n, size_t at);   // bytes of a workspace with the search's part behind `at`
BucketSetup bucket_setup_args(const void *x, uint64_t n, const SearchPlan &plan, void *ws);
// Behind the set-up: sort, sum, pick.  *fallback (device) is 1 afterwards if nothing was scored.
hipError_t launch_bucket_search(const void *x, uint64_t n, const SearchPlan &plan, void *ws, const uint32_t **fallback, hipStream_t s);

}  // namespace qp
