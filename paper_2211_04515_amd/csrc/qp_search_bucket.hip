// Step 2b for large fp32 tensors at up to 8 bit: the DS-ACIQ directed search (Sec. 3, Eq. 1) by value buckets.
//
// Eq. 1 sums e^2 over the elements, e = fl(x - x^), x^ the value of x's level on the candidate's grid.  Scoring every
// element against every candidate is 24 clocks of vector ALU work per pair and wave (qp_search.hip).  But over a short run of
// values x^ is one constant, and if e keeps its binade there too, then fl(x - x^) moves with x alone: candidates whose x^ agree
// below e's last place round x alike, e = f + E with one f for all of them, and sum e^2 = sum f^2 + 2 E sum f + n E^2.
// So the tensor is sorted into buckets of neighbouring values (equal sign, exponent and leading bits of the mantissa) and a bucket
// keeps three sums (n, sum f, sum f^2) for each of the few ways f that its elements are rounded.  All f are whole multiples of
// the bucket's last place below 2^24 of it, so these sums are exact, whatever their order: the sort need not be stable, and
// the scores are those of the element-by-element sum with equal terms grouped, bit-reproducible.
//   k_bucket_sort   a block sorts one tile of the tensor by bucket in LDS and writes it back, with the tile's table of
//                   bucket starts; then it takes its share of the buckets and lists, for each, the pieces on which a
//                   candidate's x^ and e's binade are constant, and the sums that these pieces need;
//   k_bucket_sum    blocks gather a bucket's elements from the tiles, form its sums, and add each candidate's pieces;
//                   elements outside the buckets' range (0.1 to 2 % as a rule) are scored one by one;
//   k_search_pick   adds the blocks' partial sums and takes the first minimum, as for the tile search.
// A tensor that this does not suit is left to the streaming kernel, which is launched behind.  The set-up finds most of them (NaN or
// Inf, a grid that needs the full clamp sequence, too many elements outside the buckets: see bucket_plan): the call then takes 4 to 10
// us longer than without buckets.  Lists that outgrow their room are found by k_bucket_sort, whose time is then spent: 27 us at 4.3 M
// elements, 40 at 9.7 M, 100 at 30 M.
#include "qp_bucket.hpp"

namespace qp {

struct BucketArgs {
    const float *x;             // the segment
    uint64_t n;
    uint32_t tile, tiles, ncand;
    uint32_t first_segment;     // 1: the lists are still to be made
    BucketPlan *plan;
    uint32_t *totals;           // the segment's
    uint32_t *zeros;            // elements that are zero, the segment's
    uint16_t *table;
    float *sorted;
    const Cand *cands;
    BucketRec *recs;
    uint32_t *shapes;           // of a bucket: the weight of its sums; summed by interval: classes << 16 | cuts
    uint32_t *cuts;
    BucketClass *classes;
    BucketPiece *pieces;        // a candidate's first piece of a bucket
    BucketPiece *further;       // the others
    double *partials;           // the segment's first column
    uint32_t columns;           // of all segments
};

// ---- pieces ---------------------------------------------------------------------------------------

// A bucket: elements of one sign with patterns base .. base + 2^shift - 1.
struct BucketAt {
    uint32_t base, size;
    int a;                      // exponent of its last place
    __device__ float value(uint32_t d) const { return __uint_as_float(base + d); }
};
__device__ inline BucketAt bucket_at(const BucketPlan &p, uint32_t b)
{
    const uint32_t neg = b >= p.width ? 1u : 0u, u = b - neg * p.width;
    BucketAt t;
    t.base = ((p.first + u) << p.shift) | (neg << 31);
    t.size = 1u << p.shift;
    t.a = (int)((t.base >> 23) & 0xffu) - 150;
    return t;
}
__device__ inline double pow2(int e) { return __longlong_as_double((long long)(e + 1023) << 52); }   // -1022 <= e <= 1023
// exponent of the last place that fl32 gives a difference
__device__ inline int place_of(double e)
{
    const int x = (int)((uint32_t)__double2hiint(e) >> 20 & 0x7ffu) - 1046;
    return e == 0.0 ? -2000 : (x < -149 ? -149 : x);
}
__device__ inline int place_of_value(float v)
{
    const int x = (int)(__float_as_uint(v) >> 23 & 0xffu) - 150;
    return v == 0.0f ? 2000 : (x < -149 ? -149 : x);
}
__device__ __forceinline__ float bucket_level(const Cand &c, float x)
{
    const float xc = __builtin_amdgcn_fmed3f(x, c.lo, c.hi);
    const float d = xc - c.lo;
    return rintf(d * c.inv_scale);   // the short sequence: candidate_grid has shown that it needs no upper clamp
}

// What the sums cost, in tenths of a microsecond of a block of k_bucket_sum per batch of 4096 elements, with four blocks on a
// compute unit: measured as 3.5 to 4 us with one sum, 6.5 to 7 with five of class 0, 9.4 with five of four classes, 12 with nine;
// a class by interval 8 to 20, most of it the LDS atomics and more where few intervals hold most elements.  A few hundred elements take two thirds of a batch's sums.
__device__ __forceinline__ uint32_t sum_weight(const BucketSum &m)
{
    return m.m == 0.0f ? (m.from > 0.0f ? 9u : 7u) : m.from > 0.0f ? 14u : 11u;
}
// A bucket (one class of it) of n elements: what a share of it costs at least, and the whole.  shape: see BucketArgs.
__device__ __forceinline__ uint32_t bucket_least(uint32_t shape)
{
    const uint32_t low = shape & 0xffffu;
    return shape >> 16 ? 70u + low / 4u : 30u + low * 2u / 3u;
}
__device__ __forceinline__ uint32_t bucket_cost(uint32_t n, uint32_t shape)
{
    const uint32_t low = shape & 0xffffu, batches = n / 64u;   // in 1/64
    return shape >> 16 ? bucket_least(shape) + batches * 130u / 64u : max(bucket_least(shape), 30u + batches * (28u + low) / 64u);
}

// A value that the compiler must take as new: what it would otherwise work out early or once for all (addresses, 64-bit copies)
// costs the registers of a wave.
__device__ __forceinline__ void opaque(uint32_t &v)
{
#if defined(__AMDGCN__)
    asm volatile("" : "+v"(v));
#endif
}

// A bucket's lists while 128 lanes, one a candidate, fill them.
constexpr uint32_t kBkKeyed = 128;    // classes that candidates share: place - a < 32, parity, frac 0 or a half
constexpr uint32_t kBkAsIs = 255u;    // class 0
static_assert(kBkKeyed + kBkOwnCap < kBkAsIs, "a class is a byte");
struct BucketRounding { float frac; int k2; };   // k2 = 2 k + odd
struct alignas(16) BucketLists {
    uint32_t ncut, nown, npiece, over, wanted[kBkKeyed / kWave], need[2], weight;
    uint32_t cut[kBkCutCap];          // its place in the bucket << 9 | number, so that no two are equal
    uint16_t order[kBkCutCap];        // a cut's place among the sorted ones
    uint16_t keyed[kBkKeyed];         // 1: wanted; then its number
    uint32_t owner[kBkOwnCap];        // candidate << 20 | where in the bucket
    uint8_t own_place[kBkOwnCap], own_at[kBkOwnCap];   // by owner; and which one lies there
    BucketRounding own[kBkOwnCap];
    BucketPiece piece[kBkPieceCap];
};

__device__ inline double class_round(double x, double inv, double frac, double magic) { return (fma(x, inv, -frac) + magic) - magic; }

// A class from how it rounds; f + add needs at most 2 + max(19, k - a) + 1 <= 24 bits.
constexpr int kBkFurthest = 20;   // most of k - a
__device__ inline BucketClass bucket_class(const BucketAt &t, const BucketRounding &c)
{
    const int k = c.k2 >> 1;
    const double odd = (double)(c.k2 & 1), inv = pow2(-k), frac = (double)c.frac;
    const double base = (double)t.value(0), r = class_round(base, inv, frac, 0x1.8p52 + odd);   // r(base)
    const double parity = (r != 2.0 * floor(0.5 * r)) != (odd != 0.0) ? 1.0 : 0.0;
    return BucketClass{(float)((fma(base, inv, -r) - frac) * pow2(k)), (float)((0x1.8p23 + parity) * pow2(k)), (float)inv, 0.0f};
}

// All pieces of one candidate in one bucket.
__device__ inline void candidate_pieces(const BucketAt &t, const Cand &c, uint32_t j, BucketLists &l)
{
    const double sgn = (t.base >> 31) ? -1.0 : 1.0;
    const double unit = pow2(-t.a), base = (double)t.value(0), abase = fabs(base);
    const uint32_t last = t.size - 1u;
    const float r_end = bucket_level(c, t.value(last));
    uint32_t prev = kBkNone, cut_d = 0u, cut_ref = 0u;   // the piece before; the last cut
    bool over = false;
    auto cut = [&](uint32_t d) -> uint32_t {
        if (d == 0u) return 0u;
        if (d == t.size) return kBkNone;
        if (d == cut_d) return cut_ref;
        const uint32_t i = atomicAdd(&l.ncut, 1u);
        if (i >= kBkCutCap) { over = true; return 0u; }
        l.cut[i] = d << 9 | i;
        cut_d = d;
        cut_ref = i + 1u;
        return cut_ref;
    };
    auto emit = [&](double e, uint32_t cls, int dk, uint32_t from, uint32_t to) {
        const uint32_t cf = cut(from), ct = cut(to);
        uint32_t slot = j;
        if (prev != kBkNone) {
            slot = kBkCands + atomicAdd(&l.npiece, 1u);
            if (slot >= kBkPieceCap) { over = true; return; }
            l.piece[prev].next = (uint16_t)slot;
        }
        l.piece[slot] = BucketPiece{e, (uint8_t)cls, (uint8_t)dk, (uint16_t)cf, (uint16_t)ct, (uint16_t)kBkNone};
        prev = slot;
    };
    uint32_t from = 0u;
    while (from < t.size && !over) {
        const float r = bucket_level(c, t.value(from));
        uint32_t to = t.size;
        if (r != r_end) {
            // the level's end: bisection around where it lies but for a few roundings at the size of the range's ends
            auto same = [&](uint32_t d) { return bucket_level(c, t.value(d)) == r; };
            const double at = ((double)c.lo + ((double)r + 0.5 * sgn) * (double)c.scale) * sgn;
            const double g = fmin(fmax((at - abase) * unit, 0.0), (double)last);
            const double w = 8.0 * fmax(1.0, fmax(fabs((double)c.lo), fabs((double)c.hi)) * unit * 0x1p-23);
            uint32_t lo = g - w > (double)from ? (uint32_t)(g - w) : from, hi = g + w < (double)last ? (uint32_t)(g + w) : last;
            if (lo < from || !same(lo)) lo = from;
            if (hi <= lo || same(hi)) hi = last;
            while (hi - lo > 1u) {
                const uint32_t mid = lo + (hi - lo) / 2u;
                if (same(mid)) lo = mid;
                else hi = mid;
            }
            to = hi;
        }
        const float xh = dequant_level(r, c.scale, c.lo);
        const double xd = (double)xh;
        const int low = min(t.a, place_of_value(xh));
        while (from < to && !over) {
            const double e0 = (double)t.value(from) - xd, e1 = (double)t.value(to - 1u) - xd;
            const int k = place_of(e0), k1 = place_of(e1);
            // every x - x^ is a float: nothing is rounded
            if (max(k, k1) <= low) {
                emit((base - xd) * unit, kBkAsIs, 0, from, to);
                from = to;
                continue;
            }
            uint32_t end = to;
            if (k1 != k || (e0 < 0.0) != (e1 < 0.0)) {   // the end of e's binade: |x| = |x^| +- a power of two
                auto alike = [&](uint32_t d) {
                    const double e = (double)t.value(d) - xd;
                    return place_of(e) == k && (e < 0.0) == (e0 < 0.0);
                };
                const bool grows = (e0 < 0.0) == (sgn < 0.0);
                const double at = grows ? ceil((sgn * xd + pow2(k + 24) - abase) * unit) : floor((sgn * xd - pow2(k + 23) - abase) * unit) + 1.0;
                const uint32_t g = at > (double)from && at < (double)to ? (uint32_t)at : 0u;
                uint32_t lo = from, hi = to - 1u;
                if (g > lo && g <= hi) {
                    if (alike(g - 1u)) lo = g - 1u;
                    if (!alike(g)) hi = g;
                }
                while (hi - lo > 1u) {
                    const uint32_t mid = lo + (hi - lo) / 2u;
                    if (alike(mid)) lo = mid;
                    else hi = mid;
                }
                end = hi;
            }
            // one binade: e is a whole multiple of 2^k
            const double y = xd * pow2(-k), fl = floor(y);
            double frac = y - fl;
            if (k < t.a || (k == t.a && frac != 0.5)) {   // x is one too: x^ is rounded instead
                emit((base - rint(y) * pow2(k)) * unit, kBkAsIs, 0, from, end);
            } else {
                const uint32_t odd = fl != 2.0 * floor(0.5 * fl) ? 1u : 0u;
                const double magic = 0x1.8p52 + (double)odd;
                uint32_t cls;
                if (k - t.a < 32 && (frac == 0.0 || frac == 0.5)) {
                    cls = ((uint32_t)(k - t.a) * 2u + odd) * 2u + (frac == 0.5 ? 1u : 0u);
                    l.keyed[cls] = 1u;
                } else {
                    // its digits below the bucket's last place only say on which side of a multiple of half of that it lies
                    const double q = frac * pow2(k - t.a), below = floor(q), rest = q - below;
                    frac = (below + (rest == 0.0 ? 0.0 : rest < 0.5 ? 0.25 : rest == 0.5 ? 0.5 : 0.75)) * pow2(t.a - k);   // a float up to kBkFurthest
                    const uint32_t i = atomicAdd(&l.nown, 1u);
                    if (i >= kBkOwnCap) {
                        over = true;
                    } else {
                        l.own[i] = BucketRounding{(float)frac, 2 * k + (int)odd};
                        l.owner[i] = j << 20 | from;
                    }
                    cls = kBkKeyed + i;
                }
                if (k - t.a > kBkFurthest) over = true;
                emit(class_round(base, pow2(-k), (double)(float)frac, magic) - fl, cls, k - t.a, from, end);
            }
            from = end;
        }
    }
    if (over) l.over = 1u;
}

// The block's share of the buckets, eight at a time (128 lanes each, c the lane's candidate).  Its lists go to stretches of its own.
// The classes' order is that of the candidates, not of the atomics: where a bucket is summed by interval, a class's number says
// which block's sum takes it, and with that how the score is rounded.
__device__ inline void bucket_lists(const BucketArgs &a, const BucketPlan &p, const Cand &c, BucketLists *lists, uint32_t *used /* [3], shared */)
{
    const uint32_t tid = threadIdx.x, g = tid / kBkCands, j = tid % kBkCands;
    constexpr uint32_t groups = kBkThreads / kBkCands;
    static_assert(kBkKeyed == kBkCands, "a keyed class a lane");
    const uint32_t blocks = min(gridDim.x, kBkTiles);
    BucketLists &l = lists[g];
    const bool has = j < a.ncand;
    if (tid < 3u) used[tid] = 0u;
    for (uint32_t first = blockIdx.x; first < 2u * p.width; first += blocks * groups) {
        const uint32_t b = first + g * blocks;
        const bool live = b < 2u * p.width && b != p.centre;
        if (j == 0u) {
            l.ncut = l.nown = l.npiece = l.over = l.need[0] = l.need[1] = l.weight = 0u;
        }
        l.keyed[j] = 0u;
        __syncthreads();
        const BucketAt t = bucket_at(p, live ? b : 0u);
        auto keyed_class = [&](uint32_t i) { return BucketRounding{(i & 1u) ? 0.5f : 0.0f, 2 * (t.a + (int)(i >> 2)) + (int)((i >> 1) & 1u)}; };
        if (live && has) candidate_pieces(t, c, j, l);
        __syncthreads();
        const uint32_t nc = min(l.ncut, kBkCutCap), nown = min(l.nown, kBkOwnCap), np = min(l.npiece, kBkPieceCap - kBkCands);
        {   // the keyed classes' numbers: behind class 0, so far of each wave's lanes (kept in LDS, not in registers)
            const bool want = l.keyed[j] != 0u;
            const uint64_t wanted = __ballot(want);
            if (want) l.keyed[j] = (uint16_t)(1u + (uint32_t)__popcll(wanted & ((1ull << (j % kWave)) - 1ull)));
            if (j % kWave == 0u) l.wanted[j / kWave] = (uint32_t)__popcll(wanted);
        }
        if (j < 8u && nc + j < kBkCutCap) l.cut[nc + j] = 0xffffffffu;
        __syncthreads();
        // the cuts' order
        for (uint32_t i = j; i < nc; i += kBkCands) {
            const uint32_t d = l.cut[i];
            uint32_t below = 0u;
            for (uint32_t k = 0; k < nc; k += 8u) {   // (places past the end hold larger values)
                const uint4 u = *reinterpret_cast<const uint4 *>(&l.cut[k]), v = *reinterpret_cast<const uint4 *>(&l.cut[k + 4u]);
                below += (u.x < d ? 1u : 0u) + (u.y < d ? 1u : 0u) + (u.z < d ? 1u : 0u) + (u.w < d ? 1u : 0u) + (v.x < d ? 1u : 0u) +
                         (v.y < d ? 1u : 0u) + (v.z < d ? 1u : 0u) + (v.w < d ? 1u : 0u);
            }
            l.order[i] = (uint16_t)below;
        }
        for (uint32_t i = j; i < nown; i += kBkCands) {
            uint32_t me = i;
            opaque(me);
            const uint32_t o = l.owner[me];
            uint32_t below = 0u;
#pragma unroll 1
            for (uint32_t k = 0; k < nown; ++k) below += l.owner[k] < o ? 1u : 0u;
            l.own_place[me] = (uint8_t)below;
            l.own_at[below] = (uint8_t)me;
        }
        if (j >= (uint32_t)kWave && l.keyed[j]) l.keyed[j] += (uint16_t)l.wanted[0];
        const uint32_t shared = 1u + l.wanted[0] + l.wanted[1], ncls = shared + nown;
        __syncthreads();
        if (j == 0u) {   // (a dead group has a class and nothing else)
            l.ncut = atomicAdd(&used[0], nc);
            l.nown = atomicAdd(&used[1], ncls);
            l.npiece = atomicAdd(&used[2], np);
            if (l.ncut + nc > kBkCutAll || l.nown + ncls > kBkClassAll || l.npiece + np > kBkPieceAll) l.over = 1u;
            if (live && l.over) st_dev(&a.plan->fallback, 1u);
        }
        __syncthreads();
        const uint32_t at_cut = blockIdx.x * kBkCutAll + l.ncut, at_cls = blockIdx.x * kBkClassAll + l.nown, at_piece = blockIdx.x * kBkPieceAll + l.npiece;
        const bool few = ncls * (nc + 1u) <= 64u;
        if (live && !l.over) {
            for (uint32_t i = j; i < nc; i += kBkCands) a.cuts[at_cut + l.order[i]] = l.cut[i] >> 9;
            BucketClass *cls = a.classes + at_cls;
            if (j == 0u) cls[0] = BucketClass{0.0f, 0.0f, __uint_as_float((uint32_t)(127 - t.a) << 23), 0.0f};
            if (l.keyed[j]) cls[l.keyed[j]] = bucket_class(t, keyed_class(j));
            for (uint32_t i = j; i < nown; i += kBkCands) cls[shared + l.own_place[i]] = bucket_class(t, l.own[i]);
            for (uint32_t i = j; i < kBkCands + np; i += kBkCands) {
                if (i < kBkCands && !has) continue;
                BucketPiece &q = l.piece[i];
                q.cls = (uint8_t)(q.cls == kBkAsIs ? 0u : q.cls < kBkKeyed ? l.keyed[q.cls] : shared + l.own_place[q.cls - kBkKeyed]);
                if (q.from) q.from = (uint16_t)(l.order[q.from - 1u] + 1u);
                if (q.to != kBkNone) q.to = (uint16_t)(l.order[q.to - 1u] + 1u);
                if (few) {
                    const uint32_t s0 = q.cls * (nc + 1u) + q.from;
                    atomicOr(&l.need[s0 / 32u], 1u << (s0 % 32u));
                    if (q.to != kBkNone) {
                        const uint32_t s1 = q.cls * (nc + 1u) + q.to;
                        atomicOr(&l.need[s1 / 32u], 1u << (s1 % 32u));
                    }
                }
            }
        }
        __syncthreads();
        const uint64_t need = (uint64_t)l.need[0] | ((uint64_t)l.need[1] << 32);
        // a sum in registers costs 5 to 20, a class by interval 100 (bucket_cost)
        const uint32_t nsum = few && __popcll(need) <= (int)min(kBkDirect, 8u * ncls) ? (uint32_t)__popcll(need) : 0u;
        if (live && !l.over) {
            auto place = [&](uint32_t s) { return (uint16_t)__popcll(need & ((1ull << s) - 1ull)); };
            for (uint32_t i = j; i < kBkCands + np; i += kBkCands) {
                if (i < kBkCands && !has) continue;
                BucketPiece q = l.piece[i];
                if (nsum) {
                    q.from = place(q.cls * (nc + 1u) + q.from);
                    if (q.to != kBkNone) q.to = place(q.cls * (nc + 1u) + q.to);
                }
                if (i < kBkCands) a.pieces[(uint64_t)b * kBkCands + i] = q;
                else a.further[at_piece + i - kBkCands] = q;
            }
            BucketRec &r = a.recs[b];
            if (nsum && j < 64u && (need >> j & 1ull)) {
                const uint32_t k = j / (nc + 1u), cut = j % (nc + 1u);
                BucketSum m{0.0f, 0.0f, 0.0f, __uint_as_float((uint32_t)(127 - t.a) << 23)};
                for (uint32_t i = 0; i < nc; ++i)
                    if (cut == (uint32_t)l.order[i] + 1u) m.from = fabsf(t.value(l.cut[i] >> 9) - t.value(0));   // exact: one binade
                if (k) {
                    BucketRounding how{0.0f, 0};
                    if (k >= shared) how = l.own[l.own_at[k - shared]];
                    else
                        for (uint32_t i = 0; i < kBkKeyed; ++i)
                            if (l.keyed[i] == k) how = keyed_class(i);
                    const BucketClass c = bucket_class(t, how);
                    m.add = c.add;
                    m.m = c.m;
                    m.unit = c.unit;
                }
                r.sum[place(j)] = m;
                atomicAdd(&l.weight, sum_weight(m));
            }
            if (j == 0u) {
                r.cut = at_cut;
                r.cls = at_cls;
                r.piece = at_piece;
                r.ncut = nc;
                r.ncls = ncls;
                r.nsum = nsum;
            }
        }
        __syncthreads();   // the lists are reused
        if (live && j == 0u && !l.over) a.shapes[b] = nsum ? l.weight : ncls << 16 | nc;
    }
}

// ---- sort -------------------------------------------------------------------------------------------

constexpr uint32_t kBkEarly = 7u;   // loads of a lane before the lists: their registers are held meanwhile

__global__ __launch_bounds__(kBkThreads) void k_bucket_sort(BucketArgs a)
{
    __shared__ __align__(16) float sx[kBkTileMax];
    __shared__ uint32_t cnt[kBkKeys];
    __shared__ uint32_t sh_wave[kBkThreads / kWave], sh_other[kBkThreads / kWave], sh_zero[kBkThreads / kWave];
    __shared__ uint32_t sh_bad;
    static_assert(sizeof(BucketLists) * (kBkThreads / kBkCands) <= sizeof(sx), "the lists are staged where the tile was");
    if (a.plan->unsuited) return;   // (`fallback` may change while this kernel runs)
    const BucketPlan p = *a.plan;
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const uint64_t e0 = (uint64_t)blockIdx.x * a.tile;
    const uint32_t m = (uint32_t)min((uint64_t)a.tile, a.n - e0);   // elements of this tile
    const uint32_t quads = (m + 3u) / 4u;

    // much of the tile is requested before anything else but the candidates, and the lists are made while it is on its way
    const bool listing = a.first_segment && blockIdx.x < kBkTiles;
    Cand c{0.0f, 0.0f, 0.0f, 0.0f};
    if (listing && tid % kBkCands < a.ncand) c = a.cands[tid % kBkCands];
    float v[kBkRounds][4];
    auto request = [&](uint32_t i) {
        const uint32_t q = i * kBkThreads + tid;
        if (4u * q + 4u <= m) {
            Vec4<QP_F32>::load(a.x + e0, q, v[i]);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) v[i][k] = 4u * q + k < m ? a.x[e0 + 4u * q + k] : 0.0f;   // zeros are not kept
        }
    };
#pragma unroll
    for (uint32_t i = 0; i < kBkEarly; ++i) request(i);
    if (listing) bucket_lists(a, p, c, reinterpret_cast<BucketLists *>(sx), sh_wave);
#pragma unroll
    for (uint32_t i = kBkEarly; i < kBkRounds; ++i) request(i);
    for (uint32_t i = tid; i < kBkKeys; i += kBkThreads) cnt[i] = 0u;
    if (tid == 0) sh_bad = 0u;
    __syncthreads();

    // an element's place in its bucket (any order), or among the wave's elements outside the buckets (in a fixed order: those
    // are scored one by one, and their sum depends on it)
    auto key_of = [&](float x) -> uint32_t {   // as bucket_key, whose inlining here costs two spilled registers
        const uint32_t w = __float_as_uint(x), u = ((w & 0x7fffffffu) >> p.shift) - p.first;
        const uint32_t key = u + (w >> 31) * p.width;
        return u < p.width && key != p.centre ? key : 2u * p.width;
    };
    uint32_t rank[kBkRounds][2];
    uint32_t wother = 0u, wzero = 0u, bad = 0u;
#pragma unroll
    for (uint32_t i = 0; i < kBkRounds; ++i) {
        if (i * kBkThreads < quads) {
            uint32_t r[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t key = key_of(v[i][k]);
                const bool zero = v[i][k] == 0.0f;
                r[k] = 0u;
                if (key < 2u * p.width) r[k] = atomicAdd(&cnt[key], 1u);
                const uint64_t out = __ballot(key == 2u * p.width);
                if (out) {
                    const uint64_t nul = __ballot(zero);
                    const uint64_t oth = out & ~nul;
                    if (key == 2u * p.width) {
                        r[k] = wother + (uint32_t)__popcll(oth & ((1ull << lane) - 1ull));
                        bad |= __builtin_isfinite(v[i][k]) ? 0u : 1u;
                    }
                    wother += (uint32_t)__popcll(oth);
                    wzero += (uint32_t)__popcll(nul);
                }
            }
            rank[i][0] = r[0] | (r[1] << 16);
            rank[i][1] = r[2] | (r[3] << 16);
        }
    }
    if (lane == 0) {
        sh_other[wave] = wother;
        sh_zero[wave] = wzero;
    }
    if (bad) sh_bad = 1u;
    __syncthreads();

    // ---- starts of the buckets: an exclusive scan, two of them a lane ----
    static_assert(kBkKeys <= 2u * kBkThreads && kBkKeys % 2u == 0u, "two buckets a lane");
    const bool two = 2u * tid < kBkKeys;
    const uint32_t c0 = two ? cnt[2u * tid] : 0u, c1 = two ? cnt[2u * tid + 1u] : 0u;
    uint32_t s = c0 + c1;
#pragma unroll
    for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
        const uint32_t up = __shfl_up(s, o, kWave);
        if (lane >= o) s += up;
    }
    if (lane == (uint32_t)kWave - 1u) sh_wave[wave] = s;
    __syncthreads();
    uint32_t before = 0u, kept = 0u, obefore = 0u, others = 0u, zeros = 0u;
    for (uint32_t w = 0; w < kBkThreads / kWave; ++w) {
        if (w < wave) {
            before += sh_wave[w];
            obefore += sh_other[w];
        }
        kept += sh_wave[w];
        others += sh_other[w];
        zeros += sh_zero[w];
    }
    const uint32_t start0 = before + s - (c0 + c1), start1 = start0 + c0;
    uint16_t *row = a.table + (uint64_t)blockIdx.x * kBkRow;
    if (two) {
        cnt[2u * tid] = start0;
        cnt[2u * tid + 1u] = start1;
        if (tid < p.width) reinterpret_cast<uint32_t *>(row)[tid] = start0 | (start1 << 16);
        // how much work a bucket is: of every tile, since a crowd may lie in any of them.  Two counts at a time, neither reaches
        // 2^32; on their way while the tile is written.
        if ((c0 | c1) != 0u)
            atomicAdd(reinterpret_cast<unsigned long long *>(a.totals) + tid, (unsigned long long)c0 | ((unsigned long long)c1 << 32));
    }
    if (tid == 0) {
        reinterpret_cast<uint32_t *>(row)[p.width] = kept | ((kept + others) << 16);
        const uint32_t real = zeros - ((quads + kBkThreads - 1u) / kBkThreads * kBkThreads * 4u - m);   // without the places behind the tile's end
        if (real) atomicAdd(a.zeros, real);
        if (sh_bad) st_dev(&a.plan->fallback, 1u);
        if (others > m / 8u + 64u) st_dev(&a.plan->uneven, 1u);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kBkRounds; ++i) {
        if (i * kBkThreads < quads) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t key = key_of(v[i][k]);
                const uint32_t r = (rank[i][k / 2u] >> (16u * (k % 2u))) & 0xffffu;
                if (key < 2u * p.width) sx[cnt[key] + r] = v[i][k];
                else if (v[i][k] != 0.0f) sx[kept + obefore + r] = v[i][k];
            }
        }
    }
    __syncthreads();
    float4 *out = reinterpret_cast<float4 *>(a.sorted + (uint64_t)blockIdx.x * a.tile);
    const uint32_t oq = (kept + others + 3u) / 4u;   // at most tile / 4
    for (uint32_t q = tid; q < oq; q += kBkThreads) out[q] = reinterpret_cast<const float4 *>(sx)[q];
}

// ---- sum --------------------------------------------------------------------------------------------

constexpr int kBsThreads = 256;
constexpr uint32_t kBsTiles = 512;         // most tiles of a segment
constexpr uint32_t kBsQuads = 4;           // 4-element loads of a lane per batch
constexpr uint32_t kBsPerLane = 4u * kBsQuads;
constexpr uint32_t kBsLoads = 1u << 18;    // most loads that are summed by interval at a time: n < 2^24, sum |f| < 2^40
constexpr uint32_t kBsBatch = kBsThreads * kBsQuads;   // loads of a batch
constexpr uint32_t kBsItems = 128;         // most work items that a block lists at a time

struct alignas(4) Float4U { float x, y, z, w; };   // a run starts at any element
struct alignas(2) Pair16U { uint16_t x, y; };      // a bucket's start and end in a tile, one load

// Sums of one work item: those that its pieces refer to, or one class's by interval between cuts.
struct BucketSums {
    BucketSum sum[kBkDirect];
    uint32_t n[kBkDirect];
    uint64_t f[kBkDirect], q[kBkDirect];
    uint64_t nf[kBkCutCap + 1], iq[kBkCutCap + 1];   // count << 40 | sum |f|;  sum f^2
    uint64_t wave_nf[kBsThreads / kWave], wave_q[kBsThreads / kWave];
    uint32_t cut[kBkCutCap];
    uint16_t start[257];                             // cuts at or below the start of each 1/256 of the bucket
};

__device__ __forceinline__ void opaque(float (&v)[kBsPerLane])
{
#if defined(__AMDGCN__)
#pragma unroll
    for (uint32_t i = 0; i < kBsPerLane; ++i) asm volatile("" : "+v"(v[i]));
#endif
}

// The sums that a bucket's pieces refer to, a batch of 4 NQ elements a lane, `valid` of the wave's.
template <int NQ>
__device__ __forceinline__ void bucket_batch(float (&f0)[kBsPerLane], uint32_t valid, uint32_t nsum, BucketSums &sh,
                                             uint32_t lane)
{
    for (uint32_t s = 0; s < nsum; ++s) {
        opaque(f0);
        const float from = wave_uniform(sh.sum[s].from), unit = wave_uniform(sh.sum[s].unit), m = wave_uniform(sh.sum[s].m);
        uint32_t n = valid;
        float fs = 0.0f;   // at most 2^10 elements below 2^20
        double q0 = 0.0, q1 = 0.0;
        auto sums = [&](auto value) {   // four running sums
#pragma unroll
            for (int i = 0; i < 4 * NQ; i += 2) {
                const float a = value(i), b = value(i + 1);
                fs += a;
                fs += b;
                const double d0 = (double)a, d1 = (double)b;
                q0 = fma(d0, d0, q0);
                q1 = fma(d1, d1, q1);
            }
        };
        if (from > 0.0f) {
            n = 0u;
#pragma unroll
            for (int i = 0; i < 4 * NQ; ++i) n += (uint32_t)__popcll(__ballot(fabsf(f0[i]) >= from));
        }
        if (m == 0.0f) {
            if (from > 0.0f) sums([&](int i) { return fabsf(f0[i]) >= from ? f0[i] : 0.0f; });
            else sums([&](int i) { return f0[i]; });
        } else {
            const float add = wave_uniform(sh.sum[s].add);
            if (from > 0.0f) sums([&](int i) { return fabsf(f0[i]) >= from ? ((f0[i] + add) + m) - m : 0.0f; });
            else sums([&](int i) { return ((f0[i] + add) + m) - m; });
        }
        const int fi = (int)wave_sum_u32((uint32_t)(int)(fs * unit));
        const double qs = wave_sum(q0 + q1) * ((double)unit * (double)unit);
        if (lane == 0) {
            atomicAdd(reinterpret_cast<unsigned long long *>(&sh.f[s]), (unsigned long long)(long long)fi);
            atomicAdd(reinterpret_cast<unsigned long long *>(&sh.q[s]), (unsigned long long)qs);
            atomicAdd(&sh.n[s], n);
        }
    }
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, uint32_t o)
{
    return (uint64_t)__shfl_up((uint32_t)v, o, kWave) | ((uint64_t)__shfl_up((uint32_t)(v >> 32), o, kWave) << 32);
}

// sum (f + e)^2 = q + 2 e f + n e^2 with the rounding errors of its large terms carried along: x^ may lie among the elements,
// and the sum then is small beside its terms
__device__ inline double piece_sum(double n, double f, double q, double e)
{
    const double p = n * e, pe = fma(n, e, -p);
    const double f2 = 2.0 * f, s = f2 + p, sb = s - f2, se = (f2 - (s - sb)) + (p - sb);
    const double t = e * s, te = fma(e, s, -t);
    const double r = q + t, rb = r - q, re = (q - (r - rb)) + (t - rb);
    return r + (re + (te + e * (se + pe)));
}

__global__ __launch_bounds__(kBsThreads, 4) void k_bucket_sum(BucketArgs a)
{
    __shared__ BucketSums sh;
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const BucketPlan p = *a.plan;
    if (p.fallback) return;
    const uint32_t nbuckets = 2u * p.width;
    __shared__ double sh_total[kBkCands];   // of a candidate: kept here, not in registers

    __shared__ uint32_t runs[kBsTiles], first_load[kBsTiles], loads[kBsBatch], sh_wave[kBsThreads / kWave][2];

    // ---- elements outside the buckets: one candidate a lane, two lanes a candidate ----
    {
        float *sh_v = reinterpret_cast<float *>(&sh);
        double *sh_half = reinterpret_cast<double *>(sh_v + 1024);
        static_assert(sizeof(BucketSums) >= 4096 + kBkCands * sizeof(double), "their place");
        const uint32_t c = tid % kBkCands, half = tid / kBkCands;
        Cand g{0.0f, 0.0f, 0.0f, 0.0f};
        if (c < a.ncand) g = a.cands[c];
        auto score = [&](float x) { return (double)(x - dequant_level(bucket_level(g, x), g.scale, g.lo)); };
        double acc[2] = {0.0, 0.0}, total = 0.0;
        if (blockIdx.x == 0u && half == 0u) {   // all zeros have one value
            const double e = score(0.0f);
            total = (double)*a.zeros * e * e;
        }
        // the tiles' quarters, or the block's share of them all
        uint32_t share0 = 0u, share1 = 0u;
        if (p.uneven) {
            uint32_t len[2], sum = 0u;
#pragma unroll
            for (uint32_t i = 0; i < 2u; ++i) {
                const uint32_t t = 2u * tid + i;
                const uint16_t *row = a.table + (uint64_t)min(t, a.tiles - 1u) * kBkRow + nbuckets;
                runs[t] = row[0];
                len[i] = t < a.tiles ? (uint32_t)row[1] - row[0] : 0u;
                sum += len[i];
            }
            uint32_t up = sum;
#pragma unroll
            for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
                const uint32_t v = __shfl_up(up, o, kWave);
                if (lane >= o) up += v;
            }
            if (lane == (uint32_t)kWave - 1u) sh_wave[wave][0] = up;
            __syncthreads();
            uint32_t all = 0u;
            for (uint32_t w = 0; w < kBsThreads / kWave; ++w) {
                if (w < wave) up += sh_wave[w][0];
                all += sh_wave[w][0];
            }
            first_load[2u * tid] = up - sum;
            first_load[2u * tid + 1u] = up - len[1];
            share0 = (uint32_t)((uint64_t)all * blockIdx.x / kBkSumBlocks);
            share1 = (uint32_t)((uint64_t)all * (blockIdx.x + 1u) / kBkSumBlocks);
        }
        for (uint32_t t = blockIdx.x; t < (p.uneven ? blockIdx.x + 1u : 4u * a.tiles); t += kBkSumBlocks) {
            uint32_t from = share0, to = share1;
            if (!p.uneven) {
                const uint16_t *row = a.table + (uint64_t)(t / 4u) * kBkRow;
                const uint32_t start = row[nbuckets], len = row[nbuckets + 1u] - start;
                from = start + len * (t % 4u) / 4u;
                to = start + len * (t % 4u + 1u) / 4u;
            }
            for (uint32_t at = from; at < to; at += 1024u) {
                const uint32_t nv = min(1024u, to - at), mid = nv / 8u * 4u;
                __syncthreads();
                for (uint32_t i = tid; i < nv; i += kBsThreads) {
                    uint32_t tile = t / 4u, place = at + i;
                    if (p.uneven) {   // the last tile that starts at or before it
                        uint32_t h0 = kBsTiles;
                        tile = 0u;
                        while (h0 - tile > 1u) {
                            const uint32_t mid0 = (tile + h0) / 2u;
                            if (first_load[mid0] <= place) tile = mid0;
                            else h0 = mid0;
                        }
                        place += runs[tile] - first_load[tile];
                    }
                    sh_v[i] = a.sorted[(uint64_t)tile * a.tile + place];
                }
                __syncthreads();
                const uint32_t end = half ? nv : mid;
                uint32_t i = half ? mid : 0u;
                for (; i + 8u <= end; i += 8u) {
                    const float4 u = *reinterpret_cast<const float4 *>(sh_v + i), v = *reinterpret_cast<const float4 *>(sh_v + i + 4u);
                    const double e[8] = {score(u.x), score(u.y), score(u.z), score(u.w), score(v.x), score(v.y), score(v.z), score(v.w)};
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc[k & 1] = fma(e[k], e[k], acc[k & 1]);
                }
                for (; i < end; ++i) {
                    const double e = score(sh_v[i]);
                    acc[0] = fma(e, e, acc[0]);
                }
            }
        }
        total += acc[0] + acc[1];
        __syncthreads();
        if (half) sh_half[c] = total;
        __syncthreads();
        if (!half) sh_total[c] = total + sh_half[c];
        __syncthreads();   // their place is used again
    }

    // ---- the block's share: the buckets lie end to end by what they cost, and a block takes a stretch of that.  A bucket, or a
    // class of one that is summed by interval, is an item; of one that the stretch cuts the block takes the tiles that hold that
    // share of its elements (whole tiles: which elements of a bucket come first in one is the sort's chance) ----
    struct Item { uint16_t bucket, cls; uint32_t from, to, size; };   // from..to of size
    __shared__ Item sh_items[kBsItems];
    __shared__ uint32_t sh_first, sh_count, sh_run[2][2];
    __shared__ BucketPiece sh_piece[kBkCands];
    constexpr uint32_t per = (kBkKeys + kBsThreads - 1) / kBsThreads;
    static_assert(per * kBsThreads == kBkKeys && per % 4u == 0u, "16-byte loads");
    uint32_t *sizes = reinterpret_cast<uint32_t *>(&sh);   // of a bucket or of each of its classes, where the sums will be
    uint8_t *classes_of = reinterpret_cast<uint8_t *>(sizes + kBkKeys);
    static_assert(sizeof(BucketSums) >= 5u * kBkKeys, "their place");
    const uint32_t me = blockIdx.x;
    for (uint32_t first = 0u, count = 1u; first < count; first += kBsItems) {
        {
            uint32_t s1 = 0u, s2 = 0u;   // of the lane's buckets: what they cost, items
            uint32_t mine = tid * per;
            opaque(mine);   // (else the addresses are kept from the kernel's start on, in registers that it does not have)
#pragma unroll
            for (uint32_t k = 0; k < per; k += 4u) {
                const uint4 u = reinterpret_cast<const uint4 *>(a.totals)[(mine + k) / 4u], v = reinterpret_cast<const uint4 *>(a.shapes)[(mine + k) / 4u];
                const uint32_t n[4] = {u.x, u.y, u.z, u.w}, shape[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i) {
                    const uint32_t b = mine + k + i;
                    const bool used = b < nbuckets && b != p.centre;   // (the others have no shape)
                    const uint32_t ncls = used ? max(shape[i] >> 16, 1u) : 0u, size = used ? bucket_cost(n[i], shape[i]) : 0u;
                    sizes[b] = size;
                    classes_of[b] = (uint8_t)ncls;
                    s1 += ncls * size;
                    s2 += ncls;
                }
            }
            uint32_t c = s1, i0 = s2;
#pragma unroll
            for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
                const uint32_t u1 = __shfl_up(c, o, kWave), u2 = __shfl_up(i0, o, kWave);
                if (lane >= o) {
                    c += u1;
                    i0 += u2;
                }
            }
            if (lane == (uint32_t)kWave - 1u) {
                sh_wave[wave][0] = c;
                sh_wave[wave][1] = i0;
            }
            if (tid == 0) sh_first = sh_count = 0u;
            __syncthreads();
            uint32_t all = 0u;
            c -= s1;
            i0 -= s2;
            for (uint32_t w = 0; w < kBsThreads / kWave; ++w) {
                if (w < wave) {
                    c += sh_wave[w][0];
                    i0 += sh_wave[w][1];
                }
                all += sh_wave[w][0];
            }
            const uint32_t begin = (uint32_t)((uint64_t)all * me / kBkSumBlocks), end = (uint32_t)((uint64_t)all * (me + 1u) / kBkSumBlocks);
            // the item in which the stretch begins
            if (c <= begin && begin < c + s1) {
                uint32_t c1 = c, i1 = i0;
#pragma unroll 1
                for (uint32_t b = mine; b < mine + per; ++b) {
                    const uint32_t ncls = classes_of[b], size = sizes[b];
                    if (c1 <= begin && begin < c1 + ncls * size) sh_first = i1 + (begin - c1) / size;
                    c1 += ncls * size;
                    i1 += ncls;
                }
            }
            __syncthreads();
            if (c < end && begin < c + s1) {
#pragma unroll 1
                for (uint32_t b = mine; b < mine + per && c < end; ++b) {
                    const uint32_t ncls = classes_of[b], size = sizes[b];
                    if (begin < c + ncls * size) {
                        const uint32_t scrap = min(bucket_least(a.shapes[b]) / 2u, size / 2u);
                        // a place in the stretch to one in the item that it lies in; no scraps
                        auto place_at = [&](uint32_t at, uint32_t from) -> uint32_t {
                            if (at < from + scrap + 1u) return 0u;
                            if (at + scrap >= from + size) return size;
                            return at - from;
                        };
                        for (uint32_t cls = begin > c ? (begin - c) / size : 0u; cls < ncls && c + cls * size < end; ++cls) {
                            const uint32_t at = c + cls * size, number = i0 + cls - sh_first, slot = number - first;   // (before this turn: wraps around)
                            if (slot < kBsItems) sh_items[slot] = Item{(uint16_t)b, (uint16_t)cls, place_at(begin, at), place_at(end, at), size};
                            if (end <= at + size) sh_count = number + 1u;   // the last one
                        }
                    }
                    c += ncls * size;
                    i0 += ncls;
                }
            }
        }
        __syncthreads();
        count = sh_count;
        for (uint32_t item = 0; item < kBsItems && first + item < count; ++item) {
            auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
            const uint32_t b = uniform(sh_items[item].bucket), cls = uniform(sh_items[item].cls);
            const uint32_t part0 = uniform(sh_items[item].from), part1 = uniform(sh_items[item].to), whole = uniform(sh_items[item].size);
            if (part0 == part1) continue;
            const BucketRec *rec = a.recs + b;
            const uint32_t nsum = uniform(rec->nsum), ncut = uniform(rec->ncut), cuts1 = ncut + 1u;
            const uint32_t further = uniform(rec->piece);
            const bool direct = nsum != 0u;
            const uint32_t *cuts = a.cuts + uniform(rec->cut);
            const BucketClass *classes = a.classes + uniform(rec->cls);
            if (tid < kBkDirect) sh.sum[tid] = rec->sum[tid];   // (what lies past nsum is not used)
            const BucketAt at = bucket_at(p, b);
            const float base = at.value(0);
            if (tid < a.ncand) sh_piece[tid] = a.pieces[(uint64_t)b * kBkCands + tid];   // (kept in LDS, not in registers)
            // the runs, two a lane, and where their loads come in the item's list of loads
            Pair16U row[2];
#pragma unroll
            for (uint32_t i = 0; i < 2u; ++i)   // (a tile past the last has the last one's run, and no loads of it)
                row[i] = *reinterpret_cast<const Pair16U *>(a.table + (uint64_t)min(2u * tid + i, a.tiles - 1u) * kBkRow + b);
            uint32_t nl[2], sum = 0u;
#pragma unroll
            for (uint32_t i = 0; i < 2u; ++i) {
                const uint32_t t = 2u * tid + i, from = row[i].x, len = (uint32_t)row[i].y - from;
                runs[t] = from | (len << 16);
                nl[i] = t < a.tiles ? (len + 3u) / 4u : 0u;
                sum += nl[i];
            }
            static_assert(kBsTiles <= 2u * kBsThreads, "two runs a lane");
            uint32_t up = sum;
#pragma unroll
            for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
                const uint32_t v = __shfl_up(up, o, kWave);
                if (lane >= o) up += v;
            }
            if (lane == (uint32_t)kWave - 1u) sh_wave[wave][0] = up;
            if (!direct)
                for (uint32_t i = tid; i < ncut; i += kBsThreads) sh.cut[i] = cuts[i];
            __syncthreads();
            uint32_t total_loads = 0u;
            for (uint32_t w = 0; w < kBsThreads / kWave; ++w) {
                if (w < wave) up += sh_wave[w][0];
                total_loads += sh_wave[w][0];
            }
            // the block's share: from one run's start on and to another's (the blocks next to it work out the same ones)
            auto load_at = [&](uint32_t part) { return uniform((uint32_t)((double)total_loads * (double)part / (double)whole)); };
            const uint32_t at0 = load_at(part0), at1 = load_at(part1);
            up -= sum;
#pragma unroll
            for (uint32_t i = 0; i < 2u; ++i) {
                const uint32_t t = 2u * tid + i;
                if (t < a.tiles) {
                    first_load[t] = up;
                    auto nearest = [&](uint32_t load, uint32_t (&run)[2]) {
                        if (up < load && load <= up + nl[i]) {
                            const uint32_t behind = 2u * (load - up) >= nl[i] ? 1u : 0u;
                            run[0] = t + behind;
                            run[1] = up + behind * nl[i];
                        }
                    };
                    nearest(at0, sh_run[0]);
                    nearest(at1, sh_run[1]);
                }
                up += nl[i];
            }
            if (!direct) {
                // by interval between cuts: first the cuts at or below each 1/256 of the bucket, a few steps on from there
                for (uint32_t i = tid; i <= 256u; i += kBsThreads) {
                    const uint32_t d = i << (p.shift - 8u);
                    uint32_t l0 = 0u, h0 = ncut;   // cuts below l0 are <= d, cuts from h0 on are > d
                    while (l0 < h0) {
                        const uint32_t mid = (l0 + h0) / 2u;
                        if (sh.cut[mid] <= d) l0 = mid + 1u;
                        else h0 = mid;
                    }
                    sh.start[i] = (uint16_t)l0;
                }
            }
            __syncthreads();
            // (no run holds load 0's end)
            const uint32_t run0 = at0 ? uniform(sh_run[0][0]) : 0u, run1 = at1 ? uniform(sh_run[1][0]) : 0u;
            uint32_t load0 = at0 ? uniform(sh_run[0][1]) : 0u;
            const uint32_t load1 = at1 ? uniform(sh_run[1][1]) : 0u;
            while (load0 < load1) {
                const uint32_t load_end = direct ? load1 : min(load1, load0 + kBsLoads);
                if (direct) {
                    if (tid < kBkDirect) {
                        sh.n[tid] = 0u;
                        sh.f[tid] = sh.q[tid] = 0u;
                    }
                } else {
                    for (uint32_t i = tid; i < cuts1; i += kBsThreads) sh.nf[i] = sh.iq[i] = 0u;
                }
                uint32_t share = 0u;   // 2^share lanes list a run's loads
                while (share < 6u && ((run1 - run0) << (share + 1u)) <= (uint32_t)kBsThreads) ++share;
                // a batch's loads are listed and requested before the sums of the batch before it
                Float4U x[kBsQuads];
                uint32_t have = 0u;   // elements of each, a byte
                auto request = [&](uint32_t batch) {
                    __syncthreads();   // runs and their places are there; the last batch's list has been read
                    for (uint32_t r = run0 + (tid >> share); r < run1; r += (uint32_t)kBsThreads >> share) {
                        const uint32_t run = runs[r], at0 = first_load[r], len = run >> 16, n4 = (len + 3u) / 4u;
                        if (at0 + n4 <= batch || at0 >= batch + kBsBatch) continue;
                        const uint32_t where = r * a.tile + (run & 0xffffu);
                        uint32_t q = tid & ((1u << share) - 1u);
                        if (at0 + q < batch) q += ((batch - at0 - q + (1u << share) - 1u) >> share) << share;
                        for (; q < n4 && at0 + q < batch + kBsBatch; q += 1u << share)
                            loads[at0 + q - batch] = (where + 4u * q) << 2 | min(len - 4u * q - 1u, 3u);   // where < 2^25
                    }
                    __syncthreads();
                    have = 0u;
#pragma unroll
                    for (uint32_t k = 0; k < kBsQuads; ++k) {
                        const uint32_t i = batch + k * kBsThreads + tid;
                        x[k] = Float4U{base, base, base, base};
                        if (i < load_end) {
                            const uint32_t l = loads[i - batch];
                            x[k] = *reinterpret_cast<const Float4U *>(a.sorted + (l >> 2));
                            have |= ((l & 3u) + 1u) << (8u * k);
                        }
                    }
                };
                for (uint32_t batch = load0; batch < load_end; batch += kBsBatch) {
                    request(batch);
                    const uint32_t left = min(load_end - batch, kBsBatch);
                    float f0[kBsPerLane];
                    uint32_t had[kBsQuads], valid = 0u;
#pragma unroll
                    for (uint32_t k = 0; k < kBsQuads; ++k) {
                        had[k] = have >> (8u * k) & 0xffu;
                        f0[4 * k] = x[k].x - base;
                        f0[4 * k + 1] = had[k] > 1u ? x[k].y - base : 0.0f;
                        f0[4 * k + 2] = had[k] > 2u ? x[k].z - base : 0.0f;
                        f0[4 * k + 3] = had[k] > 3u ? x[k].w - base : 0.0f;
                        valid += had[k];
                    }
                    if (direct) {
                        const uint32_t all_valid = wave_sum_u32(valid);
                        if (left <= kBsThreads) bucket_batch<1>(f0, all_valid, nsum, sh, lane);
                        else bucket_batch<4>(f0, all_valid, nsum, sh, lane);
                    } else {
                        const float unit = __uint_as_float((uint32_t)(127 - at.a) << 23);
                        const BucketClass &cl = classes[cls];
                        const float add = wave_uniform(cl.add), m = wave_uniform(cl.m), per = wave_uniform(cl.unit);
#pragma unroll
                        for (uint32_t k = 0; k < kBsQuads; ++k) {
                            uint32_t d[4], v[4];
#pragma unroll
                            for (uint32_t e = 0; e < 4u; ++e) {
                                d[e] = (uint32_t)(fabsf(f0[4u * k + e]) * unit);
                                v[e] = sh.start[d[e] >> (p.shift - 8u)];
                            }
#pragma unroll
                            for (uint32_t e = 0; e < 4u; ++e) {
                                if (e < had[k]) {
                                    while (v[e] < ncut && sh.cut[v[e]] <= d[e]) ++v[e];
                                    const uint32_t r = (uint32_t)(fabsf(((f0[4u * k + e] + add) + m) - m) * per);
                                    atomicAdd(reinterpret_cast<unsigned long long *>(&sh.nf[v[e]]), (1ull << 40) + r);
                                    atomicAdd(reinterpret_cast<unsigned long long *>(&sh.iq[v[e]]), (unsigned long long)r * r);
                                }
                            }
                            asm volatile("" ::: "memory");   // a load at a time: registers
                        }
                    }
                }
                __syncthreads();
                if (!direct) {
                    // sums from each cut on: a suffix scan, three intervals a lane, from the last interval down
                    constexpr uint32_t pl = (kBkCutCap + 1 + kBsThreads - 1) / kBsThreads;
                    uint64_t nf[pl], iq[pl], snf = 0u, sq = 0u;
#pragma unroll
                    for (uint32_t i = 0; i < pl; ++i) {
                        const uint32_t v = tid * pl + i;   // counted from the end
                        nf[i] = v < cuts1 ? sh.nf[ncut - v] : 0u;
                        iq[i] = v < cuts1 ? sh.iq[ncut - v] : 0u;
                        snf += nf[i];
                        sq += iq[i];
                    }
                    uint64_t anf = snf, aq = sq;
#pragma unroll
                    for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
                        const uint64_t unf = shfl_up_u64(anf, o), uq = shfl_up_u64(aq, o);
                        if (lane >= o) {
                            anf += unf;
                            aq += uq;
                        }
                    }
                    if (lane == (uint32_t)kWave - 1u) {
                        sh.wave_nf[wave] = anf;
                        sh.wave_q[wave] = aq;
                    }
                    __syncthreads();
                    anf -= snf;
                    aq -= sq;
                    for (uint32_t w = 0; w < wave; ++w) {
                        anf += sh.wave_nf[w];
                        aq += sh.wave_q[w];
                    }
#pragma unroll
                    for (uint32_t i = 0; i < pl; ++i) {
                        const uint32_t v = tid * pl + i;
                        anf += nf[i];
                        aq += iq[i];
                        if (v < cuts1) {
                            sh.nf[ncut - v] = anf;
                            sh.iq[ncut - v] = aq;
                        }
                    }
                    __syncthreads();
                }
                // the candidate's pieces (of the item's class)
                if (tid < a.ncand) {
                    const double sgn = (at.base >> 31) ? -1.0 : 1.0;
                    double mine = 0.0;
                    BucketPiece pc = sh_piece[tid];
                    for (;;) {
                        if (direct || pc.cls == cls) {
                            double n, f, q;
                            if (direct) {
                                uint32_t ni = sh.n[pc.from];
                                uint64_t fi = sh.f[pc.from], qi = sh.q[pc.from];
                                if (pc.to != kBkNone) {
                                    ni -= sh.n[pc.to];
                                    fi -= sh.f[pc.to];
                                    qi -= sh.q[pc.to];
                                }
                                n = (double)ni;
                                f = (double)(long long)fi;
                                q = (double)qi;
                            } else {
                                uint64_t nfi = sh.nf[pc.from], qi = sh.iq[pc.from];
                                if (pc.to != kBkNone) {
                                    nfi -= sh.nf[pc.to];
                                    qi -= sh.iq[pc.to];
                                }
                                n = (double)(nfi >> 40);
                                f = sgn * (double)(nfi & ((1ull << 40) - 1ull));
                                q = (double)qi;
                            }
                            mine += piece_sum(n, f, q, pc.e) * pow2(2 * (at.a + (int)pc.dk));
                        }
                        if (pc.next == kBkNone) break;
                        pc = a.further[further + pc.next - kBkCands];
                    }
                    sh_total[tid] += mine;
                }
                __syncthreads();   // runs and sums are reused
                load0 = load_end;
            }
        }
        __syncthreads();
    }
    if (tid < a.ncand) a.partials[(uint64_t)tid * a.columns + blockIdx.x] = sh_total[tid];
}

// ---- launch -----------------------------------------------------------------------------------------

#ifndef QP_BUCKET_MIN_N
#define QP_BUCKET_MIN_N ((1ull << 21) + 1ull)   // the tile search is there below
#endif
#ifndef QP_BUCKET_LEAST_SAVING
#define QP_BUCKET_LEAST_SAVING 0.0
#endif

// What the buckets save a call against the streaming search, in microseconds.  That one's time goes with the pairs (0.16 us a
// million); sorting, listing and summing hardly know how many candidates there are.  Sender path by streaming / by buckets, Laplace
// data at 2 bit: 9.7 M elements 81 / 106 us at t = 20, 117 / 109 at 42, 207 / 110 at 100; 4.3 M 81 / 81 at 55, 113 / 82 at 100;
// 30 M 227 / 258 at 30, 349 / 262 at 55; 2.7 M 75 / 72 at 85.  At 8 bit 9.7 M 140 / 135 at 55, 4.3 M 90 / 99 at 70, 113 / 103 at 100.
// A dense sweep (see bucket_plan) has several times the pieces.  Post-GELU data, 2 bit: 9.7 M 134 / 133 at 55, 204 / 141 at 100; 3.5 M
// 98 / 98 at 100; 8 bit: 4.3 M 113 / 125, 5 M 126 / 123 at 100.
static double bucket_saving(uint64_t n, uint32_t bits, uint32_t ncand, bool dense)
{
    const double m = 1e-6 * (double)n, segments = (double)ceil_div_u64(n, QP_BUCKET_SEGMENT);
    const double fixed = bits <= 3u ? 31.0 : bits <= 4u ? 30.0 : bits <= 6u ? 32.0 : 36.0;
    const double each = bits <= 3u ? 3.75 : bits <= 6u ? 5.25 : 6.0;
    const double more = !dense ? 0.0 : (bits <= 3u ? 10.0 : 4.0) + 2.0 * m;
    return 0.16 * m * (double)ncand - fixed - each * m - 15.0 * (segments - 1.0) - more;
}
static bool bucket_search_pays(uint64_t n, uint32_t bits, uint32_t ncand, bool dense)
{
    if (bits > 3u ? n < 2u * QP_BUCKET_MIN_N : 4u * n < 5u * QP_BUCKET_MIN_N) return false;
    return bucket_saving(n, bits, ncand, dense) >= QP_BUCKET_LEAST_SAVING;
}

bool bucket_search_eligible(uint64_t n, int dtype, const SearchPlan &plan)
{
    return plan.bucket_room && dtype == QP_F32 && plan.bits <= 8u && plan.stride <= 1u && plan.t_steps + 1u <= kBkCands &&
           bucket_search_pays(n, plan.bits, plan.t_steps + 1u, false);
}

// (2 bit is what it takes first; a longer sweep than it can take asks for no less than the longest that it can)
bool bucket_search_wanted(uint64_t n, uint32_t t_steps, uint32_t stride)
{
    return stride <= 1u && bucket_search_pays(n, 2u, min(t_steps + 1u, kBkCands), false);
}

size_t bucket_search_end(uint64_t n, size_t at) { return bucket_layout(n, at).end; }

BucketSetup bucket_setup_args(const void *x, uint64_t n, const SearchPlan &plan, void *ws)
{
    const BucketLayout l = bucket_layout(n, plan.bucket_at);
    char *w = static_cast<char *>(ws);
    // Few wide buckets cost the least to list, narrow ones keep their sums in registers.  Sender path with 256 / 512 / 1024 of a sign,
    // 9.7 M elements, t = 100: Laplace data at 2 bit 110 / 113 / 125 us, 4 bit 121 / 117 / 120, 6 bit 119 / 123 / 130, 8 bit 258 (lists
    // too long) / 147 / 143; Gauss and Laplace mixed, 6 bit 125 / 119 / 124, 8 bit 258 / 144 / 134; after GELU at 2 bit 241 / 151 / 142
    // (4.3 M elements 120 / 104 / 112), 3 bit 174 / 142 / 139, 6 bit 161 / 153 / 158.
    const uint32_t width = plan.bits <= 3u ? kBkWidth / 4u : plan.bits <= 6u ? kBkWidth / 2u : kBkWidth;
    const uint32_t dense_width = plan.bits <= 3u ? (n < (1u << 23) ? kBkWidth / 2u : kBkWidth) : width;
    return BucketSetup{reinterpret_cast<BucketPlan *>(w + l.plan), reinterpret_cast<uint32_t *>(w + l.totals),
                       l.segments * (kBkKeys + 1u), width,
                       bucket_search_pays(n, plan.bits, plan.t_steps + 1u, true) ? dense_width : 0u, static_cast<const float *>(x), n};
}

hipError_t launch_bucket_search(const void *x, uint64_t n, const SearchPlan &plan, void *ws, const uint32_t **fallback, hipStream_t s)
{
    const BucketLayout l = bucket_layout(n, plan.bucket_at);
    char *w = static_cast<char *>(ws);
    BucketArgs a;
    a.tile = l.tile;
    a.ncand = plan.t_steps + 1u;
    a.plan = reinterpret_cast<BucketPlan *>(w + l.plan);
    a.table = reinterpret_cast<uint16_t *>(w + l.table);
    a.sorted = reinterpret_cast<float *>(w + l.sorted);
    a.cands = reinterpret_cast<const Cand *>(w + kOffCands);
    a.recs = reinterpret_cast<BucketRec *>(w + l.recs);
    a.shapes = reinterpret_cast<uint32_t *>(w + l.shapes);
    a.cuts = reinterpret_cast<uint32_t *>(w + l.cuts);
    a.classes = reinterpret_cast<BucketClass *>(w + l.classes);
    a.pieces = reinterpret_cast<BucketPiece *>(w + l.pieces);
    a.further = reinterpret_cast<BucketPiece *>(w + l.further);
    a.columns = kBkColumns * l.segments;
    *fallback = &a.plan->fallback;
    const uint64_t step = (uint64_t)l.tile * l.tiles;
    for (uint32_t seg = 0; seg < l.segments; ++seg) {
        const uint64_t from = seg * step;
        a.x = static_cast<const float *>(x) + from;
        a.n = n - from < step ? n - from : step;
        a.tiles = ceil_div_u64(a.n, l.tile);
        a.totals = reinterpret_cast<uint32_t *>(w + l.totals) + (size_t)seg * kBkKeys;
        a.zeros = reinterpret_cast<uint32_t *>(w + l.totals) + (size_t)l.segments * kBkKeys + seg;
        a.partials = reinterpret_cast<double *>(w + l.partials) + (size_t)seg * kBkColumns;
        a.first_segment = seg == 0 ? 1u : 0u;
        hipLaunchKernelGGL(k_bucket_sort, dim3(a.tiles), dim3(kBkThreads), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_bucket_sum, dim3(kBkColumns), dim3(kBsThreads), 0, s, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_search_pick(reinterpret_cast<const double *>(w + l.partials), a.columns, a.ncand, n, ws,
                              reinterpret_cast<double *>(w + kOffScores), *fallback, s);
}

}  // namespace qp
