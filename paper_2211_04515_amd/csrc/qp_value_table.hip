// The value table of a large bfloat16 tensor, and what can be read off it.
//
// A bf16 tensor has at most 65536 distinct values.  counts[p] = number of elements with bit
// pattern p is built in one streaming pass (k_value_hist_bf16), and both the per-tensor
// statistics (Sec. 3: mu, b_E, the histogram D_R and its peak) and the scores of the directed
// search (Eq. 1) are sums over elements of functions of the value alone, so they can be taken
// over the 65536 table entries, each weighted by its count, instead of over the tensor: the same
// sums with equal terms grouped.  For a tensor of 151 M elements that replaces two reads of the
// tensor for the statistics and one per search round by a single read.
#include <type_traits>

#include "qp_common.hpp"

namespace qp {

bool uses_value_table(uint64_t n, int dtype) { return dtype == QP_BF16 && n >= kValueTableMinN; }
bool searches_value_table(uint64_t n, int dtype, const SearchPlan &plan)
{
    if (uses_value_table(n, dtype)) return true;
    return dtype == QP_BF16 && !plan.aciq_only && plan.stride <= 1u && n >= kValueTableSearchMinN &&
           n * (plan.t_steps + 1u) >= kValueTableMinPairs;
}

// Also clears the tickets (the search over the table has no set-up launch that could) and, for statistics, the
// histogram (nbins != 0).
__global__ __launch_bounds__(1024) void k_value_table_zero(uint32_t *__restrict__ counts, uint32_t *__restrict__ hist,
                                                           uint32_t nbins, Ctl *__restrict__ ctl)
{
    const uint32_t i = blockIdx.x * 1024u + threadIdx.x;
    reinterpret_cast<uint4 *>(counts)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (i < nbins) hist[i] = 0u;
    if (i == 0) {
        ctl->ticket_search = 0u;
        ctl->ticket_stats = 0u;
    }
}

// A block counts one sign (32768 patterns, 128 KB of LDS, plain u32 counters) of one chunk of the
// tensor; blocks b and b+8 sit on the same XCD (blocks are dealt round-robin to the 8 XCDs) and
// take the two signs of the same chunk, so the second reader of a chunk hits in that XCD's L2.
constexpr int kVhThreads = 1024;
constexpr int kVhUnroll = 4;

// The streaming loop for one sign (compile-time, so that the test of an element's sign is a single
// signed compare of the dword or of its low half).  On 151 M elements the kernel takes 65 us: 9 LDS
// increments per nanosecond and compute unit, about 4.2 per clock, i.e. 15 clocks per wave64 ds_add_u32 (64
// lanes into 32 banks at random addresses conflict about 3.5-fold, and an atomic is a read and a write).
// That rate is the bound: HBM delivers the tensor once (302 MB) at 4.6 TB/s and is not the limit, and every
// arrangement puts the same number of increments on each compute unit's LDS.  Prefetching the next tile,
// counting the other sign into dummy slots instead of branching, and one block per compute unit over all
// 65536 patterns in packed 16-bit counters (each element examined once) all measured the same or worse.
template <int SIGN>
__device__ __forceinline__ void value_hist_loop(const uint16_t *__restrict__ x, uint64_t n, uint32_t chunk,
                                                uint32_t nchunks, uint32_t *sh)
{
    const uint32_t tid = threadIdx.x;
    // both halves of a dword: the high half's sign is the dword's, the low half's that of its 16-bit value
    auto count2 = [&](uint32_t w) {
        const bool hi_neg = (int32_t)w < 0, lo_neg = (int16_t)(uint16_t)w < 0;
        if (hi_neg == (SIGN != 0)) atomicAdd(&sh[(w >> 16) & 0x7fffu], 1u);
        if (lo_neg == (SIGN != 0)) atomicAdd(&sh[w & 0x7fffu], 1u);
    };
    const uint64_t nvec = n / 8;   // 16-byte vectors of 8 elements
    const uint4 *__restrict__ x16 = reinterpret_cast<const uint4 *>(x);
    const uint64_t tile = (uint64_t)kVhThreads * kVhUnroll;
    uint64_t base = (uint64_t)chunk * tile;
    const uint64_t stride = (uint64_t)nchunks * tile;
    for (; base < nvec; base += stride) {
        uint4 v[kVhUnroll];
#pragma unroll
        for (int u = 0; u < kVhUnroll; ++u) {
            const uint64_t i = base + (uint64_t)u * kVhThreads + tid;
            v[u] = (i < nvec) ? x16[i] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kVhUnroll; ++u) {
            if (base + (uint64_t)u * kVhThreads + tid < nvec) {
                count2(v[u].x);
                count2(v[u].y);
                count2(v[u].z);
                count2(v[u].w);
            }
        }
    }
    if (chunk == 0 && tid < (uint32_t)(n - nvec * 8)) {
        const uint32_t h = x[nvec * 8 + tid];
        if ((h >> 15) == (uint32_t)SIGN) atomicAdd(&sh[h & 0x7fffu], 1u);
    }
}

// PARTS: every block also leaves the statistics' first-pass partial (sums, range, NaN/Inf) of what it counted: it has the counts in
// LDS and looks at each of them anyway.  A search alone has no use for them (its 1 M elements: 18.6 us with them, 16.9 without).
template <bool PARTS>
__global__ __launch_bounds__(kVhThreads) void k_value_hist_bf16(const uint16_t *__restrict__ x, uint64_t n,
                                                                uint32_t *__restrict__ counts, Part1 *__restrict__ part)
{
    __shared__ uint32_t sh[32768];
    __shared__ Part1 sh1[kVhThreads / kWave];
    const uint32_t tid = threadIdx.x;
    const uint32_t sign = (blockIdx.x >> 3) & 1u;
    const uint32_t chunk = ((blockIdx.x >> 4) << 3) | (blockIdx.x & 7u);
    const uint32_t nchunks = gridDim.x / 2;
    for (uint32_t i = tid; i < 32768u; i += kVhThreads) sh[i] = 0u;
    __syncthreads();
    // (counting the other sign's elements into dummy slots to avoid the branch was measured slower:
    // the LDS atomics are a scarce resource too)
    if (sign) value_hist_loop<1>(x, n, chunk, nchunks, sh);
    else value_hist_loop<0>(x, n, chunk, nchunks, sh);
    __syncthreads();
    double s = 0.0, sa = 0.0;
    float mn = INFINITY, mx = -INFINITY;
    uint32_t bad = 0u;
    for (uint32_t i = tid; i < 32768u; i += kVhThreads) {
        const uint32_t c = sh[i], pattern = (sign << 15) | i;
        if (c) {
            atomicAdd(&counts[pattern], c);
            if constexpr (PARTS) {
                const float v = __uint_as_float(pattern << 16);
                const double d = (double)v, w = (double)c;   // w d is exact: c < 2^32, v has 8 significant bits
                s = fma(w, d, s);
                sa = fma(w, fabs(d), sa);
                mn = fminf(mn, v);
                mx = fmaxf(mx, v);
                bad += __builtin_isfinite(v) ? 0u : c;
            }
        }
    }
    if constexpr (!PARTS) return;
    s = wave_sum(s);
    sa = wave_sum(sa);
    mn = wave_min(mn);
    mx = wave_max(mx);
    bad = wave_sum_u32(bad);
    if (tid % kWave == 0) sh1[tid / kWave] = Part1{s, sa, mn, mx, bad, 0u};
    __syncthreads();
    if (tid == 0) {
        Part1 t = sh1[0];
        for (int k = 1; k < kVhThreads / kWave; ++k) {
            t.sum += sh1[k].sum;
            t.sum_abs += sh1[k].sum_abs;
            t.mn = fminf(t.mn, sh1[k].mn);
            t.mx = fmaxf(t.mx, sh1[k].mx);
            t.bad += sh1[k].bad;
        }
        part[blockIdx.x] = t;
    }
}

// blocks of k_value_hist_bf16, i.e. partials that it leaves
static uint32_t value_hist_blocks(uint64_t n)
{
    const uint64_t tile = (uint64_t)kVhThreads * kVhUnroll;               // 16-byte vectors per block step
    uint64_t chunks = ((n / 8) + tile - 1) / tile;
    chunks = (chunks + 7) / 8 * 8;                                        // whole groups of 8 (one per XCD)
    if (chunks > 128) chunks = 128;                                       // two blocks (signs) per chunk: one block per compute unit
    return (uint32_t)(2 * chunks);
}
static_assert(256u <= kMaxStat1Blocks && 256u <= (uint32_t)kFinThreads, "a partial per block");

hipError_t launch_value_table(const void *x, uint64_t n, uint32_t nbins, void *ws, hipStream_t s)
{
    char *w = static_cast<char *>(ws);
    uint32_t *counts = reinterpret_cast<uint32_t *>(w + kOffValueCounts);
    hipLaunchKernelGGL(k_value_table_zero, dim3(kNumValues16 / 4096u), dim3(1024), 0, s, counts,
                       reinterpret_cast<uint32_t *>(w + kOffHist), nbins, reinterpret_cast<Ctl *>(w + kOffCtl));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    Part1 *part = reinterpret_cast<Part1 *>(w + kOffPart1);
    const uint16_t *x16 = static_cast<const uint16_t *>(x);
    if (nbins) hipLaunchKernelGGL(k_value_hist_bf16<true>, dim3(value_hist_blocks(n)), dim3(kVhThreads), 0, s, x16, n, counts, part);
    else hipLaunchKernelGGL(k_value_hist_bf16<false>, dim3(value_hist_blocks(n)), dim3(kVhThreads), 0, s, x16, n, counts, part);
    return hipGetLastError();
}

// ---- statistics from the table ---------------------------------------------------------------
// The second pass over the table, a thousand patterns per block: sum c |v - mu|, sum c (v - mu)^2 and the histogram (bin of
// the value, weight c), with exactly the per-value arithmetic of the streaming kernel (fp32 bin index, fp64 moments).  Every
// block adds the first pass's partials itself; the block that draws the last ticket makes the record, as in the streaming
// pass 2.  One block over the whole table, both passes, took 11.5 us: 64 entries per lane one after the other; spread over
// 64 blocks it is latency.
constexpr uint32_t kTsBlocks = 64, kTsPer = kNumValues16 / kTsBlocks / kFinThreads;   // entries of a lane: 2
__global__ __launch_bounds__(kFinThreads) void k_stats_from_table(const uint32_t *__restrict__ counts, uint64_t n,
                                                                  const Part1 *__restrict__ part1, uint32_t nb1,
                                                                  Part2 *__restrict__ part2, uint32_t nbins,
                                                                  uint32_t *__restrict__ hist, Ctl *__restrict__ ctl,
                                                                  qp_stats_t *__restrict__ out)
{
    __shared__ uint32_t sh_hist[kMaxBins];
    __shared__ Part1 sh1[kFinThreads / kWave];
    __shared__ Part2 sh2[kFinThreads / kWave];
    __shared__ uint32_t sh_last;
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const uint32_t first = (blockIdx.x * kFinThreads + tid) * kTsPer;   // the lane's first pattern
    static_assert(kTsPer == 2 && kTsBlocks <= kMaxStat2Blocks, "two entries a lane");
    const uint2 two = reinterpret_cast<const uint2 *>(counts)[first / 2];
    const uint32_t cnt[kTsPer] = {two.x, two.y};
    const Part1 tot = reduce_part1_block<kFinThreads>(part1, nb1, sh1);
    const double mean = tot.sum / (double)n;
    const float lo = tot.mn;
    const float range = tot.mx - lo;
    const float w_inv = (float)((double)(float)nbins / (double)range);
    const float top = (float)(nbins - 1u);
    auto bin = [&](uint32_t pattern) {
        const float tt = (__uint_as_float(pattern << 16) - lo) * w_inv;
        return (uint32_t)__builtin_amdgcn_fmed3f(tt, 0.0f, top);   // NaN -> 0
    };
    // the block's patterns are a run of values: its bins lie between those of its ends (but for NaN patterns)
    const uint32_t p0 = blockIdx.x * kFinThreads * kTsPer, ba = bin(p0), bb = bin(p0 + kFinThreads * kTsPer - 1u);
    const uint32_t b0 = min(ba, bb), b1 = max(ba, bb);
    for (uint32_t b = b0 + tid; b <= b1; b += kFinThreads) sh_hist[b] = 0u;
    __syncthreads();
    double dev = 0.0, sq = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < kTsPer; ++k) {
        const uint32_t c = cnt[k], idx = bin(first + k);
        if (c) {
            const double d = (double)__uint_as_float((first + k) << 16) - mean, w = (double)c;
            dev = fma(w, fabs(d), dev);
            sq = fma(w * d, d, sq);
        }
        // small values share a bin, whole waves of them: one increment then
        const uint32_t idx0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)idx);
        const bool one = wave_max_u32(idx != idx0 ? 1u : 0u) == 0u;
        const uint32_t all = one ? wave_sum_u32(c) : 0u;
        const uint32_t add = one ? (lane == 0 ? all : 0u) : c;
        if (add) {
            if (idx >= b0 && idx <= b1) atomicAdd(&sh_hist[idx], add);
            else atomicAdd(&hist[idx], add);
        }
    }
    dev = wave_sum(dev);
    sq = wave_sum(sq);
    if (lane == 0) sh2[wave] = Part2{dev, sq};
    __syncthreads();   // also: the block's part of the histogram is complete
    for (uint32_t b = b0 + tid; b <= b1; b += kFinThreads) {
        const uint32_t c = sh_hist[b];
        if (c) atomicAdd(&hist[b], c);
    }
    if (tid == 0) {
        Part2 p = sh2[0];
        for (int k = 1; k < kFinThreads / kWave; ++k) {
            p.dev += sh2[k].dev;
            p.sq += sh2[k].sq;
        }
        st_dev(&part2[blockIdx.x].dev, p.dev);
        st_dev(&part2[blockIdx.x].sq, p.sq);
    }
    wait_stores();     // this lane's histogram atomics and partial have arrived ...
    __syncthreads();   // ... and so have those of every lane of the block
    if (tid == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(&ctl->ticket_stats, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_last = (prev == gridDim.x - 1u) ? 1u : 0u;
    }
    __syncthreads();
    if (!sh_last) return;
    finalize_stats_block<true>(part1, nb1, part2, gridDim.x, hist, nbins, n, out);
    if (tid == 0) ctl->ticket_stats = 0u;
}

// after launch_value_table with the same nbins
hipError_t launch_stats_from_table(uint64_t n, uint32_t nbins, void *ws, hipStream_t s)
{
    char *w = static_cast<char *>(ws);
    hipLaunchKernelGGL(k_stats_from_table, dim3(kTsBlocks), dim3(kFinThreads), 0, s,
                       reinterpret_cast<const uint32_t *>(w + kOffValueCounts), n, reinterpret_cast<const Part1 *>(w + kOffPart1),
                       value_hist_blocks(n), reinterpret_cast<Part2 *>(w + kOffPart2), nbins, reinterpret_cast<uint32_t *>(w + kOffHist),
                       reinterpret_cast<Ctl *>(w + kOffCtl), reinterpret_cast<qp_stats_t *>(w + kOffStats));
    return hipGetLastError();
}

// ---- the directed search over the table ------------------------------------------------------
// Eq. 1's score of a candidate is a sum over elements of a function of the value alone, so it is taken over
// the 65536 table entries, each squared error weighted by its count: the same sum with equal terms grouped.
// One block per candidate (t + 1 blocks of 1024 lanes, 64 entries per lane, all requested before anything
// else).  A block builds its own candidate's grid (the arithmetic of setup_candidates), so there is no
// set-up launch, and hands its score to the block that draws the last ticket through device-coherent
// accesses; that block takes the first minimum and writes the control record, the result and the winner's
// grid.  Sums in a fixed order: bit-reproducible.
constexpr int kTbThreads = 1024;
__global__ __launch_bounds__(kTbThreads) void k_search_table(const uint32_t *__restrict__ counts, ModelArgs m_in,
                                                             const qp_stats_t *__restrict__ stats_dev, uint64_t n_total,
                                                             Cand *__restrict__ cands, double *__restrict__ scores,
                                                             Ctl *__restrict__ ctl, qp_search_result_t *__restrict__ res,
                                                             qp_qparams_t *__restrict__ best)
{
    __shared__ double sh[kTbThreads / kWave];
    __shared__ double sh_scores[kMaxT + 1];
    __shared__ uint32_t sh_flag;
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const uint32_t j = blockIdx.x, ncand = gridDim.x;
    constexpr uint32_t per = kNumValues16 / kTbThreads;   // 64 table entries per lane, four consecutive ones per load
    uint32_t cnt[per];
#pragma unroll
    for (uint32_t k = 0; k < per / 4; ++k) {
        const uint4 c4 = reinterpret_cast<const uint4 *>(counts)[k * kTbThreads + tid];
        cnt[4 * k] = c4.x;
        cnt[4 * k + 1] = c4.y;
        cnt[4 * k + 2] = c4.z;
        cnt[4 * k + 3] = c4.w;
    }
    const ModelArgs m = resolve_model(m_in);
    const GridModel g = grid_model(m, m.from_ws ? stats_dev : nullptr);
    int safe;
    const Cand p = candidate_grid(m, g, j, safe);
    if (tid == 0) cands[j] = p;
    const float Lf = (float)((1u << m.bits) - 1u);
    double acc = 0.0;
    auto run = [&](auto short_tag) {
        constexpr bool SHORT = decltype(short_tag)::value;
#pragma unroll
        for (uint32_t k = 0; k < per; ++k) {
            const uint32_t c = cnt[k];
            if (c) {   // patterns that do not occur contribute nothing (NaN/Inf patterns among them, for finite tensors)
                const float v = __uint_as_float((((k / 4) * kTbThreads + tid) * 4 + (k % 4)) << 16);
                float r;
                if constexpr (SHORT) {
                    const float xc = __builtin_amdgcn_fmed3f(v, p.lo, p.hi);
                    const float d = xc - p.lo;
                    const float t = d * p.inv_scale;
                    r = rintf(t);
                } else {
                    r = quant_level(v, p.lo, p.hi, p.inv_scale, Lf);
                }
                const float err = v - dequant_level(r, p.scale, p.lo);
                // count * err^2: count < 2^32 and err has 24 significant bits, so count * err is exact in fp64
                // and the term is rounded once, like an unweighted one
                const double de = (double)err;
                acc = fma((double)c * de, de, acc);
            }
        }
    };
    if (safe) run(std::true_type{});
    else run(std::false_type{});
    acc = wave_sum(acc);
    if (lane == 0) sh[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double tot = sh[0];
        for (int w = 1; w < kTbThreads / kWave; ++w) tot += sh[w];
        st_dev(&scores[j], tot);
        wait_stores();   // the score has arrived before the ticket is drawn
        const uint32_t prev = __hip_atomic_fetch_add(&ctl->ticket_search, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_flag = (prev == ncand - 1u) ? 1u : 0u;
    }
    __syncthreads();
    if (!sh_flag) return;
    // the last block: every score has arrived; read them coherently
    for (uint32_t i = tid; i < ncand; i += kTbThreads) sh_scores[i] = ld_dev(&scores[i]);
    __syncthreads();
    if (wave != 0) return;
    const uint32_t bi = first_min_wave(sh_scores, ncand, lane);
    if (lane == 0) {
        write_ctl(ctl, m, g, 1, 0u, n_total);
        write_search_result(ctl, sh_scores, ncand, bi, n_total, scores, res, best);
    }
}

hipError_t launch_table_search(uint64_t n, const SearchPlan &plan, const qp_stats_t *st, void *ws, hipStream_t s)
{
    char *w = static_cast<char *>(ws);
    const uint32_t ncand = plan.t_steps + 1u;
    hipLaunchKernelGGL(k_search_table, dim3(ncand), dim3(kTbThreads), 0, s,
                       reinterpret_cast<const uint32_t *>(w + kOffValueCounts), model_args(plan, st, kListFull, ncand, ws),
                       reinterpret_cast<const qp_stats_t *>(w + kOffStats), n, reinterpret_cast<Cand *>(w + kOffCands),
                       reinterpret_cast<double *>(w + kOffScores), reinterpret_cast<Ctl *>(w + kOffCtl),
                       reinterpret_cast<qp_search_result_t *>(w + kOffResult),
                       reinterpret_cast<qp_qparams_t *>(w + kOffQParams));
    return hipGetLastError();
}

}  // namespace qp
