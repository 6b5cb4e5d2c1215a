// Alloc-T selection and expert-sorted dispatch, as one single-workgroup "plan"
// kernel (the data is a few hundred KB at most and lives in L2).
//
// Selection (Section 3.3, Eqs. (7)-(9) and the procedure after them): every
// token keeps ranks j < K_base of its sorted candidate row; of the pool of the
// remaining T*(K-K_base) candidates the B' = B - T*K_base largest are kept,
// ties to the lower (token, rank).  Because rows are sorted, the kept ranks of
// a token form a prefix, so the result is keep_count[t].
//
// The B'-th largest pool value is found exactly by narrowing a range [lo, hi]
// of order-preserving u32 keys: each pass histograms the keys inside the range
// into <= 2048 equal-width bins in LDS (integer counts: order of the atomic
// increments cannot change the result), a block-wide suffix scan picks the bin
// that holds the wanted rank, and the range shrinks to that bin until it holds
// one key value v*.  Then a candidate is kept iff key > v*, or key == v* and
// fewer than R equal keys precede it in (token, rank) order.
//
// Dispatch: rows of the kept pairs ordered by (expert, token), with no atomics:
// for each batch of 64 tokens (lane = token) and each expert e the wave ballot
// "token keeps e" is a 64-bit word M[e][batch]; the row of pair (t, e) is
//   offset[e] + (kept pairs of e in earlier batches) + popcount(M[e][batch] below lane t).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"
#include "plan_common.hpp"

namespace allocmoe {

constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kBinsLog2 = 11;
constexpr int kBins = 1 << kBinsLog2;

struct PlanShared {
    uint32_t hist[kBins];
    uint32_t wave_tot[kPlanWaves];
    uint32_t red_lo[kPlanWaves];
    uint32_t red_hi[kPlanWaves];
    uint32_t pick_bin;     // chosen bin of a pass
    uint32_t pick_rank;    // wanted rank inside the chosen bin
    uint32_t pick_count;   // number of keys inside the chosen bin
    int32_t expert_total[kWave];
    int32_t expert_off[kWave + 1];
};

// Exclusive block-wide prefix sum of one value per thread, in thread order.
// Returns the exclusive prefix; *total (optional) receives the block sum.
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* wave_tot,
                                                    uint32_t* total) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const uint32_t incl = static_cast<uint32_t>(wave_scan_incl(static_cast<int>(v)));
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t base = 0, sum = 0;
    for (int w = 0; w < kPlanWaves; ++w) {
        const uint32_t x = wave_tot[w];
        if (w < wave) base += x;
        sum += x;
    }
    if (total) *total = sum;
    __syncthreads();
    return base + incl - v;
}

// keep_count[t] for all t.  topk_s: [T,K] rows sorted descending.
__device__ void select_phase(PlanShared& sh, const float* topk_s, int T, int K, int Kb,
                             int64_t B, int32_t* keep_count) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int P = K - Kb;                       // pool entries per token
    const int64_t n_pool = static_cast<int64_t>(T) * P;
    const int64_t want = B - static_cast<int64_t>(T) * Kb;   // B'
    if (want <= 0 || want >= n_pool) {          // nothing or everything from the pool
        const int c = want <= 0 ? Kb : K;
        for (int t = tid; t < T; t += kPlanThreads) keep_count[t] = c;
        return;
    }

    if (tid == 0) {
        sh.pick_bin = 0;
        sh.pick_rank = 1;
        sh.pick_count = 1;
    }
    // ---- pass 0: range of the pool keys
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (int t = tid; t < T; t += kPlanThreads)
        for (int j = Kb; j < K; ++j) {
            const uint32_t k = ordered_key(topk_s[static_cast<size_t>(t) * K + j]);
            lo = min(lo, k);
            hi = max(hi, k);
        }
    lo = wave_min_u32(lo);
    hi = wave_max_u32(hi);
    if (lane == 0) {
        sh.red_lo[wave] = lo;
        sh.red_hi[wave] = hi;
    }
    __syncthreads();
    lo = 0xFFFFFFFFu;
    hi = 0u;
    for (int w = 0; w < kPlanWaves; ++w) {
        lo = min(lo, sh.red_lo[w]);
        hi = max(hi, sh.red_hi[w]);
    }
    __syncthreads();

    // ---- narrowing passes: rank `r` counts from the top of [lo, hi]
    uint32_t r = static_cast<uint32_t>(want);
    uint32_t in_range = static_cast<uint32_t>(n_pool);
    while (lo < hi) {
        const uint32_t width_m1 = hi - lo;                      // >= 1
        const int bits = 32 - __builtin_clz(width_m1);          // width <= 2^bits
        const int shift = bits > kBinsLog2 ? bits - kBinsLog2 : 0;
        for (int b = tid; b < kBins; b += kPlanThreads) sh.hist[b] = 0;
        __syncthreads();
        for (int t = tid; t < T; t += kPlanThreads)
            for (int j = Kb; j < K; ++j) {
                const uint32_t k = ordered_key(topk_s[static_cast<size_t>(t) * K + j]);
                if (k >= lo && k <= hi) atomicAdd(&sh.hist[(k - lo) >> shift], 1u);
            }
        __syncthreads();
        // suffix sums over bins, two adjacent bins per thread, highest bins first:
        // thread i owns bins kBins-1-2i (first) and kBins-2-2i (second)
        const int b_first = kBins - 1 - 2 * tid, b_second = b_first - 1;
        const uint32_t c_first = sh.hist[b_first], c_second = sh.hist[b_second];
        const uint32_t above = block_scan_excl(c_first + c_second, sh.wave_tot, nullptr);
        // `above` = number of in-range keys in bins higher than b_first
        if (above < r && r <= above + c_first) {
            sh.pick_bin = b_first;
            sh.pick_rank = r - above;
            sh.pick_count = c_first;
        } else if (above + c_first < r && r <= above + c_first + c_second) {
            sh.pick_bin = b_second;
            sh.pick_rank = r - above - c_first;
            sh.pick_count = c_second;
        }
        __syncthreads();
        const uint32_t pb = sh.pick_bin;
        r = sh.pick_rank;
        in_range = sh.pick_count;
        const uint32_t new_lo = lo + (pb << shift);
        const uint32_t span_m1 = (shift == 0) ? 0u : ((1u << shift) - 1u);
        const uint32_t new_hi = (hi - new_lo < span_m1) ? hi : new_lo + span_m1;
        lo = new_lo;
        hi = new_hi;
        __syncthreads();
    }
    const uint32_t vstar = lo;      // key of the B'-th largest pool entry
    const uint32_t n_equal = in_range;
    const uint32_t R = r;           // how many of the keys == vstar are kept (1..n_equal)

    if (R == n_equal) {             // no tie is split: a plain threshold
        for (int t = tid; t < T; t += kPlanThreads) {
            int c = Kb;
            for (int j = Kb; j < K; ++j)
                c += ordered_key(topk_s[static_cast<size_t>(t) * K + j]) >= vstar ? 1 : 0;
            keep_count[t] = c;
        }
        return;
    }
    // ---- ties at the threshold: keep the first R equal keys in (token, rank)
    // order.  Tokens are visited in rounds of 1024 (thread = token), so the
    // order is (round, thread, rank); `seen` carries the equal keys of earlier
    // rounds.
    uint32_t seen = 0;
    const int rounds = (T + kPlanThreads - 1) / kPlanThreads;
    for (int it = 0; it < rounds; ++it) {
        const int t = it * kPlanThreads + tid;
        uint32_t gt = 0, eq = 0;
        if (t < T)
            for (int j = Kb; j < K; ++j) {
                const uint32_t k = ordered_key(topk_s[static_cast<size_t>(t) * K + j]);
                gt += k > vstar ? 1u : 0u;
                eq += k == vstar ? 1u : 0u;
            }
        uint32_t round_total;
        const uint32_t before = seen + block_scan_excl(eq, sh.wave_tot, &round_total);
        seen += round_total;
        if (t < T) {
            // equal keys of one token sit at consecutive ranks right after its
            // larger ones, so the first min(eq, R - before) of them are kept
            const uint32_t room = before < R ? R - before : 0u;
            keep_count[t] = Kb + static_cast<int>(gt + min(eq, room));
        }
    }
}

// Rows of the kept pairs in (expert, token) order.  words/prefix: scratch of
// 64 * ceil(T/64) entries each (u64 / i32), indexed [batch * 64 + expert].
__device__ void dispatch_phase(PlanShared& sh, const int32_t* topk_ids,
                               const int32_t* keep_count, int T, int K, int E, int64_t max_rows,
                               int32_t* expert_offsets, int32_t* row_token, int32_t* row_rank,
                               int32_t* inv_row, uint64_t* words, int32_t* prefix) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int n_batch = (T + kWave - 1) / kWave;

    // ---- A: per batch, the 64-bit "who keeps expert e" words (lane e owns word e)
    for (int b = wave; b < n_batch; b += kPlanWaves) {
        const int t = b * kWave + lane;
        uint64_t mine = 0;   // bit e: this token keeps expert e
        if (t < T) {
            const int kt = min(K, keep_count[t]);
            for (int j = 0; j < kt; ++j)
                mine |= 1ull << (topk_ids[static_cast<size_t>(t) * K + j] & (kWave - 1));
        }
        uint64_t col = 0;
        for (int e = 0; e < E; ++e) {
            const uint64_t w = __ballot((mine >> e) & 1ull);
            if (lane == e) col = w;
        }
        words[static_cast<size_t>(b) * kWave + lane] = col;
    }
    __threadfence_block();
    __syncthreads();

    // ---- B: per expert, exclusive prefix over batches; then offsets over experts.
    // thread (seg, e): 16 segments of batches per expert.
    {
        const int e = tid % kWave, seg = tid / kWave;
        const int per_seg = (n_batch + kPlanWaves - 1) / kPlanWaves;
        const int b0 = seg * per_seg, b1 = min(n_batch, b0 + per_seg);
        int local = 0;
        for (int b = b0; b < b1; ++b) local += __popcll(words[static_cast<size_t>(b) * kWave + e]);
        sh.hist[seg * kWave + e] = static_cast<uint32_t>(local);
        __syncthreads();
        int base = 0, total = 0;
        for (int s = 0; s < kPlanWaves; ++s) {
            const int v = static_cast<int>(sh.hist[s * kWave + e]);
            if (s < seg) base += v;
            total += v;
        }
        int run = base;
        for (int b = b0; b < b1; ++b) {
            prefix[static_cast<size_t>(b) * kWave + e] = run;
            run += __popcll(words[static_cast<size_t>(b) * kWave + e]);
        }
        if (seg == 0) {
            // wave 0: lane e holds expert e's row count
            const int incl = wave_scan_incl(e < E ? total : 0);
            sh.expert_off[e + 1] = incl;
            if (e == 0) sh.expert_off[0] = 0;
        }
        __threadfence_block();
        __syncthreads();
        // (offsets past the budget can only come from keep counts that sum to more than it)
        if (tid <= E) expert_offsets[tid] = min(sh.expert_off[tid], static_cast<int32_t>(max_rows));
    }

    // ---- C: place every pair
    for (int b = wave; b < n_batch; b += kPlanWaves) {
        const int t = b * kWave + lane;
        if (t >= T) continue;
        const int kt = min(K, keep_count[t]);
        const uint64_t below = lanemask_lt();
        for (int j = 0; j < K; ++j) {
            int row = -1;
            if (j < kt) {
                const int e = topk_ids[static_cast<size_t>(t) * K + j] & (kWave - 1);
                const size_t idx = static_cast<size_t>(b) * kWave + e;
                row = sh.expert_off[e] + prefix[idx] + __popcll(words[idx] & below);
                if (row < max_rows) {   // holds whenever sum_t keep_count[t] <= budget
                    row_token[row] = t;
                    row_rank[row] = j;
                } else {
                    row = -1;           // no row behind this pair: the combine skips it
                }
            }
            inv_row[static_cast<size_t>(t) * K + j] = row;
        }
    }
}

__device__ void tilemap_phase(PlanShared& sh, int E, int bm, int32_t* __restrict__ tile_info,
                              int max_rows) {
    if (threadIdx.x < kWave) write_tile_map(sh.expert_off, E, bm, tile_info, max_rows);
}

// ---------------------------------------------------------------------------
// Fast path (T <= 8192 and at most 48 pool keys per thread of 1024): the same two phases, but
// everything is read from global memory once: the pool keys into registers, where they stay
// for every pass, the candidate ids into LDS (one byte each), where the keep counts, ballot
// words and prefixes live as well.
//
// Selection: entry p of the pool (token p / P, rank Kb + p % P) belongs to thread p % NT, so
// that loads are coalesced and a wave's ballot over its entries is a word of a bit map in pool
// order.  A pass histograms the keys in [lo, hi]; every wave then finds the bin with the
// wanted rank by itself (no exchange, one barrier a pass).  As soon as a bin holds at most 64
// keys they are ranked directly, as (key, complement of p): the order (score descending, token
// ascending, rank ascending) as one number, so that ties need nothing further.  The result is
// the last pair kept; a second ballot compares all entries with it, and a token's keep count is
// the number of its bits.  More than 64 equal keys at the threshold: the last one kept is found
// by counting the bits of a ballot map of the equal ones.
// Dispatch: the 64 x 64 bit matrix "token t of the batch keeps expert e" is
// transposed with a 6-stage butterfly of lane exchanges instead of 64 ballots.
//
// Bound by latency: a chain of loads, barriers and LDS round trips on one compute unit.  Phases
// of 333 tokens with 8 candidates by time stamps inside the kernel, us: loads 2.0, range 0.6, passes
// 0.8, last bin and counts 1.5, words and prefixes 1.6, rows 1.2, together 7.6; with
// thread-contiguous slices of the pool staged through LDS, three passes that ended at a single
// key and block-wide scans 4.4, 1.0, 6.0, 2.6, 1.7, 2.0.  Whole kernel by a trace of layers without
// shared expert, then and now: 64 tokens x 6 14.2, 7.4; 333 x 8 17.3, 9.1; 500 x 4 16.2, 8.3; 777 x 4
// 18.6, 11.1; 2048 x 4 24.8, 14.4; 4096 x 6 33.8 (five launches), 23.0.
constexpr int kFastMaxT = 8192;
constexpr int kFastMaxPool = 48 * kPlanThreads;
constexpr int kCrowd = 8;          // share of the pool in one bin from which on its range is measured
constexpr int kCollect = 64;       // keys of a bin that a wave ranks directly
constexpr int kMaxK = 16;          // candidates per token the interface allows
constexpr int kPlanMaxGroups = 16;   // workgroups of a launch
constexpr int kMaxPasses = 4;      // 32 key bits, 9 or 10 a pass

template <int NT>
struct FastShared {
    static constexpr int kWaves = NT / kWave;
    // (256 and 512 threads: a token each at most)
    static constexpr int kTokens = NT == kPlanThreads ? kFastMaxT : NT;
    static constexpr int kKeys = NT == kPlanThreads ? kFastMaxPool / NT : kMaxK;   // pool entries of a thread
    static constexpr int kIds = NT == kPlanThreads ? 49152 : kTokens * kMaxK;
    static constexpr int kBinsLog2 = NT == 1024 ? 10 : 9;
    static constexpr int kWords = kKeys * kWaves;   // of a bit map over the pool
    union {
        struct {   // selection
            // (behind the bins and the collected keys a unit per lane, for the entries that are
            // not in the range: no branch)
            uint32_t hist[kMaxPasses][(1 << kBinsLog2) + kWave];
            uint64_t equal[kWords];
            alignas(16) uint64_t collected[kCollect + kWave];
        };
        uint64_t words[kTokens];       // dispatch: [batch][expert]
    };
    uint64_t bits[kWords + 1];         // pool entries kept
    uint32_t n_collected;
    uint32_t red_lo[kWaves], red_hi[kWaves];
    int32_t expert_off[kWave + 1];
    int32_t seg_tot[kWaves][kWave];
    uint8_t cnt[kTokens];              // keep_count
    uint16_t prefix[kTokens];          // [batch][expert]
    uint32_t ids[kIds / 4 + 4];        // candidate ids, one byte each, [token][rank]
};
static_assert(sizeof(FastShared<1024>) <= 160 * 1024, "LDS of a compute unit");

// f(q) for every q with entries of the pool (q a compile-time constant: the keys stay in
// registers), four at a time: a branch costs a wave that is alone on its SIMD as much as several
// entries (the last four may lie past the end: key 0, not in any range).
template <int NT, typename F, int... Q>
__device__ __forceinline__ void for_entries(int n_pool, F f, std::integer_sequence<int, Q...>) {
    f(std::integral_constant<int, 0>{});
    // (At most one entry a thread: not three idle ones beside it.  24 tokens with 3 entries each: selection
    // 5.95 us, 5.5 with it; 200 with 6: 7.2, 7.3 (7.5 with the one entry's code beside the four's); 512
    // and 1024 threads have larger pools.)
    if (NT == 256 && n_pool <= NT) return;
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    (void)((4 * (Q + 1) * NT < n_pool &&
            (f(std::integral_constant<int, 4 * Q + 4>{}), f(std::integral_constant<int, 4 * Q + 5>{}),
             f(std::integral_constant<int, 4 * Q + 6>{}), f(std::integral_constant<int, 4 * Q + 7>{}), true)) && ...);
}
template <int NT, typename F>
__device__ __forceinline__ void for_entries(int n_pool, F f) {
    constexpr int kKeys = FastShared<NT>::kKeys;
    static_assert(kKeys % 4 == 0, "whole groups");
    for_entries<NT>(n_pool, f, std::make_integer_sequence<int, kKeys / 4 - 1>{});
}

// The last pool entry kept: entries are kept iff their key is larger than `key`, or equal and
// their index is at most `index`.
struct Threshold {
    uint32_t key, index;
};

// Wave-wide: the position i with above(i) < r <= above(i) + count(i), lane l holding the counts of
// positions l * N .. + N - 1 in c.  Returns i, and in `above` the sum before it.
template <int N>
__device__ __forceinline__ int wave_find_rank(const uint32_t (&c)[N], uint32_t r, uint32_t& above) {
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) sum += c[i];
    const uint32_t incl = static_cast<uint32_t>(wave_scan_incl(static_cast<int>(sum)));
    const int src = __builtin_ctzll(__ballot(incl >= r) | (1ull << (kWave - 1)));
    uint32_t run = incl - sum;
    int at = 0;
#pragma unroll
    for (int i = 0; i < N - 1; ++i) {
        const bool past = at == i && run + c[i] < r;
        run += past ? c[i] : 0u;
        at += past ? 1 : 0;
    }
    above = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(run), src));
    return src * N + __builtin_amdgcn_readlane(at, src);
}

template <int NT>
__device__ __forceinline__ Threshold find_threshold(FastShared<NT>& sh, const uint32_t (&key)[FastShared<NT>::kKeys],
                                                    int n_pool, uint32_t want) {
    using Sh = FastShared<NT>;
    constexpr int NW = NT / kWave, kBinsLane = (1 << Sh::kBinsLog2) / kWave;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t lo = 1u, hi = 0xFFFFFFFFu, r = want, count = n_pool;
    if (count <= kCollect) __syncthreads();   // (the cleared counters)
    // ---- narrowing passes: rank r counts from the top of [lo, hi]
    bool measure = true;
    for (int pass = 0; count > kCollect && lo < hi; ++pass) {
        if (measure) {   // the range that the keys in [lo, hi] have (entries past the end hold 0, below every key)
            uint32_t first = 0xFFFFFFFFu, last = 0xFFFFFFFFu;   // (distances: keys outside wrap past all inside)
            for_entries<NT>(n_pool, [&](auto q_const) {
                constexpr int q = decltype(q_const)::value;
                first = min(first, key[q] - lo);
                last = min(last, hi - key[q]);
            });
            first = wave_min_u32(first);
            last = wave_min_u32(last);
            if (lane == 0) {
                sh.red_lo[wave] = first;
                sh.red_hi[wave] = last;
            }
            __syncthreads();
            lo += wave_min_u32(sh.red_lo[lane % NW]);
            hi -= wave_min_u32(sh.red_hi[lane % NW]);
            if (lo == hi) break;
        }
        const int bits = 32 - __builtin_clz(hi - lo);   // width <= 2^bits
        const int shift = max(0, bits - Sh::kBinsLog2);
        uint32_t* hist = sh.hist[pass];   // (bins from the top of the range)
        for_entries<NT>(n_pool, [&](auto q_const) {
            constexpr int q = decltype(q_const)::value;
            const uint32_t bin = key[q] >= lo && key[q] <= hi ? (hi - key[q]) >> shift : (1u << Sh::kBinsLog2) + lane;
            atomicAdd(&hist[bin], 1u);
        });
        __syncthreads();
        uint32_t c[kBinsLane], above;
#pragma unroll
        for (int i = 0; i < kBinsLane; i += 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(&hist[lane * kBinsLane + i]);
            c[i] = v.x;
            c[i + 1] = v.y;
            c[i + 2] = v.z;
            c[i + 3] = v.w;
        }
        const int bin = wave_find_rank(c, r, above);
        count = hist[bin];
        r -= above;
        hi -= static_cast<uint32_t>(bin) << shift;
        const uint32_t span_m1 = (1u << shift) - 1u;
        lo = hi - lo > span_m1 ? hi - span_m1 : lo;
        // Much of the pool in one bin: many equal keys (padding tokens, scores of few levels), which
        // the counter takes one by one, 64 to an instruction, in every pass that is left.  Their
        // own range ends the search at once.  6000 tokens, 3 of 4 padding, 64 experts of 512 x 256,
        // 6 candidates: layer 140 us without this, now 102 (the sequence of launches 105); no
        // padding: 87.7, 87.8.  (The measuring code stands in the loop once for both uses: with a copy
        // here the kernel grew by 2 KB, 777 tokens of a layer with a shared expert 12.4 us, now 11.7.)
        measure = count > static_cast<uint32_t>(n_pool) / kCrowd;
    }
    if (count <= kCollect) {
        // ---- rank the bin's keys directly
        if (n_pool <= kCollect) {   // (the whole pool: it sits in the first lanes)
            if (tid < n_pool)
                sh.collected[tid] = (static_cast<uint64_t>(key[0]) << 32) | ~static_cast<uint32_t>(tid);
        } else {
            uint32_t n = 0;
            for_entries<NT>(n_pool, [&](auto q_const) {
                constexpr int q = decltype(q_const)::value;
                n += key[q] >= lo && key[q] <= hi ? 1u : 0u;
            });
            uint32_t slot = n ? atomicAdd(&sh.n_collected, n) : 0u;   // (the order does not matter)
            if (__ballot(n != 0u)) {
                for_entries<NT>(n_pool, [&](auto q_const) {
                    constexpr int q = decltype(q_const)::value;
                    const bool in = key[q] >= lo && key[q] <= hi;
                    sh.collected[in && slot < kCollect ? slot : kCollect + lane] =
                        (static_cast<uint64_t>(key[q]) << 32) | ~static_cast<uint32_t>(q * NT + tid);
                    slot += in ? 1u : 0u;
                });
            }
        }
        __syncthreads();
        const uint64_t mine = sh.collected[lane];   // (cleared where nothing was written)
        const int mine_lo = static_cast<int>(static_cast<uint32_t>(mine)), mine_hi = static_cast<int>(mine >> 32);
        uint32_t before = 0;
        for (int l = 0; l < static_cast<int>(count); l += 8) {
            ulonglong2 other[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) other[i] = *reinterpret_cast<const ulonglong2*>(&sh.collected[l + 2 * i]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                before += other[i].x > mine ? 1u : 0u;
                before += other[i].y > mine ? 1u : 0u;
            }
        }
        const int last = __builtin_ctzll(__ballot(before == r - 1) | (1ull << (kWave - 1)));
        return {static_cast<uint32_t>(__builtin_amdgcn_readlane(mine_hi, last)),
                ~static_cast<uint32_t>(__builtin_amdgcn_readlane(mine_lo, last))};
    }
    if (r == count) return {lo, 0xFFFFFFFFu};   // no tie is split: a plain threshold
    // ---- more equal keys than a wave ranks: the r-th of them in pool order
    for_entries<NT>(n_pool, [&](auto q_const) {
        constexpr int q = decltype(q_const)::value;
        const uint64_t eq = __ballot(key[q] == lo);
        if (lane == 0) sh.equal[q * NW + wave] = eq;
    });
    __syncthreads();
    constexpr int kPer = Sh::kWords / kWave;
    static_assert(Sh::kWords % kWave == 0, "words per lane");
    uint32_t c[kPer], above;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int w = lane * kPer + i;
        c[i] = w * kWave < n_pool ? static_cast<uint32_t>(__popcll(sh.equal[w])) : 0u;
    }
    const int word = wave_find_rank(c, r, above);
    const uint64_t in_word = sh.equal[word];
    // (lane = bit)
    const bool hit = ((in_word >> lane) & 1ull) && __popcll(in_word & ((2ull << lane) - 1ull)) == static_cast<int>(r - above);
    return {lo, static_cast<uint32_t>(word * kWave + __builtin_ctzll(__ballot(hit) | (1ull << (kWave - 1))))};
}

// Whether two of the first n of eight bytes, mod 64, are equal.  Four bytes at a time: byte differences, at most 127, plus
// 127 have their top bit set unless they are 0 (24 instructions; a mask of 64 bits takes twice as many).
__device__ __forceinline__ bool repeats_id(const uint32_t (&ids)[2], int n) {
    uint32_t x[2], rot[2][4], all = ~0u;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        // bytes from n on: 64 + position, which equals no other byte
        const int held = min(max(n - 4 * w, 0), 4);
        const uint32_t mask = held == 4 ? ~0u : (1u << (8 * held)) - 1;
        x[w] = (ids[w] & (mask & 0x3f3f3f3fu)) | (~mask & (0x43424140u + 0x04040404u * w));
#pragma unroll
        for (int r = 0; r < 4; ++r) rot[w][r] = __builtin_amdgcn_alignbyte(x[w], x[w], r);
#pragma unroll
        for (int r = 1; r < 3; ++r) all &= (x[w] ^ rot[w][r]) + 0x7f7f7f7fu;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) all &= (x[0] ^ rot[1][r]) + 0x7f7f7f7fu;
    return (~all & 0x80808080u) != 0;
}

// SPLIT (several workgroups of 1024 threads, fast_path_runs): a workgroup owns a run of batches and forms words only
// for those; of the other batches it needs how many pairs of every expert lie before and behind its own, which LDS
// counters of its waves tell (integers: any order).  A wave has kCopies of them and its lanes take the copies in turn:
// additions of one instruction to one address come one behind the other, and a popular expert is in most tokens.
// Bound by vector instructions: with every workgroup transposing all
// batches the dispatch of 6000 x 6 candidates by 64 experts takes 13.1 us (94 transposes in each of 16 workgroups), with
// runs 11.0, whatever the skew (with one counter an expert 11.0 with even experts, 14.4 with one in every
// token, 16.2 with popularities of rank^-2.2).
template <bool SELECT, bool DISPATCH, int NT, bool SPLIT>
__global__ __launch_bounds__(NT) void plan_fast_kernel(
    const float* topk_s, const int32_t* topk_ids, int T, int K, int Kb, int64_t B, int E,
    int32_t* keep_count, int32_t* expert_offsets, int32_t* row_token, int32_t* row_rank,
    int32_t* inv_row, int bm, int32_t* tile_info) {
    using Sh = FastShared<NT>;
    __shared__ Sh sh;
    constexpr int NW = NT / kWave;            // waves
    static_assert(NT == 1024 || NT == 512 || NT == 256, "block sizes");
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // Launched as several workgroups (only where nothing else wants the compute units),
    // every workgroup runs the selection and the counting phases redundantly, on its own
    // unit and in its own LDS, with identical results and no exchange between them (SPLIT: the
    // words of its own run of batches only), and then writes its share of the placement, the one phase that
    // is bound by the number of scattered stores a single compute unit can issue (SPLIT: and of the keep
    // counts); workgroup 0 writes the rest.
    const int n_groups = gridDim.x, group = blockIdx.x;
    const bool writer = group == 0;
    const int P = K - Kb, n_pool = SELECT ? T * P : 0;
    const int64_t want = B - static_cast<int64_t>(T) * Kb;
    const bool search = SELECT && want > 0 && want < n_pool;

    // ---- all loads first: the pool's scores, then the candidate ids
    float score[Sh::kKeys];
    if (search) {
        const uint32_t inv_p = 0xFFFFFFFFu / static_cast<uint32_t>(P) + 1u;   // p / P = p inv_p >> 32 (P = 1: 0)
        for_entries<NT>(n_pool, [&](auto q_const) {
            constexpr int q = decltype(q_const)::value;
            const int i = min(q * NT + tid, n_pool - 1);
            const int t = P == 1 ? i : static_cast<int>(__umulhi(static_cast<uint32_t>(i), inv_p));
            score[q] = topk_s[static_cast<size_t>(t) * K + Kb + (i - t * P)];
        });
        if (n_pool > kCollect)
            for (int i = tid; i < static_cast<int>(sizeof(sh.hist) / 4); i += NT) (&sh.hist[0][0])[i] = 0;
        if (tid < kCollect) sh.collected[tid] = 0;
        if (tid == 0) sh.n_collected = 0;
    }
    const bool ids_held = DISPATCH && T * K <= Sh::kIds;
    if (ids_held) {
        // (four to a word, whatever the number of candidates; the last word may be partly filled)
        const int n = T * K, quads = n / 4;
        typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        constexpr int kBatch = 6;
        for (int i0 = tid; i0 < quads; i0 += kBatch * NT) {
            i32x4_any v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                v[u] = *reinterpret_cast<const i32x4_any*>(topk_ids + 4 * static_cast<size_t>(min(i0 + u * NT, quads - 1)));
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (i0 + u * NT < quads)
                    sh.ids[i0 + u * NT] = static_cast<uint32_t>((v[u][0] & 255) | ((v[u][1] & 255) << 8) |
                                                                ((v[u][2] & 255) << 16) | (v[u][3] << 24));
        }
        if (tid < n % 4) reinterpret_cast<uint8_t*>(sh.ids)[4 * quads + tid] = static_cast<uint8_t>(topk_ids[4 * quads + tid]);
    }
    if (search) {
        uint32_t key[Sh::kKeys];
        for_entries<NT>(n_pool, [&](auto q_const) {
            constexpr int q = decltype(q_const)::value;
            key[q] = q * NT + tid < n_pool ? ordered_key(score[q]) : 0u;
        });
        const Threshold last = find_threshold<NT>(sh, key, n_pool, static_cast<uint32_t>(want));
        uint64_t word = 0;   // lane q: the ballot over the wave's q-th entries
        for_entries<NT>(n_pool, [&](auto q_const) {
            constexpr int q = decltype(q_const)::value;
            const uint64_t kept = __ballot(key[q] > last.key || (key[q] == last.key && static_cast<uint32_t>(q * NT + tid) <= last.index));
            word = lane == q ? kept : word;
        });
        if (lane * NT < n_pool) sh.bits[lane * NW + wave] = word;
    }
    __syncthreads();
    // keep count of token t: its bits of the map
    auto count_of = [&](int t) -> int {
        if (!SELECT) return max(0, min(K, keep_count[t]));
        if (!search) return want <= 0 ? Kb : K;
        const uint32_t* w = reinterpret_cast<const uint32_t*>(sh.bits) + (static_cast<uint32_t>(t * P) >> 5);
        const uint64_t two = w[0] | (static_cast<uint64_t>(w[1]) << 32);
        return Kb + __popc(static_cast<uint32_t>(two >> ((t * P) & 31)) & ((1u << P) - 1u));
    };
    if (!DISPATCH) {
        for (int t = tid; t < T; t += NT) keep_count[t] = count_of(t);
        return;
    }
    // candidate ids of token t, one byte each: NJ (8 or 16) of them, those past K meaningless
    auto load_ids = [&](int t, auto& ids) {
        constexpr int NJ = 4 * (sizeof(ids) / sizeof(ids[0]));
        if (ids_held) {
            const uint32_t at = static_cast<uint32_t>(t * K), *w = sh.ids + at / 4;
            uint32_t x[NJ / 4 + 1];
#pragma unroll
            for (int i = 0; i <= NJ / 4; ++i) x[i] = w[i];
#pragma unroll
            for (int i = 0; i < NJ / 4; ++i) ids[i] = __builtin_amdgcn_alignbyte(x[i + 1], x[i], at % 4);
        } else {
            uint32_t x[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) x[j] = static_cast<uint32_t>(topk_ids[static_cast<size_t>(t) * K + min(j, K - 1)]) & 255u;
#pragma unroll
            for (int i = 0; i < NJ / 4; ++i) ids[i] = x[4 * i] | (x[4 * i + 1] << 8) | (x[4 * i + 2] << 16) | (x[4 * i + 3] << 24);
        }
    };
    const int n_batch = (T + kWave - 1) / kWave;
    // SPLIT: the batches of this workgroup and, behind their words, the waves' counters of pairs before (low half) and
    // behind them (high half); an expert has at most kFastMaxT pairs
    constexpr int kOwn = kFastMaxT / kWave / kPlanMaxGroups, kCopies = 8;
    static_assert(kFastMaxT < 1 << 16, "halves");
    const int per_group = SPLIT ? (n_batch + n_groups - 1) / n_groups : n_batch;
    const int own0 = SPLIT ? min(n_batch, group * per_group) : 0, own1 = SPLIT ? min(n_batch, own0 + per_group) : n_batch;
    // [wave][copy][expert], an expert's copies in different banks; copy 0 in the end the sum of all
    typedef uint32_t Counters[kCopies][kWave + kWave / kCopies];
    auto counters_of = [&](int w) -> Counters& { return reinterpret_cast<Counters*>(sh.words + kOwn * kWave)[w]; };
    if constexpr (SPLIT) {
        static_assert(NT == kPlanThreads && kOwn * kWave * 8 + NW * sizeof(Counters) <= sizeof(sh.words) && kOwn <= NW, "room");
#pragma unroll
        for (int c = 0; c < kCopies; ++c) counters_of(wave)[c][lane] = 0;
    }
    // ---- A: ballot words by bit-matrix transpose (lane e ends up with expert e's word)
    auto make_words = [&](auto nj_const) {
        constexpr int NJ = decltype(nj_const)::value;
        for (int b = wave; b < n_batch; b += NW) {
            const int t = b * kWave + lane, tt = min(t, T - 1);
            const int kt = t < T ? count_of(tt) : 0;
            uint32_t ids[NJ / 4];
            load_ids(tt, ids);
            if constexpr (SPLIT) {
                if (b < own0 || b >= own1) {   // uniform
                    auto expert = [&](int j) { return (ids[j / 4] >> (8 * (j % 4))) & (kWave - 1); };
                    uint32_t* counter = counters_of(wave)[lane % kCopies];
                    const uint32_t one = b < own0 ? 1u : 1u << 16;
                    if (__ballot(repeats_id(ids, kt)) == 0) {
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            if (j < kt) atomicAdd(&counter[expert(j)], one);
                    } else {   // an id that a token repeats counts once, as its bit in a word does
                        uint64_t seen = 0;
                        for (int j = 0; j < kt; ++j) {
                            uint32_t e = 0;
#pragma unroll
                            for (int i = 0; i < NJ; ++i) e = i == j ? expert(i) : e;
                            if (!(seen >> e & 1)) atomicAdd(&counter[e], one);
                            seen |= uint64_t{1} << e;
                        }
                    }
                    continue;
                }
            }
            uint64_t mine = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                mine |= static_cast<uint64_t>(j < kt ? 1u : 0u) << ((ids[j / 4] >> (8 * (j % 4))) & (kWave - 1));
            if (t < T) {
                sh.cnt[t] = static_cast<uint8_t>(kt);
                if (SELECT && (SPLIT || writer)) keep_count[t] = kt;
            }
            sh.words[(b - own0) * kWave + lane] = wave_transpose64(mine);
        }
    };
    if constexpr (SPLIT)
        make_words(std::integral_constant<int, 8>{});
    else if (K <= 8)
        make_words(std::integral_constant<int, 8>{});
    else
        make_words(std::integral_constant<int, 16>{});
    if constexpr (SPLIT) {   // (the wave's own counters)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) sum += counters_of(wave)[c][lane];
        counters_of(wave)[0][lane] = sum;
    }
    __syncthreads();
    // ---- B: per expert, exclusive prefix over batches; offsets over experts
    if constexpr (SPLIT) {
        int own[kOwn];
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += counters_of(w)[0][lane];
        int before = static_cast<int>(sum & 0xFFFFu), total = static_cast<int>(sum >> 16);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) own[i] = i < own1 - own0 ? __popcll(sh.words[i * kWave + lane]) : 0;
        total += before;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            if (i < wave) before += own[i];   // (the wave's own batch: own0 + wave)
            total += own[i];
        }
        if (wave < kOwn) sh.prefix[wave * kWave + lane] = static_cast<uint16_t>(before);
        if (wave == 0) {
            const int incl = wave_scan_incl(lane < E ? total : 0);
            sh.expert_off[lane + 1] = incl;
            if (lane == 0) sh.expert_off[0] = 0;
        }
        __syncthreads();
        if (writer && tid <= E) expert_offsets[tid] = min(sh.expert_off[tid], static_cast<int32_t>(B));
    } else {
        const int e = lane, seg = wave;
        const int per_seg = (n_batch + NW - 1) / NW;
        const int b0 = min(n_batch, seg * per_seg), b1 = min(n_batch, b0 + per_seg);
        int local = 0;
        for (int b = b0; b < b1; ++b) local += __popcll(sh.words[b * kWave + e]);
        sh.seg_tot[seg][e] = local;
        __syncthreads();
        int base = 0, total = 0;
        for (int s2 = 0; s2 < NW; ++s2) {
            const int v = sh.seg_tot[s2][e];
            if (s2 < seg) base += v;
            total += v;
        }
        int run = base;
        for (int b = b0; b < b1; ++b) {
            sh.prefix[b * kWave + e] = static_cast<uint16_t>(run);
            run += __popcll(sh.words[b * kWave + e]);
        }
        if (seg == 0) {
            const int incl = wave_scan_incl(e < E ? total : 0);
            sh.expert_off[e + 1] = incl;
            if (e == 0) sh.expert_off[0] = 0;
        }
        __syncthreads();
        if (writer && tid <= E) expert_offsets[tid] = min(sh.expert_off[tid], static_cast<int32_t>(B));
    }
    // ---- tile map, by the last wave, beside the other waves' share of phase C (with few
    // tokens the last wave has no batch of its own)
    if (writer && tile_info != nullptr && wave == NW - 1)
        write_tile_map(sh.expert_off, E, bm, tile_info, static_cast<int>(B));
    // ---- C: place every pair (token t = lane of batch b); several workgroups share the batches out: SPLIT in runs,
    // else one by one (they have computed the same counts, words and prefixes)
    auto place = [&](auto nj_const) {
        constexpr int NJ = decltype(nj_const)::value;
        for (int b = SPLIT ? own0 + wave : group + n_groups * wave; b < own1; b += SPLIT ? NW : n_groups * NW) {
            const int t = b * kWave + lane;
            if (t >= T) continue;
            const int kt = sh.cnt[t];
            const uint64_t below = lanemask_lt();
            uint32_t ids[NJ / 4];
            load_ids(t, ids);
            int row[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {   // all LDS reads first
                const int e = (ids[j / 4] >> (8 * (j % 4))) & (kWave - 1), idx = (b - own0) * kWave + e;
                row[j] = sh.expert_off[e] + sh.prefix[idx] + __popcll(sh.words[idx] & below);
            }
            int32_t* inv = inv_row + static_cast<size_t>(t) * K;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                // (row < B holds whenever sum_t keep_count[t] <= budget)
                row[j] = j < kt && row[j] < B ? row[j] : -1;
                if (row[j] >= 0) {
                    row_token[row[j]] = t;
                    row_rank[row[j]] = j;
                }
            }
            typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
            for (int j = 0; j < NJ; j += 4) {
                if (j + 4 <= K) {
                    *reinterpret_cast<i32x4_any*>(inv + j) = i32x4_any{row[j], row[j + 1], row[j + 2], row[j + 3]};
                } else {
#pragma unroll
                    for (int i = j; i < j + 3; ++i)
                        if (i < K) inv[i] = row[i];
                }
            }
        }
    };
    if constexpr (SPLIT)
        place(std::integral_constant<int, 8>{});
    else if (K <= 8)
        place(std::integral_constant<int, 8>{});
    else
        place(std::integral_constant<int, 16>{});
}

// ---------------------------------------------------------------------------
// Many tokens (selection alone from kPlanSpreadTokens on, with the dispatch from
// kPlanSpreadDispatchTokens on: kernels.hpp): the same selection and dispatch spread over workgroups, as a fixed sequence of short launches, with no global atomics and no
// waiting between workgroups (what a later launch needs from all workgroups of an
// earlier one goes through memory).
//
// Selection: exact radix select of the B'-th largest pool key on the 32 key bits, 11 +
// 11 + 10 from the top.  Pass p: each of G workgroups histograms, in LDS, the digit p of
// its share of the pool keys whose higher digits equal the ones already found, and writes
// its 2048 counts to hist[p][g]; the next launch sums the G partial histograms per bin,
// walks them from the top and finds the digit that holds the wanted rank (every workgroup
// does this redundantly, workgroup 0 records digit and remaining rank for the launches
// after it).  After three passes the key v* and the number R of keys equal to v* that
// are kept are known.  keep: thread = token; ties at v* are split in (token, rank) order:
// a workgroup takes the equal keys of earlier tokens from the last pass's partial histograms and
// counts those of the group that it begins in itself (only when a tie is split).  The same launch forms the ballot words of its batches of 64 tokens.
// place: a workgroup owns 16 batches; per expert (lane) the counts of all batches and of
// the batches before its own come from popcounts of the ballot words; then the rows.
constexpr int kSpreadThreads = 1024;   // (kPlanSpreadTokens: kernels.hpp)
constexpr int kSpreadMaxGroups = 16;
constexpr int kSpreadBins = 2048;

// Tokens of a group's histogram.  Up to 16384 those of a workgroup of the keep kernel, which then finds the equal keys
// of all earlier ones in the last pass's partial histograms.  Beyond, equal shares: in whole workgroups the largest
// share is up to twice the mean (selection of 16385 tokens, 8 candidates, with the loads of that time 49.1 us, equal
// shares 39.5; 33000 63.5, 53.9).
__host__ __device__ inline int spread_group_tokens(int T, int G) {
    return T <= kSpreadMaxGroups * kSpreadThreads ? kSpreadThreads : (T + G - 1) / G;
}

struct SpreadState {
    uint32_t b1, r1, b2, r2;
};

inline int spread_groups(int T) {
    const int g = (T + kSpreadThreads - 1) / kSpreadThreads;
    return g < kSpreadMaxGroups ? g : kSpreadMaxGroups;
}

size_t plan_spread_bytes(int T) {
    if (T < kPlanSpreadTokens) return 0;
    return 3 * static_cast<size_t>(spread_groups(T)) * kSpreadBins * sizeof(uint32_t) + 256;
}

// The bin (of the G partial histograms summed) that holds the r-th largest key counted
// from the top bin, the rank inside it and its count.  Block-wide; every thread returns
// the same values.
__device__ __forceinline__ void spread_find_bin(const uint32_t* __restrict__ partials, int G,
                                                uint32_t r, uint32_t* wave_tot, uint32_t* pick,
                                                uint32_t& bin, uint32_t& rank, uint32_t& count) {
    const int tid = threadIdx.x;
    const int b_first = kSpreadBins - 1 - 2 * tid, b_second = b_first - 1;
    // (eight groups' counts in flight; one after the other they took most of the launch)
    uint32_t c_first = 0, c_second = 0;
    constexpr int kBatch = 8;
    for (int g0 = 0; g0 < G; g0 += kBatch) {
        uint2 c[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)   // (past the end: the last group's, not counted)
            c[u] = *reinterpret_cast<const uint2*>(partials + static_cast<size_t>(min(g0 + u, G - 1)) * kSpreadBins + b_second);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            c_first += g0 + u < G ? c[u].y : 0u;
            c_second += g0 + u < G ? c[u].x : 0u;
        }
    }
    const uint32_t above = block_scan_excl(c_first + c_second, wave_tot, nullptr);
    if (above < r && r <= above + c_first) {
        pick[0] = b_first;
        pick[1] = r - above;
        pick[2] = c_first;
    } else if (above + c_first < r && r <= above + c_first + c_second) {
        pick[0] = b_second;
        pick[1] = r - above - c_first;
        pick[2] = c_second;
    }
    __syncthreads();
    bin = pick[0];
    rank = pick[1];
    count = pick[2];
    __syncthreads();
}

// f(key) for token t's pool entries, eight in flight: two 16-byte loads (of any 4-byte boundary; the last of a row ends
// with it), since single loads of lanes that lie K apart ask for the same lines again and again while they
// are on their way (selection of 4096 tokens, 8 candidates, 22.6 us: one load behind the other 30.9, four or eight at once 32.4)
template <typename F>
__device__ __forceinline__ void for_keys(const float* __restrict__ keys, int t, int K, int Kb, F f) {
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    const float* row = keys + static_cast<size_t>(t) * K;
    if (K - Kb < 4) {   // uniform, as all conditions here
        float v[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = row[min(Kb + i, K - 1)];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (Kb + i < K) f(ordered_key(v[i]));
        return;
    }
    for (int j0 = Kb; j0 < K; j0 += 8) {
        const int at[2] = {min(j0, K - 4), min(j0 + 4, K - 4)};
        f32x4_any v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) v[q] = *reinterpret_cast<const f32x4_any*>(row + at[q]);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (at[q] + i >= j0 + 4 * q) f(ordered_key(v[q][i]));
    }
}

template <int PASS>
__global__ __launch_bounds__(kSpreadThreads) void spread_hist_kernel(
    const float* __restrict__ keys, int T, int K, int Kb, int64_t B, uint32_t* __restrict__ hist,
    int G, SpreadState* __restrict__ state) {
    __shared__ uint32_t h[kSpreadBins];
    __shared__ uint32_t wave_tot[kPlanWaves];
    __shared__ uint32_t pick[3];
    const int tid = threadIdx.x;
    const int P = K - Kb;
    const int64_t n_pool = static_cast<int64_t>(T) * P, want = B - static_cast<int64_t>(T) * Kb;
    if (want <= 0 || want >= n_pool) return;   // nothing or everything from the pool: no search
    uint32_t b1 = 0, b2 = 0;
    if (PASS == 2) {
        uint32_t r1, c;
        spread_find_bin(hist, G, static_cast<uint32_t>(want), wave_tot, pick, b1, r1, c);
        if (blockIdx.x == 0 && tid == 0) {
            state->b1 = b1;
            state->r1 = r1;
        }
    } else if (PASS == 3) {
        b1 = state->b1;
        uint32_t r2, c;
        spread_find_bin(hist + static_cast<size_t>(G) * kSpreadBins, G, state->r1, wave_tot, pick, b2,
                        r2, c);
        if (blockIdx.x == 0 && tid == 0) {
            state->b2 = b2;
            state->r2 = r2;
        }
    }
    for (int b = tid; b < kSpreadBins; b += kSpreadThreads) h[b] = 0;
    __syncthreads();
    const int per = spread_group_tokens(T, G);
    const int t_begin = min(T, static_cast<int>(blockIdx.x) * per), t_end = min(T, t_begin + per);
    for (int t = t_begin + tid; t < t_end; t += kSpreadThreads)
        for_keys(keys, t, K, Kb, [&](uint32_t k) {
            if (PASS == 1)
                atomicAdd(&h[k >> 21], 1u);
            else if (PASS == 2) {
                if ((k >> 21) == b1) atomicAdd(&h[(k >> 10) & 0x7FFu], 1u);
            } else {
                if ((k >> 10) == ((b1 << 11) | b2)) atomicAdd(&h[k & 0x3FFu], 1u);
            }
        });
    __syncthreads();
    uint32_t* out = hist + (static_cast<size_t>(PASS - 1) * G + blockIdx.x) * kSpreadBins;
    for (int b = tid; b < kSpreadBins; b += kSpreadThreads) out[b] = h[b];
}

// keep_count of the workgroup's 1024 tokens (SELECT; otherwise they are read) and the ballot
// words of its 16 batches (words may be null: selection only).
template <bool SELECT>
__global__ __launch_bounds__(kSpreadThreads) void spread_keep_kernel(
    const float* __restrict__ keys, const int32_t* __restrict__ topk_ids, int T, int K, int Kb,
    int64_t B, const uint32_t* __restrict__ hist, int G, const SpreadState* __restrict__ state,
    int32_t* __restrict__ keep_count, uint64_t* __restrict__ words) {
    __shared__ uint32_t wave_tot[kPlanWaves];
    __shared__ uint32_t pick[3];
    const int tid = threadIdx.x, lane = lane_id();
    const int t0 = blockIdx.x * kSpreadThreads, t = t0 + tid;
    int keep = 0;
    if (SELECT) {
        const int P = K - Kb;
        const int64_t n_pool = static_cast<int64_t>(T) * P, want = B - static_cast<int64_t>(T) * Kb;
        if (want <= 0 || want >= n_pool) {
            keep = want <= 0 ? Kb : K;
        } else {
            uint32_t b3, R, n_equal;
            spread_find_bin(hist + 2 * static_cast<size_t>(G) * kSpreadBins, G, state->r2, wave_tot,
                            pick, b3, R, n_equal);
            const uint32_t vstar = (state->b1 << 21) | (state->b2 << 10) | b3;
            uint32_t gt = 0, eq = 0;
            if (t < T)
                for_keys(keys, t, K, Kb, [&](uint32_t k) {
                    gt += k > vstar ? 1u : 0u;
                    eq += k == vstar ? 1u : 0u;
                });
            if (R == n_equal) {   // no tie is split: a plain threshold
                keep = Kb + static_cast<int>(gt + eq);
            } else {
                // Equal keys of the tokens before this workgroup's: whole groups from the last pass's
                // histograms, the rest counted here.  (All counted here: 16000 tokens, 8 candidates,
                // scores of 64 levels, kernel 60 us, 8 now.)
                const int per = spread_group_tokens(T, G), g0 = t0 / per;
                uint32_t earlier = 0, mine = 0;
                for (int g = 0; g < g0; ++g) earlier += hist[(2 * static_cast<size_t>(G) + g) * kSpreadBins + b3];
                if (g0 * per < t0) {   // uniform
                    for (int u = g0 * per + tid; u < t0; u += kSpreadThreads)
                        for_keys(keys, u, K, Kb, [&](uint32_t k) { mine += k == vstar ? 1u : 0u; });
                    uint32_t counted;
                    block_scan_excl(mine, wave_tot, &counted);
                    earlier += counted;
                }
                const uint32_t before = earlier + block_scan_excl(eq, wave_tot, nullptr);
                // a token's equal keys sit at consecutive ranks right after its larger ones
                const uint32_t room = before < R ? R - before : 0u;
                keep = Kb + static_cast<int>(gt + min(eq, room));
            }
        }
        if (t < T) keep_count[t] = keep;
    } else if (t < T) {
        keep = keep_count[t];
    }
    if (words == nullptr) return;
    uint64_t mine = 0;   // bit e: this token keeps expert e
    if (t < T) {
        const int kt = min(K, keep);
        int ids[kMaxK];   // all loads first, so that they are in flight together
#pragma unroll
        for (int j = 0; j < kMaxK; ++j) ids[j] = j < K ? topk_ids[static_cast<size_t>(t) * K + j] : 0;
#pragma unroll
        for (int j = 0; j < kMaxK; ++j)
            if (j < kt) mine |= 1ull << (ids[j] & (kWave - 1));
    }
    const uint64_t col = wave_transpose64(mine);   // lane e: who of the batch keeps expert e
    if (t0 + (tid / kWave) * kWave < T) words[static_cast<size_t>(t / kWave) * kWave + lane] = col;
}

__global__ __launch_bounds__(kSpreadThreads) void spread_place_kernel(
    const int32_t* __restrict__ topk_ids, const int32_t* __restrict__ keep_count, int T, int K,
    int E, int64_t B, const uint64_t* __restrict__ words, int32_t* __restrict__ expert_offsets,
    int32_t* __restrict__ row_token, int32_t* __restrict__ row_rank, int32_t* __restrict__ inv_row,
    int bm, int32_t* __restrict__ tile_info) {
    __shared__ int32_t part_before[kPlanWaves][kWave];
    __shared__ int32_t part_total[kPlanWaves][kWave];
    __shared__ int32_t expert_off[kWave + 1];
    __shared__ int32_t before[kWave];
    __shared__ uint64_t wd[kPlanWaves][kWave];
    __shared__ int32_t pre[kPlanWaves][kWave];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int n_batch = (T + kWave - 1) / kWave;
    const int b0 = blockIdx.x * kPlanWaves;
    // (what does not depend on the counts comes first: the wave's own batch)
    const int b = b0 + wave, t = b * kWave + lane;
    wd[wave][lane] = b < n_batch ? words[static_cast<size_t>(b) * kWave + lane] : 0ull;
    const int kept = t < T ? keep_count[t] : 0;
    int ids[kMaxK];
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) ids[j] = j < K ? topk_ids[static_cast<size_t>(min(t, T - 1)) * K + j] : 0;
    {   // lane = expert; the waves split the batches
        const int per_seg = (n_batch + kPlanWaves - 1) / kPlanWaves;
        const int s0 = min(n_batch, wave * per_seg), s1 = min(n_batch, s0 + per_seg);
        int tot = 0, bef = 0;
        constexpr int kBatch = 8;   // loads in flight
        for (int b = s0; b < s1; b += kBatch) {
            uint64_t w[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) w[u] = words[static_cast<size_t>(min(b + u, s1 - 1)) * kWave + lane];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int c = b + u < s1 ? __popcll(w[u]) : 0;
                tot += c;
                bef += b + u < b0 ? c : 0;
            }
        }
        part_total[wave][lane] = tot;
        part_before[wave][lane] = bef;
    }
    __syncthreads();
    if (wave == 0) {
        int tot = 0, bef = 0;
        for (int w = 0; w < kPlanWaves; ++w) {
            tot += part_total[w][lane];
            bef += part_before[w][lane];
        }
        const int incl = wave_scan_incl(lane < E ? tot : 0);
        expert_off[lane + 1] = incl;
        if (lane == 0) expert_off[0] = 0;
        before[lane] = bef;
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        if (tid <= E) expert_offsets[tid] = min(expert_off[tid], static_cast<int32_t>(B));
        if (tile_info != nullptr && wave == kPlanWaves - 1)
            write_tile_map(expert_off, E, bm, tile_info, static_cast<int>(B));
    }
    {
        int p = before[lane];
        for (int w = 0; w < wave; ++w) p += __popcll(wd[w][lane]);
        pre[wave][lane] = p;
    }
    __syncthreads();
    if (t >= T) return;
    const int kt = min(K, kept);
    const uint64_t below = lanemask_lt();
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        if (j >= K) continue;
        int row = -1;
        if (j < kt) {
            const int e = ids[j] & (kWave - 1);
            row = expert_off[e] + pre[wave][e] + __popcll(wd[wave][e] & below);
            if (row < B) {   // holds whenever sum_t keep_count[t] <= budget
                row_token[row] = t;
                row_rank[row] = j;
            } else {
                row = -1;
            }
        }
        inv_row[static_cast<size_t>(t) * K + j] = row;
    }
}

// the launches of the spread selection (hist: plan_spread_bytes(T) bytes of scratch)
static void launch_spread_select(const float* keys, const int32_t* topk_ids, int T, int K, int Kb,
                                 int64_t B, void* spread, int32_t* keep_count, uint64_t* words,
                                 hipStream_t stream) {
    const int G = spread_groups(T);
    uint32_t* hist = static_cast<uint32_t*>(spread);
    SpreadState* state = reinterpret_cast<SpreadState*>(hist + 3 * static_cast<size_t>(G) * kSpreadBins);
    const dim3 block(kSpreadThreads);
    hipLaunchKernelGGL(spread_hist_kernel<1>, dim3(G), block, 0, stream, keys, T, K, Kb, B, hist, G, state);
    hipLaunchKernelGGL(spread_hist_kernel<2>, dim3(G), block, 0, stream, keys, T, K, Kb, B, hist, G, state);
    hipLaunchKernelGGL(spread_hist_kernel<3>, dim3(G), block, 0, stream, keys, T, K, Kb, B, hist, G, state);
    hipLaunchKernelGGL(spread_keep_kernel<true>, dim3((T + kSpreadThreads - 1) / kSpreadThreads), block,
                       0, stream, keys, topk_ids, T, K, Kb, B, hist, G, state, keep_count, words);
}

// 0: large sizes (generic kernels), else the block size of the fast kernel.
// A thread costs the barriers and the redundant searches little and the phases that walk batches
// of 64 tokens a wave much.  Kernel by trace: 64 tokens x 6 candidates 7.4 us with 256 threads, 7.4
// with 512, 8.9 with 1024; 200 x 6 7.9, 7.7, 9.4; 333 x 8 9.0 with 512, 10.0 with 1024; 500 x 4 8.2, 9.9.
inline int fast_path_threads(int T, int K, int Kb) {
    for (int nt : {256, 512})
        if (T <= nt) return nt;
    if (T <= kFastMaxT && static_cast<int64_t>(T) * (K - Kb) <= kFastMaxPool) return kPlanThreads;
    return 0;
}

// Workgroups of the fast kernel's launch: one beside other work (more would queue behind
// it); alone on the chip as many as leave two 64-token batches of placement to each.
inline int fast_path_groups(int T, bool alone) {
    if (!alone) return 1;
    const int n_batch = (T + kWave - 1) / kWave;
    return std::max(1, std::min(kPlanMaxGroups, n_batch / 2));
}

// Whether those workgroups own runs of batches (SPLIT).  As long as a wave has one batch, or few have a second, forming
// all words costs less than counting the other batches: layer's plan kernel of 64 experts, K = 6, all words and runs:
// 600 tokens 10.7 us, 11.0; 1000: 12.5, 12.8; 1300: 12.6, 12.9; 2000: 15.3, 14.7.  A pair costs an addition there
// and little in a word, so with many candidates a token words are the shorter way: dispatch of 2500 tokens by 64
// experts, even and skewed: K = 6 7.7 us, 6.9; 8: 7.8, 7.1; 12: 9.6, 9.9; 16 (of 16): 10.0, 10.5.
inline bool fast_path_runs(int T, int K, int nt, int groups) {
    return nt == kPlanThreads && groups > 1 && T > 3 * kPlanThreads / 2 && K <= 8;
}

template <bool SELECT, bool DISPATCH, typename... Args>
void enqueue_fast(int nt, int groups, bool runs, hipStream_t stream, Args... args) {
    const dim3 grid(groups), block(nt);
    if (nt == 256)
        hipLaunchKernelGGL((plan_fast_kernel<SELECT, DISPATCH, 256, false>), grid, block, 0, stream, args...);
    else if (nt == 512)
        hipLaunchKernelGGL((plan_fast_kernel<SELECT, DISPATCH, 512, false>), grid, block, 0, stream, args...);
    else if (DISPATCH && runs)
        hipLaunchKernelGGL((plan_fast_kernel<SELECT, DISPATCH, 1024, DISPATCH>), grid, block, 0, stream, args...);
    else
        hipLaunchKernelGGL((plan_fast_kernel<SELECT, DISPATCH, 1024, false>), grid, block, 0, stream, args...);
}

__global__ __launch_bounds__(kPlanThreads) void select_kernel(const float* topk_s, int T, int K,
                                                              int Kb, int64_t B,
                                                              int32_t* keep_count) {
    __shared__ PlanShared sh;
    select_phase(sh, topk_s, T, K, Kb, B, keep_count);
}

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(
    const float* topk_s, const int32_t* topk_ids, int T, int K, int Kb, int64_t B, int E,
    int32_t* keep_count, int32_t* expert_offsets, int32_t* row_token, int32_t* row_rank,
    int32_t* inv_row, uint64_t* words, int32_t* prefix, int bm, int32_t* tile_info) {
    __shared__ PlanShared sh;
    select_phase(sh, topk_s, T, K, Kb, B, keep_count);
    __threadfence_block();
    __syncthreads();
    dispatch_phase(sh, topk_ids, keep_count, T, K, E, B, expert_offsets, row_token, row_rank,
                   inv_row, words, prefix);
    if (tile_info != nullptr) tilemap_phase(sh, E, bm, tile_info, static_cast<int>(B));
}

hipError_t launch_select(const float* topk_s, int T, int K, int Kb, int64_t B,
                         int32_t* keep_count, void* spread, hipStream_t stream) {
    const int nt = fast_path_threads(T, K, Kb);
    if ((nt == 0 || T >= kPlanSpreadTokens) && spread != nullptr && plan_spread_bytes(T) > 0) {
        launch_spread_select(topk_s, nullptr, T, K, Kb, B, spread, keep_count, nullptr, stream);
        return hipGetLastError();
    }
    int32_t* const none = nullptr;
    if (nt != 0)
        enqueue_fast<true, false>(nt, 1, false, stream, topk_s, none, T, K, Kb, B, 0, keep_count, none, none, none, none, 0, none);
    else
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(kPlanThreads), 0, stream, topk_s, T, K, Kb,
                           B, keep_count);
    return hipGetLastError();
}

hipError_t launch_dispatch(const int32_t* topk_ids, const int32_t* keep_count, int T, int K,
                           int E, int64_t B, int32_t* expert_offsets, int32_t* row_token,
                           int32_t* row_rank, int32_t* inv_row, uint64_t* words,
                           int bm, int32_t* tile_info, bool alone, hipStream_t stream) {
    if (T >= kPlanSpreadDispatchTokens) {
        const dim3 grid((T + kSpreadThreads - 1) / kSpreadThreads), block(kSpreadThreads);
        hipLaunchKernelGGL(spread_keep_kernel<false>, grid, block, 0, stream, nullptr, topk_ids, T, K,
                           0, B, nullptr, 0, nullptr, const_cast<int32_t*>(keep_count), words);
        hipLaunchKernelGGL(spread_place_kernel, grid, block, 0, stream, topk_ids, keep_count, T, K, E,
                           B, words, expert_offsets, row_token, row_rank, inv_row, bm, tile_info);
        return hipGetLastError();
    }
    static_assert(kPlanSpreadDispatchTokens <= kFastMaxT, "one launch below");
    const int nt = fast_path_threads(T, K, K), groups = fast_path_groups(T, alone);
    enqueue_fast<false, true>(nt, groups, fast_path_runs(T, K, nt, groups), stream, static_cast<const float*>(nullptr), topk_ids, T, K,
                              0, B, E, const_cast<int32_t*>(keep_count), expert_offsets, row_token, row_rank, inv_row,
                              bm, tile_info);
    return hipGetLastError();
}

hipError_t launch_plan(const float* topk_s, const int32_t* topk_ids, int T, int K, int Kb,
                       int64_t B, int E, int32_t* keep_count, int32_t* expert_offsets,
                       int32_t* row_token, int32_t* row_rank, int32_t* inv_row, uint64_t* words,
                       int32_t* prefix, int bm, int32_t* tile_info, void* spread, bool alone,
                       hipStream_t stream) {
    const int nt = fast_path_threads(T, K, Kb);
    if ((nt == 0 || T >= kPlanSpreadDispatchTokens) && spread != nullptr && plan_spread_bytes(T) > 0) {
        launch_spread_select(topk_s, topk_ids, T, K, Kb, B, spread, keep_count, words, stream);
        const dim3 grid((T + kSpreadThreads - 1) / kSpreadThreads), block(kSpreadThreads);
        hipLaunchKernelGGL(spread_place_kernel, grid, block, 0, stream, topk_ids, keep_count, T, K, E,
                           B, words, expert_offsets, row_token, row_rank, inv_row, bm, tile_info);
        return hipGetLastError();
    }
    const int groups = fast_path_groups(T, alone);
    if (nt != 0)
        enqueue_fast<true, true>(nt, groups, fast_path_runs(T, K, nt, groups), stream, topk_s, topk_ids, T, K, Kb, B, E, keep_count,
                                 expert_offsets, row_token, row_rank, inv_row, bm, tile_info);
    else
        hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kPlanThreads), 0, stream, topk_s, topk_ids,
                           T, K, Kb, B, E, keep_count, expert_offsets, row_token, row_rank,
                           inv_row, words, prefix, bm, tile_info);
    return hipGetLastError();
}

}  // namespace allocmoe
