// Routing analytics of one layer's budgeted routing (Section 5, "Analysis of
// Expert Load Balance": expert loads under the original and the budgeted
// routing, Spearman rank correlation, normalised-entropy change and
// Jensen-Shannon divergence of the score-weighted load distributions; "Analysis
// of Budget Allocation": correlation between a token's routing entropy and the
// number of experts it keeps).
//
// "Original" routing keeps all K candidates of a token, budgeted routing the
// first keep_count[t].  No floating-point atomics: every sum has a fixed order,
// and both rank correlations are formed from exact integer sums of doubled
// average ranks (2 * rank = 2 * #smaller + #equal + 1).
#include "common.hpp"
#include "kernels.hpp"

namespace allocmoe {

namespace {

// Each kernel is a chain of a few dependent trips to memory, so a workgroup has as many
// waves as it can hold and a thread's loads go out in batches.  At 6000 tokens, 64 experts
// and 6 candidates selection, dispatch and the analytics together went from 208 to 61 us (one
// thread per token or expert with serial loads, the ranks on 24 workgroups, before).
constexpr int kStatThreads = 1024;
constexpr int kStatWaves = kStatThreads / kWave;

// H_t = -sum_e s ln s, lane = expert; a wave takes kEntropyTok tokens, whose loads and
// logarithms overlap
constexpr int kEntropyTok = 4;
constexpr int kEntropyWgTok = kStatWaves * kEntropyTok;

__device__ __forceinline__ void token_entropies(const float* __restrict__ scores, int wg, int T, int E,
                                                float* __restrict__ H) {
    const int lane = lane_id();
    const int t0 = wg * kEntropyWgTok + static_cast<int>(threadIdx.x) / kWave * kEntropyTok;
    float s[kEntropyTok];
#pragma unroll
    for (int q = 0; q < kEntropyTok; ++q)
        s[q] = (lane < E && t0 + q < T) ? scores[static_cast<size_t>(t0 + q) * E + lane] : 0.f;
#pragma unroll
    for (int q = 0; q < kEntropyTok; ++q) {
        const float h = wave_sum(s[q] > 0.f ? -s[q] * logf(s[q]) : 0.f);
        if (lane == 0 && t0 + q < T) H[t0 + q] = h;
    }
}

// one workgroup per expert: counts and score sums of its candidate pairs and of its kept
// pairs; thread-strided partial sums over the flat list of pairs, then a fixed-order tree
constexpr int kLoadQuads = 8;   // 32 pairs: a bit each

__device__ __forceinline__ void expert_load(const int32_t* __restrict__ topk_ids,
                                            const float* __restrict__ topk_s,
                                            const int32_t* __restrict__ keep_count, int e, int T, int K,
                                            int32_t* load_orig, int32_t* load_kept, float* wload_orig,
                                            float* wload_kept) {
    __shared__ int32_t cnt[2][kStatWaves];
    __shared__ float wsum[2][kStatWaves];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int pairs = T * K;   // < 2^31
    // p / K = (p M) >> 35 with M = floor(2^35 / K) + 1: the excess is at most p / 2^35 < 1/16 <= 1/K
    const uint64_t M = (1ull << 35) / K + 1;
    int co = 0, ck = 0;
    float wo = 0.f, wk = 0.f;
    auto add = [&](int p) {   // a pair of this expert
        const int t = static_cast<int>((static_cast<uint64_t>(static_cast<uint32_t>(p)) * M) >> 35);
        const float s = topk_s[p];
        const int keep = keep_count[t];
        ++co;
        wo += s;
        if (p - t * K < keep) {
            ++ck;
            wk += s;
        }
    };
    // The ids of many pairs at once, then one by one what the thread's own pairs of this expert (one in E) need.
    // (Score and keep count of every pair loaded beside its id: three times the loads, which bound a unit here.  The kernel
    // with them and now, 16000 tokens, 8 candidates: 64 even experts 22.5 us, 10.0; eight of them in every token
    // 24.1, 14.9; 8 experts 23.8, 14.9; 2 experts, 2 candidates 8.4, 8.9.  6000 x 6, 64 experts of rank^-1.1: 9.7, 7.4.  Own
    // pairs two at a time: the same; four: up to 2.4 longer.)
    typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    const int quads = pairs / 4;
    for (int64_t q0 = tid; q0 < quads; q0 += kLoadQuads * kStatThreads) {
        i32x4_any id[kLoadQuads];
#pragma unroll
        for (int u = 0; u < kLoadQuads; ++u) {
            const int64_t q = q0 + u * kStatThreads;   // (past the end: the last quad, not counted)
            id[u] = *reinterpret_cast<const i32x4_any*>(topk_ids + 4 * (q < quads ? q : quads - 1));
        }
        uint32_t mine = 0;
#pragma unroll
        for (int u = 0; u < kLoadQuads; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                mine |= id[u][i] == e && q0 + u * kStatThreads < quads ? 1u << (4 * u + i) : 0u;
        for (; mine != 0; mine &= mine - 1) {
            const int bit = __builtin_ctz(mine);
            add(4 * (static_cast<int>(q0) + (bit / 4) * kStatThreads) + bit % 4);
        }
    }
    if (tid < pairs % 4 && topk_ids[4 * quads + tid] == e) add(4 * quads + tid);
    wo = wave_sum(wo);
    wk = wave_sum(wk);
    co = __builtin_amdgcn_readlane(wave_scan_incl(co), kWave - 1);
    ck = __builtin_amdgcn_readlane(wave_scan_incl(ck), kWave - 1);
    if (lane == 0) {
        cnt[0][wave] = co;
        cnt[1][wave] = ck;
        wsum[0][wave] = wo;
        wsum[1][wave] = wk;
    }
    __syncthreads();
    if (tid == 0) {
        co = ck = 0;
        wo = wk = 0.f;
        for (int w = 0; w < kStatWaves; ++w) {
            co += cnt[0][w];
            ck += cnt[1][w];
            wo += wsum[0][w];
            wk += wsum[1][w];
        }
        load_orig[e] = co;
        load_kept[e] = ck;
        wload_orig[e] = wo;
        wload_kept[e] = wk;
    }
}

// workgroups 0 .. E-1: an expert's loads; the others: the entropies of their tokens
__global__ __launch_bounds__(kStatThreads) void load_entropy_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ topk_ids,
    const float* __restrict__ topk_s, const int32_t* __restrict__ keep_count, int T, int E, int K,
    int32_t* __restrict__ load_orig, int32_t* __restrict__ load_kept, float* __restrict__ wload_orig,
    float* __restrict__ wload_kept, float* __restrict__ H) {
    const int wg = blockIdx.x;
    if (wg < E)
        expert_load(topk_ids, topk_s, keep_count, wg, T, K, load_orig, load_kept, wload_orig, wload_kept);
    else
        token_entropies(scores, wg - E, T, E, H);
}

// Pearson correlation of two rank vectors from exact integer sums (doubled ranks)
__device__ __forceinline__ float rank_correlation(long long n, long long sa, long long sb,
                                                  long long saa, long long sbb, long long sab) {
    const double va = static_cast<double>(n) * static_cast<double>(saa) -
                      static_cast<double>(sa) * static_cast<double>(sa);
    const double vb = static_cast<double>(n) * static_cast<double>(sbb) -
                      static_cast<double>(sb) * static_cast<double>(sb);
    const double cov = static_cast<double>(n) * static_cast<double>(sab) -
                       static_cast<double>(sa) * static_cast<double>(sb);
    if (va <= 0.0 || vb <= 0.0) return 0.f;   // one side constant
    return static_cast<float>(cov / sqrt(va * vb));
}

__device__ __forceinline__ long long wave_sum_int(long long s) {   // (integers: any order)
    uint64_t v = static_cast<uint64_t>(s);
    v += lane_xor<32>(v);
    v += lane_xor<16>(v);
    v += lane_xor<8>(v);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    v += lane_xor<1>(v);
    return static_cast<long long>(v);
}

// the four summary numbers of the experts' loads; one wave, lane = expert
__device__ __forceinline__ void expert_metrics(const int32_t* __restrict__ load_orig,
                                               const int32_t* __restrict__ load_kept,
                                               const float* __restrict__ wload_orig,
                                               const float* __restrict__ wload_kept, int E,
                                               float* __restrict__ metrics) {
    const int lane = lane_id();
    const bool valid = lane < E;
    const int lo = valid ? load_orig[lane] : 0, lk = valid ? load_kept[lane] : 0;
    const float wo = valid ? wload_orig[lane] : 0.f, wk = valid ? wload_kept[lane] : 0.f;
    int ro = 1, rk = 1;   // doubled average ranks among the E loads
    for (int o = 0; o < E; ++o) {
        const int oo = __builtin_amdgcn_readlane(lo, o), ok = __builtin_amdgcn_readlane(lk, o);
        ro += oo < lo ? 2 : (oo == lo ? 1 : 0);
        rk += ok < lk ? 2 : (ok == lk ? 1 : 0);
    }
    const long long a = valid ? ro : 0, b = valid ? rk : 0;
    const float rho = rank_correlation(E, wave_sum_int(a), wave_sum_int(b), wave_sum_int(a * a),
                                       wave_sum_int(b * b), wave_sum_int(a * b));
    // weighted load distributions
    const float so = wave_sum(wo), sk = wave_sum(wk);
    const float p = so > 0.f ? wo / so : 0.f, q = sk > 0.f ? wk / sk : 0.f;
    const float norm = E > 1 ? 1.f / logf(static_cast<float>(E)) : 0.f;
    const float ho = wave_sum(p > 0.f ? -p * logf(p) : 0.f) * norm;
    const float hk = wave_sum(q > 0.f ? -q * logf(q) : 0.f) * norm;
    const float m = 0.5f * (p + q);
    const float js = 0.5f * wave_sum((p > 0.f ? p * logf(p / m) : 0.f) +
                                     (q > 0.f ? q * logf(q / m) : 0.f));
    if (lane == 0) {
        metrics[0] = rho;
        metrics[1] = ho;
        metrics[2] = hk;
        metrics[3] = js;
    }
}

// Doubled average rank of every token's entropy among all T entropies: 2 #smaller + #equal
// + 1 = #smaller + #not greater + 1.  All pairs are compared, one compare and one add with
// carry each: bound by the vector units, so the pairs are spread over all of them: a
// workgroup ranks 16 tokens (lane % 16), and its 16 waves' 64 groups of 16 lanes take
// the entropies compared with in turn, four at a time.  The last workgroup's first wave has the
// experts' summary numbers instead, which nothing here depends on.
constexpr int kRankTok = 16;
constexpr int kRankGroups = kStatThreads / kRankTok;
constexpr int kRankUnroll = 4;

__global__ __launch_bounds__(kStatThreads) void entropy_rank_kernel(
    const float* __restrict__ H, int T, int32_t* __restrict__ rank2, const int32_t* __restrict__ load_orig,
    const int32_t* __restrict__ load_kept, const float* __restrict__ wload_orig,
    const float* __restrict__ wload_kept, int E, float* __restrict__ metrics) {
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x < kWave) expert_metrics(load_orig, load_kept, wload_orig, wload_kept, E, metrics);
        return;
    }
    typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // H: any 4-byte boundary
    __shared__ int part[kStatWaves][kRankTok];
    const int tid = threadIdx.x, wave = tid / kWave;
    const int t = blockIdx.x * kRankTok + tid % kRankTok;
    const float mine = H[min(t, T - 1)];
    int below = 0;   // #smaller + #not greater
    auto compare = [&](float v) {
        below += v < mine ? 1 : 0;
        below += v <= mine ? 1 : 0;
    };
    const int quads = T / 4;
    int c = tid / kRankTok;
    for (; c + (kRankUnroll - 1) * kRankGroups < quads; c += kRankUnroll * kRankGroups) {
        f32x4_u v[kRankUnroll];
#pragma unroll
        for (int u = 0; u < kRankUnroll; ++u)
            v[u] = *reinterpret_cast<const f32x4_u*>(H + 4 * static_cast<size_t>(c + u * kRankGroups));
#pragma unroll
        for (int u = 0; u < kRankUnroll; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) compare(v[u][i]);
    }
    for (; c < quads; c += kRankGroups) {
        const f32x4_u v = *reinterpret_cast<const f32x4_u*>(H + 4 * static_cast<size_t>(c));
#pragma unroll
        for (int i = 0; i < 4; ++i) compare(v[i]);
    }
    if (tid / kRankTok == 0)
        for (int u = 4 * quads; u < T; ++u) compare(H[u]);
    below += static_cast<int>(lane_xor<16>(static_cast<uint32_t>(below)));
    below += static_cast<int>(lane_xor<32>(static_cast<uint32_t>(below)));
    if (lane_id() < kRankTok) part[wave][lane_id()] = below;
    __syncthreads();
    if (tid < kRankTok && t < T) {
        int sum = 1;
#pragma unroll
        for (int w = 0; w < kStatWaves; ++w) sum += part[w][tid];
        rank2[t] = sum;
    }
}

// one workgroup: the correlation of the tokens' entropies with the experts they keep.  A keep
// count has few values: of the tokens that keep v experts the number n_v and the sum S_v of their
// entropy ranks are all that is needed beside the sum of squared ranks (b_v being the doubled
// average rank of v: sum b = sum n_v b_v, sum a b = sum b_v S_v).
constexpr int kMetricsBatch = 6;
__global__ __launch_bounds__(kStatThreads) void token_metrics_kernel(
    const int32_t* __restrict__ keep_count, const int32_t* __restrict__ entropy_rank2, int T,
    float* __restrict__ metrics) {
    constexpr int kValues = 64;   // keep counts counted (0 .. K, K <= 16)
    // (tokens mostly keep the same few counts: neighbouring lanes add to copies of their own)
    constexpr int kCopies = kStatThreads / kValues;
    __shared__ uint32_t n_of[kCopies][kValues];
    __shared__ unsigned long long s_of[kCopies][kValues], squares;
    const int tid = threadIdx.x, lane = lane_id(), copy = tid % kCopies;
    n_of[tid / kValues][tid % kValues] = 0;
    s_of[tid / kValues][tid % kValues] = 0;
    if (tid == 0) squares = 0;
    __syncthreads();
    unsigned long long sq = 0;
    for (int t0 = tid; t0 < T; t0 += kMetricsBatch * kStatThreads) {
        int v[kMetricsBatch], r[kMetricsBatch];
#pragma unroll
        for (int u = 0; u < kMetricsBatch; ++u) {
            const int t = min(t0 + u * kStatThreads, T - 1);
            v[u] = keep_count[t] & (kValues - 1);
            r[u] = entropy_rank2[t];
        }
#pragma unroll
        for (int u = 0; u < kMetricsBatch; ++u) {
            if (t0 + u * kStatThreads >= T) continue;
            atomicAdd(&n_of[copy][v[u]], 1u);   // (integers: any order)
            atomicAdd(&s_of[copy][v[u]], static_cast<unsigned long long>(r[u]));
            sq += static_cast<unsigned long long>(r[u]) * r[u];
        }
    }
    sq = static_cast<unsigned long long>(wave_sum_int(static_cast<long long>(sq)));
    if (lane == 0) atomicAdd(&squares, sq);
    __syncthreads();
    if (tid < kWave) {   // lane = keep count
        uint32_t total = 0;
        unsigned long long ranks = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) {
            total += n_of[c][lane];
            ranks += s_of[c][lane];
        }
        const int n = static_cast<int>(total);
        const long long before = wave_scan_incl(n) - n, b = 2 * before + n + 1, s = static_cast<long long>(ranks);
        const float rho = rank_correlation(T, wave_sum_int(s), wave_sum_int(n * b), static_cast<long long>(squares),
                                           wave_sum_int(n * b * b), wave_sum_int(s * b));
        if (lane == 0) metrics[4] = rho;
    }
}

}  // namespace

hipError_t launch_routing_stats(const float* scores, const int32_t* topk_ids, const float* topk_s,
                                const int32_t* keep_count, int T, int E, int K,
                                int32_t* load_orig, int32_t* load_kept, float* wload_orig,
                                float* wload_kept, float* token_entropy, int32_t* entropy_rank2,
                                float* metrics, hipStream_t stream) {
    hipLaunchKernelGGL(load_entropy_kernel, dim3(E + (T + kEntropyWgTok - 1) / kEntropyWgTok),
                       dim3(kStatThreads), 0, stream, scores, topk_ids, topk_s, keep_count, T, E, K,
                       load_orig, load_kept, wload_orig, wload_kept, token_entropy);
    hipLaunchKernelGGL(entropy_rank_kernel, dim3((T + kRankTok - 1) / kRankTok + 1), dim3(kStatThreads), 0,
                       stream, token_entropy, T, entropy_rank2, load_orig, load_kept, wload_orig, wload_kept, E,
                       metrics);
    hipLaunchKernelGGL(token_metrics_kernel, dim3(1), dim3(kStatThreads), 0, stream, keep_count, entropy_rank2, T,
                       metrics);
    return hipGetLastError();
}

}  // namespace allocmoe
