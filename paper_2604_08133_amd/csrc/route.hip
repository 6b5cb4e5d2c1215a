// Routing scores and per-token candidates (Section 3.1, Eq. (1); Section 3.3,
// Eq. (6)): logits = x W_gate (+bias), softmax over all E experts, then each
// token's K largest scores in descending order (ties: lower expert id).
//
// Layout: one lane per expert (E <= 64).  A workgroup of WAVES waves owns kRouteTok
// tokens; the waves split the hidden dimension, each lane accumulating the
// logit of its expert, and the partial sums meet in LDS in a fixed order.
#include <type_traits>

#include <algorithm>

#include "choice.hpp"
#include "common.hpp"
#include "ffn_bf16_stream.hpp"
#include "kernels.hpp"
#include "plan_common.hpp"

namespace allocmoe {

constexpr int kRouteTok = 4;    // tokens per workgroup
constexpr int kRouteBatch = 16;   // rows of the gate matrix loaded together

// Where the selection is not on the scores themselves (include/allocmoe.h, allocmoe_selector): the
// candidates' keys [T,K], fp32, formed while the candidates are found (as a launch of their own behind it: 1
// token, 64 experts of 2048 x 1408, 35.2 us a layer, 34.1 now; 333 tokens 157.0, 154.4; selection alone of 400
// tokens 26.0, 24.7).  mode 1: minus the score mass before candidate j
// (sequential adds); mode 2: s[t,j] / s[t,0] (correctly rounded division).
struct SelKeys {
    int mode;      // 0: none
    float* keys;
};

// Sorted Top-K of N tokens' scores at once, lane = expert: larger score first, equal
// scores lower expert first.  K rounds of: the largest remaining key of the wave, the
// lowest lane that holds it stores its (expert, score) at the round's position and
// leaves.  (The N chains are independent; the compiler interleaves them.)
// at[i]: the token's first candidate in ids, s and the selector's keys.  PoolSink: where the ordered
// keys that the selection compares go besides (see plan_small); NoPool: nowhere.
struct NoPool {
    __device__ void put(size_t, int, uint32_t) const {}
};
template <int N, typename PoolSink = NoPool>
__device__ __forceinline__ void wave_topk_store_n(const float (&score)[N], bool valid, int K, int32_t* ids,
                                                  float* s, const SelKeys& sel, const size_t (&at)[N],
                                                  const bool (&live)[N], const PoolSink& pool = {}) {
    const int lane = lane_id();
    // valid lanes: key >= 1 (scores are >= 0, so ordered_key has its top bit set)
    uint32_t key[N];
    float run[N];   // selector keys: mass so far, or the first score
#pragma unroll
    for (int i = 0; i < N; ++i) {
        key[i] = valid ? ordered_key(score[i]) : 0u;
        run[i] = 0.f;
    }
    auto rounds = [&](auto keyed_const) {
        constexpr bool KEYED = decltype(keyed_const)::value;
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const uint32_t top = wave_max_u32(key[i]);
                const uint64_t holders = __ballot(key[i] == top);
                const int winner = __builtin_ctzll(holders);   // (holders != 0: every lane takes part)
                float sel_key = 0.f;
                if constexpr (KEYED) {
                    const float sk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(score[i]), winner));
                    if (sel.mode == 1) {
                        sel_key = -run[i];
                        run[i] = __fadd_rn(run[i], sk);
                    } else {
                        if (k == 0) run[i] = sk;
                        sel_key = run[i] > 0.f ? __fdiv_rn(sk, run[i]) : 0.f;
                    }
                }
                if (top != 0u && lane == winner) {
                    if (live[i]) {
                        ids[at[i] + k] = lane;
                        s[at[i] + k] = score[i];
                        if constexpr (KEYED) sel.keys[at[i] + k] = sel_key;
                        pool.put(at[i], k, KEYED ? ordered_key(sel_key) : top);
                    }
                    key[i] = 0u;
                }
            }
        }
    };
    if (sel.mode == 0)
        rounds(std::false_type{});
    else
        rounds(std::true_type{});
}

__device__ __forceinline__ void wave_topk_store(float score, bool valid, int K, int32_t* ids, float* s,
                                                const SelKeys& sel, size_t at) {
    const float sc[1] = {score};
    const size_t first[1] = {at};
    const bool live[1] = {true};
    wave_topk_store_n<1>(sc, valid, K, ids, s, sel, first, live);
}

template <typename TIn, int WAVES>
__global__ __launch_bounds__(WAVES* kWave) void route_kernel(
    const TIn* __restrict__ X, const TIn* __restrict__ Wg, const float* __restrict__ bias,
    const TIn* __restrict__ w_sg, int T, int d, int E, int K, float* __restrict__ scores,
    int32_t* __restrict__ topk_ids, float* __restrict__ topk_s, float* __restrict__ sgate, SelKeys sel) {
    __shared__ float part[WAVES][kRouteTok][kWave];
    __shared__ float gpart[WAVES][kRouteTok];

    const int lane = lane_id();
    const int wave = threadIdx.x / kWave;
    const int t0 = blockIdx.x * kRouteTok;

    // this wave's slice of the hidden dimension, in chunks of 64
    const int chunks = (d + kWave - 1) / kWave;
    const int per_wave = (chunks + WAVES - 1) / WAVES;
    const int c_begin = wave * per_wave;
    const int c_end = min(chunks, c_begin + per_wave);

    float acc[kRouteTok];
    float gacc[kRouteTok];
#pragma unroll
    for (int q = 0; q < kRouteTok; ++q) acc[q] = gacc[q] = 0.f;

    const bool lane_is_expert = lane < E;
    for (int c = c_begin; c < c_end; ++c) {
        const int h0 = c * kWave;
        const int h = h0 + lane;
        float xv[kRouteTok];
#pragma unroll
        for (int q = 0; q < kRouteTok; ++q) {
            const int t = t0 + q;
            xv[q] = (t < T && h < d) ? load_f32(X, static_cast<size_t>(t) * d + h) : 0.f;
        }
        if (w_sg != nullptr) {
            const float g = h < d ? load_f32(w_sg, h) : 0.f;
#pragma unroll
            for (int q = 0; q < kRouteTok; ++q) gacc[q] += xv[q] * g;
        }
        // the token's value of h0 + i goes to all lanes as a scalar (v_readlane: one issue
        // slot, where a shuffle is a round trip through the LDS crossbar)
        auto step = [&](int i, float wv) {
#pragma unroll
            for (int q = 0; q < kRouteTok; ++q)
                acc[q] += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(xv[q]), i)) * wv;
        };
        const int n = min(kWave, d - h0);
        const TIn* wp = Wg + static_cast<size_t>(h0) * E + (lane_is_expert ? lane : 0);
        // The next 16 rows are on their way while 16 are used (past the last one: its own again, times the token's zeros
        // there).  That fits 64 registers: eight waves a SIMD.  One 16 behind the other with the rows past the last whole
        // 16 one by one (before), all 64 of a chunk at once (98 registers), this; routing and selection, us:
        // fp32, 500 tokens, d 1132 19.4, 18.3, 18.1; 8192, d 1132 84.4, 103.6, 78.9; 30000, d 2048 401, 435, 372; 66000, d
        // 200 128, 123, 123; bf16, 500, d 2048 26.3, 23.3, 21.5; 30000, d 1024 228, 305, 222.
        float cur[kRouteBatch], ahead[kRouteBatch];
        auto load = [&](float (&rows)[kRouteBatch], int i) {
#pragma unroll
            for (int u = 0; u < kRouteBatch; ++u) rows[u] = load_f32(wp, static_cast<size_t>(min(i + u, n - 1)) * E);
        };
        load(cur, 0);
#pragma unroll
        for (int i = 0; i < kWave; i += kRouteBatch) {
            if (i >= n) break;   // uniform
            if (i + kRouteBatch < kWave) load(ahead, i + kRouteBatch);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kRouteBatch; ++u) step(i + u, i + u < n ? cur[u] : 0.f);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kRouteBatch; ++u) cur[u] = ahead[u];
        }
    }
#pragma unroll
    for (int q = 0; q < kRouteTok; ++q) {
        part[wave][q][lane] = acc[q];
        if (w_sg != nullptr) {
            const float g = wave_sum(gacc[q]);
            if (lane == 0) gpart[wave][q] = g;
        }
    }
    __syncthreads();

    // wave q finishes token t0 + q
    for (int q = wave; q < kRouteTok; q += WAVES) {
        const int t = t0 + q;
        if (t >= T) continue;
        float logit = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) logit += part[w][q][lane];
        if (bias != nullptr && lane_is_expert) logit += bias[lane];
        if (!lane_is_expert) logit = -INFINITY;
        const float m = wave_max(logit);
        const float p = lane_is_expert ? expf(logit - m) : 0.f;
        const float den = wave_sum(p);
        const float s = p / den;
        if (scores != nullptr && lane_is_expert) scores[static_cast<size_t>(t) * E + lane] = s;
        wave_topk_store(s, lane_is_expert, K, topk_ids, topk_s, sel, static_cast<size_t>(t) * K);
        if (w_sg != nullptr && lane == 0) {
            float g = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) g += gpart[w][q];
            sgate[t] = 1.f / (1.f + expf(-g));
        }
    }
}

// ---------------------------------------------------------------------------
// bf16 fast path: the gate GEMM on the matrix cores.  A workgroup of 16 waves
// owns 16 MT tokens; the waves split the hidden dimension into slices of 32-wide
// steps, each wave running v_mfma_f32_16x16x32_bf16 on its slice with the A
// operand read straight from X (64 contiguous bytes per token and step) and the
// B operand from the gate matrix re-tiled at load time (pack.hip) (one 16-byte load
// per lane).  The partial logits meet in LDS in a fixed order, then one wave
// per token does the softmax and the Top-K with one lane per expert.
//
// A workgroup is bound by the bytes that cross its compute unit's vector load path
// (64 B per clock): the whole re-tiled gate matrix (262 KB, 327 KB with the shared
// gate's column) plus 4 KB per token, about 6 us at 16 tokens, whatever the token
// count.  Up to 4096 tokens that is one round of at most 256 workgroups.  Beyond,
// MT = 2: a wave multiplies every gate fragment it loads with two 16-token
// fragments, a workgroup owns 32 tokens and the launch stays one round up to 8192
// tokens.  Under the 128 registers a wave of a 16-wave workgroup gets, the loads then
// go out as two batches of two steps instead of one of four, which gives back most of
// what the halved gate traffic saves (8192 tokens: 22.7 instead of 25 us).  The partial
// sums of 16 waves x 2 token fragments would not fit the LDS at once: the upper eight
// waves hand theirs to the lower eight, which add their own and publish the sums.
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kRmTok = 16;
// 16 waves per workgroup: a workgroup is a chain of dependent steps (loads, reduction,
// softmax, Top-K) and at most a few workgroups run per compute unit, so a wave's share of
// the hidden dimension should be one batch of loads and a wave should finish one token
constexpr int kRmWaves = 16;

// Selection, dispatch and tile map (plan.hip) of at most kRoutePlanTokens tokens by the workgroup that routed them,
// from the candidates it holds in LDS.  An entry of the pool is kept iff fewer than `want` precede it in the
// order (key descending, index ascending): with at most 256 entries every one is compared with all others, no
// search.  A chain of LDS round trips and four barriers; as a launch of its own behind the routing kernel the stage
// begins with a trip to memory for what is here already.  Layer of 64 experts of 2048 x 1408 and a shared expert: 1
// token 33.6 us, 30.8 now; 2: 45.0, 41.5; 16: 88.6, 85.2; 32 experts of 512 x 256, 2 tokens 18.2, 15.0.  From 17
// tokens on the routing would no longer be one fragment of tokens a wave: with two, 24 tokens 101.2, 103.2; 32: 148.7,
// 152.0.
struct PlanSmall {
    int Kb;
    int64_t B;
    int32_t *keep_count, *expert_offsets, *row_token, *row_rank, *inv_row;
    int bm;
    int32_t* tile_info;
};

struct PlanSmallShared {
    static constexpr int kTokens = kRoutePlanTokens, kPairs = kTokens * 16;   // (16: the most candidates of a token)
    int32_t ids[kPairs];
    float s[kPairs], keys[kPairs];
    alignas(16) uint32_t pool[kPairs];   // ordered keys, [token][rank - K_base]; 0 past the end
    uint8_t kept[kPairs];
    uint64_t words[kWave];               // of an expert: who keeps it
    int32_t expert_off[kWave + 1];
    int32_t cnt[kTokens];
    __device__ void clear() {
        if (threadIdx.x < kPairs) pool[threadIdx.x] = 0u;
    }
};

struct SmallPool {
    PlanSmallShared& sh;
    int Kb, K;
    __device__ void put(size_t first, int k, uint32_t key) const {   // first: token * K
        if (k >= Kb) sh.pool[static_cast<int>(first) / K * (K - Kb) + k - Kb] = key;
    }
};

__device__ __forceinline__ void plan_small(PlanSmallShared& sh, const PlanSmall& a, int T, int K, int E,
                                           int32_t* __restrict__ topk_ids, float* __restrict__ topk_s, const SelKeys& sel) {
    constexpr int kPer = 4;   // threads to an entry
    static_assert(kPer * PlanSmallShared::kPairs == kRmWaves * kWave, "every entry has its threads");
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int pairs = T * K, P = K - a.Kb, n_pool = T * P;
    const int64_t want = a.B - static_cast<int64_t>(T) * a.Kb;
    const bool search = want > 0 && want < n_pool;
    __syncthreads();
    if (tid < pairs) {
        topk_ids[tid] = sh.ids[tid];
        topk_s[tid] = sh.s[tid];
        if (sel.mode != 0) sel.keys[tid] = sh.keys[tid];
    }
    if (search) {
        const int p = tid / kPer;
        const uint32_t mine = sh.pool[p];
        int before = 0;
        for (int q = 4 * (tid % kPer); q < n_pool; q += 4 * kPer) {   // (entries past the end hold 0: none is larger)
            const uint4 v = *reinterpret_cast<const uint4*>(&sh.pool[q]);
            const uint32_t o[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) before += o[i] > mine || (o[i] == mine && q + i < p) ? 1 : 0;
        }
        before += static_cast<int>(lane_xor<1>(static_cast<uint32_t>(before)));
        before += static_cast<int>(lane_xor<2>(static_cast<uint32_t>(before)));
        if (tid % kPer == 0) sh.kept[p] = before < want ? 1 : 0;
        __syncthreads();
    }
    if (wave == 0) {   // lane = token, then lane = expert
        int kt = 0;
        uint64_t mine = 0;
        if (lane < T) {
            kt = want <= 0 ? a.Kb : K;
            if (search) {   // (the kept candidates of a token are its first)
                kt = a.Kb;
                for (int j = 0; j < P; ++j) kt += sh.kept[lane * P + j];
            }
            for (int j = 0; j < K; ++j)
                mine |= static_cast<uint64_t>(j < kt ? 1u : 0u) << (sh.ids[lane * K + j] & (kWave - 1));
            sh.cnt[lane] = kt;
            a.keep_count[lane] = kt;
        }
        const uint64_t word = wave_transpose64(mine);
        sh.words[lane] = word;
        const int incl = wave_scan_incl(lane < E ? __popcll(word) : 0);
        sh.expert_off[lane + 1] = incl;
        if (lane == 0) sh.expert_off[0] = 0;
        if (lane < E) a.expert_offsets[lane + 1] = incl;
        if (lane == 0) a.expert_offsets[0] = 0;
    }
    __syncthreads();
    if (wave == kRmWaves - 1) write_tile_map(sh.expert_off, E, a.bm, a.tile_info, static_cast<int>(a.B));
    if (tid < pairs) {
        const int t = tid / K, j = tid - t * K, e = sh.ids[tid] & (kWave - 1);
        int row = -1;
        if (j < sh.cnt[t]) {
            row = sh.expert_off[e] + __popcll(sh.words[e] & ((1ull << t) - 1ull));
            a.row_token[row] = t;
            a.row_rank[row] = j;
        }
        a.inv_row[tid] = row;
    }
}

// 16-column blocks of the gate matrix; partial sums that meet in LDS
constexpr int route_blocks(bool gate) { return gate ? kGateBlocks : kGateBlocks - 1; }
constexpr int route_slots(int mt) { return mt == 1 ? kRmWaves : kRmWaves / 2; }
template <bool GATE, int MT>
using RouteSums = float[route_slots(MT)][MT][route_blocks(GATE)][4][kWave];

// PLAN: the one workgroup goes on with selection and dispatch (plan_small).
template <bool GATE, int MT, bool PLAN>
__device__ __forceinline__ void route_mfma_body(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Gp, const float* __restrict__ bias,
    int T, int d, int E, int K, float* __restrict__ scores, int32_t* __restrict__ topk_ids,
    float* __restrict__ topk_s, float* __restrict__ sgate, const SelKeys& sel, const PlanSmall& plan,
    RouteSums<GATE, MT>& red) {
    static_assert(MT == 1 || MT == 2, "token fragments per wave");
    constexpr int NB = route_blocks(GATE), kSlots = route_slots(MT);
    __shared__ typename std::conditional<PLAN, PlanSmallShared, int>::type small;

    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int t0 = PLAN ? 0 : blockIdx.x * (kRmTok * MT);
    if constexpr (PLAN) small.clear();
    const int KB = d / 32;
    const int per_wave = (KB + kRmWaves - 1) / kRmWaves;
    const int s0 = min(KB, wave * per_wave), s1 = min(KB, s0 + per_wave);

    const int m = lane % 16, kg = lane / 16;
    bool a_ok[MT];
    const bf16x8* ap[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int t = t0 + kRmTok * mt + m;
        a_ok[mt] = t < T;
        ap[mt] = reinterpret_cast<const bf16x8*>(X + static_cast<size_t>(a_ok[mt] ? t : 0) * d) + kg;
    }
    const bf16x8* bp = reinterpret_cast<const bf16x8*>(Gp) + lane;

    f32x4 acc[MT][NB];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mt][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {0};
    constexpr int U = MT == 1 ? 4 : 2;   // steps per batch of loads (registers: 16 waves, 128 each)
    int s = s0;
    for (; s + U <= s1; s += U) {
        bf16x8 av[U][MT], bv[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) av[u][mt] = a_ok[mt] ? ap[mt][(s + u) * 4] : zero;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                bv[u][nb] = bp[(static_cast<size_t>(nb) * KB + s + u) * kWave];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[mt][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u][mt], bv[u][nb],
                                                                          acc[mt][nb], 0, 0, 0);
    }
    for (; s < s1; ++s) {
        bf16x8 av[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[mt] = a_ok[mt] ? ap[mt][s * 4] : zero;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const bf16x8 bv = bp[(static_cast<size_t>(nb) * KB + s) * kWave];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[mt], bv, acc[mt][nb], 0, 0, 0);
        }
    }
    // accumulator register r of lane l holds C[4*(l/16) + r][l%16]
    if (MT == 1 || wave >= kSlots) {
        const int slot = MT == 1 ? wave : wave - kSlots;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[slot][mt][nb][r][lane] = acc[mt][nb][r];
    }
    __syncthreads();
    if (MT == 2) {
        if (wave < kSlots) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        red[wave][mt][nb][r][lane] = acc[mt][nb][r] + red[wave][mt][nb][r][lane];
        }
        __syncthreads();
    }

    // wave w finishes token w of every token fragment
    const bool lane_is_expert = lane < E;
    const int r = wave % 4, lsrc = 16 * (wave / 4);
    float sc[MT];
    bool live[MT];
    size_t at[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int t = t0 + kRmTok * mt + wave;
        live[mt] = t < T;
        const size_t tt = live[mt] ? t : 0;
        at[mt] = tt * K;
        float logit = 0.f;
#pragma unroll
        for (int w = 0; w < kSlots; ++w) logit += red[w][mt][lane / 16][r][lsrc + lane % 16];
        if (bias != nullptr && lane_is_expert) logit += bias[lane];
        if (!lane_is_expert) logit = -INFINITY;
        const float mx = wave_max(logit);
        const float p = lane_is_expert ? expf(logit - mx) : 0.f;
        const float den = wave_sum(p);
        sc[mt] = p / den;
        if (live[mt] && scores != nullptr && lane_is_expert) scores[tt * E + lane] = sc[mt];
    }
    if constexpr (PLAN)
        wave_topk_store_n<MT>(sc, lane_is_expert, K, small.ids, small.s, SelKeys{sel.mode, small.keys}, at, live,
                              SmallPool{small, plan.Kb, K});
    else
        wave_topk_store_n<MT>(sc, lane_is_expert, K, topk_ids, topk_s, sel, at, live);
    if (GATE && lane == 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (!live[mt]) continue;
            float g = 0.f;
#pragma unroll
            for (int w = 0; w < kSlots; ++w) g += red[w][mt][NB - 1][r][lsrc];
            sgate[t0 + kRmTok * mt + wave] = 1.f / (1.f + expf(-g));
        }
    }
    if constexpr (PLAN) plan_small(small, plan, T, K, E, topk_ids, topk_s, sel);
}

template <bool GATE, int MT>
__global__ __launch_bounds__(kRmWaves* kWave) void route_mfma_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Gp, const float* __restrict__ bias,
    int T, int d, int E, int K, float* __restrict__ scores, int32_t* __restrict__ topk_ids,
    float* __restrict__ topk_s, float* __restrict__ sgate, SelKeys sel) {
    __shared__ RouteSums<GATE, MT> red;
    route_mfma_body<GATE, MT, false>(X, Gp, bias, T, d, E, K, scores, topk_ids, topk_s, sgate, sel, PlanSmall{}, red);
}

template <bool GATE>
__global__ __launch_bounds__(kRmWaves* kWave) void route_plan_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Gp, const float* __restrict__ bias,
    int T, int d, int E, int K, float* __restrict__ scores, int32_t* __restrict__ topk_ids,
    float* __restrict__ topk_s, float* __restrict__ sgate, SelKeys sel, PlanSmall plan) {
    __shared__ RouteSums<GATE, 1> red;
    route_mfma_body<GATE, 1, true>(X, Gp, bias, T, d, E, K, scores, topk_ids, topk_s, sgate, sel, plan, red);
}

// The same, and beside it on the other compute units the first half of the shared expert, which depends on
// nothing but X: workgroup 0 routes, selects and dispatches, the others stream.  The routing
// workgroup is a chain of dependent steps with the chip idle (9-10 us at 16 tokens, 11 with the others beside it,
// whose share of the layer's weights is a third to a tenth).  A unit has one workgroup of 16 waves, which take a
// column block's steps in turn; four steps in flight a wave are 128 KB a unit.  (Six and eight do not fit the 128
// registers: 16 tokens 83.5 and 97.4 us.  With 8-bit weights three: four registers spill with a ring of four, which takes
// the same time, 1.000 in the mean of 18 layers of 1 to 16 tokens.)  Layer of 64 experts of 2048 x 1408, shared expert of 2816, streaming behind the routing workgroup and
// beside it: 1 token 31.1 us, 30.5; 8: 69.5, 65.0; 16: 85.3, 80.8; 60 experts, shared expert of 5632: 1 token 42.1 before
// either, 34.8.  Beside the routing alone of 17 and more tokens it takes longer than the routing: 32 tokens 147.2, 150.4.
template <bool FP8>
constexpr int kSharedRing = FP8 ? 3 : 4;
template <bool GATE, bool FP8>
__global__ __launch_bounds__(kRmWaves* kWave) void route_shared_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ Gp, const float* __restrict__ bias,
    int T, int d, int E, int K, float* __restrict__ scores, int32_t* __restrict__ topk_ids,
    float* __restrict__ topk_s, float* __restrict__ sgate, SelKeys sel, PlanSmall plan, StreamArgs shared) {
    typedef float StreamSums[kRmWaves][2][16][kWave];
    __shared__ __attribute__((aligned(16))) char sums[std::max(sizeof(RouteSums<GATE, 1>), sizeof(StreamSums))];
    if (blockIdx.x == 0)
        route_mfma_body<GATE, 1, true>(X, Gp, bias, T, d, E, K, scores, topk_ids, topk_s, sgate, sel, plan,
                                       reinterpret_cast<RouteSums<GATE, 1>&>(sums));
    else
        stream_body<true, FP8, kSharedRing<FP8>, 2, kRmWaves>(shared, blockIdx.x - 1, reinterpret_cast<StreamSums&>(sums));
}

// Candidates from caller-supplied scores: one wave per token.
__global__ __launch_bounds__(256) void topk_from_scores_kernel(
    const float* __restrict__ scores, int T, int E, int K, int32_t* __restrict__ topk_ids,
    float* __restrict__ topk_s, SelKeys sel) {
    const int lane = lane_id();
    const int t = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (t >= T) return;
    const bool valid = lane < E;
    const float s = valid ? scores[static_cast<size_t>(t) * E + lane] : 0.f;
    wave_topk_store(s, valid, K, topk_ids, topk_s, sel, static_cast<size_t>(t) * K);
}

namespace {

template <typename TIn, int WAVES>
void enqueue_route(const void* X, const void* Wg, const float* bias, const void* w_sg, int T, int d,
                   int E, int K, float* scores, int32_t* topk_ids, float* topk_s, float* sgate,
                   SelKeys sel, hipStream_t stream) {
    hipLaunchKernelGGL((route_kernel<TIn, WAVES>), dim3((T + kRouteTok - 1) / kRouteTok),
                       dim3(WAVES * kWave), 0, stream, static_cast<const TIn*>(X),
                       static_cast<const TIn*>(Wg), bias, static_cast<const TIn*>(w_sg), T, d, E, K,
                       scores, topk_ids, topk_s, sgate, sel);
}

}  // namespace

hipError_t launch_route(int dtype, const void* X, const void* Wg, const float* bias,
                        const void* w_sg, int T, int d, int E, int K, float* scores,
                        int32_t* topk_ids, float* topk_s, float* sgate, int sel_mode, float* sel_keys,
                        hipStream_t stream) {
    // Waves per workgroup, splitting d.  Few tokens are a chain of loads of the gate matrix: 16
    // waves keep a wave's share of it to a chunk or two (16 tokens, d 2048: 4 waves 30.0 us, 16
    // waves 19.4; d 384: 11.9, 9.6).  From four chunks of 64 down 4 waves hold one each and the
    // others would have nothing to do but fill the compute unit (d 128: 1 token 7.7 both, 8192
    // tokens 34.0 and 44.7).  With many tokens the short chains of several small workgroups
    // overlap (d 512: 4096 tokens 35.7 and 35.9, 8192: 52.9 and 54.1, 65536: 249 and 316; d
    // 2048: 8192 tokens 130 and 126, 65536: 830 and 842).  (A launch has less than 2^32 threads:
    // 16 waves end at 2^24 tokens, 4 at 2^26.)
    const bool many = d > 4 * kWave && T < (d <= 12 * kWave ? 8192 : 65536);
    const auto enqueue = dtype == 0 ? (many ? enqueue_route<float, 16> : enqueue_route<float, 4>)
                                    : (many ? enqueue_route<bf16_t, 16> : enqueue_route<bf16_t, 4>);
    enqueue(X, Wg, bias, w_sg, T, d, E, K, scores, topk_ids, topk_s, sgate, {sel_mode, sel_keys}, stream);
    return hipGetLastError();
}

hipError_t launch_route_mfma(const void* X, const void* gate_packed, const float* bias,
                             bool with_gate, int T, int d, int E, int K, float* scores,
                             int32_t* topk_ids, float* topk_s, float* sgate, int sel_mode,
                             float* sel_keys, hipStream_t stream) {
    const SelKeys sel{sel_mode, sel_keys};
    const bf16_t* Xb = static_cast<const bf16_t*>(X);
    const bf16_t* Gp = static_cast<const bf16_t*>(gate_packed);
    const dim3 block(kRmWaves * kWave);
    // 32 tokens per workgroup where 16 would need more workgroups than compute units
    const bool wide = T > 256 * kRmTok;
    const int per_group = wide ? 2 * kRmTok : kRmTok;
    const dim3 grid((T + per_group - 1) / per_group);
#define ALLOCMOE_ROUTE_LAUNCH(gate, mt)                                                            \
    hipLaunchKernelGGL((route_mfma_kernel<gate, mt>), grid, block, 0, stream, Xb, Gp, bias, T, d,  \
                       E, K, scores, topk_ids, topk_s, sgate, sel)
    if (with_gate && wide)
        ALLOCMOE_ROUTE_LAUNCH(true, 2);
    else if (with_gate)
        ALLOCMOE_ROUTE_LAUNCH(true, 1);
    else if (wide)
        ALLOCMOE_ROUTE_LAUNCH(false, 2);
    else
        ALLOCMOE_ROUTE_LAUNCH(false, 1);
#undef ALLOCMOE_ROUTE_LAUNCH
    return hipGetLastError();
}

hipError_t launch_route_few(const void* X, const void* gate_packed, const float* bias, bool with_gate, int T,
                            int d, int E, int K, int Kb, int64_t B, float* scores, int32_t* topk_ids, float* topk_s,
                            float* sgate, int sel_mode, float* sel_keys, int32_t* keep_count,
                            int32_t* expert_offsets, int32_t* row_token, int32_t* row_rank, int32_t* inv_row, int bm,
                            int32_t* tile_info, const StreamGroup& shared, hipStream_t stream) {
    const SelKeys sel{sel_mode, sel_keys};
    const PlanSmall plan{Kb, B, keep_count, expert_offsets, row_token, row_rank, inv_row, bm, tile_info};
    const bf16_t* Xb = static_cast<const bf16_t*>(X);
    const bf16_t* Gp = static_cast<const bf16_t*>(gate_packed);
    const dim3 block(kRmWaves * kWave);
    if (shared.A == nullptr) {
        hipLaunchKernelGGL(with_gate ? route_plan_kernel<true> : route_plan_kernel<false>, dim3(1), block, 0, stream, Xb,
                           Gp, bias, T, d, E, K, scores, topk_ids, topk_s, sgate, sel, plan);
        return hipGetLastError();
    }
    const StreamArgs sh{static_cast<const char*>(shared.A), static_cast<const char*>(shared.Bp), nullptr, nullptr,
                        shared.scale, static_cast<bf16_t*>(shared.C), shared.group_stride, shared.lda, shared.ldc,
                        shared.Kd, shared.N, shared.M_dense};
    const bool fp8 = shared.scale != nullptr;
    const auto kernel = with_gate ? (fp8 ? route_shared_kernel<true, true> : route_shared_kernel<true, false>)
                                  : (fp8 ? route_shared_kernel<false, true> : route_shared_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(1 + shared.N / 32), block, 0, stream, Xb, Gp, bias, T, d, E, K, scores, topk_ids,
                       topk_s, sgate, sel, plan, sh);
    return hipGetLastError();
}

hipError_t launch_topk_from_scores(const float* scores, int T, int E, int K, int32_t* topk_ids,
                                   float* topk_s, int sel_mode, float* sel_keys, hipStream_t stream) {
    const int waves = 4;
    const dim3 grid((T + waves - 1) / waves), block(waves * kWave);
    hipLaunchKernelGGL(topk_from_scores_kernel, grid, block, 0, stream, scores, T, E, K, topk_ids,
                       topk_s, SelKeys{sel_mode, sel_keys});
    return hipGetLastError();
}

}  // namespace allocmoe
