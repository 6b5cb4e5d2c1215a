// One-time re-tiling of row-major bf16 weight matrices W[g][k][n] into the
// operand order of v_mfma_f32_32x32x16_bf16, so that the per-batch kernels load
// B fragments with one contiguous 16-byte load per lane.
//
// A fragment covers 16 k x 32 n: lane l holds the 8 values
//   W[16*kb + 8*(l/32) + i][32*nb + l%32],  i = 0..7,
// stored as 64 lanes x 16 bytes = 1 KB.  The fragments of one column block nb
// are contiguous along k (kb = 0 .. Kd/16-1).  Destination of fragment
// (g, nb, kb):  out + g*group_stride + nb*nblock_stride + base_off + kb*512.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace allocmoe {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Re-tiles the gate matrix Wg [d,E] (and, as column 64, the shared expert's
// gate vector w_sg [d]) into the B-operand order of v_mfma_f32_16x16x32_bf16:
// fragment (nb, s) = 64 lanes x 8 values, lane l holding
//   G[32 s + 8 (l/16) + i][16 nb + l%16],  i = 0..7,
// with G's columns E..63 and 65..79 zero.  Layout: [nb][s][lane][8].  Done by the first
// workgroups of the expert matrices' launch, beside them (a launch of its own behind them:
// 4-7 us).
__device__ __forceinline__ void pack_gate(const PackGate& G, int64_t idx) {
    const int KB = G.d / 32;
    if (idx >= static_cast<int64_t>(kGateBlocks) * KB * kWave) return;
    const bf16_t *Wg = static_cast<const bf16_t*>(G.Wg), *w_sg = static_cast<const bf16_t*>(G.w_sg);
    const int l = idx % kWave, s = (idx / kWave) % KB, nb = static_cast<int>(idx / (static_cast<int64_t>(kWave) * KB));
    const int n = 16 * nb + l % 16, k0 = 32 * s + 8 * (l / 16);
    bf16_t* dst = static_cast<bf16_t*>(G.out) + static_cast<size_t>(idx) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        bf16_t v = 0;
        if (n < G.E)
            v = Wg[static_cast<size_t>(k0 + i) * G.E + n];
        else if (n == 64 && w_sg != nullptr)
            v = w_sg[k0 + i];
        dst[i] = v;
    }
}

// workgroups of a launch that re-tile the gate matrix: whole rounds over the XCDs
constexpr int kPackXcds = 8;
constexpr int kPackGroup = 16;   // neighbouring column blocks of an XCD
inline int gate_workgroups(const PackGate& G, int threads) {
    const int64_t pieces = static_cast<int64_t>(kGateBlocks) * (G.d / 32) * kWave;
    return static_cast<int>((pieces + threads * kPackXcds - 1) / (threads * kPackXcds) * kPackXcds);
}

// A lane gathers its 8 values (a wave-load covers 64 bytes of a row; the four waves of a
// workgroup go down the rows) and stores them as one piece, past the caches (the packed matrices
// are larger than those).  Bound by HBM: 64 experts of 2048 x 1408 and a shared expert, 2.2 GB in
// and out, take 388 us (5.7 TB/s).  An XCD takes neighbouring column blocks, so that the halves
// of a line meet in its L2 and rows are read in runs of 1 KB (consecutive workgroups down the
// rows of one column block instead, with plain stores: 418 us; 32 experts of 1088 x 704 and a
// shared expert 70, now 46; 60 of 1472 x 1024 217, 183).  Whole 256-byte row pieces per wave,
// turned in registers, were slower (467 us).  All matrices of a layer go in one launch: with a
// launch each, a layer of 16 experts of 576 x 320 took 17.4 us instead of 12.8 (8.3 with the gate
// matrix in the launch as well).
__global__ __launch_bounds__(256) void pack_b_kernel(PackJobs jobs) {
    if (static_cast<int>(blockIdx.x) < jobs.gate.n_wg) {
        pack_gate(jobs.gate, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x);
        return;
    }
    // (XCDs as in the 8-bit kernel: an XCD takes kPackGroup neighbouring column blocks of the same
    // rows one after the other)
    const int64_t wg = static_cast<int64_t>(blockIdx.x) - jobs.gate.n_wg;
    const int xcd = wg % kPackXcds;
    const int64_t idx = wg / kPackXcds;
    int64_t bid = jobs.first_wg + (idx / kPackGroup * kPackXcds + xcd) * kPackGroup + idx % kPackGroup;
    int jn = 0;
    while (bid >= jobs.job[jn].n_wg) {
        bid -= jobs.job[jn++].n_wg;
        if (jn == jobs.n) return;
    }
    const PackJob& J = jobs.job[jn];
    const int N = J.N, NB = N / 32, KQ = J.Kd / 64;   // a workgroup: four fragments of a column block
    const int l = lane_id(), nb = static_cast<int>(bid % NB);
    const int kb = 4 * static_cast<int>(bid / NB % KQ) + threadIdx.x / kWave;
    const int g = static_cast<int>(bid / NB / KQ);
    const int n = nb * 32 + (l % 32), k0 = kb * 16 + 8 * (l / 32);
    const bf16_t* src = static_cast<const bf16_t*>(J.W) + (static_cast<size_t>(g) * J.Kd + k0) * N + n;
    bf16_t* dst = static_cast<bf16_t*>(J.out) + static_cast<size_t>(g) * J.group_stride +
                  static_cast<size_t>(nb) * J.nblock_stride + J.base_off +
                  static_cast<size_t>(kb) * 512 + static_cast<size_t>(l) * 8;
    uint32_t packed[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = src[static_cast<size_t>(2 * i) * N];
        const uint32_t hi = src[static_cast<size_t>(2 * i + 1) * N];
        packed[i] = lo | (hi << 16);
    }
    __builtin_nontemporal_store(u32x4{packed[0], packed[1], packed[2], packed[3]}, reinterpret_cast<u32x4*>(dst));
}

// ---- 8-bit expert weights (E4M3 codes, one fp32 scale per output column)

// E4M3 of the OCP 8-bit floating point format: sign, 4 exponent bits (bias 7), 3 mantissa
// bits, subnormals, no infinities, largest finite magnitude 448.  Nearest code, ties to
// the even mantissa: the conversion unit's rounding.  Byte i of the result = code of y[i].
__device__ __forceinline__ uint32_t e4m3_encode4(const float (&y)[4]) {
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], w, true);
    return static_cast<uint32_t>(w);
}

// A workgroup owns 32 columns (64 bytes of every row: one column block of fragments) of one
// matrix.  Its 8 waves hold 2048 rows of the strip in registers, so the matrix is read once:
// lane 8 b + 4 h + t of wave w has columns 8 t .. + 7 of the 16 rows that make the pieces of
// half h (lanes 32 h .. of a fragment) of k block 8 w + b.  The column maxima are formed from
// the registers (lanes, then LDS), and the codes are turned in LDS, wave by wave, so that
// they leave as whole fragments (1 KB per store).  Longer columns are read twice, in chunks
// of 2048 rows.  All six matrices of a layer go in one launch, so that the shared expert's few
// strips fill up the others' last round.  Bound by HBM: 64 experts of 2048 x 1408 and a shared
// expert, 1.7 GB in and out, take 326 us (5.2 TB/s).  Two workgroups to a unit, so that one reads
// while the other converts or writes: with strips of 64 columns, which fill a unit's registers,
// and 16-byte stores 64 bytes apart it was 455 us.  Pairs of strips to an XCD instead of groups
// of 16: 368 us, with non-temporal loads (which do not wait in L2 for the line's other half) 403;
// neighbouring strips on different XCDs 570; plain stores 375 instead of 368.
constexpr int kPackWaves = 8, kPackWaveRows = 256, kPackRows = kPackWaves * kPackWaveRows, kPackCols = 32;

__global__ __launch_bounds__(kPackWaves* kWave, 4) void pack_fp8_kernel(PackFp8Jobs jobs) {
    __shared__ uint32_t wave_max[kPackWaves][kPackCols / 2];   // two columns' magnitudes each
    __shared__ float2 col_scale[kPackCols];   // and its reciprocal
    __shared__ u32x4 turn[kPackWaves][kPackWaveRows * kPackCols / 16];
    if (static_cast<int>(blockIdx.x) < jobs.gate.n_wg) {
        pack_gate(jobs.gate, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x);
        return;
    }
    // Workgroups are dealt to the XCDs in turn: an XCD takes kPackGroup neighbouring strips one
    // after the other.  Two of them share every 128-byte line, and the rows then are read in
    // runs of 1 KB.
    const int wg = blockIdx.x - jobs.gate.n_wg, xcd = wg % kPackXcds, idx = wg / kPackXcds;
    int bid = jobs.first_strip + (idx / kPackGroup * kPackXcds + xcd) * kPackGroup + idx % kPackGroup, jn = 0;
    while (bid >= jobs.job[jn].n_strips) {
        bid -= jobs.job[jn++].n_strips;
        if (jn == jobs.n) return;
    }
    const PackFp8Job& J = jobs.job[jn];
    const int N = J.N, Kd = J.Kd, strips = N / kPackCols;
    const int g = bid / strips, n0 = bid % strips * kPackCols;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int t = lane % 4, h = lane / 4 % 2, kb = lane / 8;
    const int row_lane = kPackWaveRows * wave + 32 * kb + 8 * h;   // rows + 0 .. 7 and + 16 .. 23
    const bf16_t* src = static_cast<const bf16_t*>(J.W) + static_cast<size_t>(g) * Kd * N + n0;
    typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
    // (a matrix may start at any element)
    typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
    u32x4_any v[16];
    auto load = [&](int row0) {   // (past the end, Kd being a multiple of 32: the lane's rows of the last k block)
        const bf16_t* p = src + static_cast<size_t>(min(row0, Kd - 32 + 8 * h)) * N + 8 * t;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            v[r] = *reinterpret_cast<const u32x4_any*>(p);
            p += static_cast<size_t>(r == 7 ? 9 : 1) * N;
        }
    };
    // Magnitudes of bf16 values compare like their bit patterns.  A NaN must not count (its
    // pattern is above infinity's and would be the maximum): with 0x7F added the patterns up
    // to infinity's (0x7F80) stay below 0x8000, those of NaNs become negative.
    constexpr int16_t kShift = 0x7F;
    i16x2 m[4], low = i16x2{kShift, kShift};   // low: negative once a NaN was seen
#pragma unroll
    for (int q = 0; q < 4; ++q) m[q] = i16x2{kShift, kShift};
    for (int c = 0; c < Kd; c += kPackRows) {
        if (c + kPackWaveRows * wave >= Kd) break;   // (the wave has no rows in this chunk)
        load(c + row_lane);
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const i16x2 x = __builtin_bit_cast(i16x2, (v[r][q] & 0x7FFF7FFFu) + kShift * 0x10001u);
                m[q] = __builtin_elementwise_max(m[q], x);
                low = __builtin_elementwise_min(low, x);
            }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // over the lanes with the same columns
        auto fold = [&](uint32_t other) {
            m[q] = __builtin_elementwise_max(m[q], __builtin_bit_cast(i16x2, other));
        };
        fold(lane_xor<4>(__builtin_bit_cast(uint32_t, m[q])));
        fold(lane_xor<8>(__builtin_bit_cast(uint32_t, m[q])));
        fold(lane_xor<16>(__builtin_bit_cast(uint32_t, m[q])));
        fold(lane_xor<32>(__builtin_bit_cast(uint32_t, m[q])));
        if (lane < 4) wave_max[wave][4 * t + q] = __builtin_bit_cast(uint32_t, m[q]);
    }
    __syncthreads();
    if (tid < kPackCols) {
        uint32_t top = kShift;
#pragma unroll
        for (int w = 0; w < kPackWaves; ++w) top = max(top, (wave_max[w][tid / 2] >> (16 * (tid % 2))) & 0xFFFFu);
        const float amax = __uint_as_float((top - kShift) << 16);
        const float sc = amax > 0.f ? __fdiv_rn(amax, 448.f) : 1.f;
        col_scale[tid] = make_float2(sc, __fdiv_rn(1.f, sc));
        J.scale[static_cast<size_t>(g) * J.scale_stride + n0 + tid] = sc;
    }
    __syncthreads();
    bool plain = low[0] >= 0 && low[1] >= 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float sc = col_scale[8 * t + j].x;
        plain = plain && sc > 0x1p-80f && sc < 0x1p80f;
    }
    // Plain columns: w / sc by the quotient estimate and one correction by the exact remainder.
    // That is the correctly rounded quotient for every magnitude of w (8 significant bits) and
    // every scale a column of such magnitudes can have (128 mantissas: the pairs were compared
    // one by one, tests/test_quant.py), where the scale's exponent is moderate (a value so
    // small that a remainder underflows is far below half the smallest code and becomes zero
    // either way).  The remainder is formed with its sign turned, which keeps a zero's.  The
    // quotient's magnitude is at most 448 and an ulp, which rounds to 448.
    auto quotient = [](float w, float2 sc) {
        const float q = w * sc.y;
        return fmaf(-fmaf(q, sc.x, -w), sc.y, q);
    };
    // Others: the full division; above 448 saturates, and so does a NaN, with its sign (the
    // minimum passes over it).
    auto saturated = [](float w, float2 sc) {
        const float y = __fdiv_rn(w, sc.x);
        return copysignf(fminf(fabsf(y), 448.f), y);
    };
    char* out = static_cast<char*>(J.out) + static_cast<size_t>(g) * J.group_stride + J.base_off +
                static_cast<size_t>(n0 / kPackCols) * J.nblock_stride;
    u32x4* my = turn[wave];
    // Piece 32 h + n of a fragment stands at position p ^ x of its 64 in LDS, x such that 16
    // neighbouring lanes write 16 different 16-byte units of the 256 bytes the banks span (on
    // the way out the lanes read within the same eight units).
    const int x_in = (t >> 1) | (h << 1) | ((kb & 1) << 2), at_lane = 64 * kb + 32 * h + 8 * t;
    auto turn_codes = [&](auto fast) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float2 sc = col_scale[8 * t + j];
            uint32_t word[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t pair = v[4 * q + i][j / 2];
                    const float w = __uint_as_float((j % 2) ? (pair & 0xFFFF0000u) : (pair << 16));
                    y[i] = decltype(fast)::value ? quotient(w, sc) : saturated(w, sc);
                }
                word[q] = e4m3_encode4(y);
            }
            int at = x_in;
            asm("" : "+v"(at));   // (eight positions kept in registers would not fit beside the strip)
            my[at_lane + (j ^ at)] = u32x4{word[0], word[1], word[2], word[3]};
            __builtin_amdgcn_sched_barrier(0);   // one piece at a time: the strip fills the registers
        }
    };
    const bool all_plain = __all(plain);
    for (int c = 0; c < Kd; c += kPackRows) {
        const int first = c + kPackWaveRows * wave;
        if (first >= Kd) break;
        if (Kd > kPackRows) load(c + row_lane);
        if (all_plain)
            turn_codes(std::true_type{});
        else
            turn_codes(std::false_type{});
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < kPackWaveRows / 32; ++i) {
            if (first + 32 * i >= Kd) break;
            const int x_out = ((lane >> 4) & 1) | ((lane >> 5) << 1) | ((i & 1) << 2);
            __builtin_nontemporal_store(my[64 * i + (lane ^ x_out)],
                                        reinterpret_cast<u32x4*>(out + static_cast<size_t>(first / 32 + i) * 1024 + lane * 16));
        }
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_pack_fp8(PackFp8Jobs jobs, hipStream_t stream) {
    int64_t strips = 0;
    for (int j = 0; j < jobs.n; ++j) {
        PackFp8Job& J = jobs.job[j];
        J.n_strips = J.G * (J.N / kPackCols);
        strips += J.n_strips;
    }
    // threads of a launch: 2^32 - 1; whole rounds of groups over the XCDs
    constexpr int64_t kRound = kPackGroup * kPackXcds, kMaxWg = (1ll << 32) / (kPackWaves * kWave) - 1;
    jobs.gate.n_wg = gate_workgroups(jobs.gate, kPackWaves * kWave);
    for (int64_t first = 0; first < strips;) {
        const int64_t n = std::min((kMaxWg - jobs.gate.n_wg) / kRound, (strips - first + kRound - 1) / kRound) * kRound;
        jobs.first_strip = static_cast<int>(first);
        hipLaunchKernelGGL(pack_fp8_kernel, dim3(static_cast<unsigned>(jobs.gate.n_wg + n)),
                           dim3(kPackWaves * kWave), 0, stream, jobs);
        first += n;
        jobs.gate.n_wg = 0;   // (done by the first launch)
    }
    return hipGetLastError();
}

hipError_t launch_pack_b(PackJobs jobs, hipStream_t stream) {
    int64_t wgs = 0;
    for (int j = 0; j < jobs.n; ++j) {
        PackJob& J = jobs.job[j];
        J.n_wg = static_cast<int64_t>(J.G) * (J.N / 32) * (J.Kd / 64);
        wgs += J.n_wg;
    }
    // a launch has less than 2^32 threads: layers of 3.4e10 weights take a second one
    constexpr int64_t kRound = kPackGroup * kPackXcds, kMaxWg = (1ll << 32) / 256 - 1;
    jobs.gate.n_wg = gate_workgroups(jobs.gate, 256);
    for (jobs.first_wg = 0; jobs.first_wg < wgs;) {
        const int64_t n = std::min((kMaxWg - jobs.gate.n_wg) / kRound, (wgs - jobs.first_wg + kRound - 1) / kRound) * kRound;
        hipLaunchKernelGGL(pack_b_kernel, dim3(static_cast<unsigned>(jobs.gate.n_wg + n)), dim3(256), 0, stream, jobs);
        jobs.first_wg += n;
        jobs.gate.n_wg = 0;   // (done by the first launch)
    }
    return hipGetLastError();
}

}  // namespace allocmoe
