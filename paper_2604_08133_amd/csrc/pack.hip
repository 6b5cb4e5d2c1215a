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

// A lane gathers its 8 values (a wave-load covers 64 bytes of a row; consecutive waves go down
// the rows, the neighbouring column block finds the other half of the lines in L2) and stores
// them as one piece.  Bound by HBM: 64 experts of 2048 x 1408 and a shared expert, 2.2 GB in
// and out, take 417 us (5.5 TB/s).  Whole 256-byte row pieces per wave, turned in registers, were slower
// there (467 us).  All matrices of a layer go in one launch: with a launch each, a layer of
// 16 experts of 576 x 320 took 17.4 us instead of 12.8, 32 experts of 1088 x 704 and a shared
// expert 80.6 instead of 69.6.
__global__ __launch_bounds__(256) void pack_b_kernel(PackJobs jobs) {
    int64_t bid = jobs.first_wg + blockIdx.x;
    int jn = 0;
    while (bid >= jobs.job[jn].n_wg) bid -= jobs.job[jn++].n_wg;
    const PackJob& J = jobs.job[jn];
    const int N = J.N, KB = J.Kd / 16, NB = N / 32;
    const size_t total = static_cast<size_t>(J.G) * NB * KB * kWave;
    const size_t idx = static_cast<size_t>(bid) * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int l = idx % kWave;
    size_t f = idx / kWave;
    const int kb = f % KB;
    f /= KB;
    const int nb = f % NB;
    const int g = f / NB;
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
    *reinterpret_cast<uint4*>(dst) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
}

// ---- 8-bit expert weights (E4M3 codes, one fp32 scale per output column)

// E4M3 of the OCP 8-bit floating point format: sign, 4 exponent bits (bias 7), 3 mantissa
// bits, subnormals, no infinities, largest finite magnitude 448.  Nearest code, ties to
// the even mantissa, magnitudes above 448 saturate: the conversion unit's rounding, on
// values that were clamped before.  A NaN saturates too, with its sign (the minimum passes
// over it).  Byte i of the result = code of y[i].
__device__ __forceinline__ uint32_t e4m3_encode4(const float (&y)[4]) {
    float c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = copysignf(fminf(fabsf(y[i]), 448.f), y[i]);
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w, true);
    return static_cast<uint32_t>(w);
}

// A workgroup owns 64 columns (128 bytes of every row) of one matrix.  Lane 16 g + t of wave
// w loads columns 4 t .. + 3 of the 32 rows of k block 4 w + g, i.e. the 16 waves hold 2048
// rows of the strip in registers: the matrix is read once, the column maxima are formed
// from the registers (lanes, then LDS), and the codes leave as whole 16-byte pieces of the
// fragments.  Longer columns are read twice, in chunks of 2048 rows.  All six matrices of a
// layer go in one launch, so that the shared expert's few strips fill up the others' last
// round.  Bound by HBM: 64 experts of 2048 x 1408 and a shared expert of 2048 x 2816, 1.7 GB
// in and out, take 460 us (3.7 TB/s; a 2 GiB copy reaches 5.0, the bf16 packing 5.5: here one
// workgroup fills a unit's registers, so that a unit reads or writes).  One thread per column for
// the maxima, then a second pass that read the matrices again, took 5.9 ms: 860 us per
// matrix for a serial chain of row loads, 258 us for the codes with two full divisions.
constexpr int kPackWaves = 16, kPackRows = kPackWaves * 4 * 32, kPackCols = 64;

__global__ __launch_bounds__(kPackWaves* kWave) void pack_fp8_kernel(PackFp8Jobs jobs) {
    __shared__ uint32_t wave_max[kPackWaves][kPackCols / 2];   // two columns' magnitudes each
    __shared__ float col_scale[kPackCols];
    int bid = jobs.first_strip + blockIdx.x, jn = 0;
    while (bid >= jobs.job[jn].n_strips) bid -= jobs.job[jn++].n_strips;
    const PackFp8Job& J = jobs.job[jn];
    const int N = J.N, Kd = J.Kd, strips = N / kPackCols;
    const int g = bid / strips, n0 = bid % strips * kPackCols;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int t = lane % 16, kb = wave * 4 + lane / 16;
    const bf16_t* src = static_cast<const bf16_t*>(J.W) + static_cast<size_t>(g) * Kd * N + n0 + 4 * t;
    typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
    // (a matrix may start at any element)
    typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
    u32x2_any v[32];
    auto load = [&](int row0) {   // (past the end, Kd being a multiple of 32: the last rows again)
        const bf16_t* p = src + static_cast<size_t>(min(row0, Kd - 32)) * N;
#pragma unroll
        for (int r = 0; r < 32; ++r)
            v[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x2_any*>(p + static_cast<size_t>(r) * N));
    };
    // Magnitudes of bf16 values compare like their bit patterns.  A NaN must not count (its
    // pattern is above infinity's and would be the maximum): with 0x7F added the patterns up
    // to infinity's (0x7F80) stay below 0x8000, those of NaNs become negative.
    constexpr int16_t kShift = 0x7F;
    i16x2 m[2] = {i16x2{kShift, kShift}, i16x2{kShift, kShift}};
    for (int c = 0; c < Kd; c += kPackRows) {
        load(c + kb * 32);
#pragma unroll
        for (int r = 0; r < 32; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                m[h] = __builtin_elementwise_max(m[h], __builtin_bit_cast(i16x2, (v[r][h] & 0x7FFF7FFFu) + kShift * 0x10001u));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // over the lanes with the same columns
        m[h] = __builtin_elementwise_max(m[h], __builtin_bit_cast(i16x2, lane_xor<16>(__builtin_bit_cast(uint32_t, m[h]))));
        m[h] = __builtin_elementwise_max(m[h], __builtin_bit_cast(i16x2, lane_xor<32>(__builtin_bit_cast(uint32_t, m[h]))));
        if (lane < 16) wave_max[wave][2 * t + h] = __builtin_bit_cast(uint32_t, m[h]);
    }
    __syncthreads();
    if (tid < kPackCols) {
        uint32_t top = kShift;
#pragma unroll
        for (int w = 0; w < kPackWaves; ++w) top = max(top, (wave_max[w][tid / 2] >> (16 * (tid % 2))) & 0xFFFFu);
        const float amax = __uint_as_float((top - kShift) << 16);
        const float sc = amax > 0.f ? __fdiv_rn(amax, 448.f) : 1.f;
        col_scale[tid] = sc;
        J.scale[static_cast<size_t>(g) * J.scale_stride + n0 + tid] = sc;
    }
    __syncthreads();
    float sc[4], rc[4];
    bool moderate = true;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        sc[j] = col_scale[4 * t + j];
        rc[j] = __fdiv_rn(1.f, sc[j]);
        moderate = moderate && sc[j] > 0x1p-80f && sc[j] < 0x1p80f;
    }
    // w / sc, correctly rounded: the quotient estimate and two corrections by the exact
    // remainder, as in the full division, whose scaling for extreme exponents is not needed
    // where the scale's exponent is moderate (a value so small that a remainder underflows
    // is far below half the smallest code and becomes zero either way; the sign of a zero,
    // which the remainders lose, is put back)
    auto quotient = [&](float w, int j) {
        const float q0 = w * rc[j];
        const float q1 = fmaf(fmaf(-q0, sc[j], w), rc[j], q0);
        return copysignf(fmaf(fmaf(-q1, sc[j], w), rc[j], q1), w);
    };
    char* out = static_cast<char*>(J.out) + static_cast<size_t>(g) * J.group_stride + J.base_off;
    auto store_codes = [&](int row0, auto short_division) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + 4 * t + j;
            char* frag = out + static_cast<size_t>(n / 32) * J.nblock_stride + static_cast<size_t>(row0 / 32) * 1024;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t word[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t pair = v[16 * (q / 2) + 8 * h + 4 * (q % 2) + i][j / 2];
                        const float w = __uint_as_float((j % 2) ? (pair & 0xFFFF0000u) : (pair << 16));
                        y[i] = decltype(short_division)::value ? quotient(w, j) : __fdiv_rn(w, sc[j]);
                    }
                    word[q] = e4m3_encode4(y);
                }
                *reinterpret_cast<uint4*>(frag + (32 * h + n % 32) * 16) = make_uint4(word[0], word[1], word[2], word[3]);
                __builtin_amdgcn_sched_barrier(0);   // one piece at a time: the strip fills the registers
            }
        }
    };
    const bool all_moderate = __all(moderate);
    for (int c = 0; c < Kd; c += kPackRows) {
        const int row0 = c + kb * 32;
        if (Kd > kPackRows) load(row0);
        if (row0 >= Kd) continue;
        if (all_moderate)
            store_codes(row0, std::true_type{});
        else
            store_codes(row0, std::false_type{});
    }
}

hipError_t launch_pack_fp8(PackFp8Jobs jobs, hipStream_t stream) {
    int64_t strips = 0;
    for (int j = 0; j < jobs.n; ++j) {
        PackFp8Job& J = jobs.job[j];
        J.n_strips = J.G * (J.N / kPackCols);
        strips += J.n_strips;
    }
    constexpr int64_t kMaxStrips = (1ll << 32) / (kPackWaves * kWave) - 1;   // threads of a launch: 2^32 - 1
    for (int64_t first = 0; first < strips; first += kMaxStrips) {
        jobs.first_strip = static_cast<int>(first);
        hipLaunchKernelGGL(pack_fp8_kernel, dim3(static_cast<unsigned>(std::min(kMaxStrips, strips - first))),
                           dim3(kPackWaves * kWave), 0, stream, jobs);
    }
    return hipGetLastError();
}

hipError_t launch_pack_b(PackJobs jobs, hipStream_t stream) {
    int64_t wgs = 0;
    for (int j = 0; j < jobs.n; ++j) {
        PackJob& J = jobs.job[j];
        J.n_wg = (static_cast<int64_t>(J.G) * (J.N / 32) * (J.Kd / 16) * kWave + 255) / 256;
        wgs += J.n_wg;
    }
    // a launch has less than 2^32 threads: layers of 3.4e10 weights take a second one
    constexpr int64_t kMaxWg = (1ll << 32) / 256 - 1;
    for (jobs.first_wg = 0; jobs.first_wg < wgs; jobs.first_wg += kMaxWg)
        hipLaunchKernelGGL(pack_b_kernel, dim3(static_cast<unsigned>(std::min(kMaxWg, wgs - jobs.first_wg))),
                           dim3(256), 0, stream, jobs);
    return hipGetLastError();
}

}  // namespace allocmoe
