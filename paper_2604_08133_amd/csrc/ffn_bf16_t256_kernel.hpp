// bf16 expert networks on the matrix cores for prefill-shaped layers (Section
// 3.1: one feed-forward execution per selected pair), fp32 accumulation:
//   H = silu(A W1) * (A W3)   (SWIGLU)    or    O = A W2,   both stored as bf16.
//
// Register-blocked 256 x 256 tile on 4 waves (one per SIMD, all 512 registers).
//
// A workgroup owns <= 256 rows of one expert times 128 SwiGLU columns (128 of
// W1 and the same 128 of W3) or 256 columns of W2, fewer in the last column tile of a
// width that is no multiple of those.  Wave w owns 64 of those
// weight columns (four 16-column MFMA operands: two of W1 and two of W3 of the
// same columns, or four neighbouring ones of W2) times every 16-row block of
// the tile: up to 16 x 4 accumulators of 16x16, 256 registers.
//
//  * v_mfma_f32_16x16x32_bf16 and not the 32x32x16 form: the chip is limited by
//    power on real data, and the longer contraction per instruction moves the
//    sums half as often.  Issued back to back on N(0,1) operands the 16x16x32
//    form sustains 2.12 PFLOP/s (allocmoe_probe_mfma), the 32x32x16 form 1.85 on the
//    same box.  A 16384 x 2816 x 2048 product (second half) runs at 1.34 PFLOP/s (1.19
//    with the 32x32x16 form), 16384 x 2048 x 5632 (SwiGLU half) at 1.25 (1.15).
//  * The weights never pass through LDS: they were re-tiled once into MFMA
//    fragment order, a wave is the only consumer of its columns, so each lane
//    loads its 16 bytes per fragment straight from global memory (1 KB
//    contiguous per wave-load) into a ring of 4 to 12 steps of 32 k.
//  * The activation rows go global -> LDS directly (no VGPR staging) into a ring
//    of 4 slots of 256 rows x 64 k; lanes 8r..8r+7 fetch the eight 16-byte
//    chunks of row r (one 128-byte line per row), XOR-swizzled so that every
//    MFMA A-operand read is one conflict-free ds_read_b128.  Loads run two
//    slots ahead; one workgroup barrier per 64 k.
//  * Per 32 k a wave issues 4 MFMAs per 16-row block for one LDS read, so a tile
//    with fewer than 256 rows costs in proportion to its 16-row blocks.
//  * 8-bit weights (E4M3 codes with one fp32 scale per output column): a lane's
//    16-byte load holds its fragments of two k16 steps, i.e. all it needs of a
//    stream for 32 k; the codes are widened to bf16 (exactly) one step before the
//    MFMAs that use them and the column scales multiply the fp32 sums in the
//    epilogue.
//
// Compiled once per (half, weight format), see ffn_bf16_t256_*.hip: 16 tile heights and two
// weight rings make a variant some thousand lines of machine code each.
#pragma once
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"

namespace allocmoe {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = kTileRowsLarge;   // rows per tile
constexpr int kStepK = 64;              // contraction elements per ring slot
constexpr int kSlots = 4;
constexpr int kWaves = 4;
constexpr int kSlotBytes = kRows * kStepK * 2;
constexpr int kXcds = 8;                // accelerator dies (one L2 each) of an MI355X
// 32-k steps of weight fragments held per stream.  Tiles of up to 128 rows run where the
// weights are most of the bytes: there a shorter ring is 0.5-1 % faster (2048 tokens, 60 or
// 64 experts: 327.5 against 329 us and 223 against 225 us a layer), full tiles need the
// longer one (8192 tokens, skewed experts: 729 us, 760 us with the shorter ring everywhere).
constexpr int ring_steps(int row_blocks16, bool fp8) { return !fp8 && row_blocks16 <= 8 ? 4 : 8; }
constexpr int kRingDeep = 12;       // bf16, tiles of up to 64 rows: light ones, dense groups of few workgroups
constexpr int kLightRowBlocks = 4;  // 16-row blocks of such a tile (the plan counts the light ones: up to 64 rows)

// 8 rows x 128 B of activations, global -> LDS directly: lane l's 16 bytes land
// at M0 + 16 l (M0 holds the wave-uniform LDS base; one other instruction has to stand
// between writing M0 and the load that reads it: an MFMA, see the callers).  The base
// travels from the one to the other as a value that lives in M0: whatever the compiler
// might put there in between, it would have to put the base back.  (It does not see an MFMA
// written as asm as that other instruction: the loop has the address computation there too,
// so that it adds no idle state.)  Written as
// asm, hidden from the compiler's wait-count insertion: it treats a direct-to-LDS load as
// touching both memory paths and then drains *all* outstanding loads (vmcnt(0)) at the
// next use of any loaded register, which would serialise the weight prefetch.
// Hidden, these loads still count in vmcnt, in issue order: every wait the
// compiler emits for a weight register is then stricter than needed, never
// weaker, and the waits for the slots themselves are written by hand.
struct LdsBase {
    uint32_t m0;
};
__device__ __forceinline__ LdsBase set_lds_base(uint32_t lds_addr) {
    LdsBase b;
    asm volatile("s_mov_b32 %0, %1" : "={m0}"(b.m0) : "s"(lds_addr) : "memory");
    return b;
}
__device__ __forceinline__ void load_rows_to_lds(const bf16x8* g, LdsBase b) {
    asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(g), "{m0}"(b.m0) : "memory");
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence
// would wait for every outstanding load, i.e. also for the prefetched slots.
// What a step needs is awaited explicitly (vmcnt) before the barrier.
__device__ __forceinline__ void wg_barrier_nofence() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt_le() {
    // s_waitcnt with expcnt/lgkmcnt unconstrained; vmcnt is bits [3:0] and [15:14]
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// d += b a for a 16x16 block over 32 k, the sum staying in AGPRs.  Written as asm because
// with 64 independent four-register sums the compiler moves part of them through VGPRs on
// every pass of the loop (half as many copies as MFMAs).  NOP: two idle states first, which
// the unit needs between a vector instruction that wrote an operand and the MFMA; all other
// calls have at least one MFMA and its successor in between.
template <bool NOP>
__device__ __forceinline__ void mfma_16x16x32(f32x4& d, bf16x8 b, bf16x8 a) {
    if (NOP)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(b), "v"(a));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(b), "v"(a));
}

// f(0), f(1), ... with the index as a compile-time constant
template <typename F, int... Q>
__device__ __forceinline__ void unrolled(F f, std::integer_sequence<int, Q...>) {
    (f(std::integral_constant<int, Q>{}), ...);
}

// two E4M3 codes (half h of the dword) -> two bf16 values, exactly
template <bool HI>
__device__ __forceinline__ uint32_t widen_fp8x2(uint32_t q) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 p = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(q, 1.0f, HI);
    return __builtin_bit_cast(uint32_t, p);
}

// b0, b1: the wave's two weight streams (bf16 fragments, or with FP8 the codes: a lane's
// 16 bytes per 32 k hold its fragment of the even k16 step, then of the odd one);
// sc0, sc1: with FP8 the scales of the 32 columns of each stream.
// live: the wave's columns exist; a wave past the last column (the other waves still need its
// share of the activation loads) reads zeros in place of weights and stores nothing.
// NF: 16-row blocks of the tile.  NR: 32-k steps of weights held in registers.
template <bool SWIGLU, int NF, bool STREAM_ONCE, bool FP8, int NR>
__device__ __forceinline__ void t256_body(char* lds, const bf16_t* A, size_t lda,
                                          const int32_t* row_map, const void* b0,
                                          const void* b1, const float* sc0, const float* sc1,
                                          int KT, int wave, int lane, int row0,
                                          int rows, int nt, bool live, void* C, int ldc) {
    // acc[f][c]: 16 token rows (f) x 16 weight columns (c: two blocks per stream)
    f32x4 acc[NF][4];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[f][c] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A: per slot, wave w stages rows 32 i + 8 w .. + 7 of every 32-row block i that
    // holds real rows (NL wave-loads): lane 8 r + p fetches the chunk that belongs
    // at position p of row r.  Rows past the tile's end re-read its last row (in
    // bounds, never stored).
    constexpr int NL = (NF + 1) / 2;
    const bf16x8* arow[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int R = 32 * i + 8 * wave + lane / 8;
        const int my_row = row0 + min(R, rows - 1);
        const long src = row_map ? row_map[my_row] : my_row;
        const int q = (lane % 8) ^ ((R >> 1) & 7);   // chunk: bits 0 and 1 exchanged (see a_at)
        arow[i] = reinterpret_cast<const bf16x8*>(A + static_cast<size_t>(src) * lda) +
                  ((q & 4) | ((q & 1) << 1) | ((q >> 1) & 1));
    }
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
    typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;
    // Weight fragments come through buffer loads: a scalar descriptor per stream
    // (base, size) and the step in the lane's offset, one addition for the loads of a 32-k
    // step.  That offset is what the range check looks at (a scalar offset beside it is
    // documented as left out), so a step past the end of the stream reads zeros and touches no
    // memory.  Weights that no other tile reads are marked non-temporal: they need not displace
    // what the caches hold for tiles that share theirs.
    const int stream_bytes = live ? KT * kStepK * 32 * (FP8 ? 1 : 2) : 0;
    const __amdgpu_buffer_rsrc_t rs0 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void*>(b0), 0, stream_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs1 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void*>(b1), 0, stream_bytes, 0x00020000);
    const int lane_off = lane * 16;
    constexpr int kAux = STREAM_ONCE ? 2 : 0;   // nt
    // ring[r][j][h]: stream j, k16 step h of a 32-k step (FP8: one load holds both)
    constexpr int NH = FP8 ? 1 : 2;
    i32x4 ring[NR][2][NH];
    auto load_b = [&](int r, int j, int h, int d) {   // entry r <- 32-k step d
        ring[r][j][h] = __builtin_amdgcn_raw_buffer_load_b128(j == 0 ? rs0 : rs1, lane_off + (d * NH + h) * 1024,
                                                              0, kAux);
    };
    // The matrix instruction is 16x16x32: its operand holds row (or column) l%16 in lane l,
    // and lane group l/16 supplies 8 of the 32 k.  Which k the groups take is free as long as
    // both operands agree.  The weight fragments are packed 16 k x 32 columns, lane l holding
    // column l%32 and k half l/32; exchanging the odd 16-lane rows of the even step's fragment
    // with the even rows of the odd step's (one v_permlane16_swap per register) gives the two
    // operands of 32 k x 16 columns, groups 0..3 holding k chunks 0, 2, 1, 3 (of 8 k each).
    // The weight operand is the first one and the activation operand the second, i.e. the
    // unit forms the transposed block: register r of lane l holds the output of token row
    // l%16 at column 4 (l/16) + r, four consecutive columns, which the epilogue stores as
    // one 8-byte word of bf16 (paired to 16 bytes).
    i32x4 wide[FP8 ? 2 : 1][4];   // FP8: the widened operands of this and the next 32-k step
    auto swap_pair = [&](int& x, int& y) {
        const auto v = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = static_cast<int>(v[0]);
        y = static_cast<int>(v[1]);
    };
    constexpr int kPrep = FP8 ? 20 : 8;   // vector instructions that prepare a 32-k step's weights
    auto prepare = [&](int t, int r) {    // instruction t of entry r
        if constexpr (FP8) {
            // a lane's 16 codes: 8 of the even k16 step, then 8 of the odd one
            const int j = t / 10, u = t % 10;
            i32x4& q = ring[r][j][0];
            if (u < 2) {
                int x = q[u], y = q[u + 2];
                swap_pair(x, y);
                q[u] = x;
                q[u + 2] = y;
            } else {
                const int h = (u - 2) / 4, w = (u - 2) % 4;
                const uint32_t src = q[2 * h + w / 2];
                wide[r & 1][2 * j + h][w] = (w & 1) ? widen_fp8x2<true>(src) : widen_fp8x2<false>(src);
            }
        } else {
            const int j = t / 4, e = t % 4;
            int x = ring[r][j][0][e], y = ring[r][j][1][e];
            swap_pair(x, y);
            ring[r][j][0][e] = x;
            ring[r][j][1][e] = y;
        }
    };
    auto weights = [&](int r, int c) {   // operand of the 16 columns c of entry r
        if constexpr (FP8)
            return __builtin_bit_cast(bf16x8, wide[r & 1][c]);
        else
            return __builtin_bit_cast(bf16x8, ring[r][c / 2][c % 2]);
    };
    // A operand of 16-row block f, half slot h (32 k): lane l reads row 16 f + l%16, chunk
    // 4 h + {0, 2, 1, 3}[l/16] of the row's eight 16-byte chunks.  Chunk c is stored at
    // position c' ^ ((row/2) % 8), c' being c with bits 0 and 1 exchanged, so the lane's
    // position is (4 h + l/16) ^ ((row/2) % 8): the 16 lanes of a group hit 16 different
    // 16-byte units of the 256 bytes that the LDS banks span, and so do 8 lanes of one group
    // with the complementary 8 rows of its neighbour, which the unit serves together.
    // (An LDS instruction's offset reaches 64 KB: one address per half slot for slots 0 and
    // 1, one for 2 and 3, kept apart from each other so that no read needs an addition.)
    const int m = lane % 16, sw = (m >> 1) & 7, g4 = lane / 16;
    uint32_t a_at[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            a_at[p][h] = lds0 + p * 2 * kSlotBytes + (m * 8 + ((4 * h + g4) ^ sw)) * 16;
            asm("" : "+v"(a_at[p][h]));
        }
    auto read_a = [&](int slot, int h, int f) {
        typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
        uint32_t at;
        if constexpr (NR % 8 == 0)   // the slot is a constant
            at = a_at[slot / 2][h] + (slot & 1) * kSlotBytes;
        else
            at = a_at[0][h] + slot * kSlotBytes;
        return *reinterpret_cast<lds_bf16x8*>(at + f * (16 * 128));
    };

    // Schedule.  A slot (64 k) is four steps kc = 0 .. 3: 32-k step kc/2, and of the tile's
    // 16-row blocks the first NE (kc even) or the last NO (kc odd).  A wave has one SIMD to
    // itself and issues one instruction per 4 cycles, an MFMA takes 16: everything else goes
    // one by one into the gaps between the MFMAs (`fill`), since two or three instructions
    // in a row already leave the matrix unit idle:
    //   every step   the LDS reads of the next step's A operands
    //   even         the weight loads that refill the entry used last, for NR - 1 steps ahead
    //   odd          the lane swaps (FP8: and conversions) that prepare the next 32-k step
    //   kc = 0       the activation loads of the slot two ahead
    // The barrier stands behind kc = 2: slot s + 1 has landed (below), and every wave is done
    // with slot s - 1, which the loads of the next kc = 0 overwrite.  Slot s + 1 was issued at
    // kc = 0 of slot s - 1, its last load behind that step's weight loads; until the wait
    // behind kc = 2 of slot s follow 3 x 4 (FP8: 3 x 2) weight loads and NL loads of slot
    // s + 2 -> kWaitA (fewer in the tail, see `pass`).  The prologue issues slot 0, the weights of steps 0 .. NR - 3, slot 1
    // and the weights of step NR - 2, so that count holds from the first slot on.  Loads past
    // the end of the contraction re-read the last slot (in bounds, never multiplied) or, for
    // the weights, read zeros past the end of the buffer, which keeps the count uniform.
    // At most 63 loads can be outstanding per wave.
    constexpr int NE = (NF + 1) / 2, NO = NF / 2;
    constexpr int kWLoads = 2 * NH;   // weight loads per 32-k step
    constexpr int kWaitA = 3 * kWLoads + NL;
    static_assert(NR % 2 == 0 && NR * kWLoads + 2 * NL <= 63, "outstanding loads per wave");
    auto issue_slot = [&](int s, int slot) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const LdsBase base = set_lds_base(lds_wave + slot * kSlotBytes + i * 4096);
            asm volatile("s_nop 0");
            load_rows_to_lds(arow[i] + s * (kStepK / 8), base);
        }
    };
    issue_slot(0, 0);
#pragma unroll
    for (int r = 0; r < NR - 1; ++r) {
        if (r == NR - 2) issue_slot(min(1, KT - 1), 1);
#pragma unroll
        for (int t = 0; t < kWLoads; ++t) load_b(r, t / NH, t % NH, r);
    }
    wait_vmcnt_le<kWLoads*(NR - 1) + NL>();   // slot 0 has landed (this wave's part)
    wg_barrier_nofence();
    bf16x8 af[2][NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) af[0][i] = read_a(0, 0, i);
#pragma unroll
    for (int t = 0; t < kPrep; ++t) prepare(t, 0);

    // step kc of slot s (LDS slot `slot`), weights of ring entry r; refill: with this step's
    // weight loads (even steps)
    auto step = [&](int kc, int s, int slot, int r, bool refill) {
        const bool odd = kc & 1;
        const int M = odd ? NO : NE, f0 = odd ? NE : 0, NM = 4 * M;
        const int n_next = odd ? NE : NO;   // 16-row blocks of the next step
        const int next_slot = kc == 3 ? ((slot + 1) & 3) : slot, next_h = ((kc + 1) & 3) / 2;
        const int next_f0 = odd ? 0 : NE;
        const int far = min(s + 2, KT - 1) * (kStepK / 8), far_slot = (slot + 2) & 3;
        const bf16x8* p[NL];
        LdsBase base[NL];
        // instruction t of cnt, spread over the step, `off` MFMAs behind its share's start
        auto due = [&](int n, int t, int cnt, int off) {
            return NM == 0 ? true : n == min(NM - 1, t * NM / cnt + off);
        };
        auto fill = [&](int n) {   // what follows MFMA n
#pragma unroll
            for (int t = 0; t < n_next; ++t)
                if (due(n, t, n_next, 1)) af[!odd][t] = read_a(next_slot, next_h, next_f0 + t);
            if (odd) {
#pragma unroll
                for (int t = 0; t < kPrep; ++t)
                    if (due(n, t, kPrep, 0)) prepare(t, (r + 1) % NR);
            } else if (refill) {
#pragma unroll
                for (int t = 0; t < kWLoads; ++t)
                    if (due(n, t, kWLoads, 0))
                        load_b((r + NR - 1) % NR, t / NH, t % NH, 2 * s + kc / 2 + NR - 1);
            }
            if (kc == 0) {
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    if (due(n, i, NL, 1)) base[i] = set_lds_base(lds_wave + far_slot * kSlotBytes + i * 4096);
                    if (due(n, i, NL, 2)) p[i] = arow[i] + far;
                    if (due(n, i, NL, 3)) load_rows_to_lds(p[i], base[i]);
                }
            }
        };
        if (NM == 0) fill(0);
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            const int i = n / 4, c = n % 4;
            if (n == 0 && !odd)
                mfma_16x16x32<true>(acc[f0 + i][c], weights(r, c), af[odd][i]);
            else
                mfma_16x16x32<false>(acc[f0 + i][c], weights(r, c), af[odd][i]);
            __builtin_amdgcn_sched_barrier(0);
            fill(n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // (Copies of accumulators that the compiler makes between the passes, and the epilogue's
    // reads, depend on MFMAs it does not know: 16 idle states cover their latency.)
    auto drain = [] {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // slots [s2, s2 + SLOTS) of the contraction (s2 a multiple of NR / 2); TAIL: the last
    // ones.  The tail issues no weight load that nothing would use (the compiler would drop
    // it, and the count with it).
    auto pass = [&](int s2, auto slots_const, auto tail_const) {
        constexpr int SLOTS = decltype(slots_const)::value;
        constexpr bool TAIL = decltype(tail_const)::value;
        auto slot_body = [&](auto q_const) {
            constexpr int q = decltype(q_const)::value;
            const int s = s2 + q, slot = NR % 8 == 0 ? (q & 3) : (s & 3);
            // weight loads in the even step of 32-k step d of this pass (d < 0: an earlier one)
            auto refills = [](int d) { return !TAIL || d < 0 || d + NR - 1 < 2 * SLOTS; };
            constexpr int kIssued = (refills(2 * q - 1) + refills(2 * q) + refills(2 * q + 1)) * kWLoads;
            static_assert(TAIL || kIssued + NL == kWaitA, "the count above");
            if constexpr (TAIL && q == SLOTS - 1) {   // an odd number of slots ends one earlier
                drain();
                if (s >= KT) return;
            }
            step(0, s, slot, 2 * q, refills(2 * q));
            step(1, s, slot, 2 * q, false);
            step(2, s, slot, 2 * q + 1, refills(2 * q + 1));
            // this wave's part of the next slot has landed; after the barrier everybody's
            // has, and everybody is done with the slot before this one
            wait_vmcnt_le<kIssued + NL>();
            wg_barrier_nofence();
            step(3, s, slot, 2 * q + 1, false);
        };
        unrolled(slot_body, std::make_integer_sequence<int, SLOTS>{});
    };
    int s2 = 0;
    for (; s2 + NR / 2 <= KT; s2 += NR / 2) {
        pass(s2, std::integral_constant<int, NR / 2>{}, std::false_type{});
        drain();
    }
    static_assert(NR == 4 || NR == 8 || NR == 12, "remainder passes");
    const int rest = (KT - s2 + 1) / 2;
    if (NR == 12 && rest == 3) {
        pass(s2, std::integral_constant<int, 6>{}, std::true_type{});
        drain();
    }
    if (NR == 12 && rest == 2) {
        pass(s2, std::integral_constant<int, 4>{}, std::true_type{});
        drain();
    }
    if (NR == 8 && rest == 2) {
        pass(s2, std::integral_constant<int, 4>{}, std::true_type{});
        drain();
    }
    if (rest == 1) {
        pass(s2, std::integral_constant<int, 2>{}, std::true_type{});
        drain();
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt_le<0>();   // the surplus loads have landed before registers and LDS are reused
    // The accumulators leave the AGPRs by hand-written reads: read by ordinary vector
    // instructions, they make the compiler keep part of them in VGPRs through the loop and
    // copy them in and out around the MFMAs.
    auto sum_of = [&](int f, int c, int r) {
        float v;
        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[f][c][r]));
        return v;
    };

    // epilogue: lane l owns token row l%16 of every 16-row block; acc[f][c] holds columns
    // 16 c + 4 (l/16) .. + 3 of the wave's columns (c = 0, 1: first stream, 2, 3: second).
    // SwiGLU: the two streams are the W1 and W3 halves of the same 32 columns.
    // The two 16-column blocks of a stream are stored together: exchanging odd 16-lane rows
    // of the first with even rows of the second gives lane group g = 0..3 the 8 consecutive
    // columns from {0, 16, 8, 24}[g] on, 16 bytes per lane (a store costs by the row segments
    // it touches).
    const int cq = 4 * g4, col8 = 16 * (g4 & 1) + 8 * (g4 >> 1);
    f32x4 scale[4];   // FP8: of the lane's columns, [block]
    if constexpr (FP8) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            scale[c] = *reinterpret_cast<const f32x4*>((c < 2 ? sc0 : sc1) + 16 * (c % 2) + cq);
    }
    // w0, w1: a lane's 4 columns of the first and of the second block of a stream
    auto store_pair = [&](bf16_t* at, uint2 w0, uint2 w1) {
        const auto x = __builtin_amdgcn_permlane16_swap(w0.x, w1.x, false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(w0.y, w1.y, false, false);
        *reinterpret_cast<uint4*>(at) = make_uint4(x[0], y[0], x[1], y[1]);
    };
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int mr = f * 16 + m;
        if (mr >= rows || !live) continue;   // (the same for the four lanes of a row)
        bf16_t* out = static_cast<bf16_t*>(C) + static_cast<size_t>(row0 + mr) * ldc +
                      nt * (SWIGLU ? 128 : 256) + wave * (SWIGLU ? 32 : 64) + col8;
        if (SWIGLU) {
            uint2 w[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float av = sum_of(f, c, r), bv = sum_of(f, 2 + c, r);
                    if constexpr (FP8) {
                        av *= scale[c][r];
                        bv *= scale[2 + c][r];
                    }
                    h[r] = av * bv * __builtin_amdgcn_rcpf(1.f + __expf(-av));
                }
                // round-to-nearest-even in the conversion unit (v_cvt_pk_bf16_f32)
                w[c] = __builtin_bit_cast(uint2, __builtin_convertvector(f32x4{h[0], h[1], h[2], h[3]}, bf16x4));
            }
            store_pair(out, w[0], w[1]);
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint2 w[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    f32x4 v = {sum_of(f, 2 * j + c, 0), sum_of(f, 2 * j + c, 1),
                               sum_of(f, 2 * j + c, 2), sum_of(f, 2 * j + c, 3)};
                    if constexpr (FP8) v *= scale[2 * j + c];
                    w[c] = __builtin_bit_cast(uint2, __builtin_convertvector(v, bf16x4));
                }
                store_pair(out + 32 * j, w[0], w[1]);
            }
        }
    }
}

// How many tiles at the end of the tile map form the light class (single tiles of at most
// kLightRowBlocks 16-row blocks, spread among the others and run with the deeper weight ring):
// all of them if they are the minority, else none.  8-bit weights: none (no deeper ring for
// them, and without it spreading the light tiles only costs).
__device__ __forceinline__ int light_class_of(const int32_t* tile_info, bool fp8) {
    const int tiles = tile_info[0], light = tile_info[1];
    return (!fp8 && 2 * light <= tiles) ? light : 0;
}

template <bool SWIGLU, bool FP8>
__global__ __launch_bounds__(kWaves* kWave, 1) void ffn_bf16_t256_kernel(StreamGroup g0,
                                                                        StreamGroup g1) {
    __shared__ __attribute__((aligned(1024))) char lds[kSlots * kSlotBytes];

    // Work order.  Workgroups are dealt to the 8 XCDs round-robin by blockIdx, and
    // each XCD has its own L2: workgroup i is item i/8 of XCD i%8's list.
    //  * The dense (shared-expert) group comes first.  The XCDs form an
    //    xr x (8/xr) grid over its (row tiles, column tiles), interleaved, and an
    //    XCD's items are ordered (column tile, row tile): the workgroups of the
    //    first round start together and stay in step, so a weight stream is fetched
    //    into an L2 once for all the XCD's row tiles, an activation tile once for
    //    all its column tiles.
    //  * Then the routed tiles in the tile map's order (longest first), in pairs of
    //    neighbours: pair p runs on XCD p % 8, its items ordered (column tile, tile
    //    of the pair).  Neighbouring tiles mostly belong to one expert and cost the
    //    same, so the two workgroups of a column tile start together and share one
    //    pass over the weight stream; the column tiles that share the gathered
    //    activation rows follow within a few items.
    constexpr int kColsPerTile = SWIGLU ? 128 : 256;
    const int xcd = blockIdx.x % kXcds, idx = g1.first_item + blockIdx.x / kXcds;
    const int nt0 = g0.A ? (g0.N + kColsPerTile - 1) / kColsPerTile : 1;
    const int nt1 = g1.A ? (g1.N + kColsPerTile - 1) / kColsPerTile : 1;
    int S = 0, s_rows = 1;     // dense group: items and row tiles of this XCD
    const int xr = g1.xr, xc = kXcds / xr, xri = xcd % xr, xci = xcd / xr;
    if (g1.A != nullptr) {
        const int tiles = (g1.M_dense + g1.dense_rows - 1) / g1.dense_rows;
        s_rows = (tiles - xri + xr - 1) / xr;
        S = s_rows * ((nt1 - xci + xc - 1) / xc);
    }
    const bool first = idx >= S;
    const StreamGroup& g = first ? g0 : g1;
    int tile, nt;
    if (first) {
        if (g0.A == nullptr) return;
        int sub = idx - S;
        if (g0.tile_info != nullptr) {
            // (8-bit weights: no deeper ring for the light tiles, and without it spreading
            // them only costs: they stay at the end)
            const int tiles = g0.tile_info[0];
            const int light = light_class_of(g0.tile_info, FP8), heavy = tiles - light;
            // (pairs dealt in serpentine order: even rounds left to right, odd rounds
            // right to left, which evens out the XCDs' totals of the sorted tile costs)
            const int round = sub / (2 * nt0), in_pair = sub % (2 * nt0);
            const int q = round * kXcds + ((round & 1) ? kXcds - 1 - xcd : xcd);
            // The light tiles (single tiles of at most kLightRowBlocks 16-row blocks: the end
            // of the tile map) wait for their weights, the others for the matrix unit:
            // their pairs are spread evenly among the pairs of the others, so that both
            // kinds run side by side through the whole launch.  Of the first q + 1 pair
            // positions floor((q + 1) n_light / n_pairs) hold light pairs.
            const int hp = (heavy + 1) / 2, lp = (light + 1) / 2, np = hp + lp;
            if (q >= np) return;   // the grid is sized for the host's bound
            const int lq = static_cast<int>(static_cast<int64_t>(q + 1) * lp / np);
            const int lq0 = static_cast<int>(static_cast<int64_t>(q) * lp / np);
            int first_of_pair, end;
            if (lq > lq0) {
                first_of_pair = heavy + 2 * lq0;
                end = tiles;
            } else {
                first_of_pair = 2 * (q - lq0);
                end = heavy;
            }
            tile = first_of_pair + in_pair % 2;
            nt = in_pair / 2;
            if (tile >= end) return;
        } else {   // a dense group in the first slot: its row tiles striped over the XCDs
            const int tiles = (g0.M_dense + g0.dense_rows - 1) / g0.dense_rows;
            tile = sub / nt0 * kXcds + xcd;
            nt = sub % nt0;
            if (tile >= tiles) return;
        }
    } else {
        tile = xri + xr * (idx % s_rows);
        nt = xci + xc * (idx / s_rows);
    }

    const bf16_t* __restrict__ A = static_cast<const bf16_t*>(g.A);
    const char* __restrict__ Bp = static_cast<const char*>(g.Bp);
    const int32_t* __restrict__ row_map = g.row_map;
    const int32_t* __restrict__ tile_info = g.tile_info;
    const int lda = g.lda, Kd = g.Kd, ldc = g.ldc, M_dense = g.M_dense;
    int e, row0, rows;
    bool only_tile;   // of its expert: nobody else reads these weights
    if (tile_info != nullptr) {
        const int32_t* ent = tile_info + kTileHdr + 4 * static_cast<size_t>(tile);
        e = ent[0];
        row0 = ent[1];
        rows = ent[2];
        only_tile = ent[3] == 1;
    } else {
        e = 0;
        row0 = tile * g.dense_rows;
        rows = min(g.dense_rows, M_dense - row0);
        only_tile = M_dense <= g.dense_rows;
    }
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n_f = (rows + 15) / 16;   // 16-row blocks that hold real rows
    const bool deep_ring = g.deep_ring || (tile_info != nullptr && only_tile && light_class_of(tile_info, FP8) > 0);
    const int KT = Kd / kStepK;

    // B: the two fragment streams of this wave's 64 weight columns; a stream is
    // Kd/16 fragments of 64 lanes x 16 B (FP8: Kd/32), contiguous
    constexpr size_t kElemBytes = FP8 ? 1 : 2;
    const size_t stream_elems = static_cast<size_t>(Kd) * 32;
    // (N is a multiple of 64: a wave's columns exist all or not at all; one without columns
    // keeps addresses inside the matrix)
    constexpr int kColsPerWave = kColsPerTile / kWaves;
    const int col0 = nt * kColsPerTile + wave * kColsPerWave;
    const bool live = col0 < g.N;
    const int wcol = live ? col0 : 0;
    const size_t sidx = SWIGLU ? static_cast<size_t>(wcol / 32) * 2 : static_cast<size_t>(wcol / 32);
    // (wave-uniform pointers: the loads take a scalar base and the lane's offset)
    const char* b0 = Bp + (static_cast<size_t>(e) * g.group_stride + sidx * stream_elems) * kElemBytes;
    const char* b1 = b0 + stream_elems * kElemBytes;
    // FP8: scale[expert][stream][N]; SwiGLU: W1 and W3 scales of the wave's 32 columns,
    // plain: of its two neighbouring 32-column blocks
    const float* sc0 = nullptr;
    const float* sc1 = nullptr;
    if (FP8) {
        const float* sc = g.scale + static_cast<size_t>(e) * (SWIGLU ? 2 : 1) * g.N;
        sc0 = sc + wcol;
        sc1 = SWIGLU ? sc0 + g.N : sc0 + 32;
    }

    // The deeper weight ring is for light tiles that run among matrix-bound ones; where
    // most tiles are light (few tokens) the launch as a whole is bound by the memory
    // system, which more loads in flight per unit only crowd (measured: +3 % step time at
    // 256 tokens, +17 % on a layer whose experts all hold 128 rows).  A dense group of few
    // workgroups (StreamGroup::deep_ring) has no such crowd either: a workgroup is alone with
    // the latency of its long weight streams.  Shared expert of 16384 on 512, 130 tokens (10
    // workgroups of 32 rows in the second half): layer 146 us with the short ring, 135 with the
    // longer ones; 22528 on 2048: 221, 209; 300 tokens, 16384 on 1024 (one round): 163, 155.
#define ALLOCMOE_T256_BODY(n, ring)                                                                 \
    do {                                                                                            \
        if (only_tile)                                                                              \
            t256_body<SWIGLU, n, true, FP8, ring>(lds, A, lda, row_map, b0, b1, sc0, sc1, KT,       \
                                                  wave, lane, row0, rows, nt, live, g.C, ldc);      \
        else                                                                                        \
            t256_body<SWIGLU, n, false, FP8, ring>(lds, A, lda, row_map, b0, b1, sc0, sc1, KT,      \
                                                   wave, lane, row0, rows, nt, live, g.C, ldc);     \
    } while (0)
#define ALLOCMOE_T256_CASE(n)                                                                       \
    case n:                                                                                         \
        if constexpr (!FP8 && n <= kLightRowBlocks) {                                               \
            if (deep_ring) {                                                                        \
                ALLOCMOE_T256_BODY(n, kRingDeep);                                                   \
                break;                                                                              \
            }                                                                                       \
        } else if constexpr (!FP8 && ring_steps(n, FP8) < 8) {                                      \
            if (g.deep_ring) {                                                                      \
                ALLOCMOE_T256_BODY(n, 8);                                                           \
                break;                                                                              \
            }                                                                                       \
        }                                                                                           \
        ALLOCMOE_T256_BODY(n, ring_steps(n, FP8));                                                  \
        break;
    switch (n_f) {   // uniform over the workgroup
        ALLOCMOE_T256_CASE(1)
        ALLOCMOE_T256_CASE(2)
        ALLOCMOE_T256_CASE(3)
        ALLOCMOE_T256_CASE(4)
        ALLOCMOE_T256_CASE(5)
        ALLOCMOE_T256_CASE(6)
        ALLOCMOE_T256_CASE(7)
        ALLOCMOE_T256_CASE(8)
        ALLOCMOE_T256_CASE(9)
        ALLOCMOE_T256_CASE(10)
        ALLOCMOE_T256_CASE(11)
        ALLOCMOE_T256_CASE(12)
        ALLOCMOE_T256_CASE(13)
        ALLOCMOE_T256_CASE(14)
        ALLOCMOE_T256_CASE(15)
        default: ALLOCMOE_T256_CASE(16)
    }
#undef ALLOCMOE_T256_CASE
#undef ALLOCMOE_T256_BODY
}

}  // namespace

template <bool SWIGLU, bool FP8>
void enqueue_t256(dim3 grid, StreamGroup routed, StreamGroup shared, hipStream_t stream) {
    hipLaunchKernelGGL((ffn_bf16_t256_kernel<SWIGLU, FP8>), grid, dim3(kWaves * kWave), 0, stream,
                       routed, shared);
}

}  // namespace allocmoe
