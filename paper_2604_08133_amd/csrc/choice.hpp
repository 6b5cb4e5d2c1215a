// Which kernel and which stream the bf16 expert networks of a layer take, from the layer's sizes
// alone.  Host arithmetic only (no HIP), so that it can be compiled and checked by itself.
#pragma once
#include <cstdint>

namespace allocmoe {

struct FfnChoice {
    bool routed_tiled;   // routed experts: register-blocked tile kernel (256-row tiles), else the
    bool shared_tiled;   // shared expert:  weight-streaming kernel (32-row tiles)
    bool own_stream;     // the shared expert's launches run on the library's stream
};

// T tokens, d hidden, E experts of I, shared expert of Is (0: none), B selected pairs.
//
// Large layers (kLargeWeights or kLargeFlops) decide per group: the routed experts are
// tiled from about eight rows each on, the shared expert from about 128 tokens on, and where
// either is tiled the shared expert runs beside selection and the routed experts.
// Measured on DeepSeek-V2-Lite shapes the two kernels cross between 6 and 9 rows per
// expert for the routed group (B = 6E: 174 us a step streaming, 182 tiled; B = 9E: 200
// against 193; B = 12E: 227 against 201).
//
// Smaller layers mostly run both groups on one kernel, in one launch per half.  A fork and join
// of two streams costs some of them 5-9 us and gains others as much; two launches behind each other
// cost 6-20 us.  (Shared expert twice as wide as the experts, two pairs a token: 320 x 192, 32
// experts, 300 tokens: one launch 26 us streaming, 30 tiled, side stream 37; 1088 x 704, 777 tokens:
// 123, 77, 83; 1472 x 1344, 64 experts, 300 and 1600 tokens: 177, 144, 154 and 549, 204, 192.  36
// drawn layers that run tiled in one launch here: 1.5 % longer on two streams in the mean, 13 %
// shorter to 15 % longer.)  Tiled where the experts see ten rows or more on average
// (8 rows, 64 experts of 1472 x 1344: 143 us streaming, 149 tiled; 11.5: 172, 163) and the
// work covers the tile kernel's longer start and end.  With more than 32 rows an expert's
// weights are streamed more than once, and the tile kernel wins earlier:
//   48 and more rows: 1.9 GFLOP 54 us streaming, 56 tiled; 3.4: 60, 57; 3.7: 58, 51;
//                     4.9: 69, 59; 11: 94, 69
//   fewer:            2.1: 57, 56; 2.6: 47, 58; 4.2: 66, 63 and 62, 67; 11: 174, 161
// That average says nothing about a shared expert much wider than the routed ones, which then
// decides by itself:
//   * enough tokens and work of its own: tiled, however few rows the routed experts see
//     (1024 x 256, 64 experts, shared 8192, 300 tokens, 300 pairs, 15 GFLOP: 133 us streaming, 89
//     tiled; shared 4096, 7.7 GFLOP: 74, 62; shared 4096, 130 tokens, 3.3 GFLOP: 48, 58);
//   * nearly all of the layer and long enough to hide selection and the routed experts: a stream
//     of its own (2048 x 1408, 8 experts, shared 22528, 130 tokens: 220 us in one launch per half,
//     189 beside; 1024 x 512, 32 experts, shared 16384, 300 tokens: 159, 152);
//   * few tokens and most of the work: streaming (1152 x 1280, 7 experts, shared 2560, 128
//     tokens: 53 us, tiled 57; 2048 x 1408, 8 experts, shared 45056, 40 tokens: 376, 541).
// The same limits serve 8-bit weights.  They were chosen while the fork still stood behind the routing
// kernel (and cost 10-20 us): over 1522 layers (d 256 to 2048, 4 to 64 experts, shared
// expert 0 to 32 times the expert width, 24 to 8192 tokens, a tenth to all of T K pairs, both
// formats) the choice was 0.7 % behind the best of the combinations in the mean; the worst cases,
// 13-15 % behind, lie around 130 to 180 tokens, where all of them are close to each other.
inline FfnChoice choose_ffn(int T, int d, int E, int I, int Is, int64_t B) {
    constexpr double kLargeWeights = 4e8, kLargeFlops = 4e10;
    constexpr int64_t kRoutedTiledRowsPerExpert = 8;
    constexpr int kSharedTiledTokens = 128;
    constexpr int64_t kSmallTiledRowsPerExpert = 10, kManyRowsPerExpert = 48;
    constexpr double kTiledFlops = 4.5e9, kTiledFlopsManyRows = 3e9, kSharedTiledFlops = 7e9;
    constexpr double kOwnStreamFlops = 1.6e10, kOwnStreamShare = 10;
    constexpr int kFewTokens = 160;

    const double routed = 6.0 * d * static_cast<double>(B) * I;    // operations
    const double shared = 6.0 * d * static_cast<double>(T) * Is;
    const bool both = B > 0 && Is > 0;
    if (3.0 * d * (static_cast<double>(E) * I + Is) >= kLargeWeights || routed + shared >= kLargeFlops) {
        FfnChoice c{B >= kRoutedTiledRowsPerExpert * E, T >= kSharedTiledTokens, false};
        c.own_stream = both && (c.routed_tiled || c.shared_tiled);
        return c;
    }
    if (both && T >= kSharedTiledTokens) {
        if (shared >= kOwnStreamFlops && shared >= kOwnStreamShare * routed)
            return {B >= kRoutedTiledRowsPerExpert * E, true, true};
        if (shared >= kSharedTiledFlops) return {true, true, false};
    }
    if (both && T < kFewTokens && shared > routed) return {false, false, false};
    const int64_t rows = B + (Is > 0 ? T : 0), experts = (B > 0 ? E : 0) + (Is > 0 ? 1 : 0);
    const bool tiled = rows >= kSmallTiledRowsPerExpert * experts &&
                       routed + shared >= (rows >= kManyRowsPerExpert * experts ? kTiledFlopsManyRows : kTiledFlops);
    return {tiled, tiled, false};
}

// Tokens (one fragment of the gate GEMM's matrix instruction) that one workgroup routes, selects and dispatches
// (route.hip), and whether the shared expert's first half runs beside it in the same launch: on the
// streaming kernel, one round of workgroups with the routing one (32 columns each), and a step of the
// contraction, 16 or with 8-bit weights 32 deep, for each of a workgroup's 16 waves.
constexpr int kRoutePlanTokens = 16;
inline bool first_half_beside_route(const FfnChoice& c, int T, int d, int Is, int64_t B, bool fp8) {
    constexpr int kUnits = 256, kWaves = 16;
    return T <= kRoutePlanTokens && !c.own_stream && !c.routed_tiled && !c.shared_tiled && Is > 0 && B > 0 &&
           Is / 32 < kUnits && d >= kWaves * (fp8 ? 32 : 16);
}

// Most workgroups of a dense group on the tile kernel below which its tiles stay lower than 256 rows
// (ffn_bf16_t256.hip), for the second half of a shared expert on its own stream.
//
// That half is not waited for while the routed experts stream their weights, and a low tile holds a compute unit
// nearly as long as a high one: 600 tokens, 64 experts of 2048 x 1408, shared expert of 2816, 80 workgroups of
// 64 rows took 84 us each beside the first routed half.  With 64 instead of 128 as the limit: 400 tokens 211.3 us
// a layer, 204.9; 600: 225.2, 217.7; 1000: 242.1, 239.0; 2048: 301.4, 298.6; 8-bit weights 600: 146.2, 140.3; 32 gives 1 %
// back.  It has to end before the routed experts do, though: a workgroup's matrix instructions take
// Kd rows / 8 cycles, and about 3.5 times that beside the weight streams; the routed weights take their
// bytes at 6 TB/s.  (600 tokens, 60 experts, shared expert of 5632, 8-bit weights: 144.7 with 128, 147.3 with 64.)
constexpr int kDenseWorkgroups = 128, kHiddenDenseWorkgroups = 64;
inline int dense_tile_rows(int64_t rows, int col_tiles, int64_t most) {
    int h = 32;
    while (h < 256 && (rows + h - 1) / h * col_tiles > most) h += 32;
    return h;
}
inline int side_second_half_workgroups(int T, int d, int E, int I, int Is, int64_t B, int weight_bytes) {
    const int h = dense_tile_rows(T, (d + 255) / 256, kHiddenDenseWorkgroups);
    const double shared_us = 3.5 * Is * h / 8 / 2000;
    const double experts = static_cast<double>(E < B ? E : B);
    const double routed_us = 3.0 * experts * d * I * weight_bytes / 6e6;
    return shared_us <= routed_us ? kHiddenDenseWorkgroups : kDenseWorkgroups;
}

}  // namespace allocmoe
