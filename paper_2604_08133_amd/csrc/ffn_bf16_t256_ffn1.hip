// The tile kernel, first half, bf16 weights.
#include "ffn_bf16_t256_kernel.hpp"

namespace allocmoe {
template void enqueue_t256<true, false>(dim3, StreamGroup, StreamGroup, hipStream_t);
}
