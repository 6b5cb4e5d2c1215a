// The tile kernel, first half, 8-bit weights.
#include "ffn_bf16_t256_kernel.hpp"

namespace allocmoe {
template void enqueue_t256<true, true>(dim3, StreamGroup, StreamGroup, hipStream_t);
}
