// The tile kernel, second half, bf16 weights.
#include "ffn_bf16_t256_kernel.hpp"

namespace allocmoe {
template void enqueue_t256<false, false>(dim3, StreamGroup, StreamGroup, hipStream_t);
}
