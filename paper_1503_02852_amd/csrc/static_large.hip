// The static workspace of windows whose exchange copies come on top of RNN_STATIC_WORKSPACE_BYTES (api.cpp).
// In a code object of its own, which is loaded when such a window is first asked for: the loader fills the array, and a
// process's first rnn_forward_static takes 65 ms with it, 14 ms with the 32 MiB array alone.
#include "kernels.h"

namespace rnng {
static __device__ __align__(256) unsigned char large[STATIC_LARGE_BYTES];

hipError_t static_large_workspace(void** p) { return hipGetSymbolAddress(p, HIP_SYMBOL(large)); }
}  // namespace rnng
