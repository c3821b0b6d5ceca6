// Explicit instantiation of the wave-per-head kernels, bf16, heads of 16 features.
#include "chain_kernel.h"
namespace longer {
LONGER_CHAIN_INSTANTIATE(64)
LONGER_CHAIN_INSTANTIATE(128)
}
