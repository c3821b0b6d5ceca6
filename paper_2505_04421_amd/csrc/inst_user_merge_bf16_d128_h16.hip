// Explicit instantiation of the feature-tile-per-wave merge kernels for one (width, head width), bf16.
#include "user_kernel.h"
namespace longer {
LONGER_USER_MERGE_INSTANTIATE_128(16)
}
