// Explicit instantiation of the feature-tile-per-wave stack kernels for one (width, head width), bf16.
#include "user_kernel.h"
namespace longer {
LONGER_USER_INSTANTIATE_128(32)
}
