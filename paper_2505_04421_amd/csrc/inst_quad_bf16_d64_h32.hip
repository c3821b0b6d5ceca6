// Explicit instantiation of the four-waves-per-tile kernels for one (width, head width), bf16.
#include "quad_kernel.h"
namespace longer {
LONGER_QUAD_INSTANTIATE(64,32)
}
