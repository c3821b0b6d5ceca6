// Explicit instantiation of the merge kernel for one (width, head width).
#include "merge_kernel.h"
namespace longer {
LONGER_INSTANTIATE_MERGE(64, 32)
}
