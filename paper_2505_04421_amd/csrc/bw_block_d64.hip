// instantiations of the block backward kernel at width 64
#include "bw_block.h"
namespace longer { namespace bw {
void bw_block_launch_64(int dh, const BlockBwParams& p, hipStream_t st) { bw_block_launch_d<64>(dh, p, st); }
} }
