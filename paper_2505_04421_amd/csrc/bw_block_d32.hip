// instantiations of the block backward kernel at width 32
#include "bw_block.h"
namespace longer { namespace bw {
void bw_block_launch_32(int dh, const BlockBwParams& p, hipStream_t st) { bw_block_launch_d<32>(dh, p, st); }
} }
