// instantiations of the block backward kernel at width 128
#include "bw_block.h"
namespace longer { namespace bw {
void bw_block_launch_128(int dh, const BlockBwParams& p, hipStream_t st) { bw_block_launch_d<128>(dh, p, st); }
} }
