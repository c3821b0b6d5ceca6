// instantiation of the input generation's backward kernel at width 64
#include "bw_input.h"
namespace longer { namespace bw {
void bw_input_launch_64(const InputBwParams& p, hipStream_t st) { bw_input_launch_d<64>(p, st); }
} }
