// instantiation of the input generation's backward kernel at width 128
#include "bw_input.h"
namespace longer { namespace bw {
void bw_input_launch_128(const InputBwParams& p, hipStream_t st) { bw_input_launch_d<128>(p, st); }
} }
