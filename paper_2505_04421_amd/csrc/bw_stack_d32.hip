// instantiations of the reduced stack's training kernels at width 32
#include "bw_stack.h"
namespace longer { namespace bw {
void bw_stack_fwd_32(const StackFwd& p, const StackFwd& k, hipStream_t st) { bw_stack_fwd_d<32>(p, k, st); }
void bw_stack_bwd_32(const StackBwd& p, const StackBwd& k, hipStream_t st) { bw_stack_bwd_d<32>(p, k, st); }
} }
