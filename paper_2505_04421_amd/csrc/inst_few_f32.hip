// Instantiations and launcher of the small launches' kernel in full precision (few_f32_kernel.h).
#include "few_f32_kernel.h"
namespace longer {
template <int MODE, int W>
static void launch(const BlockParams& p, dim3 grid, hipStream_t stream) {
  constexpr int threads = 64 * kFewWaves * few_tiles(MODE);
  if (p.act == 1) hipLaunchKernelGGL((few_f32_kernel<MODE, W, true>), grid, dim3(threads), 0, stream, p);
  else hipLaunchKernelGGL((few_f32_kernel<MODE, W, false>), grid, dim3(threads), 0, stream, p);
}
int launch_few_f32(int mode, int win, const BlockParams& p, dim3 grid, hipStream_t stream) {
  if (mode == MODE_STACK) launch<MODE_STACK, 16>(p, grid, stream);
  else if (mode != MODE_MERGE) return -1;
  else if (win == 4) launch<MODE_MERGE, 4>(p, grid, stream);
  else if (win == 8) launch<MODE_MERGE, 8>(p, grid, stream);
  else launch<MODE_MERGE, 16>(p, grid, stream);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
}
