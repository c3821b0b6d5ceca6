// The key / value projections of width 128 and 256, bf16.
#include "kv_kernel.h"
namespace longer {
int launch_kv(int d, const BlockParams& p, hipStream_t stream) {
  const int tiles = p.B * p.tiles_per_user, most = kv_workgroups(d), grid = tiles < most ? tiles : most;
  if (d == 128) hipLaunchKernelGGL((kv_kernel<128>), dim3(grid), dim3(256), 0, stream, p);
  else if (d == 256) hipLaunchKernelGGL((kv_kernel<256>), dim3(grid), dim3(512), 0, stream, p);
  else return -1;
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
}
