// The key / value projections of width 128 and 256, bf16.
#include "kv_kernel.h"
namespace longer {
int launch_kv(int d, const BlockParams& p, int tiles, hipStream_t stream) {
  if (d == 128) hipLaunchKernelGGL((kv_kernel<128>), dim3(tiles < 512 ? tiles : 512), dim3(256), 0, stream, p, tiles);
  else if (d == 256) hipLaunchKernelGGL((kv_kernel<256>), dim3(tiles < 256 ? tiles : 256), dim3(512), 0, stream, p, tiles);
  else return -1;
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
}
