// The tile-stream decode kernel for bf16 pools with a head_dim other than 64 and 128.
#include <hip/hip_runtime.h>

#include "decode_mfma.h"

namespace {

using StreamKernel = void (*)(StreamArgs);
// [fused][paged], launch shape of four waves and two buffers
#define ODMA_WIDE(D32) {{decode_stream_kernel<false, 2, 4, false, STREAM_BF16_WIDE + D32>, decode_stream_kernel<true, 2, 4, false, STREAM_BF16_WIDE + D32>}, \
                        {decode_stream_kernel<false, 2, 4, true, STREAM_BF16_WIDE + D32>, decode_stream_kernel<true, 2, 4, true, STREAM_BF16_WIDE + D32>}}
struct WideKernels {
  int head_dim;
  StreamKernel kernel[2][2];
};
const WideKernels wide_kernels[] = {
    {32, ODMA_WIDE(1)},
    {96, ODMA_WIDE(3)},
    {160, ODMA_WIDE(5)},
    {192, ODMA_WIDE(6)},
    {224, ODMA_WIDE(7)},
    {256, ODMA_WIDE(8)}};
std::atomic<unsigned> wide_lds[sizeof(wide_kernels) / sizeof(wide_kernels[0])][2][2];   // dynamic LDS enabled so far

}  // namespace

hipError_t odma_launch_wide_bf16(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  for (size_t i = 0; i < sizeof(wide_kernels) / sizeof(wide_kernels[0]); ++i)
    if (wide_kernels[i].head_dim == 32 * (fmt - STREAM_BF16_WIDE))
      return launch_with_lds(wide_kernels[i].kernel[fused][paged], wide_lds[i][fused][paged], n_wg, 4, lds_bytes, s,
                             *(const StreamArgs*)args);
  return hipErrorInvalidDeviceFunction;
}
