// The tile-stream decode kernel for bf16 pools with a head_dim other than 64 and 128.
#include <hip/hip_runtime.h>

#include "decode_mfma.h"

hipError_t odma_launch_wide_bf16(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  return launch_wide<STREAM_BF16_WIDE, 1, 3, 5, 6, 7, 8>(fmt, fused, paged, n_wg, lds_bytes, s, args);
}
