// The tile-stream decode kernel for fp32 pools.
#include <hip/hip_runtime.h>

#include "decode_mfma.h"

hipError_t odma_launch_wide_f32(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  return launch_wide<STREAM_F32_WIDE, 1, 2, 3, 4, 5, 6, 7, 8>(fmt, fused, paged, n_wg, lds_bytes, s, args);
}
