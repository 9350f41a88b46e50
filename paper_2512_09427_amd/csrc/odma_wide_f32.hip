// The tile-stream decode kernel for fp32 pools, compiled once for launches that reuse a plan and once for
// launches that make it (ODMA_STREAM_PLAN).
#include <hip/hip_runtime.h>

#include "decode_mfma.h"

template <>
hipError_t odma_launch_wide_f32<ODMA_STREAM_PLAN>(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  return launch_wide<ODMA_STREAM_PLAN, STREAM_F32_WIDE, 1, 2, 3, 4, 5, 6, 7, 8>(fmt, fused, paged, n_wg, lds_bytes, s, args);
}
