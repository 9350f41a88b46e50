// The tile-stream decode kernel for bf16 pools with a head_dim other than 64 and 128, compiled once for launches that reuse a plan and once for
// launches that make it (ODMA_STREAM_PLAN).
#include <hip/hip_runtime.h>

#include "decode_mfma.h"

template <>
hipError_t odma_launch_wide_bf16<ODMA_STREAM_PLAN>(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  return launch_wide<ODMA_STREAM_PLAN, STREAM_BF16_WIDE, 1, 3, 5, 6, 7, 8>(fmt, fused, paged, n_wg, lds_bytes, s, args);
}
