// The tile-stream decode kernel for one storage format (ODMA_STREAM_FMT), for launches that reuse a plan or for launches that
// make it (ODMA_STREAM_PLAN).
#include <hip/hip_runtime.h>

#include "decode_mfma.h"
#include "device_common.h"

template <>
hipError_t odma_launch_stream<ODMA_STREAM_FMT, ODMA_STREAM_PLAN>(bool fused, bool paged, int nbuf, int wpw, int n_wg, size_t lds_bytes,
                                                                 hipStream_t s, const void* args) {
  return launch_shapes<ODMA_STREAM_FMT, ODMA_STREAM_PLAN>(fused, paged, nbuf, wpw, n_wg, lds_bytes, s, args);
}

#ifdef ODMA_DEV_TIMELINE
extern "C" int odma_dev_timeline(long long* host_dst, size_t n_values) {
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(odma_dev_timeline_buf), n_values * sizeof(long long));
  return e == hipSuccess ? ODMA_OK : hip_fail("odma_dev_timeline", e);
}
#endif
