// Host helpers shared by the translation units that launch kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "kernels_common.h"
#include "odma_internal.h"

namespace {

// ---------------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------------
inline int hip_fail(const char* where, hipError_t e) {
  odma::set_error(std::string(where) + ": " + hipGetErrorString(e));
  return ODMA_HIP_ERROR;
}

inline int device_ready(odma_pool* pool, const char* where) {
  if (!pool) {
    odma::set_error(std::string(where) + ": null pool");
    return ODMA_INVALID_ARG;
  }
  if (!pool->cfg.k_pool || !pool->cfg.v_pool) {
    odma::set_error(std::string(where) + ": pool was created without device memory");
    return ODMA_INVALID_ARG;
  }
  if (pool->n_cu == 0) {
    int dev = 0, cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(where, e);
    e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(where, e);
    pool->n_cu = cu > 0 ? cu : 256;
  }
  return ODMA_OK;
}

inline RowArgs row_args(const odma_pool* pool, int32_t layer) {
  RowArgs a;
  const int64_t head_stride = pool->pool_blocks * BLK * pool->cfg.head_dim * (int64_t)pool->elem_bytes;
  const int64_t layer_stride = head_stride * pool->cfg.n_kv_heads;
  a.k = (char*)pool->cfg.k_pool + layer * layer_stride;
  a.v = (char*)pool->cfg.v_pool + layer * layer_stride;
  a.head_stride = head_stride;
  a.Hkv = pool->cfg.n_kv_heads;
  a.D = pool->cfg.head_dim;
  return a;
}

}  // namespace
