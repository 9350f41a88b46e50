// Prompt (chunk) attention entry point of libodma for gfx950: launches the kernels in prefill_mfma.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "odma_internal.h"
#include "kernels_common.h"
#include "prefill_mfma.h"
#include "device_common.h"

extern "C" {

int odma_prefill_attention(odma_pool_t* pool, int32_t layer, int32_t n, const void* q, int64_t total_q,
                           const int64_t* q_start, const int32_t* n_q, const int64_t* offsets, const int32_t* lengths,
                           const int32_t* block_table, int32_t bt_stride, void* out, void* stream) {
  const char* where = "odma_prefill_attention";
  int rc = device_ready(pool, where);
  if (rc) return rc;
  const odma_pool_config_t& c = pool->cfg;
  if (pool->decode_kernel != ODMA_KERNEL_MFMA || c.head_dim != 128) {
    odma::set_error(std::string(where) + ": needs a bf16 or fp8 pool with head_dim 128 (the matrix-core path)");
    return ODMA_INVALID_ARG;
  }
  if (n == 0 || total_q == 0) return ODMA_OK;
  if (!c.workspace) {
    odma::set_error(std::string(where) + ": pool has no workspace");
    return ODMA_INVALID_ARG;
  }
  if (layer < 0 || layer >= c.n_layers || n < 0 || n > c.max_requests || total_q < 0 || !q || !q_start || !n_q ||
      !lengths || !out || (!block_table && !offsets) || (block_table && bt_stride <= 0)) {
    odma::set_error(std::string(where) + ": invalid argument");
    return ODMA_INVALID_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)c.workspace;
  const RowArgs ra = row_args(pool, layer);
  PrefillArgs a;
  a.k = ra.k;
  a.v = ra.v;
  a.q = (const unsigned short*)q;
  a.out = out;
  a.q_start = q_start;
  a.n_q = n_q;
  a.offsets = offsets;
  a.lengths = lengths;
  a.bt = block_table;
  a.bt_stride = bt_stride;
  a.hdr = (PrefillHeader*)(ws + pool->ws.prefill);
  a.item_start = (int32_t*)(ws + pool->ws.prefill + 256);
  a.n = n;
  a.Hq = c.n_q_heads;
  a.Hkv = c.n_kv_heads;
  a.G = c.n_q_heads / c.n_kv_heads;
  a.total_q = total_q;
  a.head_stride = ra.head_stride;
  const bool fp8 = pool->elem_bytes == 1;
  a.scale_log2 = c.sm_scale * 1.4426950408889634f * (fp8 ? c.k_scale : 1.0f);
  a.out_scale = fp8 ? c.v_scale : 1.0f;
  a.out_bf16 = c.out_dtype == ODMA_BF16;
  // column tiles per wave: 2 (128-column items, two work-groups per CU whose LDS and matrix phases overlap)
  // measured faster than 4 (256-column items, one work-group per CU) on every prompt mix tried
  const int ct = pool->prefill_ct ? pool->prefill_ct : 2;
  const int slots = pool->n_cu * (ct == 2 ? 2 : 1);
  dim3 grid((slots + PREFILL_XCDS - 1) / PREFILL_XCDS * PREFILL_XCDS);   // every queue has as many work-groups
  // There is one set of states of parts, for the null stream: its calls are ordered, whoever makes them.  A call on another
  // stream, captured ones among them, may run beside it or beside its like, so it cuts nothing and keeps nothing in the
  // workspace.
  a.part_slots = s ? 0 : (int32_t)std::min<int64_t>(pool->ws.prompt_columns / (64 * ct), odma_plan::PROMPT_MAX_PARTS);
  a.arrive = (unsigned long long*)(ws + pool->ws.prompt_arrive);
  a.part_ml = (float2*)(ws + pool->ws.prompt_ml);
  a.part_o = (float*)(ws + pool->ws.prompt_o);
  // Few items -- no more than work-groups, counted from the rows of q (rows that several requests share only make more of
  // them): planned in the attention launch.  With more, the work-groups balance through counters, which a planning launch
  // clears.
  const int64_t items = (total_q * a.G + 64 * ct - 1) / (64 * ct) * a.Hkv + (int64_t)n * a.Hkv;
  const bool here = n <= PREFILL_LDS_REQ && items <= (int64_t)grid.x;
  // Items are cut on the null stream, where a request can be long enough and there is room for two parts of every item.  How
  // many items there are is known here to within a block per request and KV head: half of that is expected.  (With room for one
  // part only, the kernel that can cut is the slower one: 30 prompts of 1 to 59 tokens, 28 / 4 heads, 10.1 -> 9.6 us, one of 1500
  // and 50 short ones, 8 / 1 heads, 41.6 -> 40.4.)  Such a launch has a work-group for every part that
  // an item can have, counted from the longest request there can be, and none beyond: they would each scan the batch and
  // hold up the end of the launch (a queue's first parts go to its first work-groups, which start first).
  const int64_t longest = block_table ? (int64_t)bt_stride * BLK : std::max<int64_t>(c.large_cap, pool->boundaries.back());
  const int64_t parts = prefill_parts((int)std::min<int64_t>(longest / (2 * BLK), 1 << 20));
  const bool cut = here && a.part_slots && parts > 1 && 2 * items - (int64_t)n * a.Hkv <= (int64_t)grid.x;
  if (cut) grid.x = (unsigned)std::min<int64_t>(grid.x, (items * parts + PREFILL_XCDS - 1) / PREFILL_XCDS * PREFILL_XCDS);
  // Long calls may be the eight-wave kernel's: the plan decides, and the other kernel ends at once.  (A pool with a tuned number of
  // column tiles keeps that, and rows that the requests cannot all have, no request having more queries than tokens, say
  // nothing about how long a call is.)
  const double items_cu = (double)total_q * c.n_q_heads / (256.0 * pool->n_cu);   // items of 256 columns for each CU
  const double least = items_cu * (total_q / n) / (4 * BLK), most = items_cu * longest / (2 * BLK);
  const bool weigh = !here && !pool->prefill_ct && total_q / n <= longest &&
                     (fp8 ? least >= PREFILL_WEIGH_FP8 || (least >= PREFILL_WEIGH_FP8_LEAST && most >= PREFILL_WEIGH_FP8_MOST) : least >= PREFILL_WEIGH_BF16);
  PrefillRule rule = fp8 ? PREFILL_EIGHT_FP8 : block_table ? PREFILL_EIGHT_BF16_PAGED : PREFILL_EIGHT_BF16;
  rule.n_cu = pool->n_cu;
  if (!here)
    hipLaunchKernelGGL(weigh ? prefill_plan_kernel<true> : prefill_plan_kernel<false>, dim3(1), dim3(PREFILL_PLAN_THREADS), 0, s, n_q, lengths,
                       q_start, total_q, n, c.n_kv_heads, a.G, 64 * ct, a.hdr, a.item_start, rule);
  // [fp8][two column tiles][paged][planned in front, here, here and cut]
#define ODMA_PREFILL(P, CT, F) {prefill_kernel<P, CT, F, false, false>, prefill_kernel<P, CT, F, true, false>, prefill_kernel<P, CT, F, true, true>}
#define ODMA_PREFILL_F(F) {{ODMA_PREFILL(false, 4, F), ODMA_PREFILL(true, 4, F)}, {ODMA_PREFILL(false, 2, F), ODMA_PREFILL(true, 2, F)}}
  static void (*const kernels[2][2][2][3])(PrefillArgs) = {ODMA_PREFILL_F(false), ODMA_PREFILL_F(true)};
  static void (*const eight_kernels[2][2])(PrefillArgs) = {   // [fp8][paged]
      {prefill_kernel<false, 2, false, false, false, 8>, prefill_kernel<true, 2, false, false, false, 8>},
      {prefill_kernel<false, 2, true, false, false, 8>, prefill_kernel<true, 2, true, false, false, 8>}};
  if (weigh)
    hipLaunchKernelGGL(eight_kernels[fp8][block_table != nullptr], dim3((pool->n_cu + PREFILL_XCDS - 1) / PREFILL_XCDS * PREFILL_XCDS), dim3(512), 0, s, a);
  hipLaunchKernelGGL(kernels[fp8][ct == 2][block_table != nullptr][here + cut], grid, dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(where, e);
  return ODMA_OK;
}

}  // extern "C"
