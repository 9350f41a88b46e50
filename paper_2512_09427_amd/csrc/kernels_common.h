// Types and small device helpers shared by every kernel of libodma.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "odma.h"
#include "plan_types.h"

namespace {

constexpr int BLK = ODMA_BLOCK_TOKENS;
constexpr int PLAN_THREADS = 1024;
constexpr int PLAN_LDS_REQ = 8192;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

// Block-table entries are read through the constant address space: with a wave-uniform index the load is then a
// scalar one (its own counter), where a load from the global address space becomes a vector load that queues behind
// the K/V tile loads in flight -- and the next tile's address would have to wait for all of them.  The table is
// written before the launch and by nobody during it.
typedef const int32_t __attribute__((address_space(4))) const_i32;
__device__ __forceinline__ const const_i32* as_constant(const int32_t* p) { return (const const_i32*)(uintptr_t)p; }

using odma_plan::PlanHeader;
using odma_plan::Item;
using odma_plan::ReqInfo;

struct DecodeArgs {
  const char* k;         // layer base of the K pool
  const char* v;
  const void* q;
  void* out;
  const int64_t* offsets;
  const int32_t* lengths;
  const int32_t* bt;
  int32_t bt_stride;
  const PlanHeader* hdr;
  const Item* items;
  const ReqInfo* req;
  float2* part_ml;
  float* part_o;
  int32_t n, Hq, Hkv, G, D;
  int64_t head_stride;   // bytes between KV-head planes of one layer
  float scale_log2;      // sm_scale * log2(e)
  int32_t out_bf16;
};

struct RowArgs {
  char* k;               // layer base
  char* v;
  int64_t head_stride;   // bytes
  int32_t Hkv, D;
};

// Where the running reference of a softmax starts: the lowest finite number, not -inf.  A column all of whose scores so
// far are -inf then has weights 2^(-inf - m) = 0 and keeps (m, 0, 0), a state that later scores, other pieces and other
// partials join by the usual rescale; from -inf the differences -inf - -inf would be NaN and stay in the sums.  Finite
// scores see no difference: 2^(m - score) is 0 from either start.
constexpr float LOWEST_REF = -__FLT_MAX__;

__device__ __forceinline__ int rfl(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  return x;
}
__device__ __forceinline__ float bf16_bits_to_float(unsigned short b) {
  return __uint_as_float((unsigned int)b << 16);
}
__device__ __forceinline__ unsigned short float_to_bf16_bits(float f) {
  __bf16 h = (__bf16)f;   // round to nearest even (v_cvt_pk_bf16_f32)
  return __builtin_bit_cast(unsigned short, h);
}

// Partial states cross from one XCD's L2 to another's inside one launch.  They are written and
// read with agent-scope accesses (write-through / coherent reads, 8 bytes at a time), which keeps
// the exchange coherent without flushing or invalidating a whole L2 -- a release or acquire fence
// at agent scope does exactly that on this part and costs tens of microseconds per launch.
__device__ __forceinline__ void store_pair_agent(float* p, float x, float y) {
  const unsigned long long v = (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
  __hip_atomic_store((unsigned long long*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_pair_agent(const float* p) {
  const unsigned long long v = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}

// Arrival counter of a cut segment: {tag, count}, count 0 between launches.  The workspace is the caller's and may hold
// anything when a launch begins (its first use, another pool's records, a caller who used it as scratch), and the launch
// that plans itself has no earlier launch to clear counters in.  So the counter carries a tag: an arrival that finds other
// bytes than the tag replaces them by {tag, 1} (compare-and-swap; whoever loses the swap adds to what the winner left).
// The usual arrival is one atomic add, as with a counter known to be zero.  The tag is a NaN pattern, which no partial
// state holds in the word that would have to hold it.  Returns the number of earlier arrivals.
constexpr unsigned ARRIVE_TAG = 0x7fd15a3cu;
__device__ __forceinline__ int count_in(unsigned long long* c) {
  unsigned long long seen = __hip_atomic_fetch_add(c, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((unsigned)(seen >> 32) == ARRIVE_TAG) return (int)(unsigned)seen;
  ++seen;                                                  // what the add left behind
  while ((unsigned)(seen >> 32) != ARRIVE_TAG) {
    if (__hip_atomic_compare_exchange_strong(c, &seen, ((unsigned long long)ARRIVE_TAG << 32) | 1ull, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return 0;
  }
  return (int)(unsigned)__hip_atomic_fetch_add(c, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace
