// Prefill (chunk) attention for gfx950: the last n_q tokens of every request each carry a
// query and attend causally to the request's slab (bf16 storage, head_dim 128, G <= 16).
//
// Unlike decode this is a dense contraction with reuse: one 16-token K/V tile serves every
// query column.  The (token, head-in-group) pairs of one (request, KV head) are flattened into
// columns  col = j * G + h  (j: query token of the chunk, h: head inside the GQA group), so any
// group size fills the 16-wide matrix tiles.  A work item is 64 CT consecutive columns of one
// (request, KV head): four waves of a work-group take CT 16-column tiles each, whose Q operands
// and O accumulators stay in registers, and share the K/V tiles the item can see through LDS.
// CT = 4 (256-column items, one work-group per CU) has the most reuse per K/V byte.  CT = 2 halves the
// registers so that two work-groups share a CU and one's LDS reads and item start run under the other's
// matrix instructions: +12 to +25 % on every prompt mix measured, and the default.  Calls of long items run 256-column items by
// eight waves of CT = 2 in two groups that take turns at the matrix cores (stream_eight), if the plan finds that this pays.
//
// The items of a call, ordered by (request, KV head, column block from the heaviest down), are cut into eight queues
// of equal cost, one per XCD (cost: the 32-token K/V pairs an item streams plus a constant for its start and end), and
// handed out through atomic counters to persistent work-groups: causal items differ in length by construction.  The
// work-groups of an XCD then read the same one or two K/V heads out of their L2 -- with one queue for the chip every XCD
// fetched every K/V byte (16 x 4096 tokens: 60 M L2 misses of 128 bytes, 12 M with eight queues).  A work-group whose
// queue is empty goes on with the fullest other one.  A call with few items may cut their keys into parts instead (prefill_parts).
#pragma once

#include <type_traits>

#include "kernels_common.h"

namespace {

constexpr int PREFILL_PLAN_THREADS = 256;

constexpr int PREFILL_XCDS = 8;
// Two kernels serve the calls that are planned in front: items of 128 columns by four waves, two work-groups per CU, and items of
// 256 by eight waves (stream_eight).  An item of the latter takes the time of two of the former less 4 % in bf16, 6 in paged bf16
// and 16 in fp8, whose widening of a tile then serves twice the columns.  But nothing hides its start, the empty half of a last
// block is computed for nobody, and the item that a call ends with takes up to half as long again as one of 128 columns that has
// its CU to itself.  So the planning kernel, which knows every request, weighs them: the items must be long on the average,
// next to none of it padding, and the longest one a part of what each CU streams.  Of 2022 calls of random heads, lengths and
// chunks these rules give 420 to eight waves: the worst took 1.03 of its time with four (bf16; 0.996 in fp8), the mean 0.96 in bf16,
// 0.94 in paged bf16, 0.85 in fp8.  Chosen by rows of q per request, all that the host knows, the worst took 1.46: one request of
// many rows beside short ones, 8 / 8 heads and blocks of 256 columns with 4 in the last, 260 items on 256 CUs.
struct PrefillRule {
  float min_pairs, slope;    // mean pairs of an item of 256 columns: min_pairs and `slope` times the longest item's part (below)
  float max_longest;         // pairs of the longest item, as a part of what each CU streams
  float max_padding;         // pairs of the items of 256 columns relative to those of 128, two of these counted as one
  int32_t n_cu;              // 0: four waves
};
constexpr PrefillRule PREFILL_EIGHT_BF16 = {28.f, 20.f, 0.8f, 1.03f, 0}, PREFILL_EIGHT_BF16_PAGED = {16.f, 20.f, 1.0f, 1.03f, 0},
                      PREFILL_EIGHT_FP8 = {13.f, 0.f, 0.9f, 1.1f, 0};
// A call that is weighed has one launch more, which finds the other kernel chosen and ends (2.4 us).  It has to be long for that, in
// pairs that each CU streams (1 us or less): at least, with every row that of a whole prompt and all prompts of one length; or
// at most, with every row the last of the longest request that there can be.  (fp8 chunks of 512 at 6000 to 9000 tokens: 14 and
// 484, 605 -> 490 us.  Below 10 a call whose chunks do have little in front of them would notice the launch.)
constexpr double PREFILL_WEIGH_BF16 = 200, PREFILL_WEIGH_FP8 = 100, PREFILL_WEIGH_FP8_LEAST = 10, PREFILL_WEIGH_FP8_MOST = 400;
// A queue's last items go out one by one, this many per work-group: a work-group holds the run it is on and the one after
// it, and with runs of four items to the end the last work-group of a call was busy 23 % longer than the mean one.  256
// prompts around 256 tokens 696 -> 659 us, the same in fp8 760 -> 687, 29 of 816 tokens on the average (fp8, 56 / 8 heads) 728 ->
// 632 (two singles 1 and 5 % longer, eight 0.7 and 5).
constexpr int PREFILL_SINGLES = 4;
// A call of few items (one chunk of a long prompt: a hundred, or eight) leaves most of the chip idle while each streams its
// keys in one serial chain.  Such a call on the null stream cuts the keys of its items into parts, one per work-group, whose
// states the last one to arrive merges.  A pair costs a lone work-group about 0.55 us and a merged state 1.2, so the best number of
// parts grows with the square root of the pairs; at 16 pairs cutting is about even.  28 / 4 heads, whole -> cut: one chunk of 128
// tokens (28 items) ending at 512 tokens 17.6 -> 17.6 to 18.3 us, at 640 20.0 -> 18.9 to 19.6; two at 1024 27.3 -> 23.3; chunks of
// 512 (112 items) at 2048 45.9 -> 36.0, at 8192 158 -> 76, at 32 768 602 -> 237; one of 128 at 5090 with 8 / 8 heads 101 -> 32.2.
// (With sqrt(0.75 pairs) parts two chunks at 1024 were 4 % longer, a whole prompt of 700 24 %.)
constexpr int PREFILL_PARTS = 32;
__host__ __device__ inline int prefill_parts(int pairs) {
  if (pairs < 16) return 1;
  const int p = (int)sqrtf(0.4f * (float)pairs);
  return p < PREFILL_PARTS ? p : PREFILL_PARTS;
}
constexpr double PREFILL_ITEM_COST = 5.0;   // start and end of an item, in K/V pairs

struct PrefillHeader {
  int32_t bound[PREFILL_XCDS + 1];          // items [bound[x], bound[x + 1]) are queue x
  int32_t next[PREFILL_XCDS];               // runs claimed of every queue beyond the first of each work-group, reset by the plan
  int32_t avg_pairs;                        // mean cost of an item
  int32_t eight;                            // the call is the eight-wave kernel's
};

struct PrefillBounds {
  int bound[PREFILL_XCDS + 1];
};

struct PrefillArgs {
  const char* k;             // layer base of the K pool
  const char* v;
  const unsigned short* q;   // [total_q][Hq][128] bf16
  void* out;                 // [total_q][Hq][128]
  const int64_t* q_start;    // [n] first row of request r in q / out
  const int32_t* n_q;        // [n] query tokens of request r (the last n_q of its lengths[r] tokens)
  const int64_t* offsets;    // [n] slab base (tokens) or nullptr when paged
  const int32_t* lengths;    // [n]
  const int32_t* bt;
  int32_t bt_stride;
  PrefillHeader* hdr;
  int32_t* item_start;       // [n] exclusive prefix of items per request
  int32_t n, Hq, Hkv, G;
  int64_t total_q;           // rows of q and out: rows at or past it are never touched
  int64_t head_stride;
  float scale_log2;          // sm_scale * log2(e) (fp8 pools: times k_scale)
  float out_scale;           // 1, or v_scale for fp8 pools
  int32_t out_bf16;
  int32_t part_slots;        // parts of cut items whose states the workspace holds (0: items stay whole)
  unsigned long long* arrive;   // [part_slots] arrival counters of cut items (count_in)
  float2* part_ml;           // [part_slots][columns of an item]: reference and sum
  float* part_o;             // [part_slots][columns of an item * 128]: outputs, lane by lane
};

// query tokens of request r that are really there: never more than the tokens it holds, never
// past the end of q
__device__ __forceinline__ int prefill_rows(const int32_t* n_q, const int32_t* lengths, const int64_t* q_start,
                                            int64_t total_q, int r) {
  int64_t rows = min(n_q[r], lengths[r]);
  const int64_t s = q_start[r];
  if (s < 0 || rows < 0) return 0;
  rows = min(rows, total_q - s);
  return rows > 0 ? (int)rows : 0;
}

// Cost of the cb cheapest column blocks of one (request, KV head): block i streams about
// (first_pos + (i + 1/2) * cols_item / G) / 32 pairs.  It only balances: any rule would give the same results.
struct PrefillCost {
  double base, slope;
  __device__ __forceinline__ PrefillCost(int first_pos, int cols_item, int G)
      : base(first_pos * (1.0 / 32) + PREFILL_ITEM_COST), slope((double)cols_item / (64.0 * G)) {}
  __device__ __forceinline__ double upto(int cb) const { return cb * (base + cb * slope); }
  __device__ __forceinline__ int block_at(double c) const {              // nearest block whose start costs c
    return (int)(0.5 + (sqrt(base * base + 4.0 * slope * c) - base) / (2.0 * slope));
  }
};
__device__ __forceinline__ int prefill_blocks(int rows, int G, int cols_item) {
  return (int)(((int64_t)rows * G + cols_item - 1) / cols_item);
}

// One work-group of PREFILL_PLAN_THREADS: exclusive prefix of items per request (item_start[0 .. n)), and in `pl` the bounds of
// the eight queues of equal cost.  LONGEST: the most tokens of a request with items as well.  WEIGH: items of cols_item or twice
// the columns, by `rule`.  Ends with a barrier.
struct PrefillPlan {
  double part_cost[2][PREFILL_PLAN_THREADS / 64];
  int part_items[2][PREFILL_PLAN_THREADS / 64], part_longest[PREFILL_PLAN_THREADS / 64];
  int bound[PREFILL_XCDS + 1], avg_pairs, longest, eight;
};
template <bool LONGEST, bool WEIGH = false>
__device__ __forceinline__ void prefill_plan(const int32_t* n_q, const int32_t* lengths, const int64_t* q_start, int64_t total_q,
                                             int32_t n, int32_t Hkv, int32_t G, int32_t cols_item, PrefillPlan& pl,
                                             int32_t* item_start, PrefillRule rule = {}) {
  constexpr int SIZES = WEIGH ? 2 : 1;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (n + PREFILL_PLAN_THREADS - 1) / PREFILL_PLAN_THREADS;
  const int r0 = min(tid * per, n), r1 = min(r0 + per, n);
  double cost[SIZES] = {};
  int items[SIZES] = {}, longest = 0;
  for (int r = r0; r < r1; ++r) {
    const int rows = prefill_rows(n_q, lengths, q_start, total_q, r);
#pragma unroll
    for (int z = 0; z < SIZES; ++z) {
      const int nb = prefill_blocks(rows, G, cols_item << z);
      cost[z] += Hkv * PrefillCost(lengths[r] - rows, cols_item << z, G).upto(nb);
      items[z] += Hkv * nb;
    }
    if (LONGEST || WEIGH) longest = max(longest, rows ? lengths[r] : 0);
  }
  double inc_cost[SIZES];
  int inc_items[SIZES];
#pragma unroll
  for (int z = 0; z < SIZES; ++z) {
    inc_cost[z] = cost[z];
    inc_items[z] = items[z];
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    if (LONGEST || WEIGH) longest = max(longest, __shfl_up(longest, o));        // (a lane below o gets its own)
#pragma unroll
    for (int z = 0; z < SIZES; ++z) {
      const double yc = __shfl_up(inc_cost[z], o);
      const int yi = __shfl_up(inc_items[z], o);
      if (lane >= o) {
        inc_cost[z] += yc;
        inc_items[z] += yi;
      }
    }
  }
  if (lane == 63) {
#pragma unroll
    for (int z = 0; z < SIZES; ++z) {
      pl.part_cost[z][wv] = inc_cost[z];
      pl.part_items[z][wv] = inc_items[z];
    }
    if (LONGEST || WEIGH) pl.part_longest[wv] = longest;
  }
  __syncthreads();
  double all_cost[SIZES] = {};
  int all_items[SIZES] = {};
#pragma unroll
  for (int z = 0; z < SIZES; ++z) {
    cost[z] = inc_cost[z] - cost[z];
    items[z] = inc_items[z] - items[z];
    for (int i = 0; i < PREFILL_PLAN_THREADS / 64; ++i) {
      if (i < wv) {
        cost[z] += pl.part_cost[z][i];
        items[z] += pl.part_items[z][i];
      }
      all_cost[z] += pl.part_cost[z][i];
      all_items[z] += pl.part_items[z][i];
    }
  }
  if (LONGEST || WEIGH)
    for (int i = 0; i < PREFILL_PLAN_THREADS / 64; ++i) longest = max(longest, pl.part_longest[i]);
  // the size of the items: everything below is about that one
  bool eight = false;
  if constexpr (WEIGH) {
    const float pairs4 = (float)(all_cost[0] - PREFILL_ITEM_COST * all_items[0]), pairs8 = (float)(all_cost[1] - PREFILL_ITEM_COST * all_items[1]);
    const float part = (float)longest * (1.f / (2 * BLK)) * (float)rule.n_cu / pairs8;
    eight = pairs8 >= (rule.min_pairs + rule.slope * part) * (float)all_items[1] && part <= rule.max_longest &&
            2.f * pairs8 <= rule.max_padding * pairs4;               // (a call without items: not a number, so four)
  }
  const int cols = cols_item << eight;
  const double total = all_cost[eight];
  const int n_items = all_items[eight];
  double at = cost[eight];
  int first = items[eight];
  // a boundary that rounding leaves to no thread keeps its share of the items
  if (tid <= PREFILL_XCDS) pl.bound[tid] = (int)((long long)n_items * tid / PREFILL_XCDS);
  if (tid == 0) {
    pl.avg_pairs = (int)(total / max(n_items, 1));
    if (LONGEST) pl.longest = longest;
    pl.eight = eight;
  }
  __syncthreads();
  // boundary x lies at cost total * x / 8, inside the request whose cost range holds it
  for (int r = r0; r < r1; ++r) {
    item_start[r] = first;
    const int rows = prefill_rows(n_q, lengths, q_start, total_q, r), nb = prefill_blocks(rows, G, cols);
    const PrefillCost pc(lengths[r] - rows, cols, G);
    const double per_head = pc.upto(nb);
    if (nb)
      for (int x = 1; x < PREFILL_XCDS; ++x) {
        const double t = total * x / PREFILL_XCDS - at;
        if (t < 0 || t >= Hkv * per_head) continue;
        const int g = min((int)(t / per_head), Hkv - 1);
        // blocks run from the last one (the dearest) down: those that cost t come after those that cost the rest
        const int left = min(max(pc.block_at(fmax(per_head - (t - g * per_head), 0.0)), 0), nb);
        pl.bound[x] = first + g * nb + nb - left;
      }
    at += Hkv * per_head;
    first += Hkv * nb;
  }
  __syncthreads();
  if (tid == 0)                                             // (two threads' ranges may meet an ulp apart)
    for (int x = 1; x <= PREFILL_XCDS; ++x) pl.bound[x] = min(max(pl.bound[x], pl.bound[x - 1]), n_items);
  __syncthreads();
}

// the plan as a launch of its own: for calls with many items or requests
template <bool WEIGH>
__global__ __launch_bounds__(PREFILL_PLAN_THREADS) void prefill_plan_kernel(const int32_t* __restrict__ n_q,
                                                                           const int32_t* __restrict__ lengths,
                                                                           const int64_t* __restrict__ q_start,
                                                                           int64_t total_q, int32_t n, int32_t Hkv, int32_t G,
                                                                           int32_t cols_item, PrefillHeader* hdr,
                                                                           int32_t* item_start, PrefillRule rule) {
  __shared__ PrefillPlan pl;
  prefill_plan<false, WEIGH>(n_q, lengths, q_start, total_q, n, Hkv, G, cols_item, pl, item_start, rule);
  const int tid = threadIdx.x;
  if (tid <= PREFILL_XCDS) hdr->bound[tid] = pl.bound[tid];
  if (tid < PREFILL_XCDS) hdr->next[tid] = 0;
  if (tid == 0) {
    hdr->avg_pairs = pl.avg_pairs;
    hdr->eight = pl.eight;
  }
}

// LDS stage of one pair of tiles (32 tokens): K of both tiles as loaded (the 16x16x32 A operands of
// S^T = K Q^T), and V rearranged into the A operands of O^T += V^T P^T over the 32 tokens: for channel
// group dt, lane (c, q) finds channels c of tokens 4q .. 4q+3 of the first tile followed by the same of
// the second tile in one 16-byte piece.
constexpr int PREFILL_STAGE_BYTES = 16384;
constexpr int PREFILL_STAGES = 2;
constexpr int PREFILL_LDS_REQ = 1024;        // requests whose item prefix a work-group keeps in LDS
typedef const int64_t __attribute__((address_space(4))) const_i64;

// two E4M3 bytes of a word -> two bf16 bit patterns in one word (exact: E4M3 values are bf16 values)
template <bool HIGH_HALF>
__device__ __forceinline__ unsigned fp8x2_to_bf16x2(unsigned w) {
  typedef float float2v __attribute__((ext_vector_type(2)));
  const float2v f = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, HIGH_HALF);
  return (__float_as_uint(f[0]) >> 16) | (__float_as_uint(f[1]) & 0xffff0000u);
}

// FP8: the pools hold E4M3 bytes (2 KiB blocks in the fp8 operand order of the decode kernel); the loader waves
// widen them to bf16 on the way into LDS and store them in the bf16 layout, everything after that is shared.
// HERE: the kernel plans for itself (a variant of its own: inside the other one the plan cost the pair loop registers, 254
// for 242, and 2 to 7 % of every long call).
// CUT: it cuts items into parts as well, where they are few and long (again a variant of its own, for calls that may: with the
// code in them calls of few items take 0.3 to 0.4 us more, 41 prompts of 1 to 250 tokens 12.05 -> 12.45).
template <bool PAGED, int CT, bool FP8, bool HERE, bool CUT, int WAVES = 4>
__global__ __launch_bounds__(64 * WAVES, CT == 4 ? 1 : 2) void prefill_kernel(PrefillArgs a) {
  constexpr bool EIGHT = WAVES == 8;
  static_assert(!EIGHT || (CT == 2 && !HERE && !CUT), "eight waves: long calls planned in front");
  constexpr int TILE_BYTES = BLK * 128 * (FP8 ? 1 : 2);
  constexpr int LOADS = TILE_BYTES / 1024;                         // 16-byte loads per lane and tile
  constexpr int STAGES = EIGHT ? 4 : PREFILL_STAGES;
  constexpr int COLS_WAVE = 16 * CT, COLS_ITEM = WAVES * COLS_WAVE;   // CT column tiles per wave
  __shared__ __attribute__((aligned(16))) char stage_mem[STAGES * PREFILL_STAGE_BYTES];
  __shared__ int run_slot[2];
  __shared__ int item_start_lds[PREFILL_LDS_REQ];
  const int lane = threadIdx.x & 63, wv = rfl(threadIdx.x >> 6);
  const int col16 = lane & 15, g4 = lane >> 4;
  const int G = a.G;
  const float NEG_INF = -INFINITY;
  // Loader role of this wave, whose tile of a pair is the first or the second one.  Four waves: 0 and 1 bring its K, 2 and 3 its V
  // (loads_v and src_base, issue and write_stage are theirs).  Eight: each brings a quarter of both (stream_eight).
  const bool loads_v = wv >= 2;
  const int which = EIGHT ? wv >> 2 : wv & 1;
  const char* src_base = loads_v ? a.v : a.k;
  const unsigned lane16 = lane * 16;

  // Work queues.  A counter in memory answers about 14 M requests a second on this part -- with thousands of small items
  // that alone would bound the kernel.  A work-group therefore takes runs of consecutive items, long enough to stream
  // about 64 K/V pairs (some 40 us) but never more than an eighth of its share of the items, so that large items still
  // balance one by one, as do the last items of a queue; its first run is its turn's (no counter is touched when that is all
  // there is), and it asks for the next one a run ahead: the answer travels while the current run is computed.
  //
  // A call whose items are few (the launch's rule) plans here instead of in a launch in front -- six microseconds of one
  // work-group's round trips and the edge between two launches -- and its work-groups take every `turns`-th item of their
  // queue: no counter has to be clear before the launch.  7 prompts of 21 to
  // 58 tokens 11.2 -> 8.3 us, 28 of 91 to 546 tokens 20.0 -> 17.5.
  __shared__ typename std::conditional<HERE, PrefillPlan, PrefillBounds>::type plan;   // (in LDS: read between runs only)
  int (&bound)[PREFILL_XCDS + 1] = plan.bound;
  __shared__ int whole_runs[PREFILL_XCDS], run_items;                  // of each queue, in front of its singles; of a run
  const bool small = a.n <= PREFILL_LDS_REQ;
  const int turns = gridDim.x / PREFILL_XCDS;                          // work-groups of an XCD
  int run = 1;
  if constexpr (HERE) {                                                // (n <= PREFILL_LDS_REQ)
    prefill_plan<CUT>(a.n_q, a.lengths, a.q_start, a.total_q, a.n, a.Hkv, a.G, COLS_ITEM, plan, item_start_lds);
  } else {
    // The plan gave the call to the other kernel: all of its waves end here.  (In paged fp8 by the instruction.  A return, which joins
    // the kernel's end, gives the stage writes another schedule: paged calls of four waves 1.016 of the time without either, 1.007 with
    // the instruction, of eight 0.843 and 0.836; contiguous ones of four 0.999 and 1.010, of eight 0.844 and 0.851.  Four column tiles
    // are never weighed.)
    if (CT == 2 && a.hdr->eight != EIGHT) {
      if constexpr (FP8 && PAGED) __builtin_amdgcn_endpgm();
      else return;
    }
    run = min(min(max(64 / max(a.hdr->avg_pairs, 1), 1), 16), max(a.hdr->bound[PREFILL_XCDS] / ((int)gridDim.x * 8), 1));
    if (threadIdx.x <= PREFILL_XCDS) bound[threadIdx.x] = a.hdr->bound[threadIdx.x];
    if (threadIdx.x == 0) run_items = run;
    if (threadIdx.x < PREFILL_XCDS)
      whole_runs[threadIdx.x] = max(a.hdr->bound[threadIdx.x + 1] - a.hdr->bound[threadIdx.x] - PREFILL_SINGLES * turns, 0) / run;
    if (small)
      for (int i = threadIdx.x; i < a.n; i += 64 * WAVES) item_start_lds[i] = a.item_start[i];
    __syncthreads();
  }
  // Most parts that an item is cut into: as many as there is room for, and no more than the longest request's items have (parts
  // that nobody has are turns of a search, a round of loads and a barrier: five prompts of 50 tokens in a pool of slabs of
  // 16 384 10.5 us with them, 9.9 without).  An item that is too short for so many leaves its last ones empty.
  const int n_items = rfl(bound[PREFILL_XCDS]);
  // (fractions with a denominator of at most 512 are 1/512 apart or more; beyond 512 items the result is at most 1 all the same)
  const float part_room = (float)min(a.part_slots, (int)gridDim.x) * __builtin_amdgcn_rcpf((float)max(n_items, 1)) + 0x1p-10f;
  int parts = 1;
  if constexpr (CUT) parts = rfl(max(min((int)part_room, prefill_parts((plan.longest + 2 * BLK - 1) / (2 * BLK))), 1));
  // Run j of a queue of len items begins at its item run_at(len, whole, j) and ends where the next one begins: the last
  // PREFILL_SINGLES items per work-group are runs of their own.  (Counted once and from LDS: divided out and held in registers
  // over the pair loop, 16 prompts of 4096 tokens took 1886 us instead of 1874, 256 around 256 663 instead of 659.)
  auto run_at = [&](int len, int whole, int j) { return min(min(j, whole) * run_items + max(j - whole, 0), len); };
  int queue = blockIdx.x % PREFILL_XCDS;                               // (work-group b runs on XCD b % 8)
  int ahead = 0;
  auto claim = [&]() {
    if (threadIdx.x == 0) ahead = atomicAdd(&a.hdr->next[queue], 1);
  };
  // wave 0: the run after the present one, in run_slot (empty when the call is over).  With its own queue empty a
  // work-group goes on with the fullest one that was longer than its work-groups' first runs.
  bool claimed = false;
  auto settle = [&]() {
    const int x = lane % PREFILL_XCDS, at = bound[x], len = bound[x + 1] - at, whole = whole_runs[x];   // lane x: queue x
    const bool more = run_at(len, whole, turns) < len;
    const unsigned longer = (unsigned)__builtin_amdgcn_ballot_w64(more);
    int start = 0, end = 0;
    auto take = [&]() {                                                // the run that `ahead` names
      const int j = turns + rfl(ahead);
      start = __builtin_amdgcn_readlane(at + run_at(len, whole, j), queue);
      end = __builtin_amdgcn_readlane(at + run_at(len, whole, j + 1), queue);
    };
    if (claimed) take();
    while (start >= end && longer != 0) {
      const int taken = __hip_atomic_load(&a.hdr->next[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int left = more ? len - run_at(len, whole, turns + taken) : 0;
      int most = left;
#pragma unroll
      for (int o = 1; o < PREFILL_XCDS; o <<= 1) most = max(most, __shfl_xor(most, o));
      most = rfl(most);
      if (most == 0) break;
      queue = __builtin_ctzll(__builtin_amdgcn_ballot_w64(left == most));
      claim();
      take();
    }
    if (lane == 0) {
      run_slot[0] = start;
      run_slot[1] = end;
    }
    claimed = start < end && ((longer >> queue) & 1) != 0;
    if (claimed) claim();
  };
  int next = 0, run_end = 0;                                           // the present run: what is left of it
  // HERE: the work-group's next part, the end of its XCD's, and the items they belong to, [first_of, first_of + n_of): all first
  // parts, then the second ones, ...  An XCD has its queue's items.  With fewer items than queues all XCDs share them: some
  // queues would be empty, and one item's parts an eighth of the work-groups' (one chunk of 128 tokens at 32 768, 4 / 1 heads,
  // 99 -> 65 us; of 16, 8 / 1 heads, 136 -> 63).
  int unit = blockIdx.x / PREFILL_XCDS, unit_end = 0, first_of = 0, n_of = n_items;
  if constexpr (HERE) {
    if (n_items < PREFILL_XCDS) {
      unit += n_items * parts * queue / PREFILL_XCDS;
      unit_end = n_items * parts * (queue + 1) / PREFILL_XCDS;
    } else {
      first_of = rfl(bound[queue]);
      n_of = rfl(bound[queue + 1]) - first_of;
      unit_end = n_of * parts;
    }
  } else {
    const int at = rfl(bound[queue]), len = rfl(bound[queue + 1]) - at, whole = rfl(whole_runs[queue]), turn = blockIdx.x / PREFILL_XCDS;
    next = at + run_at(len, whole, turn);
    run_end = at + run_at(len, whole, turn + 1);
    if (wv == 0 && next < run_end && run_at(len, whole, turns) < len) {
      claimed = true;
      claim();
    }
  }
  for (;;) {
    // ---- next item (every wave reaches the exit together)
    __syncthreads();                                       // the previous item's slot and stages are done with
    int item, part = 0;
    if constexpr (HERE) {
      if (unit >= unit_end) break;
      if (CUT) part = rfl((int)(((float)unit + 0.5f) * __builtin_amdgcn_rcpf((float)n_of)));   // (half an n_of-th or more from whole numbers)
      item = first_of + unit - part * n_of;
      unit += turns;
    } else {
      if (next >= run_end) {
        if (wv == 0) settle();
        __syncthreads();
        next = rfl(run_slot[0]);
        run_end = rfl(run_slot[1]);
        if (next >= run_end) break;
      }
      item = next++;
    }
    // Request of the item: largest r with item_start[r] <= item (item_start is non-decreasing; empty requests repeat
    // a value, so it is the last one that still has items).  In LDS, where the table fits: the number of such entries, 64 a
    // round.  In memory every round is a dependent round trip, so there the 64 lanes probe evenly spaced entries of the
    // range that is left, which is two rounds up to 4096 requests (counted 64 by 64, 4096 requests of 8 to 40 tokens took
    // 795 us instead of 429).
    // Everything else an item needs is then one round of scalar loads, all in flight together: an item of a short prompt
    // streams fewer than ten pairs, so each dependent round trip in front of it shows.
    int found = 0;
    if (small) {
      int cnt = 0;
      for (int i0 = 0; i0 < a.n; i0 += 64) {
        const bool le = i0 + lane < a.n && item_start_lds[min(i0 + lane, a.n - 1)] <= item;
        const int k = __builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
        cnt += k;
        if (k < 64) break;
      }
      found = cnt - 1;
    } else {
      int hi = a.n;                                                    // the request is in [found, hi)
      while (hi - found > 1) {
        const int span = (hi - found + 63) / 64, i = found + lane * span;
        const bool le = i < hi && a.item_start[min(i, hi - 1)] <= item;
        const int k = __builtin_popcountll(__builtin_amdgcn_ballot_w64(le));   // (at least the first)
        found += (k - 1) * span;
        hi = min(found + span, hi);
      }
    }
    const int r = rfl(found);
    const int first_item = rfl(small ? item_start_lds[r] : a.item_start[r]);
    int len = as_constant(a.lengths)[r];
    const int asked = as_constant(a.n_q)[r];
    const int64_t q_row0 = ((const const_i64*)(uintptr_t)a.q_start)[r];
    const int64_t base_block = PAGED ? 0 : ((const const_i64*)(uintptr_t)a.offsets)[r] / BLK;
    // (the request has items, so its rows exist: prefill_rows without its checks)
    const int rows = (int)min((int64_t)min(asked, len), a.total_q - q_row0);
    const int n_blocks_item = rfl((int)(((int64_t)rows * G + COLS_ITEM - 1) / COLS_ITEM));
    const int idx = item - first_item;
    const int g = rfl(idx / n_blocks_item);
    const int cb = n_blocks_item - 1 - (idx - g * n_blocks_item);    // heaviest (latest) columns first
    const int n_cols = rows * G;
    const int c0 = cb * COLS_ITEM + wv * COLS_WAVE;   // this wave's first column
    const bool active = c0 < n_cols;                                  // a wave without columns still helps to load
    const int first_pos = len - rows;                                // position of query token 0

    // ---- per-lane columns: tile ct holds column c0 + 16 ct + col16
    // keys visible to the column (of a part: from its first one on, which may be less than none)
    constexpr int ABSENT = CUT ? -(1 << 30) : 0;                      // (or less)
    int lim[CT];
    int64_t q_at[CT];                                                  // the column's row in q and out, in elements
    bf16x8 qreg[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int col = c0 + 16 * ct + col16;
      const bool ok = col < n_cols;
      const int j = ok ? col / G : 0, h = ok ? col - j * G : 0;
      lim[ct] = ok ? first_pos + j + 1 : ABSENT;
      q_at[ct] = ((q_row0 + j) * a.Hq + g * G + h) * 128;
    }
    auto load_q = [&](bf16x8 (&qq)[CT][4]) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
          qq[ct][s] = lim[ct] > ABSENT ? *(const bf16x8*)(a.q + q_at[ct] + 32 * s + 8 * g4) : z;
        }
    };
    load_q(qreg);
    // keys the item streams: up to the limit of its last column; this wave's own columns end earlier
    const int item_last_col = min((cb + 1) * COLS_ITEM, n_cols) - 1;
    const int item_lim_max = first_pos + item_last_col / G + 1;
    int lim_min = first_pos + c0 / G + 1;                             // pairs below it need no mask in this wave
    int n_tiles = (item_lim_max + BLK - 1) / BLK, skipped = 0;         // skipped: tiles in front of the part
    const int all_pairs = (n_tiles + 1) / 2;
    int n_pairs = all_pairs, n_parts = 1;
    if (CUT && parts > 1) {
      n_parts = min(prefill_parts(all_pairs), parts);
      if (part >= n_parts) continue;
      // from here on the part's first token is token 0
      const int before = all_pairs * part / n_parts;
      n_pairs = all_pairs * (part + 1) / n_parts - before;
      n_tiles -= 2 * before;
      len -= 2 * BLK * before;
      skipped = 2 * before;
      lim_min -= 2 * BLK * before;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) lim[ct] -= 2 * BLK * before;
    }

    float m[CT], lsum[CT];
    float4v O[CT][8];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      m[ct] = NEG_INF;
      lsum[ct] = 0.f;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) O[ct][dt] = float4v{0.f, 0.f, 0.f, 0.f};
    }

    const int64_t plane = (int64_t)g * a.head_stride + (PAGED ? 0 : (int64_t)skipped * TILE_BYTES);
    const const_i32* bt_row = as_constant(PAGED ? a.bt + (int64_t)r * a.bt_stride + skipped : nullptr);
    // ---- loading: this wave's tile of pair pr -> registers, 16 bytes per lane and piece -> LDS.  Pairs past the
    // end and a second tile that does not exist re-read the last tile: every step issues its loads, so the waits on
    // them stay static counts (with conditional loads the wait before a stage was written covered the loads issued a
    // moment ago as well, and the whole memory latency was exposed in every pair).  V slots at or past `len` (stale bytes,
    // maybe NaN patterns) are zeroed, and so is the V of a tile that does not exist (the last tile's may be infinite), so
    // that a weight of 0 really removes them.  (K needs nothing: scores of tokens past a column's limit are replaced, not
    // multiplied, and the tokens of such a tile lie past every column's limit.)
    auto tile_of = [&](int pr) { return min(2 * pr + which, n_tiles - 1); };
    // tokens below it have a V: with an odd number of tiles the wave of the second tiles meets the last tile only where its
    // own does not exist (one number for the whole item: decided pair by pair it cost fp8 pools 8 %)
    const int held = (which & n_tiles & 1) ? (n_tiles - 1) * BLK : len;
    int blk_next = 0;
    auto lookup = [&](int pr) {
      if (PAGED) blk_next = bt_row[tile_of(pr)];
    };

    // One pair of tiles against the wave's 64 columns.  Scores: S^T = K Q^T per tile (16x16x32 over
    // the channels).  O^T += V^T P^T contracts over the 32 tokens of the pair in one 16x16x32
    // instruction per channel group: lane (., g4) supplies tokens 4 g4 .. +3 of the first tile, then of
    // the second, which is how the score accumulators hold them and how the stage stores V.
    //
    // Softmax reference.  Softmax is invariant under the choice of the reference m subtracted in the
    // exponent, and fp32 / bf16 weights have room for 2^127: the fast pass fixes m of a column to the
    // exact maximum over the item's (or part's) first pair and never moves it, so the steady
    // state holds no cross-lane maximum, no rescale of O and no second exponential.  Should later scores
    // exceed that reference so far that a column's weight sum passes 2^90 (or turns inf / NaN), or lie so far below the
    // stand-in reference of a column whose first pair scored -inf that the sum stays under 2^-60 (in a part: 1/2), the wave
    // repeats its columns in the slow pass below, the classic online softmax that moves its references.
    auto scores_of = [&](float4v (&x)[CT][2], const bf16x8 (&qq)[CT][4], auto&& kop) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        bf16x8 kk[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) kk[s] = kop(b, s);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          float4v s4 = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < 4; ++s) s4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk[s], qq[ct][s], s4, 0, 0, 0);
          x[ct][b] = s4;                                               // raw: the scale joins the exponent
        }
      }
    };
    auto mask = [&](float4v (&x)[CT][2], int pr) {
      const int t0 = pr * 2 * BLK;
      if (t0 + 2 * BLK > lim_min) {                                    // some column cannot see the whole pair
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (t0 + 16 * b + 4 * g4 + i >= lim[ct]) x[ct][b][i] = NEG_INF;
      }
    };
    // per-lane maximum of a column tile's eight scores, in exponent units (the scale is positive)
    auto lane_max = [&](const float4v (&xc)[2]) {
      return fmaxf(fmaxf(fmaxf(xc[0][0], xc[0][1]), fmaxf(xc[0][2], xc[0][3])),
                   fmaxf(fmaxf(xc[1][0], xc[1][1]), fmaxf(xc[1][2], xc[1][3]))) * a.scale_log2;
    };
    // the V operands of a pair: requested before the scores are computed, so that the LDS reads run under
    // the matrix instructions of S^T instead of in front of those of P V
    auto read_v = [&](bf16x8 (&av)[8], int pr) {
      const char* st = stage_mem + (pr % STAGES) * PREFILL_STAGE_BYTES + lane * 16;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) av[dt] = *(const bf16x8*)(st + 8192 + dt * 1024);
    };
    auto weights = [&](const float4v (&x)[CT][2], const bf16x8 (&av)[8]) {
      bf16x8 p8[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(x[ct][b][i], a.scale_log2, -m[ct]));
            psum += pv;
            p8[ct][4 * b + i] = (__bf16)pv;
          }
        lsum[ct] += psum;
      }
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          O[ct][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[dt], p8[ct], O[ct][dt], 0, 0, 0);
    };
    auto references = [&](const float4v (&x)[CT][2]) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        float tmax = lane_max(x[ct]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        m[ct] = tmax == NEG_INF ? 0.f : tmax;
      }
    };
    // fast pass: references fixed by the first pair.  m holds a finite value from then on (0 for a
    // column that does not exist).
    auto compute_fast = [&](int pr) {
      float4v x[CT][2];
      bf16x8 av[8];
      read_v(av, pr);
      const char* st = stage_mem + (pr % STAGES) * PREFILL_STAGE_BYTES + lane * 16;
      scores_of(x, qreg, [&](int b, int s) { return *(const bf16x8*)(st + b * 4096 + s * 1024); });
      mask(x, pr);
      if (pr == 0) references(x);
      weights(x, av);
    };
    // the same zeroing in the operands
    auto mask_v = [&](bf16x8 (&av)[8], int pr) {
      const int ta = 2 * pr * BLK, held = 2 * pr + 1 < n_tiles ? len : min(len, ta + BLK);
      if (ta + 2 * BLK > held) {
        uint4v keep;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int tok = ta + (w < 2 ? 0 : BLK) + 4 * g4 + 2 * (w & 1);
          keep[w] = (tok < held ? 0x0000ffffu : 0u) | (tok + 1 < held ? 0xffff0000u : 0u);
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) av[dt] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(uint4v, av[dt]) & keep);
      }
    };
    auto join = [](uint2v lo, uint2v hi) { return __builtin_bit_cast(bf16x8, uint4v{lo[0], lo[1], hi[0], hi[1]}); };
    // ---- slow pass of this wave's columns: operands straight from memory, no stage, no barrier.  A reference moves
    // whenever a score exceeds it by more than MAX_SLACK exponent units; the sums and O are rescaled then.
    constexpr float MAX_SLACK = 12.0f;
    auto slow_pass = [&]() {
      bf16x8 qq[CT][4];
      load_q(qq);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        m[ct] = NEG_INF;
        lsum[ct] = 0.f;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) O[ct][dt] = float4v{0.f, 0.f, 0.f, 0.f};
      }
      // The loads of a pair stand in front of its scores, its block ids (paged; scalar loads) a pair further ahead, and
      // fp8's K, whose registers there is room for, as well: with each of them where it was used, a pair began with one or
      // two more exposed round trips.  17 prompts, most of them 4096 tokens, all columns repeated: fp8 4803 -> 4626 us and
      // paged 5030 -> 4674, bf16 paged 4441 -> 4031, bf16 contiguous 4190 -> 4250 (repeating the item through the LDS
      // stages instead: 4725, 4846, 4508, 4398).
      int64_t at[2], next_at[2];
      uint4v kr[2][LOADS], vr[2][LOADS];
      auto look_up = [&](int pr) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int t = min(2 * pr + b, n_tiles - 1);
          next_at[b] = plane + (PAGED ? (int64_t)bt_row[t] : base_block + t) * TILE_BYTES;
        }
      };
      auto load = [&](uint4v (&to)[2][LOADS], const char* pool, const int64_t (&from)[2]) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int s = 0; s < LOADS; ++s) to[b][s] = *(const uint4v*)(pool + from[b] + s * 1024 + lane16);
      };
      // piece s (of four) of a tile as bf16; fp8: half of a loaded piece, widened
      auto piece = [&](const uint4v (&w)[LOADS], int s) {
        if (!FP8) return w[s % LOADS];
        const unsigned w0 = w[(s >> 1) % LOADS][2 * (s & 1)], w1 = w[(s >> 1) % LOADS][2 * (s & 1) + 1];
        return uint4v{fp8x2_to_bf16x2<false>(w0), fp8x2_to_bf16x2<true>(w0), fp8x2_to_bf16x2<false>(w1), fp8x2_to_bf16x2<true>(w1)};
      };
      look_up(0);
      if (FP8) load(kr, a.k, next_at);
      for (int pr = 0; CUT ? pr < n_pairs : 2 * pr < n_tiles; ++pr) {
#pragma unroll
        for (int b = 0; b < 2; ++b) at[b] = next_at[b];
        look_up(pr + 1);
        if (!FP8) load(kr, a.k, at);
        load(vr, a.v, at);
        float4v x[CT][2];
        scores_of(x, qq, [&](int b, int s) { return __builtin_bit_cast(bf16x8, piece(kr[b], s)); });
        if (FP8) load(kr, a.k, next_at);
        mask(x, pr);
        bool moved = false;
        float local[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          local[ct] = lane_max(x[ct]);
          moved |= local[ct] > m[ct] + MAX_SLACK;                          // (m = -inf: any visible score moves it)
        }
        if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            float tmax = local[ct];
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
            const float m_new = fmaxf(m[ct], tmax);
            // a column that has seen nothing yet keeps m = -inf; 0 stands in so that no inf - inf appears
            const float alpha = __builtin_amdgcn_exp2f(m[ct] - (m_new == NEG_INF ? 0.f : m_new));
            lsum[ct] *= alpha;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) O[ct][dt] *= alpha;
            m[ct] = m_new;
          }
        }
        float keep[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          keep[ct] = m[ct];
          if (m[ct] == NEG_INF) m[ct] = 0.f;                               // stand-in while the weights are formed
        }
        bf16x8 av[8];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const uint4v w0 = piece(vr[0], s), w1 = piece(vr[1], s);          // per tile: channel groups 2 s and 2 s + 1
          av[2 * s] = join(uint2v{w0[0], w0[1]}, uint2v{w1[0], w1[1]});
          av[2 * s + 1] = join(uint2v{w0[2], w0[3]}, uint2v{w1[2], w1[3]});
        }
        mask_v(av, pr);
        weights(x, av);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) m[ct] = keep[ct];
      }
    };

    // ---- pipeline: the loads of pair p + 2 are in flight while pair p is computed; pair p + 1 sits in
    // registers until the computation of pair p is over, is written into the other stage, and one
    // work-group barrier per pair makes it visible (and tells that the stage of pair p is free again).
    auto stream = [&]() {
      auto issue = [&](uint4v (&rg)[LOADS], int pr) {
        const char* src = src_base + plane + (PAGED ? (int64_t)blk_next : base_block + tile_of(pr)) * TILE_BYTES;
#pragma unroll
        for (int s = 0; s < LOADS; ++s) rg[s] = *(const uint4v*)(src + s * 1024 + lane16);
      };
      auto write_stage = [&](uint4v (&rg)[LOADS], int pr) {
        char* st = stage_mem + (pr % STAGES) * PREFILL_STAGE_BYTES;
        const int t = tile_of(pr);
        if (FP8) {
          if (!loads_v) {
            // lane (t16, q) holds, per 64-channel half s, channels 64 s + 8 q .. +7 and 64 s + 32 + 8 q .. +7 of
            // token t16: two bf16 pieces, for channel octets 8 s + q and 8 s + 4 + q
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
              const uint4v w = rg[i];
              const int s = i;
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const uint4v o = {fp8x2_to_bf16x2<false>(w[2 * h]), fp8x2_to_bf16x2<true>(w[2 * h]),
                                  fp8x2_to_bf16x2<false>(w[2 * h + 1]), fp8x2_to_bf16x2<true>(w[2 * h + 1])};
                *(uint4v*)(st + which * 4096 + (((8 * s + 4 * h + g4) * 16 + col16) * 16)) = o;
              }
            }
          } else {
            // lane (c, q) holds, per half s, one word per channel group 4 s + i: channel c of tokens 4q .. 4q+3
            const int tok0 = t * BLK + 4 * g4;
            const bool ragged = t * BLK + BLK > held;                      // (the same for the whole wave)
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {
              const uint4v w = rg[j];
              const int s = j;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                uint2v o = {fp8x2_to_bf16x2<false>(w[i]), fp8x2_to_bf16x2<true>(w[i])};
                if (ragged) {                                             // some of the tile's tokens are not there
                  if (tok0 + 0 >= held) o[0] &= 0xffff0000u;
                  if (tok0 + 1 >= held) o[0] &= 0x0000ffffu;
                  if (tok0 + 2 >= held) o[1] &= 0xffff0000u;
                  if (tok0 + 3 >= held) o[1] &= 0x0000ffffu;
                }
                *(uint2v*)(st + 8192 + (4 * s + i) * 1024 + lane * 16 + which * 8) = o;
              }
            }
          }
        } else if (!loads_v) {
#pragma unroll
          for (int s = 0; s < LOADS; ++s) *(uint4v*)(st + which * 4096 + s * 1024 + lane * 16) = rg[s];
        } else {
          // lane (c, q) holds, per piece s, tokens 4q .. 4q+3 of channel groups 2s (low 8 bytes) and 2s+1
          if (t * BLK + BLK > held) {                                      // some of the tile's tokens are not there
            const int tok0 = t * BLK + 4 * g4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (tok0 + i >= held) {
                const unsigned keep = (i & 1) ? 0x0000ffffu : 0xffff0000u;
#pragma unroll
                for (int s = 0; s < LOADS; ++s) {
                  rg[s][i >> 1] &= keep;
                  rg[s][2 + (i >> 1)] &= keep;
                }
              }
          }
          char* dst = st + 8192 + lane * 16 + which * 8;
#pragma unroll
          for (int s = 0; s < LOADS; ++s) {
            *(uint2v*)(dst + (2 * s) * 1024) = uint2v{rg[s][0], rg[s][1]};
            *(uint2v*)(dst + (2 * s + 1) * 1024) = uint2v{rg[s][2], rg[s][3]};
          }
        }
      };
      uint4v ra[LOADS], rb[LOADS];
      lookup(0);
      issue(ra, 0);
      lookup(1);
      issue(rb, 1);
      lookup(2);
      write_stage(ra, 0);
      __syncthreads();
      auto step = [&](uint4v (&near)[LOADS], uint4v (&far)[LOADS], int pr) {     // near: pair pr + 1, far: free for pair pr + 2
        issue(far, pr + 2);
        lookup(pr + 3);
        if (active) compute_fast(pr);
        write_stage(near, pr + 1);
        __syncthreads();
      };
      for (int pr = 0;;) {
        step(rb, ra, pr);
        if (++pr == n_pairs) break;
        step(ra, rb, pr);
        if (++pr == n_pairs) break;
      }
    };
    // ---- the eight-wave pipeline.  Two groups of four waves, a wave of each on every SIMD, take neighbouring columns of one
    // item half a step apart: while one forms weights (step p's vector half), the other is in its matrix half, the scores of
    // its next pair and P V of this one.  Two work-groups of four waves drift against each other as they like, and a SIMD's two
    // waves took 967 cycles a pair each where either half alone needs 520 to 560; half a step is 930 here, of which the
    // writes into the stages take 130 and the reads 70.  A barrier ends every half; group 1 starts a half later and group 0 waits
    // for it once at the end, so both pass the same number of them.
    //
    // Halves h of a step are numbered by group 0's: it reads V of pair p and K of pair p + 1 in h = 2 p + 1 and writes pair p + 3 in
    // h = 2 p + 2, group 1 each of them one later.  Pair p + 3 takes the stage of pair p - 1, read last by group 1 in h = 2 p, and is
    // read first in h = 2 p + 5: four stages, and no read meets a write.
    auto half_done = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto stream_eight = [&]() {
      // Every wave brings an eighth of a pair's K and V: piece wv % 4 of its tile (fp8: half a piece, 8 bytes a lane).  The roles
      // are the same, so the loop has no branch on them.
      typedef typename std::conditional<FP8, uint2v, uint4v>::type Part;
      struct Parts {
        Part k, v;
      };
      const bool behind = wv >= 4;
      const int ps = FP8 ? (wv >> 1) & 1 : wv & 3, ph = wv & 1;          // piece, and which half of its 16 bytes (fp8)
      const unsigned part_at = ps * 1024 + lane16 + (FP8 ? ph * 8 : 0);
      auto fetch = [&](Parts& to, int pr) {
        const int64_t at = plane + (PAGED ? (int64_t)blk_next : base_block + tile_of(pr)) * TILE_BYTES;
        to.k = *(const Part*)(a.k + at + part_at);
        to.v = *(const Part*)(a.v + at + part_at);
      };
      uint2v keep = {0xffffffffu, 0xffffffffu};                          // which of this lane's four tokens have a V; once it is
      auto keep_of = [&](int pr) {                                        // the last tile's it stays
        const int t = tile_of(pr), tok0 = t * BLK + 4 * g4;
        if (t * BLK + BLK > held) {
#pragma unroll
          for (int w = 0; w < 2; ++w)
            keep[w] = (tok0 + 2 * w < held ? 0x0000ffffu : 0u) | (tok0 + 2 * w + 1 < held ? 0xffff0000u : 0u);
        }
      };
      auto put = [&](const Parts& from, int pr) {                         // the layouts of write_stage
        char* st = stage_mem + (pr % STAGES) * PREFILL_STAGE_BYTES;
        uint2v lo, hi;                                                   // V of two channel groups
        if constexpr (FP8) {
          *(uint4v*)(st + which * 4096 + ((8 * ps + 4 * ph + g4) * 16 + col16) * 16) =
              uint4v{fp8x2_to_bf16x2<false>(from.k[0]), fp8x2_to_bf16x2<true>(from.k[0]), fp8x2_to_bf16x2<false>(from.k[1]),
                     fp8x2_to_bf16x2<true>(from.k[1])};
          lo = uint2v{fp8x2_to_bf16x2<false>(from.v[0]), fp8x2_to_bf16x2<true>(from.v[0])};
          hi = uint2v{fp8x2_to_bf16x2<false>(from.v[1]), fp8x2_to_bf16x2<true>(from.v[1])};
        } else {
          *(uint4v*)(st + which * 4096 + ps * 1024 + lane16) = from.k;
          lo = uint2v{from.v[0], from.v[1]};
          hi = uint2v{from.v[2], from.v[3]};
        }
        char* dst = st + 8192 + (FP8 ? 4 * ps + 2 * ph : 2 * ps) * 1024 + lane16 + which * 8;
        *(uint2v*)dst = lo & keep;
        *(uint2v*)(dst + 1024) = hi & keep;
      };
      Parts next, first[3];
#pragma unroll
      for (int pr = 0; pr < 3; ++pr) {
        lookup(pr);
        fetch(first[pr], pr);
      }
      lookup(3);
#pragma unroll
      for (int pr = 0; pr < 3; ++pr) {
        keep_of(pr);
        put(first[pr], pr);
      }
      fetch(next, 3);
      lookup(4);
      __syncthreads();
      if (behind) half_done();
      float4v x[CT][2];
      bf16x8 p8[CT], kk[2][4], av[8];
      auto read_k = [&](int pr) {
        const char* st = stage_mem + (pr % STAGES) * PREFILL_STAGE_BYTES + lane16;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int s = 0; s < 4; ++s) kk[b][s] = *(const bf16x8*)(st + b * 4096 + s * 1024);
      };
      auto scores = [&]() { scores_of(x, qreg, [&](int b, int s) { return kk[b][s]; }); };
      read_k(0);
      scores();
      // (A wave without columns computes as well, for nobody, as every wave does the scores behind its last pair.)
      auto step = [&](int pr, auto is_first) {
        half_done();
        keep_of(pr + 3);
        read_v(av, pr);
        read_k(pr + 1);
        mask(x, pr);
        if (decltype(is_first)::value) references(x);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          float sum[2];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[ct][b][i], a.scale_log2, -m[ct]));
              p8[ct][4 * b + i] = (__bf16)e[i];
            }
            sum[b] = (e[0] + e[1]) + (e[2] + e[3]);
          }
          lsum[ct] += sum[0] + sum[1];
        }
        half_done();
        // fp8: its conversions stand in the matrix half, which is then the longer one and goes first (chunks of 512 over paged pools
        // 555 -> 495 us; bf16, whose vector half is the longer one, 1750 -> 1800 on 16 prompts of 4096)
        if (FP8) __builtin_amdgcn_s_setprio(2);
        scores();
        put(next, pr + 3);
        fetch(next, pr + 4);
        lookup(pr + 5);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) O[ct][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[dt], p8[ct], O[ct][dt], 0, 0, 0);
        if (FP8) __builtin_amdgcn_s_setprio(0);
      };
      step(0, std::true_type{});
      for (int pr = 1; pr < n_pairs; ++pr) step(pr, std::false_type{});
      if (!behind) half_done();
    };
    // each lane summed the weights of its own tokens: a column's total is the sum over g4
    auto column_sums = [&](float (&l)[CT]) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        l[ct] = lsum[ct];
        l[ct] += __shfl_xor(l[ct], 16);
        l[ct] += __shfl_xor(l[ct], 32);
      }
    };

    if constexpr (EIGHT) stream_eight();
    else stream();
    if (!CUT && !active) continue;
    float l[CT];
    if (CUT)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) l[ct] = 0.f;
    if (!CUT || active) {
      column_sums(l);
      // Parts: a stand-in may not lie above its state's largest score either.  In the merge it would push the others' references
      // out of the exponent's range: 0, with scores of -60, beside one of -150 whose scores grew to -61.
      const float least = CUT && n_parts > 1 ? 0.5f : 0x1p-60f;
      bool redo = false;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) redo |= lim[ct] > 0 && !(l[ct] > least && l[ct] < 0x1p90f);
      if (__builtin_amdgcn_ballot_w64(redo) != 0) {                      // this wave's columns alone
        slow_pass();
        column_sums(l);
      }
    }
    if (CUT && __builtin_expect(n_parts > 1, 0)) {         // (the merge's code stands behind the whole items')
      // ---- merge of the parts: each leaves its state (m, l, O) in the workspace, the last to arrive reads them all, its own
      // too, from the first part to the last, so that a call repeats bit for bit whatever the order of arrival.  Nobody waits
      // for anybody; order as in the decode kernel's merge: the stores are acknowledged before the barrier, the arrival is
      // counted behind it, the loads follow the full count.
      const int slot0 = item * parts, slot = slot0 + part;
      auto ml_at = [&](int of, int ct) { return (float*)(a.part_ml + (int64_t)of * COLS_ITEM + wv * COLS_WAVE + 16 * ct + col16); };
      auto o_at = [&](int of, int ct, int dt) {
        return a.part_o + ((((int64_t)of * 4 + wv) * CT + ct) * 8 + dt) * 256 + lane * 4;
      };
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        if (!(l[ct] != 0.f)) m[ct] = NEG_INF;                            // a column that saw nothing here has no reference
      if (active) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          if (g4 == 0) store_pair_agent(ml_at(slot, ct), m[ct], l[ct]);
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) {
            store_pair_agent(o_at(slot, ct, dt), O[ct][dt][0], O[ct][dt][1]);
            store_pair_agent(o_at(slot, ct, dt) + 2, O[ct][dt][2], O[ct][dt][3]);
          }
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (threadIdx.x == 0) {
        const bool last = count_in(a.arrive + item) == n_parts - 1;
        // the last arrival leaves the count at zero for the next launch
        if (last) __hip_atomic_store(a.arrive + item, (unsigned long long)ARRIVE_TAG << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        run_slot[0] = last;
      }
      __syncthreads();
      if (!run_slot[0]) continue;
      if (active) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          m[ct] = NEG_INF;
          l[ct] = 0.f;
#pragma unroll
          for (int dt = 0; dt < 8; ++dt) O[ct][dt] = float4v{0.f, 0.f, 0.f, 0.f};
        }
        for (int of = slot0; of < slot0 + n_parts; ++of) {
          float2 ml[CT];
          float4v ov[CT][8];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            ml[ct] = load_pair_agent(ml_at(of, ct));
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) {
              const float2 lo = load_pair_agent(o_at(of, ct, dt)), hi = load_pair_agent(o_at(of, ct, dt) + 2);
              ov[ct][dt] = float4v{lo.x, lo.y, hi.x, hi.y};
            }
          }
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const float m_new = fmaxf(m[ct], ml[ct].x), ref = m_new == NEG_INF ? 0.f : m_new;
            // (factors of at least the smallest number: 0 would make an infinite value NaN that is one in the whole item)
            const float keep = fmaxf(__builtin_amdgcn_exp2f(m[ct] - ref), 0x1p-149f);
            const float add = fmaxf(__builtin_amdgcn_exp2f(ml[ct].x - ref), 0x1p-149f);
            l[ct] = l[ct] * keep + ml[ct].y * add;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) O[ct][dt] = O[ct][dt] * keep + ov[ct][dt] * add;
            m[ct] = m_new;
          }
        }
      }
    }
    if (!active) continue;

    // ---- normalise and store: lane (col16, g4) holds channels 16 dt + 4 g4 .. +3 of its columns
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float inv = a.out_scale / l[ct];
      if (a.out_bf16) {
        // two channel groups at a time: the odd rows of 16 lanes swap their words of group dt for the even rows' words of
        // group dt + 1, which leaves every lane eight consecutive channels of one group -- 16-byte stores, 64 bytes
        // of a column together, half as many instructions
        unsigned short* o = (unsigned short*)a.out + q_at[ct] + (g4 & 1) * 16 + (g4 >> 1) * 8;
#pragma unroll
        for (int dt = 0; dt < 8; dt += 2) {
          uint4v pk;
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            const unsigned lo = (unsigned)float_to_bf16_bits(O[ct][dt][2 * w] * inv) | ((unsigned)float_to_bf16_bits(O[ct][dt][2 * w + 1] * inv) << 16);
            const unsigned hi = (unsigned)float_to_bf16_bits(O[ct][dt + 1][2 * w] * inv) | ((unsigned)float_to_bf16_bits(O[ct][dt + 1][2 * w + 1] * inv) << 16);
            const uint2v sw = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
            pk[w] = sw[0];
            pk[2 + w] = sw[1];
          }
          if (lim[ct] > ABSENT) *(uint4v*)(o + 16 * dt) = pk;
        }
      } else {
        float* o = (float*)a.out + q_at[ct] + 4 * g4;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
          if (lim[ct] > ABSENT) *(float4v*)(o + 16 * dt) = O[ct][dt] * inv;
      }
    }
  }
}

}  // namespace
