// Matrix-core decode attention for bf16 storage (head_dim 128 or 64), fp8 storage (head_dim 128) and, as wide formats, fp32
// storage and bf16 storage with any other head_dim; group size <= 16.
//
// Work decomposition ("tile stream").  A tile is one 16-token pool block of one KV head.
// All tiles of the batch form one sequence ordered by (request, KV head, block); the plan
// kernel cuts it into equal contiguous ranges, one per resident wavefront, so every wave
// streams the same number of bytes no matter how skewed the length distribution is.  A
// wave walks its range with two cursors: a prefetch cursor that issues the loads of the
// tile NBUF-1 steps ahead, and a compute cursor that consumes register buffers in order.
// The pipeline never drains at request boundaries.
//
// A (request, KV head) segment that lies inside one wave's range is finished by that wave
// and written straight to `out`.  A segment cut by a range boundary leaves un-normalised
// partial states (m, l, O).  The waves of a work-group (4 or 8) own consecutive ranges, so
// a cut between two of them is healed inside the work-group: a wave parks the state of its
// first piece in LDS as soon as that piece ends, and the wave that holds the segment's
// beginning (or the work-group's first wave), when it reaches the end of its range, takes
// the pieces to its right, in order, up to the one that ends inside a range, and writes the
// result.  Waves only ever wait for waves to their right, and a wave whose whole range lies
// inside the segment for nobody, so the chain cannot deadlock and needs no barrier (one
// request of 1777 tokens, four waves a piece 10.9 -> 10.0 us; folded from neighbour to
// neighbour every hop was 0.7 us behind the last tile).  Only pieces cut by a work-group boundary go to the HBM
// workspace (at most two per work-group) and are merged by the last work-group to arrive
// at the segment, or by stream_reduce_kernel when the pool asks for a launch of its own.
//
// Per tile:  S^T[16 tok x 16 heads] = K_blk[16 x 128] * Q^T[128 x 16]     4 x mfma 16x16x32 bf16
//            O^T[128 x 16 heads]   += V_blk^T[128 x 16 tok] * P^T[16 x 16] 8 x mfma 16x16x16 bf16
// Lane l holds column (query head) l%16 and rows 4*(l/16)..+3 of S^T, P^T and O^T, so the
// running max, the running sum and the rescale factor of a head live in the lanes that hold
// its column.  The pool's block format is exactly the MFMA operand order, so each wave-wide
// load is one contiguous KiB landing in the registers the MFMA reads.  P is split into
// bf16 hi + lo parts so the P*V product keeps about 16 bits of P.
#pragma once

#include <atomic>
#include <mutex>
#include <type_traits>

#include "kernels_common.h"

namespace {

using odma_plan::StreamEntry;
using odma_plan::WaveDesc;
using odma_plan::ReduceDesc;
using odma_plan::STREAM_MAX_WG;
using odma_plan::STREAM_MAX_LAUNCH_WG;

struct StreamArgs {
  const char* k;             // layer base of the K pool
  const char* v;
  const void* q;
  void* out;
  const void* k_new;         // fused step only: [n][Hkv][head_dim] rows in storage type, appended at position len-1
  const void* v_new;
  const int32_t* bt;
  int32_t bt_stride;
  StreamEntry* entries;      // the plan: read by the kernel, or written by it when it plans itself (plan_at >= 0)
  WaveDesc* waves;
  ReduceDesc* red;           // [n_workgroups + 1], the last one empty
  const int32_t* lengths;
  const int64_t* offsets;    // nullptr when paged
  int32_t plan_at;           // a launch that plans: float offset of the planning area in LDS
  odma_plan::StreamFewest fewest;   // rule of the tile ranges, as the weights (StreamShares)
  int32_t odd_xcd_weight, late_wave_weight;
  int32_t whole_extra;       // tiles beyond an equal share that a wave may get in order that no segment is cut (-1: never)
  unsigned long long* arrive;   // [n_workgroups + 1] arrival counters of the in-kernel merge (count_in)
  int32_t fuse_reduce;       // 1: the last work-group to finish a cut segment merges it; 0: stream_reduce_kernel does
  float2* part_ml;           // [2 * n_workgroups][Hq]
  float* part_o;             // [2 * n_workgroups][Hq][ch]
  int32_t n, Hq, Hkv, G;
  int32_t wpw;               // waves per attention work-group (4 or 8)
  int32_t qs, aq;            // per-wave LDS queue depths: finished pieces, appended rows
  int64_t head_stride;       // bytes between KV-head planes of one layer
  float scale_log2;          // sm_scale * log2(e) (fp8 storage: times k_scale)
  int32_t head_dim;          // stride of q and out rows
  int32_t ch;                // channels a partial state keeps per head
  float out_scale;           // factor of the final normalisation: 1, or v_scale / 256 for fp8 storage (P is carried times 256)
  int32_t out_bf16;
};

constexpr int STREAM_PLAN_THREADS = 1024;
constexpr int STREAM_PLAN_LDS = 8192;

// ---------------------------------------------------------------------------------
// plan: lengths -> entries, per-request positions, one equal tile range per wave
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(STREAM_PLAN_THREADS) void stream_plan_kernel(
    const int32_t* __restrict__ lengths, const int64_t* __restrict__ offsets, int32_t n, int32_t Hkv,
    int32_t tile_tokens, int32_t n_waves, int32_t wpw, odma_plan::StreamFewest fewest, int32_t odd_xcd_weight,
    int32_t late_wave_weight, StreamEntry* entries, WaveDesc* waves, ReduceDesc* red) {
  __shared__ int wave_tiles[STREAM_PLAN_THREADS / 64];
  __shared__ int wave_cnt[STREAM_PLAN_THREADS / 64];
  __shared__ int wave_top[STREAM_PLAN_THREADS / 64];
  __shared__ int first_lds[STREAM_PLAN_LDS];
  __shared__ int wg_pos[STREAM_MAX_WG + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (n + STREAM_PLAN_THREADS - 1) / STREAM_PLAN_THREADS;
  const int r0 = min(tid * per, n), r1 = min(r0 + per, n);
  int loc_tiles = 0, loc_cnt = 0, longest = 0;
  for (int r = r0; r < r1; ++r) {
    const int len = max(lengths[r], 0), tiles = (len + tile_tokens - 1) / tile_tokens;
    loc_tiles += tiles;
    loc_cnt += len > 0;
    longest = max(longest, tiles);
  }
  int inc_tiles = loc_tiles, inc_cnt = loc_cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int yt = __shfl_up(inc_tiles, o), yc = __shfl_up(inc_cnt, o);
    longest = max(longest, __shfl_up(longest, o));           // (a lane below o gets its own)
    if (lane >= o) {
      inc_tiles += yt;
      inc_cnt += yc;
    }
  }
  if (lane == 63) {
    wave_tiles[wv] = inc_tiles;
    wave_cnt[wv] = inc_cnt;
    wave_top[wv] = longest;
  }
  __syncthreads();
  int base_tiles = 0, base_cnt = 0, sum_tiles = 0, n_entries = 0;
  for (int i = 0; i < STREAM_PLAN_THREADS / 64; ++i) {
    if (i < wv) {
      base_tiles += wave_tiles[i];
      base_cnt += wave_cnt[i];
    }
    sum_tiles += wave_tiles[i];
    n_entries += wave_cnt[i];
    longest = max(longest, wave_top[i]);
  }
  int run_tiles = base_tiles + inc_tiles - loc_tiles, run_cnt = base_cnt + inc_cnt - loc_cnt;
  const bool use_lds = n <= STREAM_PLAN_LDS;
  for (int r = r0; r < r1; ++r) {
    const int len = max(lengths[r], 0);
    const int tiles = (len + tile_tokens - 1) / tile_tokens;
    if (len > 0) {
      StreamEntry e;
      e.r = r;
      e.tiles = tiles;
      e.first_pos = run_tiles * Hkv;
      e.len = len;
      e.base_block = offsets ? (int32_t)(offsets[r] / BLK) : 0;
      e.pad0 = e.pad1 = e.pad2 = 0;
      entries[run_cnt] = e;
      if (use_lds) first_lds[run_cnt] = e.first_pos;
      ++run_cnt;
    }
    run_tiles += tiles;
  }
  const int total = sum_tiles * Hkv;
  // one contiguous tile range per wave (rule and weights: odma_plan::StreamShares)
  const odma_plan::StreamShares shares = odma_plan::stream_shares(
      total, n_waves, wpw, fewest.of(total, longest, n_entries * Hkv, n_waves, wpw), odd_xcd_weight, late_wave_weight);
  const int used = shares.used;
  auto pos_of = [&](int W) -> int { return shares.start(W); };
  const int n_wg = n_waves / wpw;
  for (int b = tid; b <= n_wg; b += STREAM_PLAN_THREADS) wg_pos[b] = pos_of(b * wpw);   // work-group starts
  __threadfence_block();
  __syncthreads();
  auto entry_of = [&](int pos) -> int {                   // largest entry with first_pos <= pos
    int lo = 0, hi = n_entries - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      const int f = use_lds ? first_lds[mid] : entries[mid].first_pos;
      if (f <= pos) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  for (int w = tid; w < n_waves; w += STREAM_PLAN_THREADS) {
    const int ps = pos_of(w), pe = pos_of(w + 1);
    WaveDesc wd;
    wd.pos_start = ps;
    wd.pos_end = pe;
    wd.entry0 = 0;
    wd.n_entries = n_entries;
    wd.r = wd.tiles = wd.first_pos = wd.len = wd.base_block = wd.r_next = wd.pad1 = wd.pad2 = 0;
    if (ps < pe) {
      const int lo = entry_of(ps);
      const StreamEntry e = entries[lo];
      wd.entry0 = lo;
      wd.r = e.r;
      wd.tiles = e.tiles;
      wd.first_pos = e.first_pos;
      wd.len = e.len;
      wd.base_block = e.base_block;
      wd.r_next = entries[min(lo + 1, n_entries - 1)].r;
    }
    waves[w] = wd;
  }
  // merge work: the boundary in front of work-group b cuts a segment iff the segment starts
  // before it; the first boundary inside a segment owns the merge of all its partials
  auto wg_of = [&](int pos) -> int {                      // work-group whose range holds pos (pos < total)
    int lo = 0, hi = used / wpw - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (wg_pos[mid] <= pos) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  for (int b = tid; b <= n_wg; b += STREAM_PLAN_THREADS) {
    ReduceDesc rd = {0, 0, 0, 0};
    const int bpos = wg_pos[min(b, n_wg)];
    if (b > 0 && b < n_wg && bpos < total) {
      const StreamEntry e = entries[entry_of(bpos)];
      const int g = (bpos - e.first_pos) / e.tiles;
      const int start = e.first_pos + g * e.tiles;
      if (start < bpos) {
        rd.b0 = wg_of(start);
        rd.n_parts = wg_of(start + e.tiles - 1) - rd.b0 + 1;
        rd.r = e.r;
        rd.g = g;
      }
    }
    red[b] = rd;
  }
}

// ---------------------------------------------------------------------------------
// The same plan, made by the attention launch itself: every work-group scans the lengths of the batch (a few KiB that
// its XCD's L2 holds after the first reader) into an LDS table, finds its waves' ranges there, and leaves the records
// in memory for later calls that reuse the plan.  The planning launch this replaces is one work-group on an empty chip
// (6-8 us with three dependent round trips, plus the edge between two launches); the scan delays the first tile's loads
// by a few microseconds instead.  A planning call, before and after: one request of 1 777 tokens 16.0 -> 12.7 us; 64
// requests, 46 587 tokens 30.4 -> 25.9 us; 256 requests, 159 203 tokens 69.5 -> 64.6 us.  Beyond STREAM_INLINE_REQ requests
// a thread would scan more than four of them and the table would pass 20 KiB of LDS: there the launch of its own stays.
// With one wave per SIMD every instruction in front of the first tile costs 2 ns, so what the plan takes is its number of
// instructions: only the wave's range stands in front of the loads, entries are 16-byte words, and the cuts (both boundaries
// at once, one per half of the wave, work-groups found in closed form) follow under the first tile's latency, where they used
// to stand behind the last tile.  The same three calls 12.4 -> 10.9, 23.8 -> 21.4, 63.4 -> 61.8; 1 000 requests 39.1 -> 34.5.
// ---------------------------------------------------------------------------------
constexpr int STREAM_INLINE_REQ = 1024;
constexpr int STREAM_INLINE_WG = 512;
// Up to this many requests every wave scans the batch by itself, two per lane, and writes the whole table (all waves the same
// words): no barrier stands between the lengths' arrival and the wave's range.  Scanned by the work-group together -> by every
// wave: one request of 1777 tokens 11.35 -> 11.1 us, 64 (46 587 tokens) 22.0 -> 21.6, 128 paged 65.2 -> 65.3; four per lane
// is longer, 256 requests 62.0 -> 62.3, 153 in a fused fp8 step 16.9 -> 17.05.
constexpr int STREAM_WAVE_REQ = 128;
// A batch with no more (request, KV head) segments than work-groups is cut at its segments instead -- one work-group each,
// whose waves heal the cuts between them in LDS -- if that gives no wave more than STREAM_MERGE_TILES tiles beyond an equal
// share: nothing is left to merge through memory then (store, acknowledgement, counter, partial loads, all behind the last
// tile), which is worth about that many tiles.  Bf16, 4 KV heads, equal shares -> whole segments: 16 requests of 100 to 133
// tokens 13.3 -> 9.9 us, 60 of them 14.0 -> 10.4, 60 of 400 to 533 tokens 20.5 -> 16.2; but one of 900 tokens, where the
// equal shares are a sixth of a segment's, 13.5 -> 16.0: it keeps equal shares.
constexpr int STREAM_MERGE_TILES = 5;
typedef int int4v __attribute__((ext_vector_type(4)));
struct InlinePlan {          // LDS table over the non-empty requests, in batch order; 16-byte aligned, a multiple of four ints
  int4v* wave_tot;           // [waves]: tiles, entries, longest request of each wave's part of the batch
  int4v* cuts;               // [2 * waves]: every wave's copy of the segments cut at the work-group's two boundaries (ReduceDesc)
  int4v* entry;              // [n] request, tiles, tokens, base block
  int* first;                // [n] first tile of the entry
  int* wg_pos;               // [n_wg] first tile of every work-group (unequal shares only)
  __device__ InlinePlan(float* lds, int at, int wpw, int n) {
    wave_tot = (int4v*)((int*)lds + at);
    cuts = wave_tot + wpw;
    entry = cuts + 2 * wpw;
    first = (int*)(entry + n);
    wg_pos = first + ((n + 3) & ~3);
  }
};
__host__ __device__ inline int stream_inline_ints(int wpw, int n_wg, int n) {
  return 12 * wpw + 4 * n + ((n + 3) & ~3) + ((n_wg + 3) & ~3);
}
struct InlineTotals {        // what the scan gives every wave (wave-uniform)
  int total, n_entries;      // tiles and non-empty requests of the batch
  bool whole;                // work-group b takes segment b as a whole
  odma_plan::StreamShares shares;   // otherwise: its range of the tile stream
};

// Number of leading elements of the non-decreasing table tab[0 .. n) that are <= x, four per lane and round.  The lanes of a
// group of LANES (64 or 32) ask for one x; every lane gets its group's answer.
template <int LANES>
__device__ __forceinline__ int count_le(const int* tab, int n, int x) {
  const int lane = threadIdx.x & 63;
  int cnt = 0;
  for (int i0 = 0; i0 < n; i0 += 4 * LANES) {
    const int i = i0 + 4 * (lane & (LANES - 1));
    const int4v t = *(const int4v*)(tab + min(i, (n - 1) & ~3));
    int lo = 0, hi = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned long long le = __builtin_amdgcn_ballot_w64(i + k < n && t[k] <= x);
      lo += __builtin_popcount((unsigned)le);
      hi += __builtin_popcount((unsigned)(le >> 32));
    }
    cnt += LANES == 64 ? lo + hi : lane < 32 ? lo : hi;
    if ((LANES == 64 ? lo + hi : max(lo, hi)) < 4 * LANES) break;
  }
  return cnt;
}

// x of the lane CTRL away, 0 where that lane does not exist (all lanes active)
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or_zero(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}
// one step of a wave's inclusive scans of a sum and a maximum (>= 0): row shifts inside 16 lanes, then the last lane of
// a row (0x142) or of two (0x143) to the rows behind it.  Six steps of vector arithmetic; through LDS permutes
// (__shfl_up) each step is a dependent round trip, and the scan stands in front of the first tile of every launch: 0.3 us
// of each (4 fp32 requests of 16 to 128 tokens 9.2 -> 8.9 us, one of 1777 tokens in bf16 13.3 -> 13.05, 60 of up to 500
// 16.25 -> 15.9).
template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(int& sum, int& top) {
  sum += dpp_or_zero<CTRL, ROWS>(sum);
  top = max(top, dpp_or_zero<CTRL, ROWS>(top));
}

// One group of threads scans the batch into the table: the whole work-group (WAVES = WPW), or a wave for itself (WAVES = 1).
struct InlineScan {
  int sum_tiles, n_entries, top;
};
template <int WAVES, int PER, int TT>
__device__ __forceinline__ InlineScan scan_batch(const StreamArgs& a, const InlinePlan& pl) {
  constexpr int T = 64 * WAVES;
  const int tid = threadIdx.x & (T - 1), lane = tid & 63, wv = tid >> 6;
  const int n = a.n, per = (n + T - 1) / T, r0 = tid * per;   // (per: the same for every thread, rounds past it are branched over)
  int ln[PER], base[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    ln[k] = base[k] = 0;
    if (k < per) {
      const int r = min(r0 + k, n - 1);
      ln[k] = a.lengths[r];
      if (a.offsets) base[k] = (int)((unsigned long long)a.offsets[r] / BLK);
    }
  }
  int loc_tiles = 0, longest = 0, run_cnt = 0, wave_cnt = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (k < per) {
      ln[k] = r0 + k < n ? max(ln[k], 0) : 0;
      const int tiles = (int)((unsigned)(ln[k] + TT - 1) / TT);
      loc_tiles += tiles;
      longest = max(longest, tiles);
      // entries of the lanes below, and of the wave
      const unsigned long long held = __builtin_amdgcn_ballot_w64(ln[k] > 0);
      run_cnt += __builtin_amdgcn_mbcnt_hi((unsigned)(held >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)held, 0u));
      wave_cnt += __builtin_popcountll(held);
    }
  int inc_tiles = loc_tiles;
  scan_step<0x111, 0xf>(inc_tiles, longest);
  scan_step<0x112, 0xf>(inc_tiles, longest);
  scan_step<0x114, 0xf>(inc_tiles, longest);
  scan_step<0x118, 0xf>(inc_tiles, longest);
  scan_step<0x142, 0xa>(inc_tiles, longest);
  scan_step<0x143, 0xc>(inc_tiles, longest);
  InlineScan sc = {__builtin_amdgcn_readlane(inc_tiles, 63), wave_cnt, __builtin_amdgcn_readlane(longest, 63)};
  int run_tiles = inc_tiles - loc_tiles;
  if constexpr (WAVES > 1) {
    if (lane == 0) pl.wave_tot[wv] = int4v{sc.sum_tiles, sc.n_entries, sc.top, 0};
    __syncthreads();
    sc = InlineScan{0, 0, 0};
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const int4v t = pl.wave_tot[i];
      sc.top = max(sc.top, rfl(t[2]));
      run_tiles += i < wv ? t[0] : 0;
      run_cnt += i < wv ? t[1] : 0;
      sc.sum_tiles += rfl(t[0]);
      sc.n_entries += rfl(t[1]);
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (k < per && ln[k] > 0) {
      const int tiles = (int)((unsigned)(ln[k] + TT - 1) / TT);
      pl.first[run_cnt] = run_tiles * a.Hkv;
      pl.entry[run_cnt] = int4v{r0 + k, tiles, ln[k], base[k]};
      ++run_cnt;
      run_tiles += tiles;
    }
  return sc;
}

// CHOICE: formats with two numbers for the fewest tiles of a wave
template <int WPW, int TT, bool CHOICE>
__device__ __forceinline__ InlineTotals plan_in_block(const StreamArgs& a, const InlinePlan& pl) {
  constexpr int T = 64 * WPW;
  const int n_wg = gridDim.x;
  const bool alone = a.n <= STREAM_WAVE_REQ;
  const InlineScan sc = alone ? scan_batch<1, STREAM_WAVE_REQ / 64, TT>(a, pl) : scan_batch<WPW, STREAM_INLINE_REQ / T, TT>(a, pl);
  InlineTotals t;
  t.total = sc.sum_tiles * a.Hkv;
  t.n_entries = sc.n_entries;
  const int fewest = CHOICE ? a.fewest.of(t.total, sc.top, sc.n_entries * a.Hkv, n_wg * WPW, WPW) : a.fewest.q_long;
  t.shares = odma_plan::stream_shares(t.total, n_wg * WPW, WPW, fewest, a.odd_xcd_weight, a.late_wave_weight);
  t.whole = a.whole_extra >= 0 && sc.n_entries * a.Hkv <= n_wg &&
            (long long)sc.top * t.shares.used <= WPW * (t.total + (long long)a.whole_extra * t.shares.used);
  if (__builtin_expect(!t.shares.equal(), 0))                // (read behind the barrier in front of the tile stream)
    for (int b = threadIdx.x; b < n_wg; b += T) pl.wg_pos[b] = t.shares.start(b * WPW);
  if (!alone) __syncthreads();
  return t;
}

// this wave's range and its first entry
template <int WPW>
__device__ __forceinline__ WaveDesc inline_wave_desc(const StreamArgs& a, const InlinePlan& pl, const InlineTotals& t) {
  const int lane = threadIdx.x & 63, wv = rfl(threadIdx.x >> 6);
  WaveDesc wd;
  wd.entry0 = 0;
  wd.n_entries = t.n_entries;
  wd.r = wd.tiles = wd.first_pos = wd.len = wd.base_block = wd.r_next = wd.pad1 = wd.pad2 = 0;
  int e = 0;
  if (t.whole) {
    // segment b, its tiles in equal parts; with fewer tiles than waves the empty parts on the left (see StreamShares)
    const int seg = blockIdx.x;
    wd.pos_start = wd.pos_end = t.total;
    if (seg < t.n_entries * a.Hkv) {
      e = seg / a.Hkv;
      const int n = rfl(pl.entry[e][1]), at = rfl(pl.first[e]) + (seg - e * a.Hkv) * n;
      wd.pos_start = at + (n < WPW ? max(n - (WPW - wv), 0) : n * wv / WPW);
      wd.pos_end = at + (n < WPW ? max(n - (WPW - wv - 1), 0) : n * (wv + 1) / WPW);
    }
  } else {
    const int at = t.shares.start(blockIdx.x * WPW + wv + (lane & 1));   // even lanes: the start, odd lanes: the end
    wd.pos_start = __builtin_amdgcn_readlane(at, 0);
    wd.pos_end = __builtin_amdgcn_readlane(at, 1);
    if (wd.pos_start < wd.pos_end) e = rfl(count_le<64>(pl.first, t.n_entries, wd.pos_start)) - 1;
  }
  if (wd.pos_start < wd.pos_end) {
    const int4v en = pl.entry[e];
    wd.entry0 = e;
    wd.r = rfl(en[0]);
    wd.tiles = rfl(en[1]);
    wd.first_pos = rfl(pl.first[e]);
    wd.len = rfl(en[2]);
    wd.base_block = rfl(en[3]);
    wd.r_next = rfl(pl.entry[min(e + 1, t.n_entries - 1)][0]);
  }
  return wd;
}

// The segments cut by the boundaries in front of work-groups b (lanes 0 .. 31) and b + 1 (lanes 32 .. 63), the same rule as in
// stream_plan_kernel: a wave has nothing to do beside it, so the two cost as much time as one.
template <int WPW>
__device__ __forceinline__ int4v inline_cuts(const InlinePlan& pl, const InlineTotals& t, int b, int n_wg) {
  const int mine = b + ((threadIdx.x & 63) >> 5);
  int4v rd = {0, 0, 0, 0};                                   // (a ReduceDesc)
  if (t.whole || t.total == 0) return rd;
  const bool inner = mine > 0 && mine < n_wg;
  const int pos = t.shares.start(mine * WPW);
  const bool in = inner && pos < t.total;
  const int e = max(count_le<32>(pl.first, t.n_entries, in ? pos : 0) - 1, 0);
  const int first = pl.first[e];
  const int4v en = pl.entry[e];
  const int g = (int)((unsigned)((in ? pos : 0) - first) / (unsigned)en[1]), start = first + g * en[1], last = start + en[1] - 1;
  int b0, b1;
  if (__builtin_expect(t.shares.equal(), 1)) {
    b0 = t.shares.wave_of(start) / WPW;
    b1 = t.shares.wave_of(last) / WPW;
  } else {
    b0 = count_le<32>(pl.wg_pos, t.shares.used / WPW, start) - 1;
    b1 = count_le<32>(pl.wg_pos, t.shares.used / WPW, last) - 1;
  }
  if (in && start < pos) rd = int4v{b1 - b0 + 1, en[0], g, b0};
  return rd;
}

// the records that stream_plan_kernel would have left, for calls that reuse the plan
template <int WPW>
__device__ __forceinline__ void store_inline_plan(const StreamArgs& a, const InlinePlan& pl, const WaveDesc& wd, int4v cut) {
  constexpr int T = 64 * WPW;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) a.waves[blockIdx.x * WPW + wv] = wd;
  if (threadIdx.x == 0) {
    *(int4v*)&a.red[blockIdx.x] = cut;
    if (blockIdx.x == gridDim.x - 1) a.red[gridDim.x] = ReduceDesc{0, 0, 0, 0};
  }
  const int n_entries = wd.n_entries;
  for (int i = blockIdx.x * T + threadIdx.x; i < n_entries; i += gridDim.x * T) {
    const int4v en = pl.entry[i];
    StreamEntry e;
    e.r = en[0];
    e.tiles = en[1];
    e.first_pos = pl.first[i];
    e.len = en[2];
    e.base_block = en[3];
    e.pad0 = e.pad1 = e.pad2 = 0;
    a.entries[i] = e;
  }
}

// ---------------------------------------------------------------------------------
// attention over one tile stream per wave
// ---------------------------------------------------------------------------------

// LDS per work-group: one hand-off slot per wave (O[G][128], m[G], l[G], padded; slot 0 unused),
// an int per wave that says how its parked piece ends (four or eight of them: what follows is 16-byte aligned), then per wave a
// queue of finished pieces waiting to be written to global memory (qs entries of slot + 8 ints) and of appended rows (aq records of STREAM_AQ_INTS).  The host sizes
// the queues to the tiles a wave gets: a wave that runs out of queue has to write in mid-stream.
constexpr int STREAM_MERGE_BATCH = 16;   // most partials whose loads are in flight together in the in-kernel merge
// (ch: channels a state keeps per head; np: 1 KiB pieces of a K block)
__host__ __device__ inline int stream_slot_floats(int G, int ch) { return G * ch + ((2 * G + 3) & ~3); }
// appended-row record: 8 ints of header, 128 np bytes of K pieces, 256 np bytes of V pieces
__host__ __device__ constexpr int stream_aq_ints(int np) { return 8 + 96 * np; }
__host__ __device__ inline int stream_wave_queue_floats(int G, int ch, int np, int qs, int aq) {
  return qs * (stream_slot_floats(G, ch) + 8) + aq * stream_aq_ints(np);
}
__host__ inline size_t stream_lds_bytes(int G, int ch, int np, int wpw, int qs, int aq) {
  return ((size_t)wpw * stream_slot_floats(G, ch) + wpw + (size_t)wpw * stream_wave_queue_floats(G, ch, np, qs, aq)) * 4;
}

// Maximum over the four lanes that hold one column (lanes l, l ^ 16, l ^ 32, l ^ 48), in every one of them: two
// register swaps between rows of 16 lanes and between halves of the wave, no trip through the LDS crossbar.
__device__ __forceinline__ float column_max(float x) {
  const unsigned u = __float_as_uint(x);
  const uint2v r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const unsigned w = __float_as_uint(y);
  const uint2v h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
__device__ __forceinline__ float column_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const uint2v r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const unsigned w = __float_as_uint(y);
  const uint2v h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}
constexpr float LAZY_REF_LOG2 = 8.0f;
// How a parked piece ends: cut by the work-group's end, with its segment, or at the end of its wave's range, the next wave's
// first piece being the next of the segment
constexpr int PIECE_CUT = 1, PIECE_ENDS = 2, PIECE_GOES_ON = 3;   // (0: not parked yet)
constexpr float WIDE_LAZY_REF_LOG2 = 4.0f, WIDE_WEIGHT_SCALE = 0x1p-4f;   // wide formats: slack, and the factor 2^-slack of their weights

// Development builds only (-DODMA_DEV_TIMELINE): wall-clock stamps (100 MHz) per wave, read back with
// odma_dev_timeline().  Slots: 0 kernel entry, 1 range descriptor in registers, 2 stream end, 3 queued results written,
// 4 work-group end, 5 tiles streamed, 8 + i: tile i consumed.
#ifdef ODMA_DEV_TIMELINE
constexpr int TL_SLOTS = 64;
__device__ long long odma_dev_timeline_buf[4096 * TL_SLOTS];
#define TL_STAMP(slot) do { if (lane == 0 && (slot) < TL_SLOTS) tl_lds[wv][(slot)] = wall_clock64(); } while (0)
#else
#define TL_STAMP(slot) do { } while (0)
#endif

struct Window {              // 64 consecutive entries, one per lane
  int r, tiles, len, base_block;
  int r_next;                // request of the entry after this lane's
};

struct Cursor {              // wave-uniform position in the tile stream
  int e_base, ei;            // entry = e_base + ei, ei indexes the lane window
  int g, t;                  // KV head and block inside the request
  int r, tiles, len, base_block;
  int r_next;                // request of the following entry
  int blk;                   // paged layout: physical block of the cursor's tile, fetched one step ahead
  int blk2;                  // fp8, paged: the tile's second block
};

// storage formats served by the tile stream
constexpr int STREAM_BF16_D128 = 0, STREAM_FP8_D128 = 1, STREAM_BF16_D64 = 2;
// every other head_dim D of bf16 pools, and every head_dim of fp32 pools: STREAM_BF16_WIDE + D / 32, STREAM_F32_WIDE + D / 32
constexpr int STREAM_BF16_WIDE = 16, STREAM_F32_WIDE = 32;

struct StreamFormat {        // what the kernel and its launch need to know of a format
  int hd;                    // head_dim
  int eb;                    // bytes of a K/V element
  int np;                    // 1 KiB pieces of a K (or V) block
  int blocks;                // pool blocks per tile
  int ch;                    // channels a state keeps per head
};
__host__ __device__ constexpr StreamFormat stream_format(int fmt) {
  if (fmt == STREAM_BF16_D128) return {128, 2, 4, 1, 128};
  if (fmt == STREAM_FP8_D128) return {128, 1, 2, 2, 128};
  if (fmt == STREAM_BF16_D64) return {64, 2, 2, 2, 128};
  const bool f32 = fmt > STREAM_F32_WIDE;
  const int hd = 32 * (fmt - (f32 ? STREAM_F32_WIDE : STREAM_BF16_WIDE)), eb = f32 ? 4 : 2;
  return {hd, eb, hd * eb / 64, hd == 32 ? 2 : 1, hd};
}
// Waves of one SIMD that the registers leave room for: a tile of five pieces or more takes a SIMD for one wave (with room
// for two, bf16 with head_dim 160 spilled 5 registers, fused 38: 256 fused requests of 4 heads 118 -> 95 us).  It bounds the
// compiler from above as well: one wave is what the launch has for a SIMD, and in the hope of a third that would fit, the
// registers for the merge's loads were saved by waiting for them one by one.
__host__ __device__ constexpr int stream_waves(int fmt) {
  return stream_format(fmt).np * stream_format(fmt).blocks >= 5 ? 1 : 2;
}

// PLAN: the launch makes its plan (a variant of its own: with the planning code behind a run-time branch every launch that
// reuses a plan, all layers of a step but the first, was 0.3 to 0.7 us longer, and fused bf16 steps of head_dim 64 up to 7 %)
template <bool PAGED, int NBUF, int WPW, bool FUSED, int FMT, bool PLAN>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WPW, 64 * WPW), amdgpu_waves_per_eu(stream_waves(FMT), stream_waves(FMT)))) void
decode_stream_kernel(StreamArgs a) {
  constexpr bool FP8 = FMT == STREAM_FP8_D128, D64 = FMT == STREAM_BF16_D64;
  constexpr bool WIDE = FMT > STREAM_BF16_WIDE, F32 = FMT > STREAM_F32_WIDE;
  constexpr StreamFormat F = stream_format(FMT);
  constexpr bool TWO = F.blocks == 2;                        // small blocks: a tile is two of them
  constexpr int HD = F.hd;                                   // head_dim: stride of q and out rows
  constexpr int CH = F.ch, NP = F.np, NL = NP * F.blocks;    // NL: 16-byte loads per lane of a tile's K (or V)
  constexpr int NQ = WIDE ? NP : 4;                          // 16-byte pieces of the query operand
  // Two tile buffers and the output of the widest formats leave room for one query operand, not for the next one beside it
  constexpr bool LATE_Q = NQ >= 14;
  // A tile is what a wave requests per step: 4 KiB of K and 4 KiB of V.  bf16 with head_dim 128: one
  // 16-token pool block; fp8, or bf16 with head_dim 64: two of them (32 tokens), which need not be
  // neighbours in the paged layout.  (Inside the kernel every state keeps CH channels per head; with
  // bf16 head_dim 64 the upper half stays zero and is not written out.)  The wide formats -- fp32 pools, and bf16 pools
  // with another head_dim -- take one block per tile whatever its size (two of head_dim 32).
  constexpr int TT = TWO ? 32 : BLK;
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, g4 = lane >> 4;
  const int G = a.G, Hkv = a.Hkv;
  const int slot_floats = stream_slot_floats(G, CH);
  // [wave]: 0, or how the parked piece ends; read and written with work-group-scope atomics (plain LDS instructions:
  // a volatile access would be compiled as a FLAT one, which also waits for the tile loads in flight)
  int* flags = (int*)(lds + WPW * slot_floats);
  auto flag_set = [&](int i, int v) { __hip_atomic_store(flags + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto flag_get = [&](int i) -> int { return __hip_atomic_load(flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  const float NEG_INF = -INFINITY;
#ifdef ODMA_DEV_TIMELINE
  __shared__ long long tl_lds[WPW][TL_SLOTS];
  if (lane < TL_SLOTS) tl_lds[wv][lane] = 0;
  TL_STAMP(0);
#endif
  constexpr int BLOCK_BYTES = BLK * HD * F.eb;             // one pool block of K (or V)

  // the wave's range first: everything else waits for it
  const InlinePlan pl(lds, a.plan_at, WPW, a.n);
  InlineTotals totals;
  WaveDesc wd;
  // in-kernel merge: the segments cut at this work-group's two boundaries, requested now so that the
  // epilogue does not wait for them (a launch that plans derives them under its first tiles' loads)
  ReduceDesc rd_cut[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  if constexpr (PLAN) {
    totals = plan_in_block<WPW, TT, WIDE && (HD > 32)>(a, pl);
    wd = inline_wave_desc<WPW>(a, pl, totals);
  } else {
    wd = a.waves[blockIdx.x * WPW + rfl(wv)];
    if (a.fuse_reduce) {
      rd_cut[0] = a.red[blockIdx.x];
      rd_cut[1] = a.red[blockIdx.x + 1];
    }
  }
  // requested early, needed last: whether the request this thread looks after is empty
  const int r_mine = blockIdx.x * (64 * WPW) + threadIdx.x;
  const int len_mine = r_mine < a.n ? a.lengths[r_mine] : 1;
  const int pos_start = rfl(wd.pos_start), pos_end = rfl(wd.pos_end), n_entries = rfl(wd.n_entries);
  const int n_my = pos_end - pos_start;
  TL_STAMP(1);
  // ready flags must be clear before any neighbour can look at them: a wave clears its own
  // flag first thing, and a wave to its left reads it only at the end of a whole tile range,
  // so one work-group barrier at the top settles the order
  if (lane == 0) flag_set(wv, 0);
  __syncthreads();

  // A launch that plans derives the cuts and leaves its records while the first tiles are on their way (behind the last tile,
  // where everything waits for it, this was 1.5 to 2.5 us).  Every wave keeps the cuts in LDS until its end: eight scalar
  // registers held over the tile loop would be spilled.
  auto settle_plan = [&]() {
    const int4v cut = inline_cuts<WPW>(pl, totals, blockIdx.x, gridDim.x);
    if ((lane & 31) == 0) pl.cuts[2 * wv + (lane >> 5)] = cut;
    store_inline_plan<WPW>(a, pl, wd, cut);
  };
  if (PLAN && n_my <= 0) settle_plan();
  if (n_my > 0) {
    const char* kbase = a.k + lane * 16;
    const char* vbase = a.v + lane * (F32 ? 32 : 16);

    auto load_window = [&](Window& w, int e_base) {
      const int idx = min(e_base + lane, n_entries - 1);
      if constexpr (PLAN) {
        const int4v en = pl.entry[idx];
        w.r = en[0];
        w.tiles = en[1];
        w.len = en[2];
        w.base_block = en[3];
        w.r_next = pl.entry[min(idx + 1, n_entries - 1)][0];
        return;
      }
      const int4 lo = *(const int4*)&a.entries[idx];
      w.r = lo.x;
      w.tiles = lo.y;
      w.len = lo.w;
      w.base_block = a.entries[idx].base_block;
      w.r_next = a.entries[min(idx + 1, n_entries - 1)].r;
    };
    auto fetch = [&](Cursor& c, const Window& w) {
      c.r = __builtin_amdgcn_readlane(w.r, c.ei);
      c.tiles = __builtin_amdgcn_readlane(w.tiles, c.ei);
      c.len = __builtin_amdgcn_readlane(w.len, c.ei);
      c.base_block = __builtin_amdgcn_readlane(w.base_block, c.ei);
      c.r_next = __builtin_amdgcn_readlane(w.r_next, c.ei);   // every window register is read here, so
    };                                                          // none stays pending after a reload
    auto advance = [&](Cursor& c, Window& w) {
      if (++c.t == c.tiles) {
        c.t = 0;
        if (++c.g == Hkv) {
          c.g = 0;
          if (++c.ei == 64) {
            c.e_base += 64;
            c.ei = 0;
            load_window(w, c.e_base);
          }
          fetch(c, w);
        }
      }
    };
    // Paged layout: the block id of a tile is one dependent (scalar) load away from its address.
    // The prefetch cursor asks for it right after it moves, a whole step before the tile's loads
    // are issued, so the table look-up never sits in front of them.
    auto lookup_block = [&](Cursor& c) {
      if (PAGED) {
        const const_i32* row = as_constant(a.bt + (int64_t)c.r * a.bt_stride);
        if (TWO) {
          const int second = 2 * c.t + 1 < (c.len + BLK - 1) / BLK ? 2 * c.t + 1 : 2 * c.t;   // a last tile may have one block
          c.blk = row[2 * c.t];
          c.blk2 = row[second];
        } else {
          c.blk = row[c.t];
        }
      }
    };
    // physical byte offset of the cursor's tile inside a KV-head plane (fp8: of its first block)
    auto tile_offset = [&](const Cursor& c) -> int64_t {
      const int64_t blk = PAGED ? (int64_t)c.blk : (int64_t)c.base_block + c.t * (TT / BLK);
      return (int64_t)c.g * a.head_stride + blk * BLOCK_BYTES;
    };
    // fp8: byte offset of the tile's second block.  A last tile that holds 16 tokens or fewer has
    // none: its loads re-read the first block, so nothing outside the request's slab is touched.
    auto tile_offset2 = [&](const Cursor& c) -> int64_t {
      if (PAGED) return (int64_t)c.g * a.head_stride + (int64_t)c.blk2 * BLOCK_BYTES;
      const bool has = 2 * c.t + 1 < (c.len + BLK - 1) / BLK;
      return (int64_t)c.g * a.head_stride + ((int64_t)c.base_block + 2 * c.t + (has ? 1 : 0)) * BLOCK_BYTES;
    };

    Window wc, wp;                                         // compute and prefetch windows
    Cursor cc, pc;
    cc.e_base = rfl(wd.entry0);
    cc.ei = 0;
    cc.r = rfl(wd.r);
    cc.tiles = rfl(wd.tiles);
    cc.len = rfl(wd.len);
    cc.base_block = rfl(wd.base_block);
    cc.r_next = rfl(wd.r_next);
    {
      const int rel = pos_start - rfl(wd.first_pos);
      cc.g = rel / cc.tiles;
      cc.t = rel - cc.g * cc.tiles;
    }
    cc.blk = 0;
    pc = cc;
    lookup_block(pc);
    load_window(wc, cc.e_base);                            // needed only when a cursor leaves the first entry
    wp = wc;

    // The tiles' registers are words, not vectors of bf16: where a branch changes 16-bit elements (the mask of a ragged tail,
    // the appended row), the compiler takes whole vectors apart over every branch they live across, the ones whose loads
    // are in flight too, and waits for those in every tile (bf16 with head_dim 96, 10 600 tokens: 18 us or 33, by luck).
    // (fp8 has no such branch.  There the appended row's block is a reference, which costs vectors of bf16 no scratch memory as it
    // does words: 153 fused requests of 28 to 224 tokens, 20 / 4 heads, 18.7 us; words and selection by value 18.95.)
    using Piece = typename std::conditional<FP8, bf16x8, uint4v>::type;
    Piece kb[NBUF][NL], vb[NBUF][NL];
    // Loads of the prefetch cursor's tile.  They are issued in every step, so that the waits stay
    // static counts; once the whole range has been requested the surplus loads all read the first
    // block of the layer's pools, which stays in the L2 instead of costing HBM traffic.
    int to_issue = n_my;
    auto issue = [&](Piece (&kk)[NL], Piece (&vv)[NL]) {
      const int64_t off = to_issue > 0 ? tile_offset(pc) : 0;
      // two blocks per tile: the first half of the loads reads the first block, the rest the second one
      const int64_t off2 = !TWO ? 0 : (to_issue > 0 ? tile_offset2(pc) : 0);
      --to_issue;
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        // streaming loads: K/V bytes are used once, and loads that do not allocate in the caches
        // read 9 % faster on this part (measured)
        const int64_t o = j < NP ? off + j * 1024 : off2 + (j - NP) * 1024;
        kk[j] = __builtin_nontemporal_load((const Piece*)(kbase + o));
        if (F32) {
          // a lane's two fp32 pieces of 32 channels (c and 16 + c, four tokens each) are neighbours: the two loads that
          // take them share their cache lines
          const int64_t ov = j < NP ? off + (j >> 1) * 2048 + (j & 1) * 16 : off2 + ((j - NP) >> 1) * 2048 + (j & 1) * 16;
          vv[j] = *(const Piece*)(vbase + ov);
        } else {
          vv[j] = __builtin_nontemporal_load((const Piece*)(vbase + o));
        }
      }
    };
    // Q^T operand of the segment at cursor c: lane (col, g4) holds q[head col][32 j + 8 g4 .. +8] (fp32: [16 j + 4 g4 .. +4])
    auto load_q = [&](bf16x8 (&qq)[NQ], int r, int g) {
      const char* qp = (const char*)a.q + ((int64_t)r * a.Hq + g * G + col) * HD * (F32 ? 4 : 2) + 16 * g4;
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
        qq[j] = (col < G && (WIDE || 32 * j < HD)) ? *(const bf16x8*)(qp + 64 * j) : z;
      }
    };

    // The first segment's queries are requested ahead of the first tiles and adopted inside the main loop, after
    // the second tile's loads have been issued: waiting for them here would hold those loads back by a whole
    // memory round trip.  (They stay vectors of bf16, which no branch takes apart: held as words like the tiles, calls that
    // attend only were up to 2 % longer, three requests of 900 tokens, 8 / 2 heads x 256, two layers, 36.5 -> 37.5 us.)
    bf16x8 qreg[NQ], qnext[LATE_Q ? 1 : NQ];
    if constexpr (LATE_Q) load_q(qreg, cc.r, cc.g);
    else load_q(qnext, cc.r, cc.g);

    // prologue: NBUF-1 tiles in flight
    int p_left = n_my - 1;                                 // prefetch cursor may still advance this often
#pragma unroll
    for (int d = 0; d < NBUF - 1; ++d) {
      issue(kb[d], vb[d]);
      if (p_left > 0) {
        advance(pc, wp);
        lookup_block(pc);
        --p_left;
      }
    }
    if constexpr (PLAN) settle_plan();
    // fp8 storage: the queries go to the matrix cores as fp8 too.  Each query row is scaled by a
    // power of two that brings its largest magnitude into [128, 256) and split into a high and a
    // low E4M3 part (together about 8 significant bits); the inverse scale joins the softmax scale.
    long qhi[4] = {0, 0, 0, 0}, qlo[4] = {0, 0, 0, 0};
    float qfac = a.scale_log2;
    auto adopt_q = [&](const bf16x8 (&src)[NQ]) {
      if constexpr (!FP8) {
#pragma unroll
        for (int j = 0; j < NQ; ++j) qreg[j] = src[j];
        return;
      } else {
      float qf[4][8];
      float amax = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          qf[j][i] = (float)src[j][i];
          amax = fmaxf(amax, fabsf(qf[j][i]));
        }
      amax = column_max(amax);
      const int ex = (int)((__float_as_uint(amax) >> 23) & 0xffu);     // amax in [2^(ex-127), 2^(ex-126))
      const bool tiny = ex < 16;                                        // zero or next to it: leave unscaled
      const float qs = tiny ? 1.0f : __uint_as_float((unsigned)(261 - ex) << 23);     // 2^(134 - ex)
      const float qs_inv = tiny ? 1.0f : __uint_as_float((unsigned)(ex - 7) << 23);
      qfac = a.scale_log2 * qs_inv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int hi[2], lo[2];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          const float x0 = qf[j][4 * w] * qs, x1 = qf[j][4 * w + 1] * qs, x2 = qf[j][4 * w + 2] * qs, x3 = qf[j][4 * w + 3] * qs;
          int h = __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false);
          h = __builtin_amdgcn_cvt_pk_fp8_f32(x2, x3, h, true);
          int l = __builtin_amdgcn_cvt_pk_fp8_f32(x0 - __builtin_amdgcn_cvt_f32_fp8(h, 0), x1 - __builtin_amdgcn_cvt_f32_fp8(h, 1), 0, false);
          l = __builtin_amdgcn_cvt_pk_fp8_f32(x2 - __builtin_amdgcn_cvt_f32_fp8(h, 2), x3 - __builtin_amdgcn_cvt_f32_fp8(h, 3), l, true);
          hi[w] = h;
          lo[w] = l;
        }
        qhi[j] = (long)(unsigned)hi[0] | ((long)hi[1] << 32);
        qlo[j] = (long)(unsigned)lo[0] | ((long)lo[1] << 32);
      }
      }
    };
    float m = LOWEST_REF, lsum = 0.f;
    float4v O[CH / 16];
#pragma unroll
    for (int i = 0; i < CH / 16; ++i) O[i] = float4v{0.f, 0.f, 0.f, 0.f};
    bool from_start = cc.t == 0;

    // fused step: the token appended this step is the last token of its segment.  Its K/V row
    // comes from k_new/v_new, is patched into the registers of the segment's last tile and is
    // written into the pool by the wave that owns that tile (no other wave touches the slot).
    // The row is fetched with one wave-wide load (lanes 0..31 the K row, lanes 32..63 the V row,
    // 8 bytes each; 128-byte rows -- fp8 storage, or bf16 with head_dim 64: 4 bytes each) and handed to
    // the lanes that need its pieces through LDS: one entry in the load queue per segment instead of twelve.
    // (Wide formats: 16 bytes of the K row and of the V row per lane, as many lanes as the row has.)
    uint2v newrow = {0u, 0u};
    uint4v newrow_k = {0u, 0u, 0u, 0u}, newrow_v = {0u, 0u, 0u, 0u};
    bool new_ready = false;
    auto load_new = [&](int r, int g) {
      if (WIDE) {
        constexpr int ROW = HD * F.eb;
        if (lane * 16 < ROW) {
          newrow_k = *(const uint4v*)((const char*)a.k_new + ((int64_t)r * Hkv + g) * ROW + 16 * lane);
          newrow_v = *(const uint4v*)((const char*)a.v_new + ((int64_t)r * Hkv + g) * ROW + 16 * lane);
        }
        return;
      }
      const char* base = (const char*)(lane < 32 ? a.k_new : a.v_new);
      if (TWO) newrow[0] = *(const unsigned*)(base + ((int64_t)r * Hkv + g) * 128 + 4 * (lane & 31));
      else newrow = *(const uint2v*)(base + ((int64_t)r * Hkv + g) * 256 + 8 * (lane & 31));
    };
    // The patch happens in registers now; the write into the pool is queued in LDS and done after
    // the range has been streamed, for the same reason as the outputs.  What is written back is not
    // the bare row (16-byte pieces of K, 2-byte pieces of V: partial sectors, which the memory side
    // turns into read-modify-writes) but the patched registers that hold it: the K pieces of the
    // token pair {slot, slot^1} (32-byte sectors) and the V pieces of the token quad slot/4 (whole
    // 256-byte runs).  The neighbours' bytes go back unchanged; slots past the end may get stale
    // bytes again, as before.  fp8 storage: the same with the 2 KiB block that holds the token (two
    // 1 KiB pieces of K and of V instead of four).
    int* abase = (int*)(lds + WPW * slot_floats + WPW + wv * stream_wave_queue_floats(G, CH, NP, a.qs, a.aq) +
                        a.qs * (slot_floats + 8));
    constexpr int REC_V = 8 + 32 * NP;                       // where a record's V pieces begin
    int an = 0;
    // (Results leave with streaming stores: ordinary ones stay in the L2 as dirty lines that the end
    // of the kernel has to write back, which showed as 0.8 us per launch.)
    auto flush_appends = [&]() {
      for (int i = 0; i < an; ++i) {
        const int* rec = abase + i * stream_aq_ints(NP);
        const int64_t off = ((int64_t)rfl(rec[1]) << 32) | (unsigned)rfl(rec[0]);
        const int slot = rfl(rec[2]);
        const uint4v* kq = (const uint4v*)(rec + 8);
        const uint4v* vq = (const uint4v*)(rec + REC_V);
        if ((col >> 1) == (slot >> 1)) {
          char* kd = (char*)a.k + off + lane * 16;
#pragma unroll
          for (int j = 0; j < NP; ++j) __builtin_nontemporal_store(kq[(j * 4 + g4) * 2 + (col & 1)], (uint4v*)(kd + j * 1024));
        }
        if (g4 == (slot >> 2)) {
          char* vd = (char*)a.v + off + lane * (F32 ? 32 : 16);
#pragma unroll
          for (int j = 0; j < NP; ++j)
            __builtin_nontemporal_store(vq[j * 16 + col], (uint4v*)(vd + (F32 ? (j >> 1) * 2048 + (j & 1) * 16 : j * 1024)));
        }
      }
      an = 0;
    };
    // Token rr of the four that V words lo (tokens 0, 1) and hi (2, 3) hold of a channel becomes x (bf16).
    auto insert_v = [](unsigned& lo, unsigned& hi, int rr, unsigned short x) {
      const unsigned keep = (rr & 1) ? 0x0000ffffu : 0xffff0000u, put = (unsigned)x << (16 * (rr & 1));
      lo = rr < 2 ? (lo & keep) | put : lo;
      hi = rr < 2 ? hi : (hi & keep) | put;
    };
    auto insert_v_group = [&](uint4v& w, int half, int rr, unsigned short x) {   // half: which of the piece's two channel groups
      unsigned lo = w[2 * half], hi = w[2 * half + 1];
      insert_v(lo, hi, rr, x);
      w[2 * half] = lo;
      w[2 * half + 1] = hi;
    };
    // Blocks of 2 KiB (bf16 with head_dim 64; fp8 below): the row's 128 K bytes and 128 V bytes are
    // staged in the record's V area (overwritten by the patched pieces further down).  The pieces of the block that holds the
    // token, the tile's first or second, are selected by value: through a reference chosen at run time the tile's registers
    // live in scratch memory, in every tile (fused steps of 256 requests, 28 / 4 heads x 64 in bf16, config 3's lengths: 49 us
    // a layer, now 33).
    auto patch_two = [&](int* rec, int slot, auto second, uint4v (&kk)[NL], uint4v (&vv)[NL]) {
      uint4v k0 = second ? kk[NL / 2] : kk[0], k1 = second ? kk[NL / 2 + 1] : kk[1];
      uint4v v0 = second ? vv[NL / 2] : vv[0], v1 = second ? vv[NL / 2 + 1] : vv[1];
      const int rr = slot & 3;
      unsigned* stage = (unsigned*)(rec + REC_V);
      stage[lane] = newrow[0];
      const uint4v* krow = (const uint4v*)stage;          // K[0..64) as 8 pieces of 8 channels
      const unsigned short* vrow = (const unsigned short*)(stage + 32);
      if (col == slot) {                                   // K: 8 channels of the new token per k-step
        k0 = krow[g4];
        k1 = krow[4 + g4];
      }
      if (g4 == (slot >> 2)) {                             // V: this lane holds tokens 4*g4..+3 of 4 channels
#pragma unroll
        for (int k = 0; k < 4; ++k) insert_v_group(k < 2 ? v0 : v1, k & 1, rr, vrow[16 * k + col]);
      }
      if ((col >> 1) == (slot >> 1)) {                       // K pieces of the token pair, patched
        uint4v* kq = (uint4v*)(rec + 8);
        kq[g4 * 2 + (col & 1)] = k0;
        kq[(4 + g4) * 2 + (col & 1)] = k1;
      }
      if (g4 == (slot >> 2)) {                               // V pieces of the token quad, patched
        uint4v* vq = (uint4v*)(rec + REC_V);
        vq[col] = v0;
        vq[16 + col] = v1;
      }
      kk[0] = second ? kk[0] : k0;
      kk[1] = second ? kk[1] : k1;
      vv[0] = second ? vv[0] : v0;
      vv[1] = second ? vv[1] : v1;
      kk[NL / 2] = second ? k0 : kk[NL / 2];
      kk[NL / 2 + 1] = second ? k1 : kk[NL / 2 + 1];
      vv[NL / 2] = second ? v0 : vv[NL / 2];
      vv[NL / 2 + 1] = second ? v1 : vv[NL / 2 + 1];
    };
    // fp8: the same, through a reference; k0, k1 / v0, v1 are the pieces of the block that holds the token.
    auto patch_fp8 = [&](int* rec, int slot, bf16x8& k0, bf16x8& k1, bf16x8& v0, bf16x8& v1) {
      const int rr = slot & 3;
      unsigned* stage = (unsigned*)(rec + REC_V);
      stage[lane] = newrow[0];
      const uint2v* krow = (const uint2v*)stage;            // K[0..128) as 16 pieces of 8 bytes
      const unsigned char* vrow = (const unsigned char*)(stage + 32);
      if (col == slot) {                                     // K: per 64-channel half, 8 channels of each of its two k-steps
        const uint2v a0 = krow[g4], b0 = krow[4 + g4], a1 = krow[8 + g4], b1 = krow[12 + g4];
        k0 = __builtin_bit_cast(bf16x8, uint4v{a0[0], a0[1], b0[0], b0[1]});
        k1 = __builtin_bit_cast(bf16x8, uint4v{a1[0], a1[1], b1[0], b1[1]});
      }
      if (g4 == (slot >> 2)) {                               // V: byte rr of every word is the new token's channel
        uint4v w0 = __builtin_bit_cast(uint4v, v0), w1 = __builtin_bit_cast(uint4v, v1);
        const unsigned keep = ~(0xffu << (8 * rr));
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          w0[w] = (w0[w] & keep) | ((unsigned)vrow[16 * w + col] << (8 * rr));
          w1[w] = (w1[w] & keep) | ((unsigned)vrow[64 + 16 * w + col] << (8 * rr));
        }
        v0 = __builtin_bit_cast(bf16x8, w0);
        v1 = __builtin_bit_cast(bf16x8, w1);
      }
      if ((col >> 1) == (slot >> 1)) {                       // K pieces of the token pair, patched
        bf16x8* kq = (bf16x8*)(rec + 8);
        kq[g4 * 2 + (col & 1)] = k0;
        kq[(4 + g4) * 2 + (col & 1)] = k1;
      }
      if (g4 == (slot >> 2)) {                               // V pieces of the token quad, patched
        bf16x8* vq = (bf16x8*)(rec + REC_V);
        vq[col] = v0;
        vq[16 + col] = v1;
      }
    };
    // Wide formats: the same for a block of NP pieces.
    auto patch_wide = [&](int* rec, int slot, uint4v* kk, uint4v* vv) {
      constexpr int ROW16 = HD * F.eb / 16;
      const int rr = slot & 3;
      uint4v* stage = (uint4v*)(rec + REC_V);
      if (lane < ROW16) {
        stage[lane] = newrow_k;
        stage[ROW16 + lane] = newrow_v;
      }
      if (col == slot) {                                     // K: piece j of this lane is 16-byte chunk 4 j + g4 of the row
#pragma unroll
        for (int j = 0; j < NP; ++j) kk[j] = stage[4 * j + g4];
      }
      if (g4 == (slot >> 2)) {                               // V: this lane holds tokens 4*g4..+3 of HD / 16 channels
#pragma unroll
        for (int dt = 0; dt < HD / 16; ++dt) {
          if (F32) {
            const unsigned vnew = ((const unsigned*)(stage + ROW16))[16 * dt + col];
#pragma unroll
            for (int i = 0; i < 4; ++i) vv[dt % NP][i] = i == rr ? vnew : vv[dt % NP][i];
          } else {
            insert_v_group(vv[(dt >> 1) % NP], dt & 1, rr, ((const unsigned short*)(stage + ROW16))[16 * dt + col]);
          }
        }
      }
      if ((col >> 1) == (slot >> 1)) {                       // K pieces of the token pair, patched
#pragma unroll
        for (int j = 0; j < NP; ++j) ((uint4v*)(rec + 8))[(j * 4 + g4) * 2 + (col & 1)] = kk[j];
      }
      if (g4 == (slot >> 2)) {                               // V pieces of the token quad, patched
#pragma unroll
        for (int j = 0; j < NP; ++j) ((uint4v*)(rec + REC_V))[j * 16 + col] = vv[j];
      }
    };
    auto patch_and_store = [&](Piece (&kk)[NL], Piece (&vv)[NL]) {
      const int slot = (cc.len - 1) & (BLK - 1), rr = slot & 3;
      lookup_block(cc);                                      // the compute cursor looks its block up only here
      const bool second = TWO && (((cc.len - 1) / BLK) & 1);  // 32-token tiles: the token sits in the tile's second block
      const int64_t off = second ? tile_offset2(cc) : tile_offset(cc);
      if (an == a.aq) flush_appends();
      int* rec = abase + an * stream_aq_ints(NP);
      if (lane == 0) {
        rec[0] = (int)(off & 0xffffffffll);
        rec[1] = (int)(off >> 32);
        rec[2] = slot;
      }
      ++an;
      if constexpr (WIDE) {
        if constexpr (TWO) {
          uint4v k[NP], v[NP];
#pragma unroll
          for (int j = 0; j < NP; ++j) {
            k[j] = second ? kk[NP + j] : kk[j];
            v[j] = second ? vv[NP + j] : vv[j];
          }
          patch_wide(rec, slot, k, v);
#pragma unroll
          for (int j = 0; j < NP; ++j) {
            kk[j] = second ? kk[j] : k[j];
            vv[j] = second ? vv[j] : v[j];
            kk[NP + j] = second ? k[j] : kk[NP + j];
            vv[NP + j] = second ? v[j] : vv[NP + j];
          }
        } else {
          patch_wide(rec, slot, kk, vv);
        }
      } else if constexpr (FP8) {
        if (second) patch_fp8(rec, slot, kk[2], kk[3], vv[2], vv[3]);
        else patch_fp8(rec, slot, kk[0], kk[1], vv[0], vv[1]);
      } else if constexpr (TWO) {
        patch_two(rec, slot, second, kk, vv);
      } else {
      // stage the row in the record's V area (overwritten by the patched pieces further down)
      uint2v* stage = (uint2v*)(rec + REC_V);
      stage[lane] = newrow;
      const uint4v* krow = (const uint4v*)stage;            // K[0..128) as 16 pieces of 8
      const unsigned short* vrow = (const unsigned short*)stage + 128;
      if (col == slot) {                                     // K: this lane holds 8 channels of the new token per k-step
#pragma unroll
        for (int j = 0; j < 4; ++j) kk[j] = krow[4 * j + g4];
      }
      if (g4 == (slot >> 2)) {                               // V: this lane holds tokens 4*g4..+3 of 8 channels
#pragma unroll
        for (int k = 0; k < 8; ++k) insert_v_group(vv[k >> 1], k & 1, rr, vrow[16 * k + col]);
      }
      if ((col >> 1) == (slot >> 1)) {                       // K pieces of the token pair, patched
        uint4v* kq = (uint4v*)(rec + 8);
#pragma unroll
        for (int j = 0; j < 4; ++j) kq[(j * 4 + g4) * 2 + (col & 1)] = kk[j];
      }
      if (g4 == (slot >> 2)) {                               // V pieces of the token quad, patched
        uint4v* vq = (uint4v*)(rec + REC_V);
#pragma unroll
        for (int j = 0; j < 4; ++j) vq[j * 16 + col] = vv[j];
      }
      }
    };

    // fp8 tile: 32 tokens in two pool blocks b = 0, 1.  Per block S^T = K Q^T with the high and the
    // low part of Q (2 x 4 mfma 16x16x32 fp8).  P is carried times 256 and split into a high and a
    // low E4M3 part as well; O^T += V^T P^T contracts over all 32 tokens in one mfma per d-tile and
    // part, the operand of lane (., g4) holding tokens 4 g4 .. 4 g4 + 3 of block 0, then of block 1,
    // which is the order the pool's V block format and the S^T accumulator layout both give.
    auto compute_fp8 = [&](Piece (&kk)[NL], Piece (&vv)[NL]) {
      typedef long long2v __attribute__((ext_vector_type(2)));
      const int n_valid = cc.len - cc.t * TT;               // tokens of this tile in range (>= 32: all)
      const bool ragged = n_valid < TT;
      float x[2][4];
      float tmax = NEG_INF;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float4v s = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const long kop = __builtin_bit_cast(long2v, kk[2 * b + (j >> 1)])[j & 1];
          s = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(kop, qhi[j], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(kop, qlo[j], s, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float val = s[i] * qfac;
          if (ragged && 16 * b + 4 * g4 + i >= n_valid) val = NEG_INF;
          x[b][i] = val;
          tmax = fmaxf(tmax, val);
        }
      }
      tmax = column_max(tmax);
      // weights are carried times 256 in E4M3 (largest value 448), so the reference must be the exact running maximum;
      // the rescale is skipped when no column's maximum moved
      if (__builtin_amdgcn_ballot_w64(tmax > m) != 0) {
        const float m_new = fmaxf(m, tmax);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lsum *= alpha;
#pragma unroll
        for (int i = 0; i < 8; ++i) O[i] *= alpha;
      }
      float psum = 0.f;
      int ph[2], pl[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(x[b][i] - m);
          psum += pv[i];
          pv[i] *= 256.0f;
        }
        int h = __builtin_amdgcn_cvt_pk_fp8_f32(pv[0], pv[1], 0, false);
        h = __builtin_amdgcn_cvt_pk_fp8_f32(pv[2], pv[3], h, true);
        int l = __builtin_amdgcn_cvt_pk_fp8_f32(pv[0] - __builtin_amdgcn_cvt_f32_fp8(h, 0), pv[1] - __builtin_amdgcn_cvt_f32_fp8(h, 1), 0, false);
        l = __builtin_amdgcn_cvt_pk_fp8_f32(pv[2] - __builtin_amdgcn_cvt_f32_fp8(h, 2), pv[3] - __builtin_amdgcn_cvt_f32_fp8(h, 3), l, true);
        ph[b] = h;
        pl[b] = l;
      }
      lsum += psum;
      const long phi = (long)(unsigned)ph[0] | ((long)ph[1] << 32);
      const long plo = (long)(unsigned)pl[0] | ((long)pl[1] << 32);
      // bytes of tokens past the end may hold anything (0x7f is a NaN): keep 0 * x == 0
      unsigned keep0 = 0xffffffffu, keep1 = 0xffffffffu;
      if (ragged) {
        const int v0 = min(max(n_valid - 4 * g4, 0), 4), v1 = min(max(n_valid - 16 - 4 * g4, 0), 4);
        keep0 = v0 == 4 ? 0xffffffffu : (1u << (8 * v0)) - 1u;
        keep1 = v1 == 4 ? 0xffffffffu : (1u << (8 * v1)) - 1u;
      }
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {
        const unsigned w0 = __builtin_bit_cast(uint4v, vv[dt >> 2])[dt & 3] & keep0;
        const unsigned w1 = __builtin_bit_cast(uint4v, vv[2 + (dt >> 2)])[dt & 3] & keep1;
        const long av = (long)w0 | ((long)w1 << 32);
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(av, phi, O[dt], 0, 0, 0);
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(av, plo, O[dt], 0, 0, 0);
      }
    };

    // bf16 V pieces (tokens 4 g4 .. + 3 of two channel groups each): slots past the end may hold stale bytes (even NaN
    // patterns), zero them so 0 * x stays 0.  left: tokens from the piece's block on that are in range.
    auto zero_past = [&](uint4v* w, int pieces, int left) {
      const int t = 4 * g4;
      const unsigned k01 = (t < left ? 0x0000ffffu : 0u) | (t + 1 < left ? 0xffff0000u : 0u);
      const unsigned k23 = (t + 2 < left ? 0x0000ffffu : 0u) | (t + 3 < left ? 0xffff0000u : 0u);
#pragma unroll
      for (int j = 0; j < pieces; ++j) w[j] &= uint4v{k01, k23, k01, k23};
    };
    auto as_bf16 = [](uint4v w) { return __builtin_bit_cast(bf16x8, w); };

    // bf16, head_dim 64: the tile is two pool blocks of 2 KiB (32 tokens), kk / vv [0], [1] the two
    // 1 KiB pieces of the first block, [2], [3] those of the second.  Scores per block as for head_dim
    // 128 with two channel steps; P V contracts over the 32 tokens in one 16x16x32 instruction per
    // channel group, the operand of lane (., g4) holding tokens 4 g4 .. +3 of the first block, then of
    // the second.  P is carried as a high plus a low bf16 part.
    auto compute_d64 = [&](uint4v (&kk)[NL], uint4v (&vv)[NL]) {
      const int n_valid = cc.len - cc.t * TT;               // tokens of this tile in range (>= 32: all)
      const bool ragged = n_valid < TT;
      float x[2][4];
      float tmax = NEG_INF;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float4v s = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 2; ++j) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16(kk[2 * b + j]), qreg[j], s, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float val = s[i] * a.scale_log2;
          if (ragged && 16 * b + 4 * g4 + i >= n_valid) val = NEG_INF;
          x[b][i] = val;
          tmax = fmaxf(tmax, val);
        }
      }
      tmax = column_max(tmax);
      if (__builtin_amdgcn_ballot_w64(tmax > m + LAZY_REF_LOG2) != 0) {   // lazy reference, as for head_dim 128
        const float m_new = fmaxf(m, tmax);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lsum *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) O[i] *= alpha;
      }
      float psum = 0.f;
      bf16x8 phi, plo;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pv = __builtin_amdgcn_exp2f(x[b][i] - m);
          psum += pv;
          const __bf16 hi = (__bf16)pv;
          phi[4 * b + i] = hi;
          plo[4 * b + i] = (__bf16)(pv - (float)hi);
        }
      lsum += psum;
      if (ragged) {
        zero_past(vv, 2, n_valid);
        zero_past(vv + 2, 2, n_valid - BLK);
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const uint4v wa = vv[dt >> 1], wb = vv[2 + (dt >> 1)];
        const bf16x8 av = as_bf16((dt & 1) ? uint4v{wa[2], wa[3], wb[2], wb[3]} : uint4v{wa[0], wa[1], wb[0], wb[1]});
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, phi, O[dt], 0, 0, 0);
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, plo, O[dt], 0, 0, 0);
      }
    };

    // Wide formats.  fp32: both products run on the fp32 matrix instruction (16x16x4), whose operands are single elements
    // of the 16-byte pieces: element e of K piece j and of the query's is channel 16 j + 4 g4 + e, element e of V piece dt
    // is token 4 g4 + e of channel 16 dt + col, and score row 4 g4 + e is where the accumulator holds it -- no data moves
    // between lanes.  A 16-token tile of head_dim 128 takes 64 of them, 2048 cycles of the 6000 that its 16 KiB take to
    // arrive.  bf16: as head_dim 128, but P is carried as three bf16 parts (24 bits), so that no weight has fewer bits than
    // the vector-ALU kernel gave it.  That kernel was bound by its lane arithmetic (2048 operations per token and KV head):
    // batch 64, 46 587 tokens of 28 / 4 heads x 128 in fp32, 116.4 -> 41.6 us with plan and merge in the launch (193 MB,
    // 4.6 TB/s); fused step of 4 requests of 16 to 128 tokens, 23.1 -> 8.8 us.  Error against 64 bits 4.1e-7 -> 3.2e-7.
    // Weights are carried times 2^-4, the state's l and O with them, and the lazy reference may lag by 2^4: no weight exceeds
    // 1, as none did in the vector kernel, and values past 1e36 stay in the range of fp32 (at the other end, values under
    // 1e-36 lose up to four bits of it).  The factor is exact, so results are those of the unscaled weights.  (The running
    // maximum as reference, rescaled whenever it moves, cost up to 5 %; the factor inside the exponent cost accuracy, 3.2e-7 -> 3.5e-7.)
    auto compute_wide = [&](uint4v (&kk)[NL], uint4v (&vv)[NL]) {
      const int n_valid = cc.len - cc.t * TT;               // tokens of this tile in range (>= TT: all)
      const bool ragged = n_valid < TT;
      float x[F.blocks][4];
      float tmax = NEG_INF;
#pragma unroll
      for (int b = 0; b < F.blocks; ++b) {
        float4v s[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};   // two chains: half the latency
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
          if (F32) {
            const float4v kf = __builtin_bit_cast(float4v, kk[b * NP + j]), qf = __builtin_bit_cast(float4v, qreg[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[e], s[e & 1], 0, 0, 0);
          } else {
            s[j & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16(kk[b * NP + j]), qreg[j], s[j & 1], 0, 0, 0);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float val = (s[0][i] + s[1][i]) * a.scale_log2;
          if (ragged && 16 * b + 4 * g4 + i >= n_valid) val = NEG_INF;
          x[b][i] = val;
          tmax = fmaxf(tmax, val);
        }
      }
      tmax = column_max(tmax);
      if (__builtin_amdgcn_ballot_w64(tmax > m + WIDE_LAZY_REF_LOG2) != 0) {   // lazy reference, as for head_dim 128
        const float m_new = fmaxf(m, tmax);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lsum *= alpha;
#pragma unroll
        for (int i = 0; i < CH / 16; ++i) O[i] *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int b = 0; b < F.blocks; ++b) {
        float pv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(x[b][i] - m) * WIDE_WEIGHT_SCALE;
          psum += pv[i];
        }
        if (F32) {
          if (ragged) {                                       // stale slots may hold anything: keep 0 * x == 0
#pragma unroll
            for (int j = 0; j < NP; ++j)
#pragma unroll
              for (int i = 0; i < 4; ++i) vv[b * NP + j][i] = 16 * b + 4 * g4 + i >= n_valid ? 0u : vv[b * NP + j][i];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < CH / 16; ++dt)
              O[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float4v, vv[b * NP + dt % NP])[e], pv[e], O[dt], 0, 0, 0);
        } else {
          // Three parts of eight bits each, cut off and not rounded, so that none is negative, and none of a weight that is
          // not 0 is 0 (2^-40 of the weight stands in): an infinite V times the parts is that infinity, as times the weight,
          // where parts of both signs would give inf - inf and a part of 0 would give 0 * inf.
          bf16x4 part[3];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float least = pv[i] * 0x1p-40f;
            float rest = pv[i];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const float cut = __uint_as_float(__float_as_uint(k == 0 ? rest : fmaxf(rest, least)) & 0xffff0000u);
              part[k][i] = __builtin_bit_cast(__bf16, (unsigned short)(__float_as_uint(cut) >> 16));
              rest -= cut;
            }
          }
          if (ragged) zero_past(vv + b * NP, NP, n_valid - BLK * b);
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int dt = 0; dt < CH / 16; ++dt) {
              const uint4v w = vv[b * NP + (dt >> 1) % NP];
              const uint2v half = (dt & 1) ? uint2v{w[2], w[3]} : uint2v{w[0], w[1]};
              O[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, half),
                                                                __builtin_bit_cast(short4v, part[k]), O[dt], 0, 0, 0);
            }
        }
      }
      lsum += psum;
    };

    auto compute = [&](Piece (&kk)[NL], Piece (&vv)[NL]) {
      if constexpr (WIDE) {
        compute_wide(kk, vv);
      } else if constexpr (FP8) {
        compute_fp8(kk, vv);
      } else if constexpr (D64) {
        compute_d64(kk, vv);
      } else {
      float4v s = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16(kk[j]), qreg[j], s, 0, 0, 0);
      const int n_valid = cc.len - cc.t * BLK;              // tokens of this block in range (>= 16: all)
      const bool ragged = n_valid < BLK;
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = s[i] * a.scale_log2;
      if (ragged) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * g4 + i >= n_valid) x[i] = NEG_INF;
      }
      const float tmax = column_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      // The reference of the running softmax moves only when a column's scores pass it by more than 2^LAZY_REF_LOG2:
      // the state (m, l, O) is valid for any reference, weights up to 2^LAZY_REF_LOG2 are exact enough in fp32 and in the
      // high + low bf16 pair, and the usual tile then needs no rescale of O and no second exponential.
      if (__builtin_amdgcn_ballot_w64(tmax > m + LAZY_REF_LOG2) != 0) {
        const float m_new = fmaxf(m, tmax);
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        lsum *= alpha;
#pragma unroll
        for (int i = 0; i < 8; ++i) O[i] *= alpha;
      }
      float psum = 0.f;
      bf16x4 phi, plo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pv = __builtin_amdgcn_exp2f(x[i] - m);
        psum += pv;
        const __bf16 hi = (__bf16)pv;
        phi[i] = hi;
        plo[i] = (__bf16)(pv - (float)hi);
      }
      lsum += psum;
      if (ragged) zero_past(vv, NL, n_valid);
      const short4v bh = __builtin_bit_cast(short4v, phi);
      const short4v bl = __builtin_bit_cast(short4v, plo);
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {
        const uint4v w = vv[(dt >> 1) % NL];
        const uint2v half = (dt & 1) ? uint2v{w[2], w[3]} : uint2v{w[0], w[1]};
        const short4v av = __builtin_bit_cast(short4v, half);
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bh, O[dt], 0, 0, 0);
        O[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bl, O[dt], 0, 0, 0);
      }
      }
    };

    // Finished pieces are not stored to global memory right away: stores share the in-order
    // vmcnt queue with the tile loads, and a store in the middle of the stream makes the next
    // tile wait for the store's acknowledgement.  They are queued in LDS (a separate counter)
    // and written when the wave has streamed its whole range (or when the queue is full).
    float* qbase = lds + WPW * slot_floats + WPW + wv * stream_wave_queue_floats(G, CH, NP, a.qs, a.aq);
    const int qstride = slot_floats + 8;
    int qn = 0;
    // A state in LDS: O[G][CH], m[G], l[G].  The 16-byte pieces of a head's row are permuted in groups of eight by the head, so that
    // the lanes that hold the same channels of eight heads meet different banks (in rows as they are they all meet one, and a
    // hand-off between waves, a store and a load of a whole state behind the last tile, took 0.4 us of it).
    const int row = col < G ? col * CH : 0;
    const int sw[2] = {row + 4 * (g4 ^ (col & 7)), row + 4 * ((4 + g4) ^ (col & 7))};
    auto o_at = [&](float* state, int dt) -> float4v& { return *(float4v*)(state + sw[dt & 1] + 32 * (dt >> 1)); };
    // a finished piece's outputs, or its un-normalised state, to global memory
    auto put = [&](int kind, int r, int g, int gslot, const float4v (&o4)[CH / 16], float m_e, float l_e) {
      if (col >= G) return;
      if (kind == 0) {                                       // final: normalise and write to `out`
        const float inv = a.out_scale / l_e;
        const int64_t o_base = ((int64_t)r * a.Hq + g * G + col) * HD + 4 * g4;
        if (a.out_bf16) {
          unsigned short* o = (unsigned short*)a.out + o_base;
#pragma unroll
          for (int dt = 0; dt < HD / 16; ++dt) {
            uint2v pk;
            pk[0] = (unsigned)float_to_bf16_bits(o4[dt][0] * inv) | ((unsigned)float_to_bf16_bits(o4[dt][1] * inv) << 16);
            pk[1] = (unsigned)float_to_bf16_bits(o4[dt][2] * inv) | ((unsigned)float_to_bf16_bits(o4[dt][3] * inv) << 16);
            __builtin_nontemporal_store(pk, (uint2v*)(o + 16 * dt));
          }
        } else {
          float* o = (float*)a.out + o_base;
#pragma unroll
          for (int dt = 0; dt < HD / 16; ++dt) __builtin_nontemporal_store(o4[dt] * inv, (float4v*)(o + 16 * dt));
        }
      } else {                                               // un-normalised state to the HBM workspace
        const int64_t pi = (int64_t)gslot * a.Hq + g * G + col;
        float* o = a.part_o + pi * CH + 4 * g4;
#pragma unroll
        for (int dt = 0; dt < CH / 16; ++dt) {
          store_pair_agent(o + 16 * dt, o4[dt][0], o4[dt][1]);
          store_pair_agent(o + 16 * dt + 2, o4[dt][2], o4[dt][3]);
        }
        if (g4 == 0) store_pair_agent((float*)&a.part_ml[pi], m_e, l_e);
      }
    };
    auto flush_outputs = [&]() {
      for (int i = 0; i < qn; ++i) {
        float* e = qbase + i * qstride;
        const int* meta = (const int*)(e + slot_floats);
        const int kind = rfl(meta[0]), r = rfl(meta[1]), g = rfl(meta[2]), gslot = rfl(meta[3]);
        float4v o4[CH / 16];
#pragma unroll
        for (int dt = 0; dt < CH / 16; ++dt) o4[dt] = o_at(e, dt);
        const int c = col < G ? col : 0;
        put(kind, r, g, gslot, o4, e[G * CH + c], e[G * CH + G + c]);
      }
      qn = 0;
    };
    auto enqueue = [&](int kind, int gslot, float l_all) {
      if (qn == a.qs) flush_outputs();
      float* e = qbase + qn * qstride;
      if (col < G) {
#pragma unroll
        for (int dt = 0; dt < CH / 16; ++dt) o_at(e, dt) = O[dt];
        if (g4 == 0) {
          e[G * CH + col] = m;
          e[G * CH + G + col] = l_all;
        }
      }
      if (lane == 0) {
        int* meta = (int*)(e + slot_floats);
        meta[0] = kind;
        meta[1] = cc.r;
        meta[2] = cc.g;
        meta[3] = gslot;
      }
      ++qn;
    };
    auto park = [&](float l_all, int ends) {                  // leave this wave's first piece for the wave that begins the chain
      float* so = lds + wv * slot_floats;
      if (col < G) {
#pragma unroll
        for (int dt = 0; dt < CH / 16; ++dt) o_at(so, dt) = O[dt];
        if (g4 == 0) {
          so[G * CH + col] = m;
          so[G * CH + G + col] = l_all;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) {
        flag_set(wv, ends);
      }
    };

    // The last piece of segment (cc.r, cc.g) is finished, and the wave has more to stream.  A piece that spans its whole segment
    // is final; otherwise it belongs to a chain of pieces of neighbouring waves (see the header comment), and the wave that
    // began it (or, for wave 0, the work-group on the left through the workspace) takes it.
    auto emit = [&]() {
      const float l_all = column_sum(lsum);
      if (from_start) enqueue(0, 0, l_all);
      else if (wv == 0) enqueue(1, 2 * blockIdx.x, l_all);
      else park(l_all, PIECE_ENDS);
    };
    // The last piece of the wave's range, whose state is still in registers.
    auto finish = [&]() {
      bool to_end = cc.t == cc.tiles - 1;
      float l_all = column_sum(lsum);
      if (!to_end && wv < WPW - 1) {
        // the segment continues in the right-hand neighbour's range
        if (!from_start && wv > 0) {                           // and began to the left: whoever began it takes both pieces
          park(l_all, PIECE_GOES_ON);
          return;
        }
        // take the neighbours' first pieces, up to the one that does not fill its whole range: their references first, then
        // the outputs, each scaled once
        const int c = col < G ? col : 0;
        const int w0 = rfl(wv) + 1;
        float m_new = m;
        int ends, w1 = w0;
#pragma nounroll
        for (;; ++w1) {
          while ((ends = rfl(flag_get(w1))) == 0) __builtin_amdgcn_s_sleep(1);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
          m_new = fmaxf(m_new, lds[w1 * slot_floats + G * CH + c]);
          if (ends != PIECE_GOES_ON) break;
        }
        const float a1 = __builtin_amdgcn_exp2f(m - m_new);
        l_all *= a1;
#pragma unroll
        for (int dt = 0; dt < CH / 16; ++dt) O[dt] *= a1;
#pragma nounroll
        for (int w = w0; w <= w1; ++w) {
          float* so = lds + w * slot_floats;
          const float a2 = __builtin_amdgcn_exp2f(so[G * CH + c] - m_new);
          l_all = fmaf(so[G * CH + G + c], a2, l_all);
#pragma unroll
          for (int dt = 0; dt < CH / 16; ++dt) {
            O[dt] += o_at(so, dt) * a2;
            if (LATE_Q && (dt & 1)) __builtin_amdgcn_sched_barrier(0);   // (no registers for all of the piece at once)
          }
        }
        m = m_new;
        to_end = ends == PIECE_ENDS;
      }
      // (past the work-group's end: its slot of the segment that starts here and ends in a later one, or that began before it)
      if (from_start || wv == 0) put(from_start && to_end ? 0 : 1, cc.r, cc.g, 2 * blockIdx.x + (from_start ? 1 : 0), O, m, l_all);
      else park(l_all, to_end ? PIECE_ENDS : PIECE_CUT);
    };

    // main loop: NBUF tiles per trip so that buffer indices are compile-time constants.
    // Order inside a step matters because vmcnt retires in order: the queries of the next
    // segment are requested BEFORE this step's tile loads and adopted one step later AFTER
    // that step's tile loads, so waiting for them never drains the tile pipeline.
    // (LATE_Q: they are requested right behind the last tile of the segment before, and the next tile waits for them;
    // fp32 with head_dim 256 spilled 98 registers, fused 314, with the second operand.  64 requests of 4 heads 184 -> 102 us,
    // fused 141 -> 110; one of 300 tokens 55 -> 33, as long as on the vector kernel)
    bool q_pending = !LATE_Q;                                // the first segment's queries wait in qnext
    for (int i = 0; i < n_my; i += NBUF) {
#pragma unroll
      for (int u = 0; u < NBUF; ++u) {
        const bool active = i + u < n_my;
        const bool seg_end = active && cc.t == cc.tiles - 1;
        const bool more = i + u + 1 < n_my;
        if (q_pending && seg_end && more) {
          // a one-tile segment: its successor's queries are requested below, so the ones waiting
          // in qnext must be adopted first (this wait can stall; the common case is further down)
          if constexpr (!LATE_Q) adopt_q(qnext);
          q_pending = false;
        }
        if (!LATE_Q && seg_end && more) {
          const int ng = cc.g + 1 == Hkv ? 0 : cc.g + 1;
          const int nr = cc.g + 1 == Hkv ? cc.r_next : cc.r;
          if constexpr (!LATE_Q) load_q(qnext, nr, ng);
        }
        if (FUSED && active) {
          // fetch the appended row one tile before it is needed when the segment allows it
          if (seg_end ? !new_ready : (more && cc.t + 2 == cc.tiles)) {
            load_new(cc.r, cc.g);
            new_ready = true;
          }
        }
        issue(kb[(u + NBUF - 1) % NBUF], vb[(u + NBUF - 1) % NBUF]);
        if (p_left > 0) {
          advance(pc, wp);
          lookup_block(pc);
          --p_left;
        }
        if (q_pending) {
          // adopted after this step's tile loads were issued: waiting for the queries (requested a
          // step ago) then costs no more than waiting for the tile computed next
          if constexpr (!LATE_Q) adopt_q(qnext);
          q_pending = false;
        }
        if (active) {
          if (FUSED && seg_end) {
            patch_and_store(kb[u], vb[u]);
            new_ready = false;
          }
          compute(kb[u], vb[u]);
          TL_STAMP(8 + i + u);
#ifdef ODMA_DEV_TIMELINE
          if (lane == 0 && seg_end) tl_lds[wv][6] |= 1ll << (i + u);
          if (lane == 0 && qn == a.qs && (seg_end || !more)) tl_lds[wv][7] |= 1ll << (i + u);
#endif

          if (more) {
            if (seg_end) emit();
            advance(cc, wc);
            if (seg_end) {
              if constexpr (LATE_Q) load_q(qreg, cc.r, cc.g);
              else q_pending = true;
              m = LOWEST_REF;
              lsum = 0.f;
#pragma unroll
              for (int k = 0; k < CH / 16; ++k) O[k] = float4v{0.f, 0.f, 0.f, 0.f};
              from_start = true;
            }
          }
        }
      }
    }
    // the range is streamed: write what was queued
    finish();
    TL_STAMP(2);
    flush_outputs();
    if (FUSED) flush_appends();
    TL_STAMP(3);
#ifdef ODMA_DEV_TIMELINE
    if (lane == 0) tl_lds[wv][5] = n_my;
#endif
  }

  // Outputs of empty requests are zeros: thread i of the grid looks after request i, i + grid size, ...
  for (int r = r_mine; r < a.n; r += gridDim.x * (64 * WPW)) {
    if ((r == r_mine ? len_mine : a.lengths[r]) <= 0) {
      const int64_t o = (int64_t)r * a.Hq * HD;
      if (a.out_bf16) {
        uint2v* p = (uint2v*)((unsigned short*)a.out + o);
        for (int i = 0; i < a.Hq * (HD / 4); ++i) p[i] = uint2v{0u, 0u};
      } else {
        float4v* p = (float4v*)((float*)a.out + o);
        for (int i = 0; i < a.Hq * (HD / 4); ++i) p[i] = float4v{0.f, 0.f, 0.f, 0.f};
      }
    }
  }

#ifdef ODMA_DEV_TIMELINE
  auto tl_flush = [&]() {
    TL_STAMP(4);
    const int w = blockIdx.x * WPW + wv;
    if (w < 4096 && lane < TL_SLOTS) odma_dev_timeline_buf[w * TL_SLOTS + lane] = tl_lds[wv][lane];
  };
#else
  auto tl_flush = [&]() {};
#endif
  if (!a.fuse_reduce) {
    tl_flush();
    return;
  }
  // Merge of segments cut by work-group boundaries.  Every work-group a cut segment spans has by
  // now written one partial state to the workspace.  It then counts itself in at the segment's
  // counter; the work-group that arrives last sees all partials and merges them:
  //   m* = max m_i, w_i = 2^(m_i - m*), out = sum w_i O_i / sum w_i l_i.
  // Nobody waits for anybody.  Order: a wave's partial stores (write-through, agent scope) are
  // acknowledged (vmcnt 0) before the work-group barrier, the counter update comes after the
  // barrier, and the merging work-group reads the partials with agent-scope loads after it has
  // seen the full count.
  const int b = blockIdx.x;
  if constexpr (PLAN) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int4v c = pl.cuts[2 * wv + i];
      rd_cut[i] = ReduceDesc{rfl(c[0]), rfl(c[1]), rfl(c[2]), rfl(c[3])};
    }
  }
  // a work-group whose range begins and ends on segment boundaries has written no partial and counts in nowhere:
  // its waves leave as they finish (the descriptors are the same for every wave, so all of them take this exit)
  if (rd_cut[0].n_parts == 0 && !(rd_cut[1].n_parts > 0 && rd_cut[1].b0 == b)) {
    tl_flush();
    return;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  int* merges_here = flags;                                // chain hand-off flags are dead now
  if (threadIdx.x < 2) {
    const ReduceDesc rda = rd_cut[0], rdb = rd_cut[1];       // the segments cut at this work-group's two boundaries
    // thread 0 counts the work-group in at the segment cut in front of it (it holds a piece of that
    // segment), thread 1 at the segment that starts here and runs into the next work-group; both
    // counter updates travel together
    const bool second = threadIdx.x == 1;
    const int n_parts = second ? rdb.n_parts : rda.n_parts;
    const int owner = (second ? b : rda.b0) + 1;
    const bool in = second ? (rdb.n_parts > 0 && rdb.b0 == b) : rda.n_parts > 0;
    int last = 0;
    if (in) {
      last = count_in(a.arrive + owner) == n_parts - 1;
      // the last arrival leaves the count at zero for the next launch
      if (last) __hip_atomic_store(a.arrive + owner, (unsigned long long)ARRIVE_TAG << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    merges_here[threadIdx.x] = last;
  }
  __syncthreads();
  const bool do_a = merges_here[0] != 0, do_b = merges_here[1] != 0;
  if (!do_a && !do_b) {
    tl_flush();
    return;
  }
  // partial i of a segment sits in slot 2 (b0 + i), the first one in its work-group's "starts here" slot 2 b0 + 1
  auto part_at = [&](const ReduceDesc& rd, int i) -> int64_t { return (int64_t)(2 * (rd.b0 + i) + (i == 0 ? 1 : 0)) * a.Hq + rd.g * G; };
  auto write_merged = [&](const ReduceDesc& rd, int h, int d4, float4v acc, float l) {
    if (4 * d4 >= HD) return;                                  // head_dim 64: the upper channels are padding
    const float inv = a.out_scale / l;
    const int64_t o = ((int64_t)rd.r * a.Hq + rd.g * G + h) * HD + 4 * d4;
    if (a.out_bf16) {
      uint2v pk;
      pk[0] = (unsigned)float_to_bf16_bits(acc[0] * inv) | ((unsigned)float_to_bf16_bits(acc[1] * inv) << 16);
      pk[1] = (unsigned)float_to_bf16_bits(acc[2] * inv) | ((unsigned)float_to_bf16_bits(acc[3] * inv) << 16);
      *(uint2v*)((unsigned short*)a.out + o) = pk;
    } else {
      *(float4v*)((float*)a.out + o) = acc * inv;
    }
  };
  const int n_a = do_a ? rd_cut[0].n_parts : 0, n_b = do_b ? rd_cut[1].n_parts : 0;
  // partials whose loads are in flight together: the usual cut has two parts, a long request spans tens of work-groups; loads
  // past the last part would only repeat it, so the batch fits the count
  auto merge = [&](auto cuts_tag, auto batch_tag, int which, int thread, int threads) {
    constexpr int CUTS = decltype(cuts_tag)::value, BATCH = decltype(batch_tag)::value;
    // thread -> (head, four channels)
    for (int idx = thread; idx < G * (CH / 4); idx += threads) {
      const int h = idx / (CH / 4), d4 = idx - h * (CH / 4);
      float m_run[CUTS], l_run[CUTS];
      float4v acc[CUTS];
#pragma unroll
      for (int c = 0; c < CUTS; ++c) {
        m_run[c] = -INFINITY;
        l_run[c] = 0.f;
        acc[c] = float4v{0.f, 0.f, 0.f, 0.f};
      }
      const int most = CUTS == 2 ? max(n_a, n_b) : which == 0 ? n_a : n_b;
      for (int i0 = 0; i0 < most; i0 += BATCH) {
        float2 ml[CUTS][BATCH];
        float4v ov[CUTS][BATCH];
#pragma unroll
        for (int c = 0; c < CUTS; ++c) {
          const bool first = CUTS == 2 ? c == 0 : which == 0;
          const ReduceDesc rd = first ? rd_cut[0] : rd_cut[1];
          const int n = first ? n_a : n_b;
#pragma unroll
          for (int u = 0; u < BATCH; ++u) {
            const int64_t pi = part_at(rd, min(i0 + u, n - 1)) + h;
            ml[c][u] = load_pair_agent((const float*)&a.part_ml[pi]);
            const float2 lo = load_pair_agent(a.part_o + pi * CH + 4 * d4);
            const float2 hi = load_pair_agent(a.part_o + pi * CH + 4 * d4 + 2);
            ov[c][u] = float4v{lo.x, lo.y, hi.x, hi.y};
          }
        }
        asm volatile("" ::: "memory");                         // every load of the batch is issued before the first is waited for
#pragma unroll
        for (int c = 0; c < CUTS; ++c) {
          const int n = (CUTS == 2 ? c == 0 : which == 0) ? n_a : n_b;
          float m_new = m_run[c];
#pragma unroll
          for (int u = 0; u < BATCH; ++u)
            if (i0 + u < n) m_new = fmaxf(m_new, ml[c][u].x);
          const float keep = __builtin_amdgcn_exp2f(m_run[c] - m_new);
          acc[c] *= keep;
          l_run[c] *= keep;
#pragma unroll
          for (int u = 0; u < BATCH; ++u)
            if (i0 + u < n) {
              const float w = __builtin_amdgcn_exp2f(ml[c][u].x - m_new);
              acc[c] += ov[c][u] * w;
              l_run[c] = fmaf(w, ml[c][u].y, l_run[c]);
            }
          m_run[c] = m_new;
        }
      }
#pragma unroll
      for (int c = 0; c < CUTS; ++c) {
        const bool first = CUTS == 2 ? c == 0 : which == 0;
        write_merged(first ? rd_cut[0] : rd_cut[1], h, d4, acc[c], l_run[c]);
      }
    }
  };
  // More than eight parts: what bounds the merge are its load instructions, and a third of those brought every thread the same few
  // references and sums.  Here a row of 16 lanes holds those of 16 parts of one head -- 64 threads of outputs belong to four heads at
  // most, with 64 channels or more -- and the threads get the parts' weights from it.  Together with the halves below, launches that
  // reuse a plan: 7 requests of 3 352 to 14 405 tokens, 14 / 2 heads 18.7 -> 16.6 us, two around 16 000, 6 / 3 heads 18.0 -> 13.9; in fp32,
  // 64 channels, two of 6 633 and 5 210, 4 / 2 heads 18.4 -> 11.5.
  auto merge_many = [&](int which, int wave, int waves) {
    constexpr int BATCH = 16;
    const ReduceDesc rd = which == 0 ? rd_cut[0] : rd_cut[1];
    const int n = which == 0 ? n_a : n_b, size = G * (CH / 4);
    auto over_row = [](float x, auto op) {
      x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)));   // (rotations by 8, 4, 2, 1)
      x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false)));
      x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, false)));
      return op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, false)));
    };
    for (int t0 = 64 * wave; t0 < size; t0 += 64 * waves) {     // (every lane of a wave that has any: they hold the others' weights)
      const int idx = min(t0 + lane, size - 1), h = idx / (CH / 4), d4 = idx - h * (CH / 4), h0 = t0 / (CH / 4);
      const int row = 16 * (h - h0), row_h = min(h0 + (lane >> 4), G - 1);
      float m_run = -INFINITY, l_run = 0.f;                     // of the row's head
      float4v acc = float4v{0.f, 0.f, 0.f, 0.f};
      for (int i0 = 0; i0 < n; i0 += BATCH) {
        const bool held = i0 + (lane & 15) < n;
        const float2 ml = load_pair_agent((const float*)&a.part_ml[part_at(rd, min(i0 + (lane & 15), n - 1)) + row_h]);
        float4v ov[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const int64_t pi = part_at(rd, min(i0 + u, n - 1)) + h;
          const float2 lo = load_pair_agent(a.part_o + pi * CH + 4 * d4);
          const float2 hi = load_pair_agent(a.part_o + pi * CH + 4 * d4 + 2);
          ov[u] = float4v{lo.x, lo.y, hi.x, hi.y};
        }
        asm volatile("" ::: "memory");                         // every load of the batch is issued before the first is waited for
        const float m_new = fmaxf(m_run, over_row(held ? ml.x : -INFINITY, [](float x, float y) { return fmaxf(x, y); }));
        const float keep = __builtin_amdgcn_exp2f(m_run - m_new), w = held ? __builtin_amdgcn_exp2f(ml.x - m_new) : 0.f;
        l_run = fmaf(l_run, keep, over_row(held ? w * ml.y : 0.f, [](float x, float y) { return x + y; }));
        m_run = m_new;
        acc *= __shfl(keep, row);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const float w_u = __shfl(w, row + u);
          if (i0 + u < n) acc += ov[u] * w_u;
        }
      }
      const float l = __shfl(l_run, row);
      if (t0 + lane < size) write_merged(rd, h, d4, acc, l);
    }
  };
  // (One after the other, two cuts of a late work-group were two round trips: fp8, 64 requests 17.0 -> 16.2 us, 256 fused 115.8
  // -> 113.0 for four layers.  More than four parts of both cuts at once are slower again: 7 parts of one, 10.0 -> 10.6.)
  using std::integral_constant;
  const int t = threadIdx.x;
  if (do_a && do_b && max(n_a, n_b) <= 2) {                    // the usual two cuts: their loads travel together
    merge(integral_constant<int, 2>{}, integral_constant<int, 2>{}, 0, t, 64 * WPW);
  } else if (do_a && do_b && max(n_a, n_b) <= 4) {
    merge(integral_constant<int, 2>{}, integral_constant<int, 4>{}, 0, t, 64 * WPW);
  } else {
#pragma nounroll
    for (int which = 0; which < 2; ++which) {
      const int n = which == 0 ? n_a : n_b;
      if (n == 0) continue;
      if (n <= 2) merge(integral_constant<int, 1>{}, integral_constant<int, 2>{}, which, t, 64 * WPW);
      else if (n <= 4) merge(integral_constant<int, 1>{}, integral_constant<int, 4>{}, which, t, 64 * WPW);
      else if (n <= 8) merge(integral_constant<int, 1>{}, integral_constant<int, 8>{}, which, t, 64 * WPW);
      else {
        // Two cuts of many parts, and half of the waves are threads enough: one half for each.  (Of a few long requests the work-group
        // between two is often the last of both: it has two pieces to store.  Decided here: a number of waves that is a variable in
        // front of the short merges costs every one of them 0.1 us, and so does a second copy of the long one.)
        const bool halves = min(n_a, n_b) > 8 && G * (CH / 4) <= 32 * WPW;
        const int waves = halves ? WPW / 2 : WPW, mine = rfl(wv) & (waves - 1);
        if (halves && rfl(wv) / (WPW / 2) != which) continue;
        if constexpr (CH >= 64) merge_many(which, mine, waves);
        else merge(integral_constant<int, 1>{}, integral_constant<int, STREAM_MERGE_BATCH>{}, which, 64 * mine + lane, 64 * waves);
      }
    }
  }
  tl_flush();
}

// ---------------------------------------------------------------------------------
// cross-work-group reduction as a launch of its own.  A segment cut by work-group boundaries left one partial per
// work-group it spans: the first in that group's "starts here" slot 2b+1, the others in slot
// 2b.  The plan kernel marks, for the boundary in front of every attention work-group, whether
// a segment straddles it and this is the first boundary inside that segment; if so the
// (boundary, head) work-group of this kernel merges all partials of the segment:  m* = max m_i, w_i = 2^(m_i - m*), out = sum w_i O_i / sum w_i l_i.
// ---------------------------------------------------------------------------------
// Merges n_parts partial states of one head, BATCH partials at a time with all their loads in
// flight at once; batches are chained with a running maximum.  Thread d owns channel d.
template <int BATCH, class PartFn>
__device__ __forceinline__ float merge_parts(const StreamArgs& a, PartFn part, int n_parts, int d) {
  float m_run = -INFINITY, l_run = 0.f, acc = 0.f;
  for (int i0 = 0; i0 < n_parts; i0 += BATCH) {
    float2 ml[BATCH];
    float ov[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int64_t pi = part(min(i0 + u, n_parts - 1));
      ml[u] = a.part_ml[pi];
      ov[u] = a.part_o[pi * a.ch + d];
    }
    float m_new = m_run;
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (i0 + u < n_parts) m_new = fmaxf(m_new, ml[u].x);
    const float keep = __builtin_amdgcn_exp2f(m_run - m_new);
    acc *= keep;
    l_run *= keep;
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (i0 + u < n_parts) {
        const float w = __builtin_amdgcn_exp2f(ml[u].x - m_new);
        acc = fmaf(w, ov[u], acc);
        l_run = fmaf(w, ml[u].y, l_run);
      }
    m_run = m_new;
  }
  return acc * (a.out_scale / l_run);
}

// grid: n_wg * G work-groups (boundary, head) of one thread per channel of a state; no LDS, no
// barrier.  Used when the in-kernel merge of decode_stream_kernel is switched off.
__global__ __launch_bounds__(256) void stream_reduce_kernel(StreamArgs a, int n_wg) {
  const int G = a.G, d = threadIdx.x;
  const int b = blockIdx.x / G, h = blockIdx.x - b * G;
  const ReduceDesc rd = a.red[b];
  const int n_parts = rd.n_parts;
  if (n_parts == 0 || rd.b0 != b - 1) return;               // nothing cut here, or an earlier boundary owns the merge
  const int g = rd.g, b0 = rd.b0;
  // partial i of this segment: the first sits in its work-group's "starts here" slot
  auto part = [&](int i) -> int64_t { return (int64_t)(2 * (b0 + i) + (i == 0 ? 1 : 0)) * a.Hq + g * G + h; };
  // most cut segments span two work-groups; a long request spans tens
  const float val = n_parts <= 4 ? merge_parts<4>(a, part, n_parts, d) : merge_parts<16>(a, part, n_parts, d);
  if (d >= a.head_dim) return;                               // head_dim 64: the upper channels are padding
  const int64_t o = ((int64_t)rd.r * a.Hq + g * G + h) * a.head_dim + d;
  if (a.out_bf16) __builtin_nontemporal_store(float_to_bf16_bits(val), (unsigned short*)a.out + o);
  else __builtin_nontemporal_store(val, (float*)a.out + o);
}

// Launch with lds_bytes of dynamic LDS; `allowed`: the largest size enabled for the kernel so far (the default limit is
// 64 KiB).  Checking, setting and recording a larger size are one step: of two callers that raise it at once, the smaller
// size must not be the one set last.
inline hipError_t launch_with_lds(void (*kernel)(StreamArgs), std::atomic<unsigned>& allowed, int n_wg, int wpw, size_t lds_bytes,
                                  hipStream_t s, const StreamArgs& a) {
  if (lds_bytes > 64 * 1024 && lds_bytes > allowed.load(std::memory_order_acquire)) {
    static std::mutex raising;
    std::lock_guard<std::mutex> lock(raising);
    if (lds_bytes > allowed.load(std::memory_order_relaxed)) {
      const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
      if (e != hipSuccess) return e;
      allowed.store((unsigned)lds_bytes, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL(kernel, dim3(n_wg), dim3(64 * wpw), lds_bytes, s, a);
  return hipSuccess;
}

// Every launch shape of a format: register buffers per wave (3 or 2), waves per work-group (8 or 4).
template <int FMT, bool PLAN>
hipError_t launch_shapes(bool fused, bool paged, int nbuf, int wpw, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  // [fused][paged][3 - nbuf][wpw == 4]
#ifdef ODMA_DEV_MINIMAL_VARIANTS
  // development builds: only the default shape is compiled; the launch of another fails with an error
#define ODMA_SHAPES(U, P) {{nullptr, nullptr}, {nullptr, decode_stream_kernel<P, 2, 4, U, FMT, PLAN>}}
#else
#define ODMA_SHAPES(U, P) {{decode_stream_kernel<P, 3, 8, U, FMT, PLAN>, decode_stream_kernel<P, 3, 4, U, FMT, PLAN>}, \
                           {decode_stream_kernel<P, 2, 8, U, FMT, PLAN>, decode_stream_kernel<P, 2, 4, U, FMT, PLAN>}}
#endif
  static void (*const kernels[2][2][2][2])(StreamArgs) = {{ODMA_SHAPES(false, false), ODMA_SHAPES(false, true)},
                                                          {ODMA_SHAPES(true, false), ODMA_SHAPES(true, true)}};
#undef ODMA_SHAPES
  static std::atomic<unsigned> allowed[2][2][2][2];          // dynamic LDS enabled so far (nothing: zero-initialised)
  const auto kernel = kernels[fused][paged][3 - nbuf][wpw == 4];
  if (!kernel) return hipErrorInvalidDeviceFunction;
  return launch_with_lds(kernel, allowed[fused][paged][3 - nbuf][wpw == 4], n_wg, wpw, lds_bytes, s, *(const StreamArgs*)args);
}

// The wide formats of one storage type, in the launch shape of four waves and two buffers: BASE + D32 for every D32 given
// (head_dim 32 D32).  Instantiated in a unit of its own per storage type.
template <bool PLAN, int BASE, int... D32>
hipError_t launch_wide(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args) {
  struct Entry {
    int fmt;
    void (*kernel[2][2])(StreamArgs);                        // [fused][paged]
  };
  static const Entry entries[] = {
      {BASE + D32,
       {{decode_stream_kernel<false, 2, 4, false, BASE + D32, PLAN>, decode_stream_kernel<true, 2, 4, false, BASE + D32, PLAN>},
        {decode_stream_kernel<false, 2, 4, true, BASE + D32, PLAN>, decode_stream_kernel<true, 2, 4, true, BASE + D32, PLAN>}}}...};
  static std::atomic<unsigned> allowed[sizeof...(D32)][2][2];   // dynamic LDS enabled so far (nothing: zero-initialised)
  for (size_t i = 0; i < sizeof...(D32); ++i)
    if (entries[i].fmt == fmt)
      return launch_with_lds(entries[i].kernel[fused][paged], allowed[i][fused][paged], n_wg, 4, lds_bytes, s, *(const StreamArgs*)args);
  return hipErrorInvalidDeviceFunction;
}

}  // namespace

// The kernels are compiled in units of their own, one per format (or family of wide formats) and PLAN: odma_stream.hip,
// odma_wide_f32.hip and odma_wide_bf16.hip.  args: a StreamArgs, whose type is local to every unit.
template <int FMT, bool PLAN>
hipError_t odma_launch_stream(bool fused, bool paged, int nbuf, int wpw, int n_wg, size_t lds_bytes, hipStream_t s, const void* args);
template <bool PLAN>
hipError_t odma_launch_wide_f32(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args);
template <bool PLAN>
hipError_t odma_launch_wide_bf16(int fmt, bool fused, bool paged, int n_wg, size_t lds_bytes, hipStream_t s, const void* args);
#define ODMA_STREAM_UNIT(FMT, PLAN) \
  template <> hipError_t odma_launch_stream<FMT, PLAN>(bool, bool, int, int, int, size_t, hipStream_t, const void*);
#define ODMA_WIDE_UNITS(PLAN) \
  template <> hipError_t odma_launch_wide_f32<PLAN>(int, bool, bool, int, size_t, hipStream_t, const void*); \
  template <> hipError_t odma_launch_wide_bf16<PLAN>(int, bool, bool, int, size_t, hipStream_t, const void*);
ODMA_STREAM_UNIT(STREAM_BF16_D128, false) ODMA_STREAM_UNIT(STREAM_BF16_D128, true)
ODMA_STREAM_UNIT(STREAM_FP8_D128, false) ODMA_STREAM_UNIT(STREAM_FP8_D128, true)
ODMA_STREAM_UNIT(STREAM_BF16_D64, false) ODMA_STREAM_UNIT(STREAM_BF16_D64, true)
ODMA_WIDE_UNITS(false) ODMA_WIDE_UNITS(true)
#undef ODMA_STREAM_UNIT
#undef ODMA_WIDE_UNITS
