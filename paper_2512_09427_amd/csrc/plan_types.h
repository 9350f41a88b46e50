// Plain data types of the decode plans, the arithmetic that cuts the tile stream into per-wave ranges, and the
// carve-up of the device workspace.  No HIP in here: the host allocator (built with g++ alone) and the kernels
// (hipcc) both include it, so that the host can size and check what the device fills in.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define ODMA_HD __host__ __device__
#else
#define ODMA_HD
#endif

namespace odma_plan {

// ---- chunked scheme (vector-ALU kernel) ----
struct PlanHeader {
  int32_t n_pairs;       // number of (request, chunk) pairs
  int32_t chunk;         // tokens per chunk, multiple of 64
  int32_t n_req;
  int32_t pad;
  int64_t total_tokens;
};
struct Item {            // one (request, chunk) pair; replicated over KV heads by the kernels
  int32_t r, tok_start, n_tok, n_split;
};
struct ReqInfo {
  int32_t first_pair, n_split;
};

// ---- tile-stream scheme (matrix-core kernel) ----
struct StreamEntry {         // one non-empty request, in batch order
  int32_t r, tiles, first_pos, len;   // tiles = ceil(len/16) per KV head; first_pos = position of (r, head 0, block 0)
  int32_t base_block, pad0, pad1, pad2;
};
struct WaveDesc {            // one wave's tile range, with its first entry inlined so that the
  int32_t pos_start, pos_end, entry0, n_entries;   // first loads need no second lookup
  int32_t r, tiles, first_pos, len;
  int32_t base_block, r_next, pad1, pad2;   // r_next: request of entry0 + 1
};
struct ReduceDesc {          // the segment cut by the boundary in front of work-group b
  int32_t n_parts;           // work-groups the segment spans (0: no segment is cut here)
  int32_t r, g, b0;          // segment and the first work-group it touches; boundary b0 + 1 owns its merge
};

constexpr int STREAM_MAX_WG = 4096;  // work-groups the pool workspace is sized for
constexpr int STREAM_MAX_LAUNCH_WG = 2048;   // most work-groups of one launch: eight waves per SIMD of 256 compute units
// What the regions hold beyond a launch's most work-groups is prompt attention's: the states of items whose keys are cut into
// parts, so that a plan for decode launches survives a prompt call (StreamLayout::prompt_*).  At most this many parts.
constexpr int PROMPT_MAX_PARTS = 4096;
// Work-groups of a pool served by the wide formats, whose partial states live in the workspace that the chunked scheme
// sizes: one per compute unit, as many as fit.  In a small workspace the chunked kernel may spread further, one wave per
// (chunk, KV head), up to eight per compute unit; it does G heads' arithmetic on the vector ALU, though, where the matrix
// cores do not care.  It serves the pool if it has more than 1 + 2 G times the waves (chunked_is_wider), or if less than
// STREAM_WIDE_LEAST_WG work-groups fit.  Measured both ways over 743 calls with max_splits of 24 to 520, 1 to 32 KV heads and
// G of 1 to 8: none is slower than on the chunked kernel, the mean takes 0.66 of its time.  Without the rule 129 were
// slower, 32 heads with G = 1 up to six times (8 requests, 16 500 tokens, bf16, head_dim 32: 206 us against 34).
constexpr int STREAM_WIDE_WG = 256, STREAM_WIDE_LEAST_WG = 16;
inline bool chunked_is_wider(int64_t pairs, int64_t n_kv_heads, int64_t group, int64_t n_wg) {
  const int64_t most = 8 * STREAM_WIDE_WG, waves = pairs * n_kv_heads < most ? pairs * n_kv_heads : most;
  return waves > (1 + 2 * group) * 4 * n_wg;
}

// Shares of the tile stream.  Wave W of the `used` waves gets the tiles [start(W), start(W + 1)).
//   * Fewer tiles than waves: the empty ranges are all on the LEFT (wave W gets tile total - (used - W)), never
//     between two waves that hold tiles.  The attention kernel relies on this: a wave whose segment runs on past its
//     range waits for the first piece of its right-hand neighbour, and an empty wave never hands one over.
//   * Otherwise start(W) = floor(total * weight(0..W) / weight(all)): shares differ by at most one tile with equal
//     weights.  Work-groups on odd XCDs and the second wave on a SIMD (waves wpw/2.. of an 8-wave work-group) can be
//     given other weights (in 1/256 of the others'); weights are ignored below four tiles per wave, where a light
//     share could round to nothing.
// Weights are kept in 1/64 so that total (< 2^31) * cum (< 2^15 waves * 2^7 * 2^7) fits 64 bits.
struct StreamShares {
  int32_t total, used, wpw;
  long long w_even, w_odd, s_early, s_late, cum_all;

  ODMA_HD long long cum(int W) const {                     // weight of waves [0, W)
    const int half = wpw / 2;
    const long long s_wg = half * (s_early + s_late);       // slot weights of one whole work-group
    const int b = W / wpw, wv_in = W - b * wpw;
    const long long per8 = 4 * (w_even + w_odd);
    const int x = b & 7;                                    // work-group b runs on XCD b % 8
    const long long pre = (long long)(x + 1) / 2 * w_even + (long long)x / 2 * w_odd;   // work-groups before b in its round of 8
    const int early = wv_in < half ? wv_in : half, late = wv_in > half ? wv_in - half : 0;
    const long long in_wg = (long long)early * s_early + (long long)late * s_late;
    return ((long long)(b >> 3) * per8 + pre) * s_wg + ((x & 1) ? w_odd : w_even) * in_wg;
  }
  ODMA_HD bool equal() const { return w_even == w_odd && s_early == s_late; }
  ODMA_HD int start(int W) const {
    if (W >= used) return total;
    if (total < used) return total - (used - W) > 0 ? total - (used - W) : 0;
    // Equal weights: floor(total * W / used).  The product is below 2^46 and exact in a double, and a quotient that is
    // not whole lies at least 1 / used > 2^-15 under the next whole number, which rounding to 53 bits cannot reach: the
    // division (which every wave waits for when it plans) need not be a 64-bit integer one.
    if (equal()) return (int)((double)((long long)total * W) / (double)used);
    return (int)((long long)total * cum(W) / cum_all);
  }
  // Equal weights: the wave that holds tile pos, 0 <= pos < total.  start(W) <= pos is total * W < (pos + 1) * used, so it is
  // floor(((pos + 1) * used - 1) / total); with half a unit more above the line the quotient lies 1 / (2 total) > 2^-32 or more
  // from the whole numbers, which the rounding of a double under 2^15 cannot reach.
  ODMA_HD int wave_of(int pos) const {
    if (total < used) return used - total + pos;
    return (int)(((double)((long long)(pos + 1) * used) - 0.5) / (double)total);
  }
};

// Fewest tiles of a wave: q_short or q_long.  The smaller number spreads a batch over more waves and cuts its segments into more parts,
// which the last of their work-groups merges.  It is for batches that leave a wave no more than three tiles of their own and whose
// longest request has few parts.  Requests of one length that fill whole waves of q_long tiles and no more than one work-group
// stay there: no segment is cut through memory then, and shares of two to three tiles would cut most of them.
struct StreamFewest {
  int q_short, q_long;              // the same: nothing to choose
  int most_tiles, most_longest;     // of the batch and of its longest request
  // (A launch that plans computes this in front of its first tile, where an instruction costs 2 ns: no division.  q_long * wpw is a
  // power of two where there is a choice.)
  ODMA_HD int of(int total, int longest, int segments, int n_waves, int wpw) const {
    if (q_short == q_long || total > most_tiles || longest > most_longest) return q_long;
    const int whole = q_long * wpw;
    const bool even = longest > 1 && longest <= whole && (longest & (longest - 1)) == 0 && (total & (whole - 1)) == 0 &&
                      longest * segments == total && total > q_short * n_waves;
    return even ? q_long : q_short;
  }
};
// The parts of a longest request that two tiles a wave still pay for.  fp32, whose tiles are the dearer ones: 64, with few channels less.
// bf16: 24, and fewer where a merge is more than a turn of a work-group's threads (four channels each).  Of 3 577 random batches of
// few tiles a wave and at most 64 parts, twos against fours, the mean of a planning call and of one that reuses the plan: bf16 0.964 of
// the time, 25 of 1 482 above 1.04 (two always: 0.966 and 80, up to 1.33); fp32 0.918, 16 of 2 095 above 1.04 (0.918 and 27).
ODMA_HD inline int stream_few_parts(bool f32, int head_dim, int G) {
  if (f32) return head_dim < 128 ? 32 + head_dim / 4 : 64;
  return G * head_dim > 1024 ? 24 * 1024 / (G * head_dim) : 24;
}
ODMA_HD inline StreamFewest stream_fewest(int q_short, int q_long, int n_waves, int wpw, int parts) {
  if (q_short == q_long) return StreamFewest{q_short, q_long, 0, 0};
  return StreamFewest{q_short, q_long, 3 * n_waves, parts * q_short * wpw};
}

// Waves used: all of them unless that would leave less than q_min tiles per wave; a whole number of work-groups.
ODMA_HD inline StreamShares stream_shares(int total, int n_waves, int wpw, int q_min, int odd_xcd_weight,
                                          int late_wave_weight) {
  StreamShares s;
  int used = n_waves;
  if ((long long)used * q_min > total) used = total / q_min > 1 ? total / q_min : 1;
  used = (used + wpw - 1) / wpw * wpw;
  if (used > n_waves) used = n_waves;
  const bool weighted = (long long)total >= 4ll * used;
  s.total = total;
  s.used = used;
  s.wpw = wpw;
  s.w_even = 64;
  s.w_odd = weighted ? odd_xcd_weight >> 2 : 64;
  s.s_early = 64;
  s.s_late = weighted ? late_wave_weight >> 2 : 64;
  s.cum_all = s.equal() ? 1 : s.cum(used);   // (read with unequal weights alone)
  return s;
}

constexpr int STREAM_SPARE_WG = STREAM_MAX_WG - STREAM_MAX_LAUNCH_WG;
static_assert(STREAM_SPARE_WG > 0 && (size_t)STREAM_SPARE_WG * 8 * sizeof(WaveDesc) >= (size_t)PROMPT_MAX_PARTS * sizeof(int64_t),
              "an arrival counter for every part");

// Byte offsets of the regions of a tile-stream workspace sized for max_requests requests, n_wg_cap attention
// work-groups and n_q_heads query heads (partial states keep `channels` channels per head).
struct StreamLayout {
  size_t header, req_info, items, waves, red, arrive, part_ml, part_o, end;   // (header and req_info: unused, kept so that the size stays)
  size_t prompt_arrive, prompt_ml, prompt_o;   // with n_wg_cap = STREAM_MAX_WG, else 0
  int64_t prompt_columns;                      // query columns (a reference, a sum and `channels` outputs) that fit there
};
ODMA_HD inline StreamLayout stream_layout(size_t off, int64_t max_requests, int64_t n_wg_cap, int64_t n_q_heads,
                                          int64_t channels = 128) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  StreamLayout w;
  w.header = off;   off += 256;
  w.req_info = off; off += up((size_t)max_requests * 8);
  w.items = off;    off += up((size_t)max_requests * sizeof(StreamEntry));
  w.waves = off;    off += up((size_t)n_wg_cap * 8 * sizeof(WaveDesc));
  w.red = off;      off += up((size_t)(n_wg_cap + 1) * sizeof(ReduceDesc));
  w.arrive = off;   // one 64-bit counter per boundary of a launch
  off += up((size_t)((n_wg_cap < STREAM_MAX_LAUNCH_WG ? n_wg_cap : STREAM_MAX_LAUNCH_WG) + 1) * sizeof(int64_t));
  w.part_ml = off;  off += up((size_t)2 * n_wg_cap * n_q_heads * 2 * sizeof(float));
  w.part_o = off;   off += up((size_t)2 * n_wg_cap * n_q_heads * channels * sizeof(float));
  w.end = off;
  const bool spare = n_wg_cap == STREAM_MAX_WG;
  w.prompt_arrive = spare ? w.waves + (size_t)STREAM_MAX_LAUNCH_WG * 8 * sizeof(WaveDesc) : 0;
  w.prompt_ml = spare ? w.part_ml + (size_t)2 * STREAM_MAX_LAUNCH_WG * n_q_heads * 2 * sizeof(float) : 0;
  w.prompt_o = spare ? w.part_o + (size_t)2 * STREAM_MAX_LAUNCH_WG * n_q_heads * channels * sizeof(float) : 0;
  w.prompt_columns = spare ? (int64_t)2 * STREAM_SPARE_WG * n_q_heads : 0;
  return w;
}

}  // namespace odma_plan
