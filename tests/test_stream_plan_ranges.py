"""Host logic: the tile ranges the matrix-core plan gives its waves (odma_stream_plan_ranges, the same arithmetic the
plan kernel runs on the device).

The attention kernel lets a wave whose segment runs on past its range wait for the first piece of its right-hand
neighbour inside the work-group; an empty wave hands nothing over, so a range that holds tiles must never have an
empty range to its right among the used waves.  These tests pin that, and the plain properties of a partition,
over small totals, both work-group sizes, every tile minimum and the whole range of the share weights.
"""
import itertools
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2512_09427_amd import binding as B


def ranges(total, n_waves, wpw, q_min, odd=256, late=256):
    start, used = B.odma_stream_plan_ranges(total, n_waves, wpw, q_min, odd, late)
    return start.astype(np.int64), used


def check_partition(total, n_waves, wpw, q_min, odd=256, late=256):
    start, used = ranges(total, n_waves, wpw, q_min, odd, late)
    what = f"total={total} n_waves={n_waves} wpw={wpw} q_min={q_min} odd={odd} late={late}"
    assert start[0] == 0 and start[-1] == total, what
    assert (np.diff(start) >= 0).all(), what
    assert 1 <= used <= n_waves and used % wpw == 0, what
    assert (start[used:] == total).all(), what                      # waves past `used` hold nothing
    sizes = np.diff(start)[:used]
    holding = np.nonzero(sizes > 0)[0]
    if len(holding):
        # empty ranges form a prefix of the used waves
        assert (sizes[holding[0]:] > 0).all(), what + f" sizes={sizes.tolist()}"
    return sizes, used


@pytest.mark.parametrize("wpw", [4, 8])
def test_no_empty_range_right_of_a_range_with_tiles_small_totals(wpw):
    for n_waves in (wpw, 2 * wpw, 1024):
        for q_min in (1, 2, 4, 8):
            for total in range(0, 6 * wpw * 4 + 3):
                sizes, used = check_partition(total, n_waves, wpw, q_min)
                if total >= used:
                    assert sizes.max() - sizes.min() <= 1              # equal weights: shares differ by at most a tile


def test_the_shapes_that_used_to_interleave_empty_ranges():
    # one request of two tiles on one KV head, default shape: two tiles over a four-wave work-group
    sizes, used = check_partition(2, 1024, 4, 4)
    assert used == 4 and sizes.tolist() == [0, 0, 1, 1]
    # eight-wave work-groups, 2..6 tiles
    for total in range(2, 7):
        sizes, used = check_partition(total, 2048, 8, 4)
        assert used == 8 and sizes.tolist() == [0] * (8 - total) + [1] * total


@pytest.mark.parametrize("wpw", [4, 8])
def test_weighted_shares_never_round_to_nothing(wpw):
    rng = np.random.default_rng(7)
    weights = [128, 160, 232, 256, 300, 512]
    for odd, late in itertools.product(weights, weights):
        for n_waves in (wpw, 8 * wpw, 1024):
            totals = np.unique(np.concatenate([np.arange(0, 5 * n_waves + 2, max(1, n_waves // 16)),
                                               rng.integers(0, 40 * n_waves, 12)]))
            for q_min in (1, 2, 4):
                for total in totals:
                    sizes, used = check_partition(int(total), n_waves, wpw, q_min, odd, late)
                    if total >= 4 * used:
                        assert sizes.min() >= 1


def test_full_size_shares_are_even_and_weights_shift_them():
    total = 26240                                                     # about config 3: 104 745 tokens, 4 KV heads
    sizes, used = check_partition(total, 1024, 4, 4)
    assert used == 1024 and sizes.sum() == total and sizes.max() - sizes.min() <= 1
    light, _ = check_partition(total, 1024, 4, 4, odd=232)
    wg = light.reshape(256, 4).sum(axis=1)
    assert wg[1::2].mean() < wg[0::2].mean()                          # odd work-groups (odd XCDs) got less
    assert abs(wg[1::2].mean() / wg[0::2].mean() - 232 / 256) < 0.01


def test_invalid_arguments_are_refused():
    for args in [(-1, 8, 4, 4), (10, 0, 4, 4), (10, 6, 4, 4), (10, 8, 5, 4), (10, 8, 4, 0)]:
        with pytest.raises(B.OdmaError):
            B.odma_stream_plan_ranges(*args)
    with pytest.raises(B.OdmaError):
        B.odma_stream_plan_ranges(10, 8, 4, 4, 100, 256)


WAVE_OF = r"""
#include <cstdio>
#include <initializer_list>
#include "plan_types.h"
int check(int total, int n_waves, int wpw, int pos) {
  const odma_plan::StreamShares s = odma_plan::stream_shares(total, n_waves, wpw, 4, 256, 256);
  const int w = s.wave_of(pos);
  if (s.equal() && w >= 0 && w < s.used && s.start(w) <= pos && pos < s.start(w + 1)) return 0;
  std::printf("total %d n_waves %d wpw %d used %d pos %d: wave %d\n", total, n_waves, wpw, s.used, pos, w);
  return 1;
}
int main() {
  int bad = 0;
  for (int wpw = 4; wpw <= 8; wpw += 4)
    for (int n_waves : {wpw, 3 * wpw, 1024, 4096}) {
      for (int total = 1; total < 300; ++total)                        // every tile, fewer tiles than waves among them
        for (int pos = 0; pos < total; ++pos) bad += check(total, n_waves, wpw, pos);
      for (int total : {1023, 1024, 1025, 4095, 4097, 11649, 26240, 1 << 20, 0x7ffffffe, 0x7fffffff}) {
        const odma_plan::StreamShares s = odma_plan::stream_shares(total, n_waves, wpw, 4, 256, 256);
        for (int w = 0; w < s.used; ++w)                                 // the first and the last tile of every wave
          for (int pos : {s.start(w), s.start(w + 1) - 1}) if (pos >= s.start(w)) bad += check(total, n_waves, wpw, pos);
      }
    }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_the_wave_that_holds_a_tile(tmp_path):
    """StreamShares::wave_of is the inverse of StreamShares::start for equal shares."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_09427_amd", "csrc")
    (tmp_path / "t.cpp").write_text(WAVE_OF)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")], check=True, timeout=120)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]


FEWEST = r"""
#include <cstdio>
#include <initializer_list>
#include "plan_types.h"
int bad = 0;
void check(bool ok, const char* what, int wpw, int n_waves, int total, int longest, int segments, int got) {
  if (ok) return;
  std::printf("%s: wpw %d n_waves %d total %d longest %d segments %d: %d\n", what, wpw, n_waves, total, longest, segments, got);
  ++bad;
}
int main() {
  const int big = 0x7fffffff;
  for (int wpw : {4, 8})
    for (int n_waves : {3 * wpw, 1024, 4096}) {
      // a tuned minimum, up to 2^31 - 64 tokens: nothing to choose, nothing to overflow
      for (int q : {1, 4, big / 64 * 4})
        for (int total : {0, 1, n_waves, big})
          for (int longest : {0, 1, total}) {
            const int got = odma_plan::stream_fewest(q, q, n_waves, wpw, 32).of(total, longest, 1, n_waves, wpw);
            check(got == q, "tuned", wpw, n_waves, total, longest, 1, got);
          }
      for (int d : {32, 64, 96, 128, 256})
        for (int G : {1, 5, 16}) {
          const int parts = odma_plan::stream_few_parts(d == 64, d, G);
          const auto f = odma_plan::stream_fewest(2, 4, n_waves, wpw, parts);
          check(parts >= 6 && parts <= 64, "parts", wpw, n_waves, d, G, 0, parts);
          // both lines, with segments of other lengths beside the longest one
          const int line = 3 * n_waves, most = parts * 2 * wpw;
          for (int total : {0, 1, line - 1, line, line + 1, big})
            for (int longest : {0, 1, 7, most - 1, most, most + 1, big}) {
              const int got = f.of(total, longest, 3, n_waves, wpw);
              if ((long long)longest * 3 == total) continue;
              check(got == (total > line || longest > most ? 4 : 2), "line", wpw, n_waves, total, longest, 3, got);
            }
          // segments of one length: four tiles where two would be cut to fractions and four end with the segments
          for (int longest = 1; longest <= 4 * wpw + 1; ++longest)
            for (int segments = 1; segments * longest <= line && segments < 5000; ++segments) {
              const int total = segments * longest, got = f.of(total, longest, segments, n_waves, wpw);
              const auto s = odma_plan::stream_shares(total, n_waves, wpw, 4, 256, 256);
              bool uncut = total > 2 * n_waves && longest > 1;         // no segment reaches over a work-group's end, shares are whole
              for (int w = 0; w < s.used && uncut; ++w) uncut = s.start(w + 1) - s.start(w) == 4 && (w % wpw || s.start(w) % longest == 0);
              check(got == (uncut ? 4 : 2), "even", wpw, n_waves, total, longest, segments, got);
            }
        }
    }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_the_fewest_tiles_of_a_wave(tmp_path):
    """StreamFewest on both sides of its lines and for segments of one length, without overflow at the largest tuned minimum."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_09427_amd", "csrc")
    (tmp_path / "t.cpp").write_text(FEWEST)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", csrc, str(tmp_path / "t.cpp"),
                    "-o", str(tmp_path / "t")], check=True, timeout=120)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-2000:]
