"""Bulk append and export of whole 16-token groups: every storage type with small, odd and large head_dims (rows of less
than one staging chunk up to several), groups that are cut, appends that start inside a block, both layouts; and the slots
of a block past the appended rows, which must keep what they hold."""
import numpy as np
import pytest

import workloads as wl
from tests import harness as H
from tests.test_gpu_parity import small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("kvd,d,hkv", [("f32", 32, 1), ("f32", 64, 3), ("f32", 128, 4), ("f32", 256, 8), ("bf16", 32, 1),
                                       ("bf16", 64, 4), ("bf16", 96, 3), ("bf16", 128, 2), ("bf16", 256, 5), ("fp8", 128, 4)])
def test_append_in_two_calls_then_export(kvd, d, hkv, paged):
    lens = np.array([1, 15, 16, 17, 33, 250, 64, 700])
    first = np.array([1, 3, 16, 16, 20, 0, 32, 511])          # the second call starts on and inside blocks
    w = small_workload(lens, kv_dtype=kvd, hq=hkv, hkv=hkv, d=d, seed=d + hkv, bounds=(64, 1024), large_cap=1024)
    dp = H.make_pool(w)
    kv = [wl.request_kv(w, 0, r) for r in range(len(lens))]
    where = dict(block_table=wl.shuffled_block_table(lens, w.pool_tokens // 16, 16, seed=3)) if paged else \
        dict(offsets=H.assign_perfect(dp, lens)[0])
    H.fill(dp, 0, [(k[:c], v[:c]) for (k, v), c in zip(kv, first)], **where)
    H.fill(dp, 0, [(k[c:], v[c:]) for (k, v), c in zip(kv, first)], positions=first, **where)
    for r, n in enumerate(lens):
        for m in {int(n), 1, max(1, int(n) - 1)}:
            at = dict(block_row=where["block_table"][r]) if paged else {}
            gk, gv = H.gather(dp, 0, 0 if paged else int(where["offsets"][r]), m, **at)
            np.testing.assert_array_equal(gk, kv[r][0][:m])
            np.testing.assert_array_equal(gv, kv[r][1][:m])


@pytest.mark.parametrize("kvd,d", [("f32", 64), ("bf16", 64), ("bf16", 256)])
@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 15])
def test_rewriting_the_first_rows_of_a_block_keeps_the_others(kvd, d, rows):
    lens = np.array([48])
    w = small_workload(lens, kv_dtype=kvd, hq=2, hkv=2, d=d, seed=7, bounds=(64, 1024), large_cap=1024)
    dp = H.make_pool(w)
    k, v = wl.request_kv(w, 0, 0)
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, [(k, v)], offsets=off)
    k2, v2 = wl.request_kv(w, 1, 0)
    H.fill(dp, 0, [(k2[:rows], v2[:rows])], offsets=off, positions=np.array([16]))
    k, v = k.copy(), v.copy()
    k[16:16 + rows], v[16:16 + rows] = k2[:rows], v2[:rows]
    gk, gv = H.gather(dp, 0, int(off[0]), 48)
    np.testing.assert_array_equal(gk, k)
    np.testing.assert_array_equal(gv, v)


@pytest.mark.parametrize("kvd,d,hkv,n_tok", [("f32", 128, 32, 33), ("bf16", 128, 20, 18), ("bf16", 96, 11, 40), ("f32", 32, 1, 70001),
                                             ("bf16", 32, 3, 66000)])
def test_rows_of_many_chunks_and_more_groups_than_the_grid(kvd, d, hkv, n_tok):
    """Rows of up to 16 KiB, the last chunk partial; exports and appends of more 16-token groups than work-groups in a grid row."""
    lens = np.array([n_tok])
    w = small_workload(lens, kv_dtype=kvd, hq=hkv, hkv=hkv, d=d, seed=11, bounds=(64, 1 << 17), large_cap=1 << 17, main=1 << 17,
                       safety=1 << 17)
    dp = H.make_pool(w)
    kv = wl.request_kv(w, 0, 0)
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, [kv], offsets=off)
    gk, gv = H.gather(dp, 0, int(off[0]), n_tok)
    np.testing.assert_array_equal(gk, kv[0])
    np.testing.assert_array_equal(gv, kv[1])
