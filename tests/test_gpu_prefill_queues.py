"""Prompt attention where its item queues can go wrong: fewer items than queues, one request that fills several of them,
empty requests around the boundaries, more requests than the item table in LDS holds, and bf16 output rows whose last
wave has columns of some lanes only.  Bounds of tests/test_gpu_prefill.py."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import attention as oa
from paper_2512_09427_amd import binding as B
from tests import harness as H
from tests.test_gpu_parity import small_workload
from tests.test_gpu_prefill import P_ROUNDING, TIGHT, chunk_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("column_tiles", [2, 4])
@pytest.mark.parametrize("lens,hq,hkv", [
    ([1], 1, 1),                                             # one item of one column
    ([0, 0, 5, 0], 7, 1),                                    # empty requests on both sides
    ([18, 19], 7, 1),                                        # an item that is just full, and one column more
    ([2000, 1, 1, 0, 1], 8, 1),                              # one request holds all boundaries of the queues
    ([1] * 70, 3, 3),                                        # two hundred items of one pair
    ([0, 300, 0, 700, 0, 0, 31, 0], 8, 4),
])
def test_item_queues(lens, hq, hkv, column_tiles):
    for out_dtype in (B.F32, B.BF16):
        chunk_case(lens, lens, hq=hq, hkv=hkv, sharp=True, seed=91, column_tiles=column_tiles, out_dtype=out_dtype)


@pytest.mark.parametrize("n", [1024, 1025])
def test_requests_around_the_size_of_the_item_table(n):
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 24, n)
    lens[n // 2] = 900
    chunk_case(lens, lens, hq=2, hkv=1, sharp=True, seed=92, bounds=(64, 512, 1024), large_cap=1024, main=1 << 17)


@pytest.mark.parametrize("n", [1500, 4096, 4097])
def test_requests_found_in_memory(n):
    """The 64-way search: one whole round and a part, two rounds, and one request more; a third of the requests empty,
    at both ends too, so that values repeat across the probes."""
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, n)
    lens[rng.random(n) < 1 / 3] = 0
    lens[:70] = lens[-70:] = 0
    lens[n // 3] = 300
    chunk_case(lens, lens, hq=2, hkv=1, sharp=True, seed=93, bounds=(64, 512, 1024), large_cap=1024, main=n * 64 + 4096)


@pytest.mark.parametrize("n", [800, 1030, 2100])
def test_runs_of_items_and_single_ones(n):
    """More items than eight per work-group, so that they go out in runs of one to four, the last of every queue alone; one
    request has a queue's share by itself."""
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, n)
    lens[n // 5] = 700
    chunk_case(lens, lens, hq=8, hkv=8, sharp=True, seed=94, bounds=(64, 512, 1024), large_cap=1024, main=n * 64 + 4096)


@pytest.mark.parametrize("column_tiles", [2, 4])
@pytest.mark.parametrize("kvd,paged", [("bf16", False), ("bf16", True), ("fp8", False), ("fp8", True)])
@pytest.mark.parametrize("lens,n_q,hq,hkv", [
    ([480, 481, 512, 513], [5, 37, 64, 1], 8, 8),            # 15 pairs (whole) and 16 (two parts), odd and even numbers of tiles
    ([5090], [128], 8, 8),                                   # one chunk, eight parts
    ([1000, 31], [1000, 31], 7, 1),                          # late parts that some columns see nothing of; short items whole
    ([4000, 0, 2500, 17], [19, 0, 18, 17], 7, 1),            # empty request, a block that is just full, one column more
    ([9000, 3000], [20, 300], 1, 1),                         # fewer states than parts in the workspace
    ([6000] + list(range(1, 41)), [128] + list(range(1, 41)), 7, 1),   # a long chunk beside many short prompts
    (list(range(30, 60)), [5] * 30, 4, 4),                   # short ones alone
])
def test_items_cut_into_parts(lens, n_q, hq, hkv, kvd, paged, column_tiles):
    for out_dtype in (B.F32, B.BF16):
        chunk_case(lens, n_q, hq=hq, hkv=hkv, sharp=True, seed=96, column_tiles=column_tiles, out_dtype=out_dtype, kv_dtype=kvd,
                   paged=paged, bounds=(512, 16384), large_cap=16384, main=1 << 17)


@pytest.mark.parametrize("lens,n_q,hq,hkv", [
    ([6000], [16], 8, 1),                                    # one item, eight parts for eight XCDs
    ([700, 3000], [30, 20], 4, 1),                           # two, of two and six parts
    ([2500], [70], 7, 7),                                    # seven: one fewer than queues
    ([2500], [130], 8, 4),                                   # twelve: queues again
])
def test_fewer_items_than_queues(lens, n_q, hq, hkv):
    chunk_case(lens, n_q, hq=hq, hkv=hkv, sharp=True, seed=101, bounds=(512, 8192), large_cap=8192, main=1 << 14)


def test_parts_whatever_the_workspace_holds():
    """Arrival counters and states in a workspace of arbitrary bytes, and again in what the call before left there; a graph's
    replays beside them."""
    lens, n_q = np.array([3000, 700]), np.array([40, 700])
    w = small_workload(lens, hq=8, hkv=8, seed=97, bounds=(512, 4096), large_cap=4096, main=1 << 14)
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    q, _ = wl.draw_values(np.random.default_rng(97), (int(n_q.sum()), 8, 128), 1.0, "bf16")
    q_start = np.array([0, 40])
    off = H.assign_perfect(dp, lens)[0]
    H.fill(dp, 0, kv, offsets=off)
    ref = np.concatenate([oa.attend_chunk(q[a:a + m], kv[r][0], kv[r][1], 1.0 / np.sqrt(128.0)) for r, (a, m) in enumerate(zip(q_start, n_q))])
    ref_abs = np.concatenate([oa.attend_chunk(q[a:a + m], kv[r][0], kv[r][1] & 0x7fff, 1.0 / np.sqrt(128.0))
                              for r, (a, m) in enumerate(zip(q_start, n_q))])
    for fill in (0, 0xff, 0x7f, None, None):                 # None: as the last call left it
        if fill is not None:
            dp.workspace.fill_(fill)
        got = H.prefill(dp, 0, q, q_start, n_q, lens, offsets=off)
        H.check(got, ref, TIGHT[0] + P_ROUNDING * ref_abs, TIGHT[1], what=f"workspace of {fill}")
    args = [H.to_dev(x) for x in (q, q_start.astype(np.int64), n_q.astype(np.int32), np.asarray(off, np.int64), lens.astype(np.int32))]
    out = torch.zeros(q.shape, dtype=torch.float32, device=H.DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dp.pool.odma_prefill_attention(0, 2, args[0], len(q), args[1], args[2], args[3], args[4], None, 0, out,
                                       torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        H.check(out.cpu().numpy(), ref, TIGHT[0] + P_ROUNDING * ref_abs, TIGHT[1], what="replay")


def test_items_cut_into_parts_repeat_bit_for_bit():
    """The states of an item are merged in the order of its keys, whichever work-group comes last."""
    lens, n_q = np.array([5090, 3000]), np.array([128, 40])
    w = small_workload(lens, hq=8, hkv=8, seed=98, bounds=(512, 8192), large_cap=8192, main=1 << 14)
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    q, _ = wl.draw_values(np.random.default_rng(98), (int(n_q.sum()), 8, 128), 1.0, "bf16")
    off = H.assign_perfect(dp, lens)[0]
    H.fill(dp, 0, kv, offsets=off)
    first = H.prefill(dp, 0, q, np.array([0, 128]), n_q, lens, offsets=off)
    for _ in range(20):
        np.testing.assert_array_equal(H.prefill(dp, 0, q, np.array([0, 128]), n_q, lens, offsets=off), first)


@pytest.mark.parametrize("waves_per_cu", [4, 32])
def test_a_plan_for_decode_launches_survives_a_prompt_call(waves_per_cu):
    """A planning decode call, a prompt call that cuts its items, a decode call that reuses the plan: the latter's output is what
    it is without the prompt call between.  4: the usual launch; 32: as many work-groups as a launch can have."""
    lens, n_q = np.array([5090, 3000, 700, 0, 33]), np.array([128, 40, 1, 0, 33])
    w = small_workload(lens, hq=8, hkv=8, seed=102, bounds=(512, 8192), large_cap=8192, main=1 << 15)
    dp = H.make_pool(w, out_dtype=B.F32)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_CU, waves_per_cu)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    off = H.assign_perfect(dp, lens)[0]
    H.fill(dp, 0, kv, offsets=off)
    rows, _ = wl.draw_values(np.random.default_rng(102), (int(n_q.sum()), 8, 128), 1.0, "bf16")
    q = wl.queries(w, 0, sharp=True)
    prompt = lambda: H.prefill(dp, 0, rows, np.concatenate([[0], np.cumsum(n_q)[:-1]]), n_q, lens, offsets=off)
    decode = lambda flags: H.decode(dp, 0, q, lens, offsets=off, flags=flags)
    planned = decode(0)
    reused, cut = decode(B.REUSE_PLAN), prompt()
    np.testing.assert_array_equal(reused, planned)
    for _ in range(3):
        np.testing.assert_array_equal(decode(B.REUSE_PLAN), reused)
        np.testing.assert_array_equal(prompt(), cut)


def test_calls_on_other_streams_are_independent():
    """Calls of few items on streams of their own leave the workspace alone, so they may overlap."""
    lens, n_q = np.array([5090, 3000]), np.array([128, 40])
    w = small_workload(lens, hq=8, hkv=8, seed=99, bounds=(512, 8192), large_cap=8192, main=1 << 14)
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    q_start = np.array([0, 128])
    off = H.assign_perfect(dp, lens)[0]
    H.fill(dp, 0, kv, offsets=off)
    where = [H.to_dev(x) for x in (q_start.astype(np.int64), n_q.astype(np.int32), np.asarray(off, np.int64), lens.astype(np.int32))]
    qs = [wl.draw_values(np.random.default_rng(seed), (int(n_q.sum()), 8, 128), 1.0, "bf16")[0] for seed in (99, 100)]
    sides = [torch.cuda.Stream() for _ in qs]
    dev = [H.to_dev(q) for q in qs]
    outs = [torch.zeros(q.shape, dtype=torch.float32, device=H.DEV) for q in qs]

    def call(i):
        dp.pool.odma_prefill_attention(0, 2, dev[i], len(qs[i]), where[0], where[1], where[2], where[3], None, 0, outs[i], sides[i])

    dp.workspace.fill_(0x5a)
    alone = []
    for i, q in enumerate(qs):
        torch.cuda.synchronize()
        call(i)
        torch.cuda.synchronize()
        alone.append(outs[i].clone())
        for r, (a, m) in enumerate(zip(q_start, n_q)):
            rows = slice(a, a + m)
            ref = oa.attend_chunk(q[rows], kv[r][0], kv[r][1], 1.0 / np.sqrt(128.0))
            ref_abs = oa.attend_chunk(q[rows], kv[r][0], kv[r][1] & 0x7fff, 1.0 / np.sqrt(128.0))
            H.check(alone[i][rows].cpu().numpy(), ref, TIGHT[0] + P_ROUNDING * ref_abs, TIGHT[1], what=f"request {r}")
    assert bool((dp.workspace == 0x5a).all())
    for _ in range(10):
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        for _ in range(4):
            call(0)
            call(1)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], alone[0]) and torch.equal(outs[1], alone[1])


@pytest.mark.parametrize("column_tiles", [2, 4])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("kvd", ["bf16", "fp8"])
def test_columns_that_are_repeated(kvd, paged, column_tiles):
    """Scores of standard deviation 64: most columns outgrow their first pair's reference and are repeated; requests of one
    tile, odd and even numbers of tiles, whole prompts and late chunks."""
    lens, n_q = np.array([16, 37, 48, 64, 700, 333]), np.array([16, 37, 1, 64, 90, 333])
    w = small_workload(lens, kv_dtype=kvd, hq=7, hkv=1, seed=95)
    dp = H.make_pool(w, out_dtype=B.F32)
    dp.pool.odma_pool_tune(B.TUNE_PREFILL_COLUMN_TILES, column_tiles)
    f, sign_off = (wl.FP8_SCALE, 0x7f) if kvd == "fp8" else (1.0, 0x7fff)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    q, _ = wl.draw_values(np.random.default_rng(95), (int(n_q.sum()), 7, 128), 64.0, "bf16")
    q_start = np.concatenate([[0], np.cumsum(n_q)[:-1]])
    where = dict(block_table=wl.shuffled_block_table(lens, w.pool_tokens // 16, 16, seed=79)) if paged else \
        dict(offsets=H.assign_perfect(dp, lens)[0])
    H.fill(dp, 0, kv, **where)
    got = H.prefill(dp, 0, q, q_start, n_q, lens, **where)
    for r in range(len(lens)):
        rows = slice(q_start[r], q_start[r] + n_q[r])
        ref = oa.attend_chunk(q[rows], kv[r][0], kv[r][1], f / np.sqrt(128.0)) * f
        ref_abs = oa.attend_chunk(q[rows], kv[r][0], kv[r][1] & sign_off, f / np.sqrt(128.0)) * f
        # scores up to 400, summed in fp32 over 128 channels: an error of 400 * 2^-24 * 8 in the exponent, twice over |V|
        H.check(got[rows], ref, TIGHT[0] + (P_ROUNDING + 4e-4) * ref_abs, TIGHT[1], what=f"request {r}")
