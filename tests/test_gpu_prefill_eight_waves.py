"""Prompt attention by eight waves per item, bounds of tests/test_gpu_prefill.py.  The plan gives it calls whose items are long on
the average, so most tests here have further requests with many rows in their call (and rows of q that nobody uses), beside which
prompts of a few tokens run it too: one to a few pairs of tiles, odd numbers of tiles, ragged ends, waves without columns."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as wl
from paper_2512_09427_amd import binding as B
from tests import harness as H
from tests import test_gpu_infinite_values as infinite
from tests import test_gpu_prefill as prefill
from tests.test_gpu_parity import small_workload
from tests.test_gpu_prefill import P_ROUNDING, chunk_case

pytestmark = pytest.mark.gpu

FURTHER_ROWS, FURTHER_LEN = 512, 2400


def run_by_eight_waves(lens, n_q, hq, hkv, kv_dtype, paged, slack=1.0):
    """The plan's rule (mean pairs of an item, the longest item beside what a CU streams, padding), with some slack."""
    lens, n_q, n_cu = np.asarray(lens, np.float64), np.asarray(n_q, np.int64), torch.cuda.get_device_properties(0).multi_processor_count
    group = hq // hkv
    pairs, items = [], []
    for cols in (128, 256):
        blocks = -(-n_q * group // cols)
        pairs.append(float((hkv * blocks * ((lens - n_q) / 32 + blocks * cols / (64 * group))).sum()))
        items.append(int(hkv * blocks.sum()))
    least, slope, longest, padding = (13, 0, 0.9, 1.1) if kv_dtype == "fp8" else (16, 20, 1.0, 1.03) if paged else (28, 20, 0.8, 1.03)
    part = lens[n_q > 0].max() / 32 * n_cu / pairs[1]
    return (pairs[1] >= slack * (least + slope * part) * items[1] and slack * part <= longest
            and 2 * pairs[1] <= (1 + (padding - 1) / slack) * pairs[0])


@pytest.fixture
def many_rows(monkeypatch):
    """Calls have further requests of many rows behind those of the test, all of them the same (tokens, rows and results): as many as
    it takes, or up to the number of requests that a test sets in the dict it gets."""
    make_pool, prefill, room, want = H.make_pool, H.prefill, 2048, {"requests": None}

    def pool(w, **kw):
        # (behind the tokens that the test knows of: its slabs and its block tables stay where they were)
        dp = make_pool(dataclasses.replace(w, safety_tokens=w.safety_tokens + FURTHER_LEN), max_requests=w.n_requests + room, **kw)
        g = torch.Generator(device="cuda").manual_seed(5)
        for rows in (dp.k_pool, dp.v_pool):
            rows = rows.view(w.n_kv_heads, -1)[:, -FURTHER_LEN * w.head_dim:]
            x = torch.randn(rows.shape, generator=g, device="cuda")
            rows.copy_(x.to(torch.float8_e4m3fn).view(torch.uint8) if w.kv_dtype == "fp8" else x.to(torch.bfloat16).view(torch.int16))
        return dp

    def call(dp, layer, q, q_start, n_q, lengths, offsets=None, block_table=None):
        w, n, rows, paged = dp.w, len(n_q), len(q), block_table is not None
        at = w.pool_tokens - FURTHER_LEN
        for m in range(1, room) if want["requests"] is None else [want["requests"] - n]:
            more = lambda x, y, t: np.concatenate([np.asarray(x, t), np.full(m, y, t)])
            nq, lens = more(n_q, FURTHER_ROWS, np.int64), more(lengths, FURTHER_LEN, np.int64)
            if run_by_eight_waves(lens, nq, w.n_q_heads, w.n_kv_heads, w.kv_dtype, paged, slack=1.1):
                break
        else:
            raise AssertionError("too few further requests")
        more_q, _ = wl.draw_values(np.random.default_rng(6), (FURTHER_ROWS, w.n_q_heads, w.head_dim), 1.0, "bf16")
        table = None
        if paged:
            table = np.full((n + m, max(FURTHER_LEN // 16, block_table.shape[1])), -1, np.int32)
            table[:n, :block_table.shape[1]] = block_table
            table[n:, :FURTHER_LEN // 16] = at // 16 + np.arange(FURTHER_LEN // 16)
        # (rows of q enough for the call to be weighed: 200 pairs per compute unit)
        total = int(1.1 * (200 * 64 * 256 * 256 * (n + m) / w.n_q_heads) ** 0.5)
        got = []
        for column_tiles in (2, 0):
            dp.pool.odma_pool_tune(B.TUNE_PREFILL_COLUMN_TILES, column_tiles)
            got.append(prefill(dp, layer, np.concatenate([q, more_q]), more(q_start, rows, np.int64), nq, lens,
                               offsets=None if paged else more(offsets, at, np.int64), block_table=table,
                               total_q=max(total, rows + FURTHER_ROWS)))
        # the further requests' rows: four waves add a column's weights in another order
        finite, same = np.isfinite(got[1][rows:]).all(), np.array_equal(got[0][rows:], got[1][rows:])
        assert finite and (dp.out_dtype == B.BF16 or not same)
        return got[1][:rows]

    monkeypatch.setattr(H, "make_pool", pool)
    monkeypatch.setattr(H, "prefill", call)
    return want


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("hq,hkv", [(7, 1), (28, 4), (3, 3), (16, 1)])
def test_whole_prompts_and_chunks(many_rows, kv_dtype, paged, hq, hkv):
    lens = [1, 16, 17, 32, 33, 47, 64, 65, 96, 97, 129, 300, 0, 200, 500, 31]
    n_q = [1, 16, 17, 32, 33, 47, 64, 65, 96, 97, 129, 300, 0, 17, 70, 1]
    for out_dtype in (B.F32, B.BF16):
        chunk_case(lens, n_q, paged=paged, sharp=True, hq=hq, hkv=hkv, seed=101, kv_dtype=kv_dtype, out_dtype=out_dtype)


@pytest.mark.parametrize("n", [1024, 1025])
def test_requests_around_the_size_of_the_item_table(many_rows, n):
    many_rows["requests"] = n
    lens = np.random.default_rng(n).integers(0, 60, n - 620)
    chunk_case(lens, lens, hq=4, hkv=2, sharp=True, seed=102, bounds=(64, 512, 2048), large_cap=2048, main=1 << 17)


@pytest.mark.parametrize("gain", [3.0, 5.0])
def test_columns_that_are_repeated(many_rows, gain):
    prefill.test_scores_that_outgrow_the_first_pair_are_redone_with_moving_references(gain, 0)


@pytest.mark.parametrize("grow", [False, True])
@pytest.mark.parametrize("paged", [False, True])
def test_infinite_values(many_rows, paged, grow):
    infinite.test_infinite_values_of_a_prompt_with_an_odd_number_of_tiles(paged, grow)


@pytest.mark.parametrize("out_dtype", [B.F32, B.BF16])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("paged", [False, True])
def test_late_chunks_of_long_requests(many_rows, kv_dtype, paged, out_dtype):
    """A hundred pairs of tiles and more, against the oracle."""
    chunk_case([5001, 3333, 2400, 4096, 1777], [70, 33, 1, 128, 200], paged=paged, sharp=True, hq=8, hkv=2, seed=105, kv_dtype=kv_dtype,
               out_dtype=out_dtype, bounds=(1024, 4096, 8192), large_cap=8192)


def whole_prompts(lens, kv_dtype, hq, hkv, paged):
    """Outputs of whole prompts as the plan chooses and by four waves."""
    w = small_workload(lens, kv_dtype=kv_dtype, hq=hq, hkv=hkv, seed=103, bounds=(256, 1024, 2048, 16384), large_cap=16384,
                       main=(int(2 * lens.sum()) + 16384) // 256 * 256)
    q, _ = wl.draw_values(np.random.default_rng(104), (int(lens.sum()), hq, 128), 1.0, "bf16")
    q_start = np.concatenate([[0], np.cumsum(lens)[:-1]])
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    where = dict(block_table=wl.shuffled_block_table(lens, w.pool_tokens // 16, 16, seed=79)) if paged else \
        dict(offsets=H.assign_perfect(dp, lens)[0])
    H.fill(dp, 0, kv, **where)
    got = []
    for column_tiles in (0, 2):
        dp.pool.odma_pool_tune(B.TUNE_PREFILL_COLUMN_TILES, column_tiles)
        got.append(H.prefill(dp, 0, q, q_start, lens, lens, **where))
    return got


@pytest.mark.parametrize("kv_dtype,n_tok,step", [("bf16", 2120, 2), ("fp8", 1000, 1)])
def test_long_prompts_against_four_waves(kv_dtype, n_tok, step):
    """Prompts long enough by themselves.  The weights, their bf16 values and the sums of P V are the same for both, a column's sum of
    weights is added in another order: eight weights for each pair of tiles in a lane, then four lanes, each addition within 2^-24 of the sum,
    and so are the division, the product and its store."""
    lens = np.arange(n_tok, n_tok + 56, step)
    assert run_by_eight_waves(lens, lens, 8, 4, kv_dtype, True, slack=1.05)
    got = whole_prompts(lens, kv_dtype, 8, 4, True)
    finite, same = np.isfinite(got[0]).all(), np.array_equal(got[0], got[1])
    assert finite and not same                               # (the same bits: four waves twice)
    np.testing.assert_allclose(got[0], got[1], rtol=2 * (8 * lens.max() / 32 + 7) * 2.0 ** -24, atol=0)


# whole prompts that eight waves are slower on: one request is most of the call's time; blocks of 256 columns mostly empty; short ones
SLOWER = [("bf16", 4, 1, [1800] * 60 + [16000]), ("fp8", 4, 1, [600] * 60 + [9000]), ("fp8", 8, 8, [516] * 75), ("bf16", 8, 8, [1804] * 40),
          ("fp8", 8, 2, [200] * 150)]


@pytest.mark.parametrize("kv_dtype,hq,hkv,lens", SLOWER)
def test_calls_that_stay_with_four_waves(kv_dtype, hq, hkv, lens):
    lens = np.array(lens)
    assert not run_by_eight_waves(lens, lens, hq, hkv, kv_dtype, False)
    got = whole_prompts(lens, kv_dtype, hq, hkv, False)
    np.testing.assert_array_equal(got[0], got[1])
