"""Prompt attention by eight waves per item (calls of long prompts), bounds of tests/test_gpu_prefill.py.  What selects it are
the rows of q per request; most tests here name more rows than their requests use (rows past a request's own are never
touched), so that prompts of a few tokens run it too: one to a few pairs of tiles, odd numbers of tiles, ragged ends, waves
without columns."""
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

@pytest.fixture
def many_rows(monkeypatch):
    """As many rows of q as the requests could have: 2048 each and more."""
    real = H.prefill

    def call(dp, layer, q, q_start, n_q, lengths, offsets=None, block_table=None):
        longest = dp.w.large_cap
        if block_table is not None:
            longest = 4096
            block_table = np.pad(block_table, ((0, 0), (0, 256 - block_table.shape[1])), constant_values=-1)
        return real(dp, layer, q, q_start, n_q, lengths, offsets=offsets, block_table=block_table, total_q=len(n_q) * longest)

    monkeypatch.setattr(H, "prefill", call)


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
    lens = np.random.default_rng(n).integers(0, 60, n)
    chunk_case(lens, lens, hq=4, hkv=2, sharp=True, seed=102, bounds=(64, 512, 2048), large_cap=2048, main=1 << 17)


@pytest.mark.parametrize("gain", [3.0, 5.0])
def test_columns_that_are_repeated(many_rows, gain):
    prefill.test_scores_that_outgrow_the_first_pair_are_redone_with_moving_references(gain, 0)


@pytest.mark.parametrize("grow", [False, True])
@pytest.mark.parametrize("paged", [False, True])
def test_infinite_values(many_rows, paged, grow):
    infinite.test_infinite_values_of_a_prompt_with_an_odd_number_of_tiles(paged, grow)


@pytest.mark.parametrize("kv_dtype,n_tok", [("bf16", 2100), ("fp8", 700)])
def test_long_prompts_against_four_waves(kv_dtype, n_tok):
    """Prompts long enough by themselves.  Both sides round every weight to bf16 and divide the same sums, in other orders: a
    weight differs by 2^-8 of itself at most, so an output by 2 * 2^-8 of the largest value, here under 5."""
    lens = np.arange(n_tok, n_tok + 60, 6 if kv_dtype == "bf16" else 3)   # (more than 512 items of 128 columns)
    w = small_workload(lens, kv_dtype=kv_dtype, hq=8, hkv=4, seed=103, bounds=(1024, 4096), large_cap=4096, main=1 << 16)
    rng = np.random.default_rng(104)
    total = int(lens.sum())
    q, _ = wl.draw_values(rng, (total, 8, 128), 1.0, "bf16")
    q_start = np.concatenate([[0], np.cumsum(lens)[:-1]])
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    got = []
    for column_tiles in (0, 2):
        dp = H.make_pool(w, out_dtype=B.F32)
        dp.pool.odma_pool_tune(B.TUNE_PREFILL_COLUMN_TILES, column_tiles)
        off, _ = H.assign_perfect(dp, lens)
        H.fill(dp, 0, kv, offsets=off)
        got.append(H.prefill(dp, 0, q, q_start, lens, lens, offsets=off))
    assert np.isfinite(got[0]).all() and not np.array_equal(got[0], got[1])
    np.testing.assert_allclose(got[0], got[1], rtol=0, atol=2 * P_ROUNDING * 5)
