"""Prompt attention where its item queues can go wrong: fewer items than queues, one request that fills several of them,
empty requests around the boundaries, more requests than the item table in LDS holds, and bf16 output rows whose last
wave has columns of some lanes only.  Bounds of tests/test_gpu_prefill.py."""
import numpy as np
import pytest

from paper_2512_09427_amd import binding as B
from tests.test_gpu_prefill import chunk_case

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
