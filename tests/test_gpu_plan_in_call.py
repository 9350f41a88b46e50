"""Decode calls that plan inside the attention launch: batch sizes around the work-group's scan width and the limit of
the in-launch plan, plans left behind for calls that reuse them, and workspaces that hold arbitrary bytes when a call
begins.  Against the oracle with the bounds of tests/test_gpu_parity.py; a reused plan must give the same bits."""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_2512_09427_amd import binding as B
from tests import harness as H
from tests.test_gpu_parity import TIGHT_F32, small_workload

pytestmark = pytest.mark.gpu


def make(lens, seed, **kw):
    lens = np.asarray(lens, dtype=np.int64)
    w = small_workload(lens, hq=4, hkv=2, seed=seed, bounds=(64, 1024, 8192), large_cap=8192, **kw)
    dp = H.make_pool(w, out_dtype=B.F32)
    off, _ = H.assign_perfect(dp, np.maximum(lens, 1))
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    H.fill(dp, 0, kv, offsets=off)
    q = wl.queries(w, 0, sharp=True)
    ref = H.oracle_out(w, q, kv)
    ref[lens == 0] = 0.0
    return dp, q, lens, off, ref


@pytest.mark.parametrize("wpw", [4, 8])
@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 513, 1024, 1025])
def test_batch_sizes_around_the_scan_width(n, wpw):
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 40, n)
    lens[rng.integers(0, n)] = 5000                          # cut over many work-groups
    dp, q, lens, off, ref = make(lens, seed=71, main=n * 64 + 16384)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_WG, wpw)
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, ref, *TIGHT_F32, what=f"n={n}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)


@pytest.mark.parametrize("odd_xcd_weight", [256, 232])
@pytest.mark.parametrize("n", [1, 127, 128, 129, 300])
def test_scans_by_a_wave_and_by_a_work_group(n, odd_xcd_weight):
    """Both ways to scan the batch, with equal shares (the work-group of a tile in closed form) and unequal ones (a table)."""
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 60, n)
    lens[[0, n // 2, n - 1]] = [700, 5000, 33]               # (the last entry's neighbours: none behind, empty ones in between)
    lens[n // 3:n // 3 + n // 8] = 0
    dp, q, lens, off, ref = make(lens, seed=74, main=n * 64 + 32768)
    dp.pool.odma_pool_tune(B.TUNE_ODD_XCD_WEIGHT, odd_xcd_weight)
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, ref, *TIGHT_F32, what=f"n={n}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)


@pytest.mark.parametrize("wpw", [4, 8])
@pytest.mark.parametrize("lens", [[64], [130], [176], [250], [400], [641], [1000], [300, 900], [1100, 1300, 700], [2100, 90, 2500], [6000, 500]])
def test_pieces_of_a_segment_over_waves_and_work_groups(lens, wpw):
    """Segments over two to all waves of a work-group, cut at none, one or both of its ends, into two, four, eight and more parts."""
    dp, q, lens, off, ref = make(lens, seed=75, main=32768)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_WG, wpw)
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, ref, *TIGHT_F32, what=str(lens))
    for _ in range(3):                                       # whoever arrives last, the same bits
        np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off), got)
        np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)


@pytest.mark.parametrize("lens", [[0], [0, 0, 0], [1], [0, 16, 0, 17, 0]])
def test_batches_with_next_to_no_tiles(lens):
    dp, q, lens, off, ref = make(lens, seed=72, main=16384)
    H.check(H.decode(dp, 0, q, lens, offsets=off), ref, *TIGHT_F32, what=str(lens))


def test_workspace_contents_do_not_matter():
    dp, q, lens, off, ref = make([7000, 3, 4000, 0, 2500, 64], seed=73, main=32768)
    g = torch.Generator(device=H.DEV).manual_seed(1)
    want = None
    for fill in (0x00, 0xff, 0x7f, 0x3c, None, None):
        if fill is None:
            dp.workspace.random_(0, 256, generator=g)
        else:
            dp.workspace.fill_(fill)
        got = H.decode(dp, 0, q, lens, offsets=off)
        H.check(got, ref, *TIGHT_F32, what=f"workspace of {fill}")
        want = got if want is None else want
        np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off), got)
        np.testing.assert_array_equal(got[1], want[1])


def test_two_pools_on_one_workspace():
    dp1, q1, lens1, off1, ref1 = make([7000, 3, 4000, 0, 2500, 64], seed=74, main=32768)
    lens2 = np.array([900, 8000, 31], np.int64)
    w2 = small_workload(lens2, hq=8, hkv=2, seed=75, bounds=(64, 1024, 8192), large_cap=8192, main=32768)
    dp2 = H.make_pool(w2, out_dtype=B.F32)
    # the second pool over the first one's workspace: other offsets of every region
    args = dict(n_layers=1, n_q_heads=8, n_kv_heads=2, head_dim=128, kv_dtype=B.BF16, out_dtype=B.F32,
                main_tokens=w2.main_tokens, safety_tokens=w2.safety_tokens, large_cap=w2.large_cap,
                boundaries=w2.boundaries, max_requests=3, align_tokens=w2.align_tokens)
    shared = torch.empty(max(dp1.workspace.numel(), dp2.workspace.numel()), dtype=torch.uint8, device=H.DEV)
    cfg, keep = B.make_config(**args, k_pool=dp2.k_pool, v_pool=dp2.v_pool, workspace=shared)
    dp2 = H.DevicePool(B.Pool(cfg, keep), dp2.k_pool, dp2.v_pool, shared, w2, B.F32)
    args1 = dict(args, n_q_heads=4, main_tokens=dp1.w.main_tokens, safety_tokens=dp1.w.safety_tokens, max_requests=6)
    cfg, keep = B.make_config(**args1, k_pool=dp1.k_pool, v_pool=dp1.v_pool, workspace=shared)
    dp1b = H.DevicePool(B.Pool(cfg, keep), dp1.k_pool, dp1.v_pool, shared, dp1.w, B.F32)
    off2, _ = H.assign_perfect(dp2, lens2)
    kv2 = [wl.request_kv(w2, 0, r, sharp=True) for r in range(3)]
    H.fill(dp2, 0, kv2, offsets=off2)
    q2 = wl.queries(w2, 0, sharp=True)
    ref2 = H.oracle_out(w2, q2, kv2)
    for _ in range(3):
        H.check(H.decode(dp1b, 0, q1, lens1, offsets=off1), ref1, *TIGHT_F32, what="first pool")
        H.check(H.decode(dp2, 0, q2, lens2, offsets=off2), ref2, *TIGHT_F32, what="second pool")


def test_planning_call_in_a_replayed_graph():
    """A captured call plans on every replay: lengths that grow between replays are honoured."""
    dp, q, lens, off, _ = make([3000, 40, 0, 700], seed=76, main=32768)
    n = len(lens)
    qd, od = H.to_dev(q), H.to_dev(np.asarray(off, np.int64))
    ld = H.to_dev((lens // 2).astype(np.int32))
    out = torch.zeros(n, 4, 128, dtype=torch.float32, device=H.DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        dp.pool.odma_decode_attention(0, n, qd, od, ld, None, 0, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dp.pool.odma_decode_attention(0, n, qd, od, ld, None, 0, out)
    for part in (2, 3, 1):
        now = lens // part
        ld.copy_(H.to_dev(now.astype(np.int32)))
        g.replay()
        torch.cuda.synchronize()
        got = out.cpu().numpy().copy()
        np.testing.assert_array_equal(got, H.decode(dp, 0, q, now, offsets=off))


@pytest.mark.parametrize("wpw", [4, 8])
@pytest.mark.parametrize("lens", [
    [1], [16], [17, 33, 49, 64],                             # fewer tiles than waves: empty parts on the left
    list(range(1, 65)),                                      # 128 segments of one to four tiles
    [300] * 60, [575, 576, 577],                             # near the longest segment that one work-group takes
    [5] * 128, [5] * 129,                                    # as many segments as work-groups, and two more
    [0, 40, 0, 0, 2000, 16],                                 # one long request: equal shares
])
def test_small_batches_cut_at_their_segments_or_not(lens, wpw):
    dp, q, lens, off, ref = make(lens, seed=77, main=65536)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_WG, wpw)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_CU, wpw)         # one work-group per compute unit
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, ref, *TIGHT_F32, what=str(lens[:6]))
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)
