"""Decode of fp32 pools and of bf16 pools with a head_dim other than 64 and 128, every head_dim, on the tile-stream kernel
(what ODMA_KERNEL_AUTO takes): attention, fused steps across block boundaries with the rows read back, both layouts, the
largest group, the separate reduction, workspaces too small for it, and the vector-ALU kernel beside it.

Bound: products and sums are fp32 (bf16 products are exact in it) and the weights keep 24 bits, so both kernels stay
within 1e-5 + 1e-5 |oracle|, the bound the suite uses for fp32 pools."""
import numpy as np
import pytest

import workloads as wl
from paper_2512_09427_amd import binding as B
from tests import harness as H
from tests.test_gpu_fp8 import TIGHT_FP8
from tests.test_gpu_parity import TIGHT_F32, small_workload

pytestmark = pytest.mark.gpu

FORMATS = [("f32", d) for d in range(32, 257, 32)] + [("bf16", d) for d in (32, 96, 160, 192, 224, 256)]
TOL = (1e-5, 1e-5)


def make(lens, kvd, d, hq, hkv, extra=0, paged=False, sharp=True, **pool_args):
    lens = np.asarray(lens, np.int64)
    w = small_workload(lens, kv_dtype=kvd, hq=hq, hkv=hkv, d=d, seed=d, bounds=(96, 1024, 4096),
                       main=65536)
    dp = H.make_pool(w, out_dtype=B.F32, **pool_args)
    kv = [wl.request_kv(w, 0, r, n_tokens=int(lens[r]) + extra, sharp=sharp) for r in range(len(lens))]
    held = [(k[:n], v[:n]) for (k, v), n in zip(kv, lens)]
    where = dict(block_table=wl.shuffled_block_table(lens + extra, w.pool_tokens // 16, 16, seed=5)) if paged else \
        dict(offsets=H.assign_perfect(dp, np.maximum(lens + extra, 1))[0])
    H.fill(dp, 0, held, **where)
    return w, dp, lens, kv, held, where


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("kvd,d", FORMATS)
def test_attention(kvd, d, paged):
    w, dp, lens, _, kv, where = make([0, 1, 15, 16, 17, 31, 32, 33, 700, 2500, 48], kvd, d, 14, 2, paged=paged)
    q = wl.queries(w, 0, sharp=True)
    ref = H.oracle_out(w, q, kv)
    ref[lens == 0] = 0.0
    got = H.decode(dp, 0, q, lens, **where)
    H.check(got, ref, *TOL, what=f"{kvd} {d}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, flags=B.REUSE_PLAN, **where), got)
    dp.pool.odma_pool_tune(B.TUNE_FUSE_REDUCE, 0)
    H.check(H.decode(dp, 0, q, lens, **where), ref, *TOL, what=f"{kvd} {d}, separate reduction")


@pytest.mark.parametrize("kvd,d", FORMATS)
def test_fused_steps(kvd, d):
    steps = 18
    lens0 = np.array([0, 1, 14, 15, 16, 30, 31, 600], np.int64)
    for paged in (False, True):
        w, dp, lens, kv, _, where = make(lens0, kvd, d, 3, 1, extra=steps, paged=paged)
        lens = lens.copy()
        for s in range(steps):
            k_new = np.stack([kv[r][0][lens[r]] for r in range(len(lens))])
            v_new = np.stack([kv[r][1][lens[r]] for r in range(len(lens))])
            lens += 1
            q = wl.queries(w, 0, step=s, sharp=True)
            got = H.decode_step(dp, 0, q, k_new, v_new, lens, **where)
            H.check(got, H.oracle_out(w, q, [(k[:n], v[:n]) for (k, v), n in zip(kv, lens)]), *TOL, what=f"{kvd} {d} step {s}")
        for r in (0, 3, 5, 7):
            at = dict(block_row=where["block_table"][r]) if paged else {}
            gk, gv = H.gather(dp, 0, 0 if paged else int(where["offsets"][r]), int(lens[r]), **at)
            np.testing.assert_array_equal(gk, kv[r][0][:lens[r]])
            np.testing.assert_array_equal(gv, kv[r][1][:lens[r]])


@pytest.mark.parametrize("kvd,d", [("f32", 256), ("f32", 64), ("bf16", 256), ("bf16", 32)])
def test_largest_group_and_many_requests(kvd, d):
    rng = np.random.default_rng(d)
    w, dp, lens, _, kv, where = make(rng.integers(0, 90, 200), kvd, d, 16, 1)
    q = wl.queries(w, 0, sharp=True)
    ref = H.oracle_out(w, q, kv)
    ref[lens == 0] = 0.0
    H.check(H.decode(dp, 0, q, lens, **where), ref, *TOL, what=f"{kvd} {d}")


@pytest.mark.parametrize("max_splits", [1, 40, 400, 0])
def test_small_workspaces(max_splits):
    """The workspace is sized by max_splits; whatever kernel it leaves room for must serve the call."""
    w, dp, lens, _, kv, where = make([4000, 3, 900], "f32", 64, 4, 2, max_splits=max_splits)
    q = wl.queries(w, 0, sharp=True)
    dp.workspace.fill_(0xff)
    H.check(H.decode(dp, 0, q, lens, **where), H.oracle_out(w, q, kv), *TOL, what=f"max_splits={max_splits}")


@pytest.mark.parametrize("kvd,d", [("f32", 64), ("f32", 128), ("bf16", 96), ("bf16", 256)])
def test_no_less_exact_than_the_vector_kernel(kvd, d):
    """Scores of standard deviation one, as a model has them: near-uniform softmax over long requests, where the order of
    the sums shows most."""
    errs = []
    for kernel in (B.KERNEL_VALU, B.KERNEL_AUTO):
        w, dp, lens, _, kv, where = make([3000, 777, 64, 2048], kvd, d, 8, 2, decode_kernel=kernel)
        assert dp.pool.odma_pool_decode_kernel() == B.KERNEL_VALU
        q = wl.queries(w, 0, sharp=True)
        ref = H.oracle_out(w, q, kv)
        got = H.decode(dp, 0, q, lens, **where)
        H.check(got, ref, *TOL, what=f"{kvd} {d} kernel {kernel}")
        errs.append(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"{kvd} {d}: relative error vector kernel {errs[0]:.2e}, matrix cores {errs[1]:.2e}")
    assert errs[1] <= 1.2 * errs[0] + 1e-8


@pytest.mark.parametrize("step", [False, True])
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("kernel", [B.KERNEL_AUTO, B.KERNEL_VALU])
@pytest.mark.parametrize("kvd,d", [("f32", 64), ("f32", 160), ("bf16", 96), ("bf16", 128), ("bf16", 256)])
def test_both_kernels_in_both_layouts(kvd, d, kernel, paged, step):
    """The tile stream (AUTO) and the chunked kernel (VALU: a step appends, then attends)."""
    w, dp, lens, kv, held, where = make([1, 15, 16, 17, 700, 2500, 48, 333], kvd, d, 6, 2, extra=1, paged=paged, decode_kernel=kernel)
    tol = TOL if kernel == B.KERNEL_VALU or (kvd, d) != ("bf16", 128) else (2e-5, 2e-4)
    q = wl.queries(w, 0, sharp=True)
    if not step:
        H.check(H.decode(dp, 0, q, lens, **where), H.oracle_out(w, q, held), *tol, what=f"{kvd} {d}")
        return
    k_new, v_new = (np.stack([kv[r][i][lens[r]] for r in range(len(lens))]) for i in (0, 1))
    H.check(H.decode_step(dp, 0, q, k_new, v_new, lens + 1, **where), H.oracle_out(w, q, kv), *tol, what=f"{kvd} {d}")
    for r in range(len(lens)):
        at = dict(block_row=where["block_table"][r]) if paged else {}
        gk, gv = H.gather(dp, 0, 0 if paged else int(where["offsets"][r]), int(lens[r]) + 1, **at)
        np.testing.assert_array_equal(gk, kv[r][0])
        np.testing.assert_array_equal(gv, kv[r][1])


@pytest.mark.parametrize("max_splits", [24, 72, 200, 520])
@pytest.mark.parametrize("hq,hkv", [(8, 1), (8, 8), (16, 4)])
def test_small_workspaces_by_either_kernel(hq, hkv, max_splits):
    """Which kernel a small workspace is served by depends on the heads (tests/test_host_dispatch.py): either serves it, attention
    and fused step, whatever the workspace holds."""
    w, dp, lens, kv, held, where = make([4000, 3, 900], "f32", 64, hq, hkv, extra=1, max_splits=max_splits)
    q = wl.queries(w, 0, sharp=True)
    dp.workspace.fill_(0xff)
    H.check(H.decode(dp, 0, q, lens, **where), H.oracle_out(w, q, held), *TOL, what=f"max_splits={max_splits}")
    k_new, v_new = (np.stack([kv[r][i][lens[r]] for r in range(3)]) for i in (0, 1))
    H.check(H.decode_step(dp, 0, q, k_new, v_new, lens + 1, **where), H.oracle_out(w, q, kv), *TOL, what=f"max_splits={max_splits}")


@pytest.mark.parametrize("lens", [[33], [63, 0, 1], [512], [1000, 24], [250, 260, 16, 1], [2040], [300] * 30])
@pytest.mark.parametrize("kvd,d", [("f32", 32), ("f32", 64), ("f32", 256), ("bf16", 32), ("bf16", 96)])
def test_fewest_tiles_of_a_wave(kvd, d, lens):
    """Batches in which a wave's share lies around the fewest tiles it may get (two, or four with 32 channels)."""
    w, dp, lens, _, kv, where = make(lens, kvd, d, 8, 2)
    q = wl.queries(w, 0, sharp=True)
    ref = H.oracle_out(w, q, kv)
    ref[lens == 0] = 0.0
    got = H.decode(dp, 0, q, lens, **where)
    H.check(got, ref, *TOL, what=f"{kvd} {d} {lens}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, flags=B.REUSE_PLAN, **where), got)


@pytest.mark.parametrize("wpw", [4, 8])
@pytest.mark.parametrize("lens", [[6100, 5900], [2300, 9000, 700, 4100]])
@pytest.mark.parametrize("kvd,d", [("f32", 32), ("f32", 64), ("f32", 160), ("f32", 256), ("bf16", 96), ("bf16", 224), ("bf16", 64), ("bf16", 128),
                                   ("fp8", 128)])
def test_cuts_of_many_parts(kvd, d, lens, wpw):
    """Segments over nine to tens of work-groups and next to each other, so that one work-group may merge the cuts at both of its
    ends: batches of 16 parts and less, one to four heads in the threads of a wave, half of the waves and all of them."""
    lens = np.array(lens)
    for hq, hkv in [(1, 1), (5, 1), (14, 2), (16, 1)]:
        w = small_workload(lens, kv_dtype=kvd, hq=hq, hkv=hkv, d=d, seed=d, bounds=(1024, 4096, 16384), large_cap=16384, main=65536)
        dp = H.make_pool(w, out_dtype=B.F32)
        dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_WG, wpw)
        dp.pool.odma_pool_tune(B.TUNE_MIN_CHUNK, 64)
        kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
        off, _ = H.assign_perfect(dp, lens)
        H.fill(dp, 0, kv, offsets=off)
        q = wl.queries(w, 0, sharp=True)
        got = H.decode(dp, 0, q, lens, offsets=off)
        tol = TIGHT_FP8 if kvd == "fp8" else TOL if kvd == "f32" or d not in (64, 128) else TIGHT_F32
        H.check(got, H.oracle_out(w, q, kv), *tol, what=f"{kvd} {d} {hq}/{hkv}")
        for _ in range(2):                                   # whoever arrives last, the same bits
            np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)


@pytest.mark.parametrize("wpw", [4, 8])
@pytest.mark.parametrize("lens", [[8192], [8193], [16384], [16385], [895] * 32, [897] * 32, [16] * 1030 + [8200], [16] * 200 + [8000],
                                  [3072], [3073], [6144], [6145], [768] * 32, [769] * 32, [16] * 1030 + [3100], [64] * 300, [63] * 300, [128] * 140, [64] * 301,
                                  [32] * 560, [256] * 72, [32] * 1040])
@pytest.mark.parametrize("kvd,d", [("f32", 64), ("bf16", 96)])
def test_fewest_tiles_where_the_rule_changes(kvd, d, lens, wpw):
    """Longest requests of 24, 48 and 64 parts and one tile more, shares of 3 and 3.5 tiles and a little more, requests of one length
    that fill waves of four tiles or do not, planned in the launch and in front of it."""
    lens = np.array(lens)
    w = small_workload(lens, kv_dtype=kvd, hq=4, hkv=2, d=d, seed=d, bounds=(64, 1024, 16400), large_cap=16400, main=1 << 18)
    dp = H.make_pool(w, out_dtype=B.F32)
    dp.pool.odma_pool_tune(B.TUNE_WAVES_PER_WG, wpw)
    kv = [wl.request_kv(w, 0, r, sharp=True) for r in range(len(lens))]
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, kv, offsets=off)
    q = wl.queries(w, 0, sharp=True)
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, H.oracle_out(w, q, kv), *TOL, what=f"{kvd} {d}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)
