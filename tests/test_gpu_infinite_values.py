"""Infinite scores: K rows that score -inf (what a caller uses to switch tokens off), for whole tiles, whole ranges of a
wave or a work-group, and for some heads of a group only.  The oracle gives these tokens weight 0; the outputs are held
to the bounds of the finite cases, since the tokens that remain are ordinary.  Infinite values: channels in which a V row
is infinite come out infinite, the others as ever."""
import numpy as np
import pytest

import workloads as wl
from paper_2512_09427_amd import binding as B
from tests import harness as H
from tests.test_gpu_parity import small_workload

pytestmark = pytest.mark.gpu

FORMATS = [("f32", 64, B.KERNEL_AUTO), ("f32", 64, B.KERNEL_VALU), ("f32", 256, B.KERNEL_AUTO), ("bf16", 32, B.KERNEL_AUTO),
           ("bf16", 96, B.KERNEL_AUTO), ("bf16", 96, B.KERNEL_VALU), ("bf16", 64, B.KERNEL_AUTO), ("bf16", 128, B.KERNEL_AUTO)]
# lengths, and per request the tokens that are switched off
LENS = [64, 40, 700, 5000, 5000, 33]
OFF = [slice(0, 16), slice(0, 32), slice(0, 650), slice(0, 4400), slice(300, 5000), slice(1, 33)]


def bits(kvd, x):
    x = np.float32(x)
    return x if kvd == "f32" else np.uint16(x.view(np.uint32) >> 16)


def case(kvd, d, kernel, edit, hq=4, hkv=2):
    lens = np.array(LENS)
    w = small_workload(lens, kv_dtype=kvd, hq=hq, hkv=hkv, d=d, seed=d, bounds=(64, 1024, 8192), large_cap=8192, main=1 << 15)
    dp = H.make_pool(w, out_dtype=B.F32, decode_kernel=kernel)
    kv = [wl.request_kv(w, 0, r) for r in range(len(lens))]
    q = wl.queries(w, 0)
    edit(q, kv)
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, kv, offsets=off)
    return w, dp, q, kv, lens, off


def tolerance(kvd, d):
    return (1e-5, 1e-5) if kvd == "f32" or d not in (64, 128) else (2e-5, 2e-4)


@pytest.mark.parametrize("some_heads", [False, True])
@pytest.mark.parametrize("kvd,d,kernel", FORMATS)
def test_tokens_switched_off(kvd, d, kernel, some_heads):
    """K of channel 0 is -inf; or, for some heads, so low that their queries' product overflows while the others' is 0."""
    def edit(q, kv):
        for r, tokens in enumerate(OFF):
            kv[r][0][:, :, 0] = bits(kvd, 0.0)
            kv[r][0][tokens, :, 0] = bits(kvd, -3e38 if some_heads else -np.inf)
        q[:, :, 0] = bits(kvd, 1.0)
        if some_heads:
            q[:, 0::2, 0] = bits(kvd, 1e10)
            q[:, 1::2, 0] = bits(kvd, 0.0)

    w, dp, q, kv, lens, off = case(kvd, d, kernel, edit)
    ref = H.oracle_out(w, q, kv)
    got = H.decode(dp, 0, q, lens, offsets=off)
    H.check(got, ref, *tolerance(kvd, d), what=f"{kvd} {d} kernel {kernel}")
    np.testing.assert_array_equal(H.decode(dp, 0, q, lens, offsets=off, flags=B.REUSE_PLAN), got)
    dp.pool.odma_pool_tune(B.TUNE_FUSE_REDUCE, 0)
    H.check(H.decode(dp, 0, q, lens, offsets=off), ref, *tolerance(kvd, d), what=f"{kvd} {d}, separate reduction")


@pytest.mark.parametrize("kvd,d,kernel", FORMATS)
def test_a_request_without_a_finite_score_touches_no_other(kvd, d, kernel):
    """All tokens of request 2 are off: its softmax has no value, the others keep theirs."""
    def edit(q, kv):
        for r in range(len(LENS)):
            kv[r][0][:, :, 0] = bits(kvd, -np.inf if r == 2 else 0.0)
        q[:, :, 0] = bits(kvd, 1.0)

    w, dp, q, kv, lens, off = case(kvd, d, kernel, edit)
    got = H.decode(dp, 0, q, lens, offsets=off)
    assert np.isnan(got[2]).all()
    keep = [r for r in range(len(LENS)) if r != 2]
    H.check(got[keep], H.oracle_out(w, q, [kv[r] if r != 2 else kv[0] for r in range(len(LENS))])[keep], *tolerance(kvd, d))


def check_with_infinities(got, ref, tol, what):
    inf = np.isinf(ref)
    assert inf.any() and not np.isnan(ref).any()
    np.testing.assert_array_equal(got[inf], ref[inf], err_msg=what)
    H.check(np.where(inf, 0.0, got), np.where(inf, 0.0, ref), *tol, what=what)


@pytest.mark.parametrize("kvd,d,kernel", [("f32", 32, B.KERNEL_AUTO), ("f32", 256, B.KERNEL_AUTO), ("f32", 96, B.KERNEL_VALU)] +
                         [("bf16", d, B.KERNEL_AUTO) for d in (32, 96, 160, 192, 224, 256)] + [("bf16", 96, B.KERNEL_VALU)])
def test_infinite_values(kvd, d, kernel):
    """One token's V is +inf in some channels, another's -inf in others, of ordinary weight, in requests that one wave
    finishes and that several do; also a weight of exactly 1 (request 5 holds one token)."""
    lens = np.array([1 if r == 5 else n for r, n in enumerate(LENS)])
    w = small_workload(lens, kv_dtype=kvd, hq=4, hkv=2, d=d, seed=d, bounds=(64, 1024, 8192), large_cap=8192, main=1 << 15)
    dp = H.make_pool(w, out_dtype=B.F32, decode_kernel=kernel)
    kv = [wl.request_kv(w, 0, r) for r in range(len(lens))]
    for r, n in enumerate(lens):
        kv[r][1][n // 2, :, 3::7] = bits(kvd, np.inf)
        if n > 1:
            kv[r][1][n - 1, :, 5::7] = bits(kvd, -np.inf)
    q = wl.queries(w, 0)
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, kv, offsets=off)
    check_with_infinities(H.decode(dp, 0, q, lens, offsets=off), H.oracle_out(w, q, kv), tolerance(kvd, d), f"{kvd} {d} kernel {kernel}")


@pytest.mark.parametrize("grow", [False, True])
@pytest.mark.parametrize("paged", [False, True])
def test_infinite_values_of_a_prompt_with_an_odd_number_of_tiles(paged, grow):
    """The last query sees the infinite V of its own token; the tile after the last one does not exist.  With `grow` the
    scores outgrow the first pair's reference, so the columns are repeated."""
    lens, n_q = np.array([48, 20, 5, 16, 300]), np.array([48, 4, 5, 1, 20])
    w = small_workload(lens, hq=7, hkv=1, seed=6)
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r) for r in range(len(lens))]
    rng = np.random.default_rng(6)
    q, _ = wl.draw_values(rng, (int(n_q.sum()), 7, 128), w.data_scale, "bf16")
    q[:, :, 0] = bits("bf16", 1.0)
    for r, n in enumerate(lens):
        kv[r][0][:, :, 0] = bits("bf16", 0.0)
        if grow:
            kv[r][0][-1, :, 0] = bits("bf16", 2048.0)
        kv[r][1][-1, :, 3::7] = bits("bf16", np.inf)
    where = dict(block_table=wl.shuffled_block_table(lens, w.pool_tokens // 16, 16, seed=5)) if paged else \
        dict(offsets=H.assign_perfect(dp, lens)[0])
    H.fill(dp, 0, kv, **where)
    q_start = np.concatenate([[0], np.cumsum(n_q)[:-1]])
    got = H.prefill(dp, 0, q, q_start, n_q, lens, **where)
    for r, n in enumerate(lens):
        last = q_start[r] + n_q[r] - 1
        ref = H.oracle_out(w, q[last:last + 1], [kv[r]])
        # (the weights of a prompt are bf16: 2^-8 of the values they average)
        check_with_infinities(got[last:last + 1], ref, (2.0 ** -8 * w.data_scale * 4, 2e-2), f"request {r}")


@pytest.mark.parametrize("score", [-300.0, -3.0, 200.0])
def test_prompt_whose_first_tokens_are_switched_off(score):
    """The first pair of tiles, and more, scores -inf; what follows lies far below, near and far above zero."""
    lens, n_q, off = np.array([64, 200, 333]), np.array([20, 1, 200]), np.array([40, 64, 100])
    w = small_workload(lens, hq=7, hkv=1, seed=8)
    dp = H.make_pool(w, out_dtype=B.F32)
    kv = [wl.request_kv(w, 0, r) for r in range(len(lens))]
    q, _ = wl.draw_values(np.random.default_rng(8), (int(n_q.sum()), 7, 128), w.data_scale, "bf16")
    q[:, :, 0] = bits("bf16", 1.0)
    for r in range(len(lens)):
        kv[r][0][:, :, 0] = bits("bf16", score * np.log(2.0) * np.sqrt(128.0))
        kv[r][0][:off[r], :, 0] = bits("bf16", -np.inf)
    where = dict(offsets=H.assign_perfect(dp, lens)[0])
    H.fill(dp, 0, kv, **where)
    q_start = np.concatenate([[0], np.cumsum(n_q)[:-1]])
    got = H.prefill(dp, 0, q, q_start, n_q, lens, **where)
    for r, n in enumerate(lens):
        for j in range(max(0, int(off[r] - (n - n_q[r]))), n_q[r]):       # queries that see a token that is on
            seen = int(n - n_q[r] + j + 1)
            ref = H.oracle_out(w, q[q_start[r] + j:q_start[r] + j + 1], [(kv[r][0][:seen], kv[r][1][:seen])])
            # (the weights of a prompt are bf16: 2^-8 of the values they average)
            H.check(got[q_start[r] + j:q_start[r] + j + 1], ref, 2.0 ** -8 * w.data_scale * 4, 2e-2, what=f"request {r} query {j}")


@pytest.mark.parametrize("size", [1e-37, 1e37])
@pytest.mark.parametrize("kvd,d,kernel", [("f32", 64, B.KERNEL_AUTO), ("f32", 128, B.KERNEL_AUTO), ("f32", 64, B.KERNEL_VALU),
                                          ("bf16", 32, B.KERNEL_AUTO), ("bf16", 96, B.KERNEL_AUTO), ("bf16", 256, B.KERNEL_AUTO)])
def test_values_near_the_ends_of_the_range(kvd, d, kernel, size):
    """Values of 1e37 and 1e-37: the weights that multiply them are at most 1, the largest of a request is 1.  (Few tokens of
    like weight, so that their sum stays in range.)"""
    lens = np.array([1, 2, 17, 40, 300])
    w = small_workload(lens, kv_dtype=kvd, hq=4, hkv=2, d=d, seed=d, bounds=(64, 1024), large_cap=1024, main=1 << 13)
    dp = H.make_pool(w, out_dtype=B.F32, decode_kernel=kernel)
    kv = []
    for r in range(len(lens)):
        k, _ = wl.request_kv(w, 0, r, sharp=True)
        v, _ = wl.draw_values(np.random.default_rng([7, r]), k.shape, size, kvd)
        kv.append((k, v))
    q, _ = wl.draw_values(np.random.default_rng(7), (len(lens), 4, d), 4.0, kvd)
    off, _ = H.assign_perfect(dp, lens)
    H.fill(dp, 0, kv, offsets=off)
    got = H.decode(dp, 0, q, lens, offsets=off)
    assert np.isfinite(got).all()
    # (values of 1e-37 sit at the bottom of the normal range, where sums lose up to eight bits)
    tol = (1e-5, 1e-5) if size > 1 else (1e-4, 1e-4)
    H.check(got.astype(np.float64) / size, H.oracle_out(w, q, kv) / size, *tol, what=f"{kvd} {d}")


# One request of 32 pairs of tiles, cut behind pairs 10 and 21: per case its scores, as (first token, token behind the last,
# score), later entries over earlier ones, and the tokens whose V is infinite.
PARTS = {
    # the middle part begins with tokens that are switched off and goes on far below zero (2^-59.5 in all); one token of the
    # first part holds a tenth of that, 89 powers of two above those it began with
    "low behind tokens that are off": ([(0, 320, -152), (100, 101, -62.7), (320, 352, -np.inf), (352, 672, -67.8), (672, 1024, -np.inf)], []),
    "a part that is off": ([(320, 672, -np.inf)], []),
    "all but the last part off": ([(0, 700, -np.inf)], []),
    "infinite values of ordinary weight": ([], [40, 500, 1000]),
    # 2^-90 of the weight that the sums began with, 2^-140 of the largest
    "an infinite value of little weight": ([(320, 672, -100), (500, 501, -90), (672, 1024, 50)], [500]),
}


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("name", list(PARTS))
def test_prompt_whose_keys_are_cut_into_parts(name, paged):
    scores, infinite = PARTS[name]
    n, n_q = 1024, 4
    w = small_workload([n], hq=7, hkv=1, seed=9, main=1 << 14)
    dp = H.make_pool(w, out_dtype=B.F32)
    k, v = wl.request_kv(w, 0, 0)
    q = np.zeros((n_q, 7, 128), np.uint16)                     # (scores as they are given, nothing beside them)
    q[:, :, 0] = bits("bf16", 1.0)
    k[:, :, 0] = bits("bf16", 0.0)
    for a, b, score in scores:
        k[a:b, :, 0] = bits("bf16", score * np.log(2.0) * np.sqrt(128.0))
    v[infinite, :, 3::7] = bits("bf16", np.inf)
    where = dict(block_table=wl.shuffled_block_table([n], w.pool_tokens // 16, 16, seed=5)) if paged else \
        dict(offsets=H.assign_perfect(dp, np.array([n]))[0])
    H.fill(dp, 0, [(k, v)], **where)
    got = H.prefill(dp, 0, q, np.array([0]), np.array([n_q]), np.array([n]), **where)
    for j in range(n_q):
        seen = n - n_q + j + 1
        ref = H.oracle_out(w, q[j:j + 1], [(k[:seen], v[:seen])])
        # (the weights of a prompt are bf16: 2^-8 of the values they average)
        tol = (2.0 ** -8 * w.data_scale * 4, 2e-2)
        if infinite:
            check_with_infinities(got[j:j + 1], ref, tol, f"{name}, query {j}")
        else:
            H.check(got[j:j + 1], ref, *tol, what=f"{name}, query {j}")
