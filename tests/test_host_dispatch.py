"""The host side of the device calls, on a stand-in HIP runtime (no GPU): what a planning call leaves behind when its launch
fails, and the dynamic LDS size when two threads raise it.  Each case runs in a process of its own (tests/fake_runtime.py)."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake_hip")
    (d / "map").write_text("hip_4.2 { global: hip*; __hip*; fake_*; local: *; };\n")
    so = str(d / "libamdhip64.so.7")
    subprocess.run([CXX, "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-Wl,-soname,libamdhip64.so.7",
                    f"-Wl,--version-script={d / 'map'}", os.path.join(ROOT, "tests", "native", "fake_hip.cpp"), "-o", so],
                   check=True, capture_output=True, text=True, timeout=120)
    return so


def run(runtime, code):
    env = dict(os.environ, FAKE_HIP=runtime, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", "from tests.fake_runtime import *\n" + textwrap.dedent(code)], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]


POOLS = [
    ("make_pool()", 5, False),                               # planned in the attention launch
    ("make_pool()", 1500, False),                            # by a launch in front of it
    ("make_pool()", 5, True),                                # static scratch
    ("make_pool(kv_dtype=B.F32)", 5, False),                 # wide format
    ("make_pool(kv_dtype=B.FP8)", 5, False),
]


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("pool,n,static", POOLS)
def test_a_planning_launch_that_failed_left_no_plan(runtime, pool, n, static, first):
    """`first`: the pool's first call fails; otherwise one that replaces the plan of another batch."""
    run(runtime, f"""
        n = {n}
        call = lambda p, m, flags=0: decode(p, m, flags, static={static})
        other = {pool}
        planning = launched(lambda: call(other, n))
        reusing = launched(lambda: call(other, n, B.REUSE_PLAN))
        assert planning != reusing and len(reusing) == 1, (planning, reusing)
        p = {pool}
        if not {first}:
            call(p, n - 1)
        hip.fake_fail_launch(len(planning) - 1)              # the attention launch
        assert fails(lambda: call(p, n))
        assert launched(lambda: call(p, n, B.REUSE_PLAN)) == planning
        assert launched(lambda: call(p, n, B.REUSE_PLAN)) == reusing
    """)


@pytest.mark.parametrize("pool,static", [(p, s) for p, n, s in POOLS if n == 5])
def test_a_planning_call_refused_its_lds_left_no_plan(runtime, pool, static):
    run(runtime, f"""
        call = lambda n, flags=0: decode(p, n, flags, static={static})
        p = {pool}
        call(3)
        hip.fake_fail_attribute(0)
        assert fails(lambda: call(1000))                     # (a longer planning table: more LDS)
        again = launched(lambda: call(1000, B.REUSE_PLAN))
        assert again == launched(lambda: call(1000))
        assert again != launched(lambda: call(1000, B.REUSE_PLAN))
    """)


@pytest.mark.parametrize("pool", ["make_pool(hq=32)", "make_pool(hq=32, kv_dtype=B.F32)", "make_pool(hq=32, kv_dtype=B.FP8)"])
def test_two_threads_raise_the_lds_size(runtime, pool):
    """A call that asked for the smaller size is overtaken by one that asks for a larger: the larger stays allowed."""
    run(runtime, f"""
        import threading, time
        p, p2 = {pool}, {pool}
        hip.fake_hold_first_attribute()
        slow = threading.Thread(target=lambda: decode(p, 300))
        slow.start()
        while hip.fake_attribute_calls() < 1:
            time.sleep(0.001)
        decode(p2, 1000)
        slow.join()
        assert hip.fake_attribute_calls() == 2
        decode(p, 900)
        decode(p2, 1000)
    """)


def test_kernels_that_serve_a_pool(runtime):
    """AUTO: the tile stream, in its wide formats where head_dim or storage ask for them; VALU: the chunked kernel.  A fused
    step is one launch on the tile stream, an append and three launches on the chunked kernel."""
    run(runtime, """
        stream, chunked = ["decode_stream_kernel"], ["plan_kernel", "decode_valu_kernel", "reduce_kernel"]
        names = lambda call: [k for k, *_ in launched(call)]
        formats = [(B.F32, d) for d in range(32, 257, 32)] + [(B.BF16, d) for d in range(32, 257, 32)] + [(B.FP8, 128)]
        for kv, d in formats:
            for paged in (False, True):
                p = make_pool(kv_dtype=kv, head_dim=d)
                assert names(lambda: decode(p, 6, paged=paged)) == stream
                assert names(lambda: step(p, 6, paged=paged)) == stream
                assert names(lambda: step(p, 6, B.REUSE_PLAN, paged=paged)) == stream
                if kv == B.FP8:
                    continue
                p = make_pool(kv_dtype=kv, head_dim=d, decode_kernel=B.KERNEL_VALU)
                assert p.odma_pool_decode_kernel() == B.KERNEL_VALU
                assert names(lambda: decode(p, 6, paged=paged)) == chunked
                assert names(lambda: step(p, 6, paged=paged)) == ["append_kernel"] + chunked
        p = make_pool(kv_dtype=B.F32)
        assert names(lambda: decode(p, 1024)) == stream
        assert names(lambda: decode(p, 1025)) == ["stream_plan_kernel"] + stream
    """)


def test_kernels_that_serve_a_pool_with_a_small_workspace(runtime):
    """max_splits sizes the workspace: the wide formats take as many work-groups as fit, from 16 up, unless the chunked kernel
    has more than 1 + 2 G times their waves there."""
    run(runtime, """
        seen = set()
        for kv, d, hq, hkv in [(B.F32, 64, 4, 2), (B.F32, 128, 28, 4), (B.F32, 128, 8, 8), (B.F32, 128, 32, 32), (B.F32, 256, 16, 8),
                               (B.BF16, 96, 16, 4), (B.BF16, 32, 32, 32), (B.BF16, 32, 16, 1)]:
            served = []
            for max_splits in [1, 8, 24, 32, 40, 56, 72, 100, 136, 200, 264, 400, 520, 700, 1032, 8192]:
                p = make_pool(kv_dtype=kv, head_dim=d, hq=hq, hkv=hkv, max_requests=8, max_splits=max_splits)
                got = launched(lambda: decode(p, 6))
                if got[0][0] == "plan_kernel":
                    assert [k for k, *_ in got] == ["plan_kernel", "decode_valu_kernel", "reduce_kernel"]
                    served.append(0)
                    continue
                assert len(got) == 1
                n_wg = got[0][1][0]
                assert 16 <= n_wg <= 256 and min((8 + max_splits) * hkv, 2048) <= (1 + 2 * hq // hkv) * 4 * n_wg, got
                served.append(n_wg)
            assert served[0] == 0 and served[-2:] == [256, 256], served
            seen.add(tuple(served))
        # many KV heads, one query head each: chunked as long as the workspace is small
        assert any(s[8] == 0 for s in seen) and any(s[3] > 0 for s in seen), seen
    """)


@pytest.mark.parametrize("kv,d", [("BF16", 128), ("BF16", 64), ("FP8", 128), ("F32", 128), ("BF16", 96)])
def test_launches_that_plan_are_kernels_of_their_own(runtime, kv, d):
    """One kernel per (planning, fused, paged); a batch planned by a launch in front runs the one that reuses a plan."""
    run(runtime, f"""
        def kernel(call):
            at = hip.fake_launches()
            call()
            return [hip.fake_name(i) for i in range(at, hip.fake_launches()) if b"decode_stream_kernel" in hip.fake_name(i)]
        p = make_pool(kv_dtype=B.{kv}, head_dim={d})
        seen = {{}}
        for paged in (False, True):
            for f in (decode, step):
                plans, = kernel(lambda: f(p, 9, paged=paged))
                reuses, = kernel(lambda: f(p, 9, B.REUSE_PLAN, paged=paged))
                seen[f, paged, True], seen[f, paged, False] = plans, reuses
                assert kernel(lambda: f(p, 1200, paged=paged)) == [reuses]
        assert len(set(seen.values())) == 8, seen
    """)


def test_prompt_calls_that_may_be_cut(runtime):
    """The variant that cuts items into parts: calls of few items on the null stream, of pools (or block tables) whose requests can
    hold 16 pairs of tiles.  It has a work-group for every part there can be; the others of such calls have all of them."""
    run(runtime, """
        def prompt(p, n=1, rows=16, stream=0, paged=None):
            at = hip.fake_launches()
            p.odma_prefill_attention(0, n, Q, rows, OFFS, NEW, None if paged else OFFS, LENS, TABLE if paged else None, paged or 0, OUT,
                                     stream)
            return [(hip.fake_name(i).decode(), hip.fake_grid(i, 0)) for i in range(at, hip.fake_launches())]

        variant = lambda paged, here, cut: f"prefill_kernelILb{int(paged)}ELi2ELb0ELb{int(here)}ELb{int(cut)}E"
        def check(got, paged, here, cut, grid=512):
            assert len(got) == (1 if here else 2) and variant(paged, here, cut) in got[-1][0] and got[-1][1] == grid, got

        p = make_pool()                                      # requests of up to 4096 tokens: up to 7 parts
        check(prompt(p), False, True, True, 32)              # 2 + 2 items at most, 28 parts
        check(prompt(p, stream=77), False, True, False)
        check(prompt(p, paged=32), True, True, True, 8)      # 512 tokens: 2 parts
        check(prompt(p, paged=31), True, True, False)
        check(prompt(p, paged=1 << 30), True, True, True, 128)
        check(prompt(p, n=200), False, True, True)
        check(prompt(p, n=254), False, True, True)           # 2 items of rows and one a request expected: 256, two parts of each
        check(prompt(p, n=255), False, True, False)
        check(prompt(p, n=300), False, False, False)
        check(prompt(p, rows=1 << 20), False, False, False)
        check(prompt(p, rows=1 << 20, stream=77), False, False, False)
    """)


def test_prompt_calls_that_may_run_eight_waves(runtime):
    """Calls that are long by what the host knows launch a plan that weighs them, the kernel of eight waves and the one of four; the
    others, and those of a pool with a set number of column tiles, a plan that does not and the kernel of four."""
    run(runtime, """
        def prompt(p, n, rows, paged=None):
            at = hip.fake_launches()
            p.odma_prefill_attention(0, n, Q, rows, OFFS, NEW, None if paged else OFFS, LENS, TABLE if paged else None, paged or 0, OUT, 0)
            return [(hip.fake_name(i).decode(), hip.fake_grid(i, 0)) for i in range(at, hip.fake_launches())]

        def check(got, weighed, fp8, paged, ct=2):
            kernel = lambda c, w: f"prefill_kernelILb{int(paged)}ELi{c}ELb{int(fp8)}ELb0ELb0ELi{w}E"
            want = [(f"prefill_plan_kernelILb{int(weighed)}E", 1)] + [(kernel(2, 8), 256)] * weighed + [(kernel(ct, 4), 512 if ct == 2 else 256)]
            assert len(got) == len(want) and all(w in g and x == y for (g, x), (w, y) in zip(got, want)), (got, want)

        # 16 heads: a call of n * m rows has n * m / 4096 items of 256 columns for each of 256 CUs, of at least m / 64 pairs
        for paged in (False, True):
            stride = 256 if paged else None                  # (requests of up to 4096 tokens in both layouts)
            p = make_pool(hq=16)
            check(prompt(p, 16, 16 * 1792, stride), False, False, paged)
            check(prompt(p, 16, 16 * 1811, stride), True, False, paged)          # 200.2 pairs: 16 * 1811^2 / 2^18
            check(prompt(p, 14, 14 * 4096, stride), True, False, paged)
            check(prompt(p, 14, 14 * 4097, stride), False, False, paged)         # rows that the requests cannot all have
            for ct in (2, 4):
                p.odma_pool_tune(B.TUNE_PREFILL_COLUMN_TILES, ct)
                check(prompt(p, 14, 14 * 4096, stride), False, False, paged, ct)
            p = make_pool(kv_dtype=B.FP8, hq=16)
            check(prompt(p, 16, 16 * 404, stride), False, True, paged)
            check(prompt(p, 16, 16 * 405, stride), False, True, paged)           # 10 pairs at least, 202 at most
            check(prompt(p, 32, 32 * 404, stride), True, True, paged)            # 19.9 and 404
            check(prompt(p, 31, 31 * 410, stride), False, True, paged)           # 19.9 and 397
            check(prompt(p, 16, 16 * 1279, stride), True, True, paged)           # 99.8 and 639
            check(prompt(p, 128, 128 * 142, stride), False, True, paged)         # 9.8 and 568
            check(prompt(p, 128, 128 * 144, stride), True, True, paged)          # 10.1 and 576
        # requests of up to 1024 tokens: the most is no more than four times the least
        p = make_pool(kv_dtype=B.FP8, hq=16)
        check(prompt(p, 32, 32 * 800, 64), False, True, True)    # 78 and 200
        check(prompt(p, 32, 32 * 906, 64), True, True, True)     # 100.2
    """)
