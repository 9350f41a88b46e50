"""The library on a stand-in HIP runtime (tests/native/fake_hip.cpp): which kernels a call launches, and what it does when
a launch fails.  Imported in a process of its own (tests/test_host_dispatch.py starts it) before anything that loads the
real runtime; FAKE_HIP names the stand-in's shared object.  No kernel runs and no device address is ever read."""
import ctypes as C
import os
import sys

sys.modules["torch"] = None                      # (the binding loads torch's runtime if it can)
hip = C.CDLL(os.environ["FAKE_HIP"], mode=C.RTLD_GLOBAL)
hip.fake_name.restype = C.c_char_p
hip.fake_lds.restype = C.c_uint64
hip.fake_grid.restype = C.c_uint32

from paper_2512_09427_amd import binding as B  # noqa: E402

Q, OUT, K, V, WS, LENS, OFFS, TABLE, NEW = ((i + 1) << 32 for i in range(9))    # addresses nobody reads


def make_pool(*, kv_dtype=B.BF16, head_dim=128, hq=8, hkv=2, max_requests=4096, **kw):
    args = dict(n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=head_dim, kv_dtype=kv_dtype, out_dtype=B.F32,
                main_tokens=1 << 20, safety_tokens=1 << 12, large_cap=4096, boundaries=[64, 4096], max_requests=max_requests,
                quantiles=[(1, 2), (1, 1)], **kw)
    cfg, keep = B.make_config(**args)
    cfg.workspace_bytes = B.odma_workspace_bytes(cfg)
    cfg.k_pool, cfg.v_pool, cfg.workspace = K, V, WS
    return B.Pool(cfg, keep)


def launched(call):
    """The launches of a call: [(kernel, grid, dynamic LDS bytes)], the kernel as its plain name."""
    at = hip.fake_launches()
    call()
    res = []
    for i in range(at, hip.fake_launches()):
        mangled = hip.fake_name(i).decode()
        name = max((k for k in KERNELS if k in mangled), key=len, default=mangled)
        res.append((name, tuple(hip.fake_grid(i, a) for a in range(3)), hip.fake_lds(i)))
    return res


KERNELS = ["decode_stream_kernel", "stream_plan_kernel", "stream_reduce_kernel", "decode_valu_kernel", "plan_kernel",
           "reduce_kernel", "append_kernel", "append_fp8_kernel", "append_bf16_d128_kernel", "gather_kernel", "prefill_kernel",
           "prefill_plan_kernel"]


def decode(p, n, flags=0, paged=False, static=False, stream=0):
    fn = p.odma_decode_attention_static if static else p.odma_decode_attention
    return fn(0, n, Q, None if paged else OFFS, LENS, TABLE if paged else None, 8 if paged else 0, OUT, flags, stream)


def step(p, n, flags=0, paged=False):
    return p.odma_decode_step(0, n, Q, NEW, NEW, None if paged else OFFS, LENS, TABLE if paged else None, 8 if paged else 0, OUT,
                              flags, 0)


def fails(call):
    try:
        call()
    except B.OdmaError as e:
        assert e.code == B.HIP_ERROR, e
        return True
    return False
