"""The C-ABI library without a GPU: it loads, exports every symbol the header declares, and rejects bad
arguments on the host before anything is launched (these calls never reach a kernel)."""
import ctypes
import re
from pathlib import Path

import numpy as np
import pytest

from paper_2506_19830_amd import binding as B

ROOT = Path(__file__).resolve().parent.parent


def good_desc(**kw):
    d = dict(num_requests=1, num_q_heads=40, num_kv_heads=8, head_dim=128, gamma=8, branch_len=64, block_size=16,
             max_blocks_per_request=2048, q_dtype="bf16", kv_dtype="fp8_e4m3", branch_kv_dtype="fp8_e4m3",
             out_dtype="bf16", softmax_scale=128 ** -0.5)
    d.update(kw)
    return B.make_attn_desc(**d)


def _declared(header_name):
    header = (ROOT / "include" / header_name).read_text()
    return set(re.findall(r"LA_API[^;(]*?\b(la_\w+)\s*\(", header))


def _exported(path):
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", str(path)], capture_output=True, text=True, check=True).stdout
    return {line.split()[-1] for line in out.splitlines() if " T " in line}


def test_library_exports_every_declared_symbol():
    """The product library exports exactly what la_verify.h declares; the benchmark library that and the aids of
    la_verify_bench.h; neither exports anything else."""
    declared = _declared("la_verify.h")
    aids = _declared("la_verify_bench.h")
    assert declared == set(B.EXPORTED_SYMBOLS) and aids == set(B.BENCH_SYMBOLS)
    lib, bench = B.load("product"), B.load("bench")
    for name in declared:
        assert hasattr(lib, name) and hasattr(bench, name), name
    for name in aids:
        assert hasattr(bench, name) and not hasattr(lib, name), name
    assert _exported(B.LIB_PATH) == declared
    assert _exported(B.BENCH_LIB_PATH) == declared | aids


def test_struct_layouts_match_the_header():
    assert ctypes.sizeof(B.la_attn_desc) == 15 * 4
    assert ctypes.sizeof(B.la_attn_plan) == 7 * 4
    assert ctypes.sizeof(B.la_accept_desc) == 7 * 4
    assert ctypes.sizeof(B.la_layer_strides) == 8 + 4 * 8        # int32 padded to the int64 that follows


def test_status_strings():
    assert B.status_string(0) == "ok"
    assert "workspace" in B.status_string(3)
    assert B.status_string(99) == "unknown status"


def test_workspace_query_and_plan():
    ws = B.la_verify_attention_workspace(good_desc(), [32768])
    rows = 8 * 64 * 40
    assert ws > 0 and ws % (rows * 130 * 4) < 512          # whole partial slots (O[128] + m + l per row)
    assert B.la_verify_attention_workspace(good_desc(kv_split_tokens=32768), [32768]) < ws
    f32 = good_desc(q_dtype="f32", kv_dtype="f32", branch_kv_dtype="f32", out_dtype="f32", head_dim=64)
    assert B.la_verify_attention_workspace(f32, [32768]) == 0
    acc = B.make_accept_desc(num_branches=8, num_draft=8, vocab=152064, logits_dtype="bf16")
    assert B.la_spec_accept_workspace(acc) > 8 * 17 * 19 * 8


def test_planner_deals_unequal_requests_as_the_hardware_does():
    """Configuration 4's batch: four requests of 8K..32K keys on a bf16 cache, 3072 rows per KV head.  One chunk per
    request and chunks of a quarter of the longest need the same number of rounds x longest-chunk steps; dealt out in
    launch order the first leaves the chip half empty while the longest request runs (measured 1.17 against 1.04 ms).
    The plan must be the balanced one; a single request keeps the plan that rounds x longest gives."""
    kw = dict(num_requests=4, num_q_heads=64, num_kv_heads=8, gamma=8, branch_len=48, kv_dtype="bf16",
              branch_kv_dtype="bf16", max_blocks_per_request=2060)
    plan = B.la_verify_attention_plan(good_desc(**kw), [8192, 16384, 24576, 32768])
    assert plan["chunk_tokens"] == 8192 and plan["chunks_total"] == 10
    one = B.la_verify_attention_plan(good_desc(), [32768])
    assert one["kernel_shape"] == 1 and one["chunk_tokens"] == 10944 and one["workgroups"] == 240
    # every la_verify_attention call plans on the host before it enqueues anything: the plan must stay cheap
    import time
    few_rows = good_desc(num_requests=4, branch_len=4, max_blocks_per_request=2060)
    t0 = time.perf_counter()
    for _ in range(50):
        B.la_verify_attention_plan(few_rows, [8192, 16384, 24576, 32768])
    assert (time.perf_counter() - t0) / 50 < 5e-4          # observed 13 us; an allocating version of the model took 3 ms


def _plan_status(desc, lens, chain_len=0):
    try:
        return 0, B.la_verify_attention_plan(desc, lens, chain_len)
    except B.LaError as e:
        return e.status, None


def test_split_that_only_the_row_tiles_hold():
    """The streaming shapes keep 2048 block ids of a chunk, the row tiles 4096: a bf16 call that asks for a chunk length
    between the two runs on the row tiles, whatever its prefixes are."""
    bf16 = dict(kv_dtype="bf16", branch_kv_dtype="bf16", num_q_heads=64, branch_len=48, max_blocks_per_request=4096)
    for block, split, streams in ((16, 32448, True), (16, 32512, False), (16, 65024, False), (32, 65536, False)):
        desc = good_desc(**bf16, block_size=block, kv_split_tokens=split)
        for lens in ([100], [32000]):
            plan = B.la_verify_attention_plan(desc, lens)
            assert (plan["kernel_shape"] >= 3) == streams
            assert B.la_verify_attention_workspace(desc, lens) > 0


@pytest.mark.parametrize("kw,lens,shape", [
    (dict(gamma=6, branch_len=9), [20011], 3),                                                      # fp8, few rows
    (dict(gamma=15, branch_len=9, kv_dtype="bf16", branch_kv_dtype="bf16"), [12345], 6),
    (dict(kv_dtype="fp8_e4m3", branch_kv_dtype="bf16"), [900], 1),
])
def test_what_the_plan_of_a_nested_call_names_can_be_forced(kw, lens, shape):
    """The shape la_verify_attention_plan reports, given back as kernel_shape, is the same plan again, for flat calls and
    for calls with a chain, and the call itself gets as far as its workspace."""
    plan = B.la_verify_attention_plan(good_desc(**kw), lens, 135)
    assert plan["kernel_shape"] == shape
    pinned = good_desc(**kw, kernel_shape=shape)
    assert B.la_verify_attention_plan(pinned, lens, 135) == plan == B.la_verify_attention_plan(pinned, lens, 0)
    assert B.la_verify_attention_workspace(pinned, lens) == B.la_verify_attention_workspace(good_desc(**kw), lens)
    vp, vis = ctypes.c_void_p, (ctypes.c_int32 * pinned.gamma)()
    call = lambda desc: B.load().la_verify_attention_nested(
        ctypes.byref(desc), vp(256), vp(256), vp(256), vp(0), vp(256), (ctypes.c_int32 * 1)(*lens), vp(256), vp(256), vp(256),
        vp(256), ctypes.c_int32(135), vp(256), vis, vp(0), vp(0), vp(256), vp(0), vp(256), ctypes.c_size_t(1024), vp(0))
    assert call(pinned) == 3
    wrong = 6 if kw.get("kv_dtype") != "bf16" else 3                    # the other storage type's shape
    assert call(good_desc(**kw, kernel_shape=wrong)) == 2


def test_plans_of_several_short_requests_stay_cheap():
    """Dealing the workgroups of several requests out costs host time per candidate plan; candidates that cannot win are
    left out by a bound.  Eight requests of 1500 keys: 50 us per plan without it, 6 with it; one of them alone 4 us."""
    import time

    def plan_time(n):
        desc = good_desc(num_requests=n, gamma=1, branch_len=1)
        lens, out, lib = (ctypes.c_int32 * n)(*[1250 + 50 * (i % 8) for i in range(n)]), B.la_attn_plan(), B.load()
        best = 1.0
        for _ in range(10):
            t0 = time.perf_counter()
            for _ in range(100):
                lib.la_verify_attention_plan(ctypes.byref(desc), lens, 60, ctypes.byref(out))
            best = min(best, (time.perf_counter() - t0) / 100)
        return best

    assert plan_time(8) < 5 * plan_time(1)


def test_plan_of_the_general_path():
    """What the general kernel would launch (head dimensions 64 and 256, fp32), as with the workspace of the query."""
    kw = dict(num_q_heads=64, num_kv_heads=8, head_dim=64, gamma=4, branch_len=16, kv_dtype="bf16", branch_kv_dtype="bf16")
    plan = B.la_verify_attention_plan(good_desc(**kw), [8190])
    assert plan["path"] == 1 and plan["kernel_shape"] == 0
    assert plan["rows_per_workgroup"] == 32 and plan["row_tiles"] == 16             # 512 rows per KV head
    n = -(-8190 // plan["chunk_tokens"])
    assert n > 1 and plan["chunks_total"] == n and plan["workgroups"] == 8 * 16 * n
    rows = 4 * 16 * 64
    assert B.la_verify_attention_workspace(good_desc(**kw), [8190]) == n * rows * (64 + 2) * 4
    assert B.la_verify_attention_plan(good_desc(**kw), [8190], 40) == plan
    short = B.la_verify_attention_plan(good_desc(**kw, num_requests=2), [100, 0])
    assert short["chunk_tokens"] == 0 and short["chunks_total"] == 2 and short["workgroups"] == 2 * 8 * 16
    split = B.la_verify_attention_plan(good_desc(**kw, num_requests=2, kv_split_tokens=64), [100, 0])
    assert split["chunk_tokens"] == 64 and split["chunks_total"] == 3
    f32 = dict(q_dtype="f32", kv_dtype="f32", branch_kv_dtype="f32", out_dtype="f32", num_q_heads=4, num_kv_heads=2)
    plan = B.la_verify_attention_plan(good_desc(**f32, gamma=2, branch_len=9), [256])
    assert plan == dict(path=1, kernel_shape=0, rows_per_workgroup=16, row_tiles=3, chunk_tokens=0, chunks_total=1,
                        workgroups=6)


@pytest.mark.parametrize("seed", range(8))
def test_the_planner_refuses_only_what_no_shape_runs(seed):
    """Left to itself the library runs a call exactly where some kernel shape, forced, runs it (random descriptors)."""
    import random
    rng = random.Random(seed)
    seen = set()
    for _ in range(250):
        kv, br = rng.choice((("bf16", "bf16"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "bf16")))
        hkv = rng.choice((1, 2, 8, 64))
        block = 1 << rng.randint(4, 18)
        n_req = rng.randint(1, 10)
        blocks = rng.randint(1, 4096)
        lens = [int(min(blocks * block, 400000) * rng.random() ** 3) for _ in range(n_req)]
        if blocks * block > 1 << 30:
            continue
        kw = dict(num_requests=n_req, num_kv_heads=hkv, num_q_heads=hkv * rng.choice((1, 5, 8)), gamma=rng.randint(1, 16),
                  branch_len=rng.choice((1, 9, 64, 700, 30000)), block_size=block, max_blocks_per_request=blocks,
                  kv_dtype=kv, branch_kv_dtype=br, kv_split_tokens=64 * rng.choice((0, 0, 1, 100, 500, 520, 900, 1024, 3000)))
        if kw["gamma"] * kw["branch_len"] * kw["num_q_heads"] * n_req > 1 << 30:
            continue
        status, plan = _plan_status(good_desc(**kw), lens)
        forced = [_plan_status(good_desc(**kw, kernel_shape=k), lens)[0] for k in range(1, 8)]
        assert status == (0 if 0 in forced else 2), (kw, lens, forced)
        assert status or forced[plan["kernel_shape"] - 1] == 0
        seen.add(status)
    assert seen == {0, 2}


@pytest.mark.parametrize("kw,lens,status", [
    (dict(num_q_heads=41), [100], 1),
    (dict(block_size=8), [100], 1),
    (dict(softmax_scale=0.0), [100], 1),
    (dict(kv_split_tokens=100), [100], 1),
    (dict(gamma=0), [100], 1),
    (dict(), [-1], 1),
    (dict(max_blocks_per_request=4), [65], 1),
    (dict(head_dim=96), [100], 2),
    (dict(head_dim=64, kernel_shape=1), [100], 2),
    (dict(q_dtype="f32"), [100], 2),
    (dict(kv_dtype="bf16", branch_kv_dtype="fp8_e4m3"), [100], 2),
    (dict(out_dtype="fp8_e4m3"), [100], 2),
])
def test_attention_rejects_bad_descriptors(kw, lens, status):
    with pytest.raises(B.LaError) as e:
        B.la_verify_attention_workspace(good_desc(**kw), lens)
    assert e.value.status == status


def _call_attention(desc, lens, ptrs, ws_bytes):
    lib = B.load()
    arr = (ctypes.c_int32 * len(lens))(*lens)
    vp = ctypes.c_void_p
    return lib.la_verify_attention(ctypes.byref(desc), vp(ptrs.get("q", 256)), vp(ptrs.get("k", 256)),
                                   vp(ptrs.get("v", 256)), vp(0), vp(ptrs.get("lens", 256)), arr,
                                   vp(ptrs.get("kb", 256)), vp(ptrs.get("vb", 256)), vp(0), vp(0),
                                   vp(ptrs.get("out", 256)), vp(0), vp(ptrs.get("ws", 256)),
                                   ctypes.c_size_t(ws_bytes), vp(0))


def test_attention_call_rejects_before_launch():
    """Fake (never dereferenced) device addresses: each call must fail validation on the host."""
    d = good_desc()
    assert _call_attention(d, [32768], {"q": 0}, 1 << 40) == 1           # required pointer missing
    assert _call_attention(d, [32768], {"k": 0}, 1 << 40) == 1           # prefix present but no cache
    assert _call_attention(d, [32768], {"out": 264}, 1 << 40) == 1       # not 16-byte aligned
    assert _call_attention(d, [32768], {}, 1024) == 3                    # workspace too small
    assert _call_attention(d, [32768], {"ws": 0}, 0) == 3


def test_nested_attention_call_rejects_before_launch():
    """Chain arguments are validated on the host: length, pointers, alignment, visibility within 0..C."""
    lib = B.load()
    d = good_desc()
    vp = ctypes.c_void_p
    lens = (ctypes.c_int32 * 1)(32768)
    n_vis = d.num_requests * d.gamma

    def call(chain_len, k_chain=256, v_chain=256, vis_dev=256, vis=None, vis_host_null=False, ws_bytes=1024):
        vis_arr = (ctypes.c_int32 * n_vis)(*(vis if vis is not None else [0] * n_vis))
        host = ctypes.POINTER(ctypes.c_int32)() if vis_host_null else vis_arr
        return lib.la_verify_attention_nested(ctypes.byref(d), vp(256), vp(256), vp(256), vp(0), vp(256), lens,
                                              vp(256), vp(256), vp(k_chain), vp(v_chain), ctypes.c_int32(chain_len),
                                              vp(vis_dev), host, vp(0), vp(0), vp(256), vp(0), vp(256),
                                              ctypes.c_size_t(ws_bytes), vp(0))

    assert call(-1) == 1
    assert call(4, k_chain=0) == 1
    assert call(4, v_chain=264) == 1                       # not 16-byte aligned
    assert call(4, vis_dev=0) == 1
    assert call(4, vis_host_null=True) == 1
    assert call(4, vis=[0] * (n_vis - 1) + [5]) == 1       # sees more than the chain holds
    assert call(4, vis=[-1] + [0] * (n_vis - 1)) == 1
    # valid chain arguments get as far as the workspace check (nothing is launched: the workspace is too small)
    assert call(4, vis=[4] * n_vis) == 3
    assert call(0, k_chain=0, v_chain=0, vis_dev=0, vis_host_null=True) == 3


def test_kv_commit_rejects_before_launch():
    lib = B.load()
    vp = ctypes.c_void_p
    lens = (ctypes.c_int32 * 1)(32768)

    def call(desc, chain_len=8, strides=None, **ptrs):
        g = lambda k, dflt=256: vp(ptrs.get(k, dflt))
        return lib.la_kv_commit(ctypes.byref(desc), g("kc"), g("vc"), vp(0), g("lens"), lens, g("kb"), g("vb"),
                                g("kch"), g("vch"), ctypes.c_int32(chain_len), g("src"), g("nch"), g("nown"), vp(0),
                                vp(0), g("new", 512), ctypes.byref(strides) if strides is not None else None, vp(0))

    roomy = good_desc(max_blocks_per_request=2048 + 8)           # 32768 + 128 positions
    assert call(good_desc()) == 1                                # table maps exactly the prefix: no room
    assert call(roomy, kc=0) == 1
    assert call(roomy, kch=0) == 1                               # chain_len 8 without a chain
    assert call(roomy, chain_len=-1) == 1
    assert call(roomy, kb=264) == 1                              # not 16-byte aligned
    assert call(roomy, new=256, lens=256) == 1                   # new lengths alias the old ones
    assert call(good_desc(max_blocks_per_request=2048 + 8, kv_dtype="bf16", branch_kv_dtype="bf16",
                          head_dim=100)) == 2
    assert call(good_desc(max_blocks_per_request=2048 + 8, q_dtype="f32", kv_dtype="f32",
                          branch_kv_dtype="bf16", out_dtype="f32")) == 2   # no such conversion
    bad = B.la_layer_strides(num_layers=0)
    assert call(roomy, strides=bad) == 1
    odd = B.la_layer_strides(num_layers=2, cache_stride=1 << 20, branch_stride=7, chain_stride=1 << 10)
    assert call(roomy, strides=odd) == 1                         # layer 1 of the branch tensors would be unaligned


def test_kv_commit_tree_rejects_before_launch():
    lib = B.load()
    vp = ctypes.c_void_p
    lens = (ctypes.c_int32 * 1)(32768)

    def call(desc, pool_len=8, **ptrs):
        g = lambda k, dflt=256: vp(ptrs.get(k, dflt))
        return lib.la_kv_commit_tree(ctypes.byref(desc), g("kc"), g("vc"), vp(0), g("lens"), lens, g("kb"), g("vb"),
                                     g("kp"), g("vp"), ctypes.c_int32(pool_len), g("seg"), g("mask"), g("src"),
                                     g("nown"), vp(0), vp(0), g("new", 512), None, vp(0))

    roomy = good_desc(max_blocks_per_request=2048 + 8)
    assert call(good_desc()) == 1                                # no room behind the prefix
    assert call(roomy, mask=0) == 1
    assert call(roomy, mask=260) == 1                            # 64-bit masks on a 4-byte boundary
    assert call(roomy, seg=0) == 1                               # a pool without node labels
    assert call(roomy, kp=0) == 1
    assert call(roomy, pool_len=-1) == 1
    assert call(roomy, src=0) == 1
    assert call(roomy, new=256, lens=256) == 1


def test_accept_rejects_bad_arguments():
    for kw, status in [(dict(num_branches=0), 1), (dict(num_draft=0), 1), (dict(vocab=0), 1),
                       (dict(temperature=0.0), 1), (dict(logits_dtype="fp8_e4m3"), 2),
                       (dict(num_branches=40000, num_draft=8), 2), (dict(top_k=-1), 1), (dict(top_p=0.0), 1),
                       (dict(top_p=1.5), 1)]:
        base = dict(num_branches=8, num_draft=8, vocab=152064, logits_dtype="bf16")
        base.update(kw)
        with pytest.raises(B.LaError) as e:
            B.la_spec_accept_workspace(B.make_accept_desc(**base))
        assert e.value.status == status
    lib = B.load()
    d = B.make_accept_desc(num_branches=8, num_draft=8, vocab=152064, logits_dtype="bf16")
    vp = ctypes.c_void_p
    args = [vp(256)] * 7 + [vp(0)]
    assert lib.la_spec_accept(ctypes.byref(d), *args, vp(256), ctypes.c_size_t(16), vp(0)) == 3
    args[0] = vp(0)
    assert lib.la_spec_accept(ctypes.byref(d), *args, vp(256), ctypes.c_size_t(1 << 30), vp(0)) == 1


@pytest.mark.parametrize("make", [
    lambda rows: rows, lambda rows: tuple(map(tuple, rows)), lambda rows: (r for r in rows),
    lambda rows: (iter(r) for r in rows), lambda rows: (map(float, r) for r in rows),
    lambda rows: iter([rows[0], iter(map(float, rows[1])), tuple(rows[2])]),
    lambda rows: iter([rows[0], iter([rows[1][0], float(rows[1][1]), rows[1][2]]), rows[2]]),
])
def test_host_rows_takes_what_iterates_once(make):
    """Labels and visible lengths on the host: any nesting of iterables of numbers, also ones that can be walked once
    only and whose later rows are not plain ints; what does not fit 32 bits wraps as a C conversion does."""
    rows = [[1, 2, 3], [4, 5, 6], [7, 8, 9]]
    assert list(B._host_rows(make(rows))) == list(range(1, 10))


def test_host_rows_odd_values():
    import numpy as np
    import torch
    assert list(B._host_rows(np.arange(6, dtype=np.int64).reshape(2, 3))) == list(range(6))
    assert list(B._host_rows(torch.arange(6).reshape(2, 3))) == list(range(6))
    assert list(B._host_rows([[2 ** 32 + 5, -1], [2 ** 31]])) == [5, -1, -2 ** 31]
    assert list(B._host_rows([])) == [0] == list(B._host_rows([[], []]))


def test_product_package_does_not_import_the_oracle():
    for f in (ROOT / "paper_2506_19830_amd").rglob("*"):
        if f.suffix in (".py", ".hip", ".hpp", ".h", ".cpp"):
            text = f.read_text()
            assert "import oracle" not in text and "from oracle" not in text and "la_oracle" not in text, f


@pytest.mark.parametrize("lens,gamma,L,hq,hkv,kv,shape,chunk,total", [
    ((5120,), 1, 4, 16, 4, "fp8_e4m3", 3, 192, 27),
    ((6531,), 1, 4, 16, 4, "bf16", 7, 192, 35),
    ((131072,), 1, 1, 8, 8, "bf16", 7, 4096, 32),
    ((1,), 1, 1, 8, 8, "bf16", 7, 64, 1),
    ((577, 576), 8, 64, 40, 8, "bf16", 6, 640, 2),
    ((3553, 1018, 7148), 1, 5, 40, 8, "fp8_e4m3", 3, 448, 27),
    ((2476, 1833), 1, 74, 40, 8, "fp8_e4m3", 4, 512, 9),
    ((375, 856, 5016, 843, 2495, 420), 3, 8, 16, 4, "fp8_e4m3", 3, 448, 24),
    ((700, 64, 0, 9000), 8, 48, 64, 8, "bf16", 6, 1856, 8),
    ((24576, 8192, 16384), 6, 64, 40, 8, "fp8_e4m3", 1, 4096, 12),
])
def test_pinned_plans(lens, gamma, L, hq, hkv, kv, shape, chunk, total):
    """What the planner's model takes to be the cheapest (which need not be what measures fastest)."""
    desc = good_desc(num_requests=len(lens), num_q_heads=hq, num_kv_heads=hkv, gamma=gamma, branch_len=L, block_size=16,
                     max_blocks_per_request=(max(lens) + 15) // 16, kv_dtype=kv, branch_kv_dtype=kv)
    plan = B.la_verify_attention_plan(desc, list(lens))
    assert (plan["kernel_shape"], plan["chunk_tokens"], plan["chunks_total"]) == (shape, chunk, total)


@pytest.mark.parametrize("lens,gamma,L,hq,hkv", [
    ((822,), 1, 6, 32, 8), ((1,), 1, 1, 8, 8), ((28431, 307), 8, 1, 16, 2), ((2585,), 1, 64, 2, 2),
])
def test_fp8_calls_of_one_64_row_tile(lens, gamma, L, hq, hkv):
    """At most 64 rows per KV head run on the streaming shape of 64 rows; with a chunk length asked for on no wider
    streaming shape; a forced shape is taken as before."""
    kw = dict(num_requests=len(lens), num_q_heads=hq, num_kv_heads=hkv, gamma=gamma, branch_len=L, block_size=16,
              max_blocks_per_request=(max(lens) + 15) // 16, kv_dtype="fp8_e4m3", branch_kv_dtype="fp8_e4m3")
    shape = lambda **k: B.la_verify_attention_plan(good_desc(**kw, **k), list(lens))["kernel_shape"]
    assert shape() == 3 and shape(kernel_shape=4) == 4
    assert shape(kv_split_tokens=64) not in (4, 5)


def draw_plan_call(rng):
    """A head-dimension-128 call for the planner: 1 to 16 ragged requests (empty ones, lengths around a key tile, around
    multiples of nine tiles and of 9 to 72 tiles, where eight and nine chunks are one length), block sizes whose tables clamp the chunk length, now and then a chunk length or a shape."""
    requests, hkv = int(rng.choice([1, 1, 2, 3, 4, 6, 8, 10, 16])), int(rng.choice([1, 2, 4, 8, 16]))
    log_int = lambda lo, hi: int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))
    longest = int(rng.choice([log_int(1, 200000), 576 * log_int(1, 300) + int(rng.integers(-1, 2)), 64 * rng.integers(9, 73)]))
    lens = [int(rng.choice([0, 1, 63, 64, 65, longest, max(1, longest // 2), log_int(1, longest + 1), longest]))
            for _ in range(requests)]
    kv, br = [("bf16", "bf16"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "bf16")][rng.integers(4)]
    block = int(rng.choice([16, 16, 32, 64, 128]))
    kw = dict(num_requests=requests, num_q_heads=hkv * int(rng.choice([1, 4, 5, 8])), num_kv_heads=hkv, head_dim=128,
              gamma=int(rng.choice([1, 2, 4, 6, 8])), branch_len=log_int(1, 120), block_size=block,
              max_blocks_per_request=(max(lens) + block - 1) // block + 1, kv_dtype=kv, branch_kv_dtype=br)
    if rng.random() < 0.2:
        kw["kv_split_tokens"] = 64 * log_int(1, 3000)
    if rng.random() < 0.3:
        kw["kernel_shape"] = int(rng.integers(1, 8))
    return kw, lens


def test_plan_search_misses_nothing():
    """The search passes over chunk counts that round to a chunk length it has modelled, stops at a lower bound of what is
    still to come and bounds the dealing out of unequal workgroups: the plans are those of a search that models every count
    (until the modelled time rises with every slot in use, as both do)."""
    B.select_library("bench")

    def plans(exhaustive):
        rng = np.random.default_rng(77)
        B.la_selftest_exhaustive_plans(exhaustive)
        out = []
        try:
            for _ in range(4000):
                kw, lens = draw_plan_call(rng)
                try:
                    desc = good_desc(**kw)
                    out.append((B.la_verify_attention_plan(desc, lens, int(rng.choice([0, 0, 70, 400]))),
                                B.la_verify_attention_workspace(desc, lens)))
                except B.LaError as e:
                    out.append(str(e))
        finally:
            B.la_selftest_exhaustive_plans(False)
        return out
    try:
        fast, full = plans(False), plans(True)
    finally:
        B.select_library("product")
    assert sum(not isinstance(x, str) for x in full) > 3000
    assert fast == full


@pytest.mark.parametrize("NB,K,V,T,top_k,top_p,draft,table", [
    (32, 8, 152064, 1.0, 0, 1.0, True, True), (15, 8, 152064, 1.0, 0, 1.0, True, False),      # 1200 slices of a row
    (16, 8, 152064, 1.0, 0, 1.0, True, True), (2000, 1, 32000, 1.0, 0, 1.0, True, False),     # rows of 32 slices
    (32, 8, 152064, 1.0, 0, 1.0, False, False), (6, 8, 152064, 0.6, 0, 0.95, False, True),
    (3, 8, 152064, 0.6, 0, 0.95, False, False), (400, 8, 10240, 0.6, 0, 0.95, False, False),  # 2048 slices; rows of six
    (32, 8, 152064, 0.6, 20, 0.95, False, False), (32, 8, 152064, 0.1, 0, 1.0, True, False),
    (600, 8, 10241, 0.6, 0, 0.95, True, True),
])
def test_calls_with_a_table_of_masses(NB, K, V, T, top_k, top_p, draft, table):
    """Which accept calls look their masses up: where the table is worth its copy to every workgroup."""
    for dtype in ("bf16", "f32"):
        desc = B.make_accept_desc(num_branches=NB, num_draft=K, vocab=V, logits_dtype=dtype, temperature=T, top_k=top_k,
                                  top_p=top_p)
        assert B.la_selftest_accept_table(desc, draft)[0] == (table and dtype == "bf16")


def test_room_for_top_p_candidates():
    """A target row's candidate segments share the row's part of the workspace, 4096 / (K + 1) bytes per 2048 tokens and call
    branch; the table of masses, where a call has one, takes no more than a sixteenth of it, and short last groups of slices
    waste nothing: a row that a call without a table could hold is not sent the long way."""
    rng = np.random.default_rng(5)
    for _ in range(2000):
        NB, K = int(rng.integers(1, 65)), int(rng.choice([1, 2, 3, 4, 6, 8, 12, 20]))
        V = int(np.exp(rng.uniform(np.log(100), np.log(300000))))
        dtype = str(rng.choice(["bf16", "f32"]))
        desc = B.make_accept_desc(num_branches=NB, num_draft=K, vocab=V, logits_dtype=dtype, temperature=0.8, top_k=0, top_p=0.9)
        table, room = B.la_selftest_accept_table(desc, False)
        slices = (V + 2047) // 2048
        key = 2 if dtype == "bf16" else 4
        most = min(1024, (16384 // (K + 1) // 16 * 16 - 16) // key) / 4                   # per slice
        assert room >= (15 / 16 if table else 0.97) * most * slices - 16, (NB, K, V, dtype, table, room, most * slices)
