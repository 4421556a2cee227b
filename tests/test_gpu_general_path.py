"""The general attention path (fp32 tensors; bf16 / fp8 storage at head dimensions 64 and 256) at the edges of its tiles:
row blocks of 16 and 32, key blocks of 16 and 32, chunks, with and without the optional workspace."""
import numpy as np
import pytest
import torch

from gpu_util import attn_desc, row_errors, upload_attention
from paper_2506_19830_amd import binding as B
from paper_2506_19830_amd import workloads as W
from test_gpu_attention import check_full, check_nested, check_tree

pytestmark = pytest.mark.gpu

BF16, FP8 = ("bf16", "bf16", "bf16"), ("bf16", "fp8_e4m3", "fp8_e4m3")
MIXED, F32 = ("bf16", "fp8_e4m3", "bf16"), ("f32", "f32", "f32")


def _case(name, prefix, gamma, L, hq, hkv, d, storage, out="f32", **kw):
    return W.AttnCase(name, prefix, gamma, L, hq, hkv, d, *storage, out, seed=len(name) + d, **kw)


CASES = [
    _case("rows_16", (31,), 2, 8, 2, 2, 64, BF16),                        # one full row block, a partial key block
    _case("rows_17", (32,), 1, 17, 1, 1, 64, BF16),                       # two row blocks, the second nearly empty
    _case("rows_33_chunks", (700, 0, 65), 3, 11, 2, 2, 64, BF16, paged=True),
    _case("split_small_block", (2049,), 1, 1, 4, 1, 64, FP8, paged=True),
    _case("split_large_block", (1537, 300), 2, 3, 4, 2, 64, FP8, paged=True, block_size=64),
    _case("mixed_chunks", (1100,), 2, 9, 5, 1, 64, MIXED, paged=True),
    _case("wide_chunks", (1025,), 1, 3, 4, 2, 256, BF16, paged=True, block_size=32),
    _case("wide_fp8", (900, 16), 2, 9, 2, 1, 256, FP8),
    _case("wide_mixed", (513,), 1, 33, 1, 1, 256, MIXED, paged=True),
    _case("f32_15", (15,), 1, 15, 1, 1, 64, F32),
    _case("f32_d128", (257, 16), 2, 5, 4, 2, 128, F32, paged=True),
    _case("f32_d256", (33,), 2, 17, 2, 1, 256, F32),
]


@pytest.mark.parametrize("split", [0, 64, 320])
@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_general_path_edges(oracle, case, split):
    """Against the fp64 oracle at the fp32 bar of the path (1e-5 of a row's largest element): operands are exact, sums
    fp32 over at most 2100 keys.  The unsplit result (no workspace) and the split one are both checked."""
    inp = W.make_attention_inputs(case)
    dev = upload_attention(case, inp)
    desc = attn_desc(case, split)
    lens = [int(x) for x in inp["prefix_lens"]]
    ref, ref_lse = oracle.verify_attention(**inp, q_dtype=case.q_dtype, kv_dtype=case.kv_dtype,
                                           branch_kv_dtype=case.branch_kv_dtype, block_size=case.block_size,
                                           scale=case.scale)
    size = B.la_verify_attention_workspace(desc, lens)
    assert size == 0 or case.kv_dtype != "f32"
    for ws in ([None] if size == 0 else [None, torch.empty(size, dtype=torch.uint8, device="cuda")]):
        out = B.empty_out(ref.shape, case.out_dtype).fill_(float("nan"))
        lse = torch.full(ref.shape[:-1], float("nan"), device="cuda")
        B.la_verify_attention(desc, dev["q"], dev["k_cache"], dev["v_cache"], dev["block_tables"], dev["prefix_lens"], lens,
                              dev["k_branch"], dev["v_branch"], dev["k_scale"], dev["v_scale"], out, lse, ws)
        torch.cuda.synchronize()
        assert row_errors(out.double().cpu().numpy(), ref).max() <= 1e-5
        assert np.abs(lse.double().cpu().numpy() - ref_lse).max() <= 1e-5


@pytest.mark.parametrize("storage", [BF16, FP8, MIXED, F32], ids=["bf16", "fp8", "mixed", "f32"])
def test_single_stage_over_many_blocks(oracle, storage):
    """Head dimension 256 keeps one K stage per wavefront, which every block overwrites: unsplit, 17 to 33 blocks each."""
    case = _case("wide_long", (4130,), 1, 5, 3, 1, 256, storage, paged=True)
    check_full(oracle, case, 1e-5, 0 if storage is F32 else 8192, lse_tol=1e-5)


FORMS = [
    # every storage type and head dimension: row blocks of 16 and 32, ragged and empty prefixes, tails of 1 to 63 keys
    *[_case(f"forms_d{d}_{name}", (700, 0, 65, 333), 3, 11, 4, 2, d, storage, paged=True)
      for d in (64, 256) for name, storage in (("bf16", BF16), ("fp8", FP8), ("mixed", MIXED))],
    _case("forms_d64_rows16", (1100, 31), 2, 2, 8, 2, 64, MIXED, block_size=64),
    _case("forms_f32_d64", (130, 0, 63), 3, 9, 4, 2, 64, F32, paged=True),
    _case("forms_f32_d256", (130, 17), 3, 5, 4, 2, 256, F32),
]


@pytest.mark.parametrize("split", [0, 64, 320])
@pytest.mark.parametrize("case", FORMS, ids=lambda c: c.name)
def test_nested_and_tree(oracle, case, split):
    """Chains around a key block of 32 (fp32: 16), visible parts of any length; trees of two shapes.  The last chunk takes
    the prefix's tail, the chain or pool and the rows' own tokens in this order."""
    rng = np.random.default_rng(split + case.seed)
    for chain_len in (1, 15, 31, 32, 33, 130):
        vis = rng.integers(0, chain_len + 1, size=(case.B, case.gamma))
        vis[0, 0], vis[-1, -1] = 0, chain_len
        check_nested(oracle, case, chain_len, 1e-5, vis, split)
    for width, depth, step_len in ((2, 2, 11), (3, 1, 32)):
        check_tree(oracle, case, width, depth, step_len, 1e-5, split)


@pytest.mark.parametrize("idx", range(18))
def test_random_shapes(oracle, idx):
    """Flat, nested and tree calls of low-precision storage at head dimensions 64 and 256, everything else drawn."""
    rng = np.random.default_rng(3000 + idx)
    hkv, g = int(rng.choice([1, 2, 4])), int(rng.choice([1, 2, 5, 8]))
    gamma, L = int(rng.choice([1, 2, 3, 5])), int(rng.choice([1, 2, 7, 16, 33, 90]))
    prefix = tuple(int(x) for x in rng.choice([0, 1, 15, 64, 65, 200, 513, 1100], size=int(rng.choice([1, 2, 3, 10]))))
    while len(prefix) * gamma * L * hkv * g > 4000:
        L = max(1, L // 2)
    case = _case("random", prefix, gamma, L, hkv * g, hkv, (64, 256)[idx % 2], (BF16, FP8, MIXED)[idx // 2 % 3],
                 block_size=int(rng.choice([16, 32, 128])), paged=bool(rng.integers(0, 2)))
    split = int(rng.choice([0, 64, 128, 448]))
    kind = idx // 6
    if kind == 0:
        check_full(oracle, case, 1e-5, split, lse_tol=1e-5)
    elif kind == 1:
        chain_len = int(rng.choice([1, 5, 64, 65, 130]))
        check_nested(oracle, case, chain_len, 1e-5, rng.integers(0, chain_len + 1, size=(case.B, gamma)), split)
    else:
        check_tree(oracle, case, *((2, 2), (2, 3), (3, 2))[int(rng.integers(0, 3))], int(rng.choice([1, 4, 17])), 1e-5, split)


def _empty_last_chunk(case, split):
    """Does some request's last chunk hold no prefix key?  (The tiles of 64 keys are dealt out evenly, the last chunk
    counted as carrying the branch-private ones.)"""
    rows = case.gamma * case.L * case.Hq
    r = rows // case.Hkv
    size = B.la_verify_attention_workspace(attn_desc(case, split), list(case.prefix_lens))
    s_max = round(size / (case.B * rows * (case.D + 2) * 4))
    tile = 32 if case.D == 64 and r > 16 else 16
    last_short = -(-min(tile + case.L, case.gamma * case.L) // 64)
    longest = max(case.prefix_lens)
    chunk = split or min(-(-longest // n) + 63 & ~63 for n in range(1, 65) if -(-longest // (-(-longest // n) + 63 & ~63)) == s_max)
    for p in case.prefix_lens:
        n, tiles = max(1, -(-p // chunk)), -(-p // 64)
        if n > 1 and (n - 1) * (tiles + last_short) // n >= tiles:
            return True
    return False


EMPTY_LAST = [
    # (case, kv_split_tokens): prefixes that end 1 .. 32 tokens into a key tile, beside branches of several tiles
    (_case("empty_p70", (70,), 2, 48, 8, 1, 64, BF16), 64),
    (_case("empty_p96_paged", (96, 0, 640), 2, 64, 2, 1, 64, BF16, paged=True), 64),
    (_case("empty_p80_fp8", (80,), 4, 40, 8, 2, 64, FP8), 64),
    (_case("empty_p65_mixed", (65,), 3, 70, 2, 1, 64, MIXED, paged=True), 64),
    (_case("empty_auto", (1055,), 1, 512, 4, 1, 64, BF16), 0),
    (_case("empty_wide", (70,), 2, 64, 2, 1, 256, BF16, paged=True), 64),
    (_case("empty_wide_auto", (450,), 1, 512, 4, 1, 256, BF16), 0),
    (_case("empty_wide_auto_fp8", (715,), 2, 320, 2, 1, 256, FP8), 0),
]


@pytest.mark.parametrize("form", ["flat", "nested", "tree"])
@pytest.mark.parametrize("case,split", EMPTY_LAST, ids=lambda v: getattr(v, "name", str(v)))
def test_last_chunk_without_prefix_keys(oracle, case, split, form):
    """Its workgroups start with the chain / pool or the branches' own tokens; every one of those keys counts."""
    assert _empty_last_chunk(case, split)
    if form == "flat":
        check_full(oracle, case, 1e-5, split, lse_tol=1e-5)
    elif form == "nested":
        check_nested(oracle, case, 75, 1e-5, None, split)
    else:
        check_tree(oracle, case, 2, 2, 11, 1e-5, split)


@pytest.mark.parametrize("d,storage", [(64, BF16), (64, FP8), (256, BF16)], ids=["d64_bf16", "d64_fp8", "d256_bf16"])
@pytest.mark.parametrize("requests", [9, 64, 65, 130])
def test_many_requests(oracle, requests, d, storage):
    """More requests than the kernel arguments hold (8): each workgroup finds its own, 64 at a time.  Ragged prefixes, some
    empty, cut into chunks and uncut; the last request's are the longest in the batch."""
    rng = np.random.default_rng(requests + d)
    prefix = [int(x) for x in rng.choice([0, 1, 40, 64, 65, 129, 300], size=requests)]
    prefix[-1], prefix[0] = 391, 0
    case = _case("many", tuple(prefix), 1, 2, 2, 1, d, storage, paged=True)
    for split in (0, 64, 192):
        check_full(oracle, case, 1e-5, split, lse_tol=1e-5)
    check_nested(oracle, case, 40, 1e-5, None, 128)


def _by_rows(case, chain_len=0):
    return B.la_verify_attention_plan(attn_desc(case), list(case.prefix_lens), chain_len)["row_tiles"] == 0


ROWS = [
    # (case, by rows in the flat call): units of 1 to 8 rows, prefixes up to the last length one round of 64 keys holds
    (_case("rows_f32", (0, 15, 16, 3, 0, 1, 7, 12), 1, 1, 128, 128, 64, F32, paged=True), True),
    (_case("rows_f32_d128", tuple([9, 0, 17, 1] * 3), 2, 1, 200, 100, 128, F32), True),
    (_case("rows_f32_d256", (62, 5, 62, 0), 1, 1, 1024, 1024, 256, F32, paged=True), True),
    (_case("rows_f32_past", (64, 5, 62, 0), 1, 1, 1024, 1024, 256, F32, paged=True), False),
    (_case("rows_bf16", (7, 16, 2), 1, 2, 500, 500, 64, BF16, out="bf16"), True),
    (_case("rows_bf16_d256", (11, 0, 30, 4), 1, 1, 750, 250, 256, BF16, paged=True, block_size=32), True),
    (_case("rows_fp8", (13, 5), 1, 1, 600, 600, 64, FP8), True),
    (_case("rows_fp8_d256", (9, 14), 2, 2, 400, 400, 256, FP8, paged=True), True),
    (_case("rows_mixed", (6, 0, 11), 3, 1, 400, 400, 64, MIXED, paged=True), True),
    (_case("rows_mixed_d256", (3, 8, 1), 2, 2, 800, 400, 256, MIXED, out="bf16"), True),
    (_case("rows_nine", (3, 8, 1), 3, 3, 400, 400, 64, F32), False),
    (_case("rows_few_units", (3, 8, 1), 1, 1, 40, 40, 64, F32), False),
]


@pytest.mark.parametrize("case,flat_by_rows", ROWS, ids=lambda v: getattr(v, "name", ""))
def test_one_wavefront_per_row(oracle, case, flat_by_rows):
    """Many requests or KV heads with a few rows of a few keys each: a kernel of its own, on both sides of its rule."""
    assert _by_rows(case) == flat_by_rows
    tol = 1e-5 if case.out_dtype == "f32" else 5e-3
    check_full(oracle, case, tol, lse_tol=1e-5)
    check_full(oracle, case, tol, 64, lse_tol=1e-5)
    assert not _by_rows(case, 75) and (not flat_by_rows or case.name == "rows_f32_d256" or _by_rows(case, 1))
    vis = np.random.default_rng(case.seed).integers(0, 5, size=(case.B, case.gamma))
    check_nested(oracle, case, 4, tol, vis)
    check_nested(oracle, case, 75, tol)
    check_tree(oracle, case, 2, 1, 2, tol)


def test_more_workgroups_than_one_grid_dimension_takes():
    """4.2 million requests of one row: more threads than one dimension of a launch may have (2^32).  All requests share
    one prefix, through the block table, so the reference is a plain product."""
    n, prefix, d, bs = (1 << 22) + 5, 100, 64, 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    q, kb, vb = draw(n, 1, 1, 1, d), draw(n, 1, 1, 1, d), draw(n, 1, 1, 1, d)
    blocks = -(-prefix // bs)
    kc, vc = draw(blocks, 1, bs, d), draw(blocks, 1, bs, d)
    table = torch.arange(blocks, dtype=torch.int32, device="cuda").repeat(n, 1)
    desc = B.make_attn_desc(num_requests=n, num_q_heads=1, num_kv_heads=1, head_dim=d, gamma=1, branch_len=1, block_size=bs,
                            max_blocks_per_request=blocks, q_dtype="f32", kv_dtype="f32", branch_kv_dtype="f32",
                            out_dtype="f32", softmax_scale=d ** -0.5)
    lens = [prefix] * n
    assert B.la_verify_attention_plan(desc, lens)["workgroups"] == n
    out = torch.full_like(q, float("nan"))
    B.la_verify_attention(desc, q, kc, vc, table, torch.full((n,), prefix, dtype=torch.int32, device="cuda"), lens, kb, vb,
                          None, None, out, None, None)
    k, v = kc.reshape(-1, d)[:prefix], vc.reshape(-1, d)[:prefix]
    for at in range(0, n, 1 << 20):
        x, y, z = (t[at:at + (1 << 20)].reshape(-1, d) for t in (q, kb, vb))
        p = torch.softmax(torch.cat([x @ k.T, (x * y).sum(1, keepdim=True)], 1) * d ** -0.5, 1)
        ref = p[:, :prefix] @ v + p[:, prefix:] * z
        err = (out[at:at + (1 << 20)].reshape(-1, d) - ref).abs().amax(1) / ref.abs().amax(1)
        assert float(err.max()) <= 1e-5
