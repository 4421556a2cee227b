"""Nested and tree calls on the streaming shapes (fp8 and bf16 caches): chain and pool lengths around a key tile, row
tiles that straddle branches, prefixes that are empty, shorter than a tile, ragged; both attempts of the kernels."""
import numpy as np
import pytest

from paper_2506_19830_amd import workloads as W
from test_gpu_attention import TOL_LOWP, check_full, check_nested, check_tree

pytestmark = pytest.mark.gpu


def make_case(kv, prefix, gamma, L, hq, hkv, paged, seed, out="bf16"):
    return W.AttnCase(f"forms_{kv}_{len(prefix)}", prefix, gamma, L, hq, hkv, 128, "bf16", kv, kv, out, paged=paged,
                      seed=seed)


# (prefixes, gamma, L, Hq, Hkv, paged): 45 rows, 135 rows over two requests, 384 rows (several row tiles of every shape)
SHAPES = [((700,), 3, 3, 10, 2, True), ((0, 333), 3, 9, 10, 2, False), ((1100,), 4, 12, 16, 2, True),
          ((5,), 6, 1, 8, 2, False)]


def streams(case):
    from paper_2506_19830_amd import binding as B
    desc = B.make_attn_desc(num_requests=case.B, num_q_heads=case.Hq, num_kv_heads=case.Hkv, head_dim=case.D,
                            gamma=case.gamma, branch_len=case.L, block_size=case.block_size,
                            max_blocks_per_request=case.max_blocks, q_dtype=case.q_dtype, kv_dtype=case.kv_dtype,
                            branch_kv_dtype=case.branch_kv_dtype, out_dtype=case.out_dtype, softmax_scale=case.scale)
    return B.la_verify_attention_plan(desc, [int(x) for x in case.prefix_lens], 1)["kernel_shape"] >= 3


@pytest.mark.parametrize("kv", ["fp8_e4m3", "bf16"])
@pytest.mark.parametrize("chain_len", [1, 63, 64, 65, 300])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_nested(oracle, kv, chain_len, shape):
    case = make_case(kv, *SHAPES[shape], seed=300 + shape)
    assert streams(case)
    rng = np.random.default_rng(chain_len + shape)
    vis = rng.integers(0, chain_len + 1, size=(case.B, case.gamma)).astype(np.int32)
    vis[0, 0], vis[-1, -1] = 0, chain_len                     # one branch sees nothing, one everything
    for split in (0, 128):
        check_nested(oracle, case, chain_len, TOL_LOWP, vis, split)


@pytest.mark.parametrize("kv", ["fp8_e4m3", "bf16"])
@pytest.mark.parametrize("width,depth,step_len", [(2, 1, 1), (2, 2, 21), (3, 2, 16), (1, 3, 64)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_tree(oracle, kv, width, depth, step_len, shape):
    case = make_case(kv, *SHAPES[shape], seed=340 + shape, out="f32" if shape == 1 else "bf16")
    assert streams(case)
    for split in (0, 128):
        check_tree(oracle, case, width, depth, step_len, TOL_LOWP, split)


@pytest.mark.parametrize("kv", ["fp8_e4m3", "bf16"])
@pytest.mark.parametrize("shape", [1, 2])
def test_second_attempt(oracle, kv, shape):
    """Every workgroup reduces its chunk again in the general form (a hook of the benchmark library)."""
    from paper_2506_19830_amd import binding as B
    case = make_case(kv, *SHAPES[shape], seed=380 + shape)
    B.select_library("bench")
    try:
        B.la_selftest_second_attempt(True)
        try:
            check_nested(oracle, case, 130, TOL_LOWP)
            check_tree(oracle, case, 2, 2, 21, TOL_LOWP)
        finally:
            B.la_selftest_second_attempt(False)
    finally:
        B.select_library("product")


@pytest.mark.parametrize("split", [32448, 32512, 65024])
def test_split_around_the_streaming_limit(oracle, split):
    """Chunk lengths asked for that the streaming shapes' table of block ids can just, and can no longer hold."""
    case = make_case("bf16", (700, 0, 130), 3, 20, 16, 2, True, seed=395)
    check_full(oracle, case, TOL_LOWP, split)
    check_nested(oracle, case, 60, TOL_LOWP, None, split)


FORCED = [("fp8_e4m3", 3), ("fp8_e4m3", 4), ("fp8_e4m3", 5), ("bf16", 6), ("bf16", 7)]


@pytest.mark.parametrize("kv,kernel_shape", FORCED)
def test_forced_shape(oracle, kv, kernel_shape, monkeypatch):
    """Every streaming shape forced on nested and tree calls, and a chain or pool that no branch sees: the flat call's
    bits."""
    from gpu_util import run_attention, run_attention_nested, run_attention_tree
    monkeypatch.setattr("gpu_util.KERNEL_SHAPE", kernel_shape)
    for i, shape in enumerate(SHAPES):
        case = make_case(kv, *shape, seed=400 + i)
        for split in (0, 192):
            check_nested(oracle, case, 130, TOL_LOWP, None, split)
            check_tree(oracle, case, 2, 2, 21, TOL_LOWP, split)
            inp = W.make_attention_inputs(case)
            flat, flat_lse = run_attention(case, inp, split)
            chain = W.make_chain_inputs(case, 70, inp, np.zeros((case.B, case.gamma), dtype=np.int32))
            tree = W.make_tree_inputs(case, 2, 2, 17, inp)
            tree["seg_mask"][:] = 0
            for got, lse in (run_attention_nested(case, inp, chain, split), run_attention_tree(case, inp, tree, split)):
                assert np.array_equal(got, flat) and np.array_equal(lse, flat_lse)


@pytest.mark.parametrize("kv", ["fp8_e4m3", "bf16"])
@pytest.mark.parametrize("requests", [9, 64, 65, 130])
def test_many_requests(oracle, requests, kv):
    """More requests than the kernel arguments hold (8): ragged prefixes, some empty, cut into chunks and uncut."""
    rng = np.random.default_rng(requests)
    prefix = [int(x) for x in rng.choice([0, 1, 40, 64, 65, 129, 300], size=requests)]
    prefix[-1], prefix[0] = 391, 0
    case = make_case(kv, tuple(prefix), 2, 2, 4, 2, True, seed=410)
    for split in (0, 64, 192):
        check_full(oracle, case, TOL_LOWP, split)
    check_nested(oracle, case, 70, TOL_LOWP, None, 128)
    check_tree(oracle, case, 2, 2, 9, TOL_LOWP, 128)


def sink_inputs(case):
    """Rows whose first key's score lies 19 to 22 nats above N(0, 2), the scores of the others."""
    inp = W.make_attention_inputs(case)
    rng = np.random.default_rng(case.seed)
    u = rng.choice([-1.0, 1.0], size=(case.Hkv, case.D)) / np.sqrt(case.D)
    q = rng.standard_normal((case.B, case.gamma, case.L, case.Hkv, case.Hq // case.Hkv, case.D))
    q -= (q * u[:, None]).sum(-1, keepdims=True) * u[:, None]
    q += np.sqrt(case.D) * rng.uniform(0.95, 1.1, size=q.shape[:-1] + (1,)) * u[:, None]
    inp["q"] = W.encode(q.reshape(inp["q"].shape).astype(np.float32), "bf16")
    inp["k_cache"][0, :, 0] = W.encode((20.0 * u).astype(np.float32), "bf16")
    return inp


@pytest.mark.parametrize("split", [0, 192])
@pytest.mark.parametrize("kernel_shape", [6, 7])
def test_first_key_holds_the_row(oracle, kernel_shape, split, monkeypatch):
    """A first token that draws all attention: as the maximum of the first tile its probability is 2^0, which bf16 holds, so
    the output is its V to fp32 accuracy.  The other 760 keys weigh 760 e^(1 - 19) = 1.2e-5 together, and their scores and
    probabilities are right to a part in a hundred (Q times the score scale and the probabilities rounded to bf16)."""
    from gpu_util import row_errors, run_attention
    from test_gpu_attention import oracle_attention
    monkeypatch.setattr("gpu_util.KERNEL_SHAPE", kernel_shape)
    case = make_case("bf16", (700,), 3, 20, 16, 2, False, seed=420, out="f32")
    inp = sink_inputs(case)
    got, _ = run_attention(case, inp, split)
    ref, _ = oracle_attention(oracle, case, inp)
    assert row_errors(got, ref).max() <= 1e-5
