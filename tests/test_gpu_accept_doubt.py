"""Resampling after a rejection where the sign of the residual p - q is decided late: tokens whose target and draft
masses agree so closely that the first pass lists them, lists that overflow, and rows where nothing is left."""
import numpy as np
import pytest

from paper_2506_19830_amd import workloads as W

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("accept_tables")]

# vocabularies around a wavefront's 512 tokens, a 2048-token slice, rows without 16-byte alignment
VOCABS = (64, 513, 2048, 2049, 6000, 20003)


def swapped(V, dtype, share, seed, NB=12, shift=0.0):
    """Target rows, and draft rows with the same logits in another order except for a `share` of the tokens, which keep
    theirs: both rows have one normaliser (up to the order of summation), so exactly those tokens are in doubt.  shift: added
    to all draft logits."""
    rng = np.random.default_rng(seed)
    t = (rng.standard_normal((NB, 2, V)) * 2).astype(np.float32)
    d = t[:, :1].copy()
    tok = np.zeros((NB, 1), dtype=np.int32)
    for nb in range(NB):
        moved = np.flatnonzero(rng.random(V) >= share)
        moved = np.union1d(moved, rng.choice(V, 2, replace=False))
        d[nb, 0, moved] = np.roll(t[nb, 0, moved], 1)
        tok[nb, 0] = moved[np.argmax(d[nb, 0, moved] - t[nb, 0, moved])]   # drafted where q exceeds p most
        d[nb] += np.float32(shift)
    return {"target_logits": W.encode(t, dtype), "draft_logits": W.encode(d, dtype), "draft_tokens": tok,
            "u_accept": np.full((NB, 1), 0.999, np.float32),
            "u_sample": rng.random(NB).astype(np.float32)}


def close(V, noise, rest, seed, NB=12):
    """fp32 rows that differ by `noise` at every token and by 1 at a share `rest` of them: the residual is made of tokens
    in doubt, or of both kinds."""
    rng = np.random.default_rng(seed)
    t = (rng.standard_normal((NB, 2, V)) * 2).astype(np.float32)
    d = t[:, :1] + (rng.standard_normal((NB, 1, V)) * noise).astype(np.float32)
    d += ((rng.random(d.shape) < rest) * rng.standard_normal(d.shape)).astype(np.float32)
    tok = rng.integers(0, V, (NB, 1)).astype(np.int32)
    for nb in range(NB):
        d[nb, 0, tok[nb, 0]] = t[nb, 0, tok[nb, 0]] + 3.0   # rejected: u just below 1 times a larger q
    return {"target_logits": t, "draft_logits": d, "draft_tokens": tok,
            "u_accept": np.full((NB, 1), 0.999, np.float32), "u_sample": rng.random(NB).astype(np.float32)}


def check(oracle, inp, dtype, V, temperature=1.0, **warp):
    from gpu_util import compare_accept, run_accept
    NB = inp["draft_tokens"].shape[0]
    case = W.AcceptCase("doubt", NB, 1, V, dtype, temperature=temperature, **warp)
    got = run_accept(case, inp)
    ref = oracle.spec_accept(**inp, logits_dtype=dtype, temperature=temperature, top_k=case.top_k,
                             top_p=float(np.float32(case.top_p)))
    assert (ref["accepted_len"] == 0).sum() >= NB // 2      # the rows do get resampled
    bad_n, bad_tok, near = compare_accept(got, ref)
    assert bad_n == 0 and bad_tok == 0 and near <= 1, f"{bad_n} lengths, {bad_tok} tokens differ, {near} set aside"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("share", [0.0, 0.03, 0.09, 0.5, 1.0])   # 48 of 512 fit a list: 0.09 lies on both sides of that
@pytest.mark.parametrize("V", VOCABS)
def test_equal_masses(oracle, V, share, dtype):
    check(oracle, swapped(V, dtype, share, seed=900 + V), dtype, V)


@pytest.mark.parametrize("noise,rest", [(3e-6, 0.0), (3e-5, 0.0), (3e-6, 0.5), (3e-4, 0.1)])
@pytest.mark.parametrize("V", VOCABS)
def test_close_masses(oracle, V, noise, rest):
    check(oracle, close(V, noise, rest, seed=950 + V), "f32", V)
    check(oracle, close(V, noise, rest, seed=951 + V), "f32", V, temperature=0.3)


@pytest.mark.parametrize("warp", [{"top_k": 40}, {"top_p": 0.9}, {"top_k": 300, "top_p": 0.95}], ids=str)
def test_equal_masses_warped(oracle, warp):
    """The draft is used as given, so the target's smaller normaliser lifts every kept token's residual above zero."""
    check(oracle, swapped(6000, "bf16", 0.5, seed=990), "bf16", 6000, temperature=0.6, **warp)


@pytest.mark.parametrize("shift", [-0.5, 100.0, 3000.0])
@pytest.mark.parametrize("V", (2049, 20003))
def test_equal_masses_shifted(oracle, V, shift):
    """A constant added to the draft's logits: by half, exact for most of them; by more, differences that fp32 rounds to one
    value although no two of them are equal, so that no sum can stand for such tokens."""
    for share in (0.3, 0.9):
        check(oracle, swapped(V, "f32", share, seed=970 + V, shift=shift), "f32", V)


@pytest.mark.parametrize("temperature", [1.0, 0.11, 0.05])
@pytest.mark.parametrize("step", [1, 3])
def test_few_differences(oracle, step, temperature):
    """bf16 rows of the same values in another order for a few tokens, and for the others the same logit or one a few bf16
    steps away: several values of the difference among the tokens in doubt, at logits of 2^-14 and above."""
    V = 6000
    inp = swapped(V, "bf16", 0.9, seed=980 + step)
    t = W._decode_for_sampling(inp["target_logits"], "bf16")
    d = W._decode_for_sampling(inp["draft_logits"], "bf16")
    rng = np.random.default_rng(step)
    small = rng.random(d.shape) < 0.5
    bits = W.encode(rng.choice([2.0 ** -14, 2.0 ** -13, 2.0 ** -12], d.shape).astype(np.float32), "bf16")
    tb, db = inp["target_logits"].copy(), inp["draft_logits"].copy()
    tb[:, :1][small] = bits[small]
    db[small] = (bits + rng.integers(0, step + 1, d.shape).astype(np.uint16))[small]
    for nb in range(d.shape[0]):
        tok = inp["draft_tokens"][nb, 0]
        tb[nb, 0, tok], db[nb, 0, tok] = inp["target_logits"][nb, 0, tok], inp["draft_logits"][nb, 0, tok]
    del t
    check(oracle, dict(inp, target_logits=tb, draft_logits=db), "bf16", V, temperature=float(np.float32(temperature)))
