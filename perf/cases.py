"""The work that the verification path does for its users, as measurable cases.

A case is one call a program makes while it verifies drafted steps: attention of one layer (flat, nested or tree
form), the accept / resample step over the vocabulary, or the KV commit of all layers.  ``listed()`` holds named
points, ``draw()`` further ones of the same ranges; sizes are the benchmark configurations of this repository
(``paper_2506_19830_amd.workloads``) and generic ones around them.  Everything goes through the package's binding.
"""
from __future__ import annotations

import math

import torch

from paper_2506_19830_amd import binding as B
from paper_2506_19830_amd import workloads as W

_SIZE = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.float8_e4m3fn}
_FP8_MAX = 448.0

# Upper bounds of what a drawn case may cost (see draw()).
_MAX_FLOPS = 3.4e11            # configuration 5's attention, one layer
_MAX_FLOPS_OTHER_HEADS = 8e9   # head dimensions 64 and 256
_MAX_FLOPS_F32 = 4e9
_MAX_LOGIT_BYTES = 1.65e8      # configuration 4's accept call


def _verify(form, prefix, gamma, L, hq, hkv, d, kv="bf16", br="bf16", q="bf16", out="bf16", block=16, paged=False,
            extra=0, width=1, depth=1):
    """extra: tokens of the drafted chain (nested) or of one tree node (tree)."""
    return {"kind": "verify", "form": form, "prefix": ",".join(str(p) for p in prefix), "gamma": gamma, "L": L,
            "Hq": hq, "Hkv": hkv, "D": d, "q": q, "kv": kv, "branch": br, "out": out, "block": block, "paged": paged,
            "extra": extra, "width": width, "depth": depth}


def _accept(nb, k, v, dtype, temperature=1.0, top_k=0, top_p=1.0, lookup=False, target_std=3.0, peak=14.0):
    """peak: added to the target logit of a token proposed by lookup, so that it is accepted about every other time."""
    return {"kind": "accept", "NB": nb, "K": k, "V": v, "dtype": dtype, "T": temperature, "top_k": top_k,
            "top_p": top_p, "lookup": lookup, "target_std": target_std, "peak": peak}


def _commit(layers, prefix, gamma, L, hkv, d, kv, br, chain, kept_chain, kept_own, tree=False, block=16):
    """tree: the drafted tokens are a pool of 14 equal nodes (two alternatives, three positions), the path
    0 - 2 - 6 is kept; else a chain of `chain` tokens of which the first `kept_chain` are kept."""
    return {"kind": "commit", "layers": layers, "prefix": prefix, "gamma": gamma, "L": L, "Hkv": hkv, "D": d,
            "kv": kv, "branch": br, "chain": chain, "kept_chain": kept_chain, "kept_own": kept_own, "tree": tree,
            "block": block}


def listed():
    cases = {
        # a small model in reference precision: one short prompt, the call a first test of an integration makes
        "f32_tiny": _verify("flat", (256,), 2, 8, 4, 1, 64, kv="f32", br="f32", q="f32", out="f32"),
        # one token per branch against a long fp8 prefix: plain decoding of eight continuations, bound by the cache
        "decode_fp8": _verify("flat", (32768,), 8, 1, 40, 8, 128, kv="fp8_e4m3", br="fp8_e4m3"),
        # the paper's own operating point: six speculative steps, nine tokens of each per target pass
        "step_fp8": _verify("flat", (32768,), 6, 9, 40, 8, 128, kv="fp8_e4m3", br="fp8_e4m3"),
        # whole drafted steps against a long fp8 prefix (the benchmark's headline configuration)
        "long_steps_fp8": _verify("flat", (32768,), 8, 64, 40, 8, 128, kv="fp8_e4m3", br="fp8_e4m3"),
        # early in a generation, bf16 cache
        "short_prefix_bf16": _verify("flat", (4096,), 4, 32, 64, 8, 128),
        # four requests of different age in one batch, paged bf16 cache: a serving batch
        "ragged_batch_bf16": _verify("flat", (8192, 16384, 24576, 32768), 8, 48, 64, 8, 128, paged=True),
        # Algorithm 1's own prefixes: each branch sees the drafted steps before it (five steps of 27 tokens)
        "nested_fp8": _verify("nested", (20011,), 6, 9, 40, 8, 128, kv="fp8_e4m3", br="fp8_e4m3", paged=True, extra=135),
        # a draft tree: two alternatives per position, three positions, every tree prefix continued (15 branches)
        "tree_bf16": _verify("tree", (12345,), 15, 9, 40, 8, 128, paged=True, extra=27, width=2, depth=3),
        # a model with heads of 64
        "head64_bf16": _verify("flat", (8190,), 4, 16, 64, 8, 64),
        # token-level acceptance with draft logits for a serving batch: the largest vocabulary scan
        "accept_dense": _accept(32, 8, 152064, "bf16"),
        # token-level acceptance as the paper samples: prompt-lookup drafts, temperature 0.6, top-p 0.95
        "accept_lookup_top_p": _accept(6, 8, 152064, "bf16", 0.6, 0, 0.95, True),
        # what survives a pass joins the cache of all layers
        "commit_fp8": _commit(64, 4096, 8, 64, 8, 128, "fp8_e4m3", "fp8_e4m3", 448, 192, 64),
    }
    return [dict(c, name=n) for n, c in cases.items()]


# ------------------------------------------------------------------------------------------------ drawing

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_form(rng, c):
    """Turn a flat case into a nested or tree one, sometimes."""
    form = rng.choice(("flat", "flat", "nested", "tree"))
    if form == "nested":
        return dict(c, form=form, extra=_log_int(rng, 8, 448))
    if form == "tree":
        width, depth = rng.choice(((2, 2), (2, 3), (3, 2), (4, 1)))
        return dict(c, form=form, extra=_log_int(rng, 4, 64), width=width, depth=depth)
    return c


def _draw_verify(rng):
    hq, hkv = rng.choice(((40, 8), (64, 8), (32, 8), (32, 4), (16, 2)))
    kv, br = rng.choice((("bf16", "bf16"), ("bf16", "bf16"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "fp8_e4m3"),
                         ("fp8_e4m3", "bf16")))
    prefix = tuple(_log_int(rng, 256, 32768) for _ in range(rng.choice((1, 1, 1, 2, 3, 4, 6))))
    c = _verify("flat", prefix, rng.randint(1, 8), _log_int(rng, 1, 64), hq, hkv, 128, kv=kv, br=br,
                out=rng.choice(("bf16", "bf16", "bf16", "f32")), block=rng.choice((16, 16, 32, 64)),
                paged=rng.random() < 0.6)
    return _draw_form(rng, c)


def _draw_other_heads(rng):
    hq, hkv = rng.choice(((64, 8), (32, 8), (16, 4), (8, 1), (14, 2)))
    kv, br = rng.choice((("bf16", "bf16"), ("bf16", "bf16"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "bf16")))
    prefix = tuple(_log_int(rng, 128, 8192) for _ in range(rng.choice((1, 1, 2, 3))))
    c = _verify("flat", prefix, rng.randint(1, 8), _log_int(rng, 1, 32), hq, hkv, rng.choice((64, 256)), kv=kv, br=br,
                out=rng.choice(("bf16", "bf16", "f32")), block=rng.choice((16, 32)), paged=rng.random() < 0.6)
    return _draw_form(rng, c)


def _draw_f32(rng):
    hq, hkv = rng.choice(((4, 1), (8, 2), (16, 4), (12, 4)))
    prefix = tuple(_log_int(rng, 16, 2048) for _ in range(rng.choice((1, 1, 2))))
    c = _verify("flat", prefix, rng.randint(1, 4), _log_int(rng, 1, 16), hq, hkv, rng.choice((64, 128, 256)), kv="f32",
                br="f32", q="f32", out="f32", paged=rng.random() < 0.5)
    return _draw_form(rng, c)


def _draw_accept(rng):
    top_k, top_p = rng.choice(((0, 1.0), (0, 1.0), (0, 0.95), (20, 0.95), (50, 1.0)))
    return _accept(_log_int(rng, 1, 32), rng.randint(1, 8), rng.choice((152064, 152064, 128000, 32003, _log_int(rng, 512, 152064))),
                   rng.choice(("bf16", "bf16", "f32")), rng.choice((0.6, 1.0)), top_k, top_p, rng.random() < 0.5)


def _draw_commit(rng):
    kv, br = rng.choice((("bf16", "bf16"), ("fp8_e4m3", "fp8_e4m3"), ("fp8_e4m3", "bf16")))
    tree, L = rng.random() < 0.4, _log_int(rng, 1, 64)
    chain = 14 * rng.randint(1, 32) if tree else rng.randint(0, 448)
    kept = 3 * (chain // 14) if tree else rng.randint(0, chain)
    return _commit(_log_int(rng, 1, 64), _log_int(rng, 64, 4096), rng.randint(1, 8), L, rng.choice((4, 8)),
                   rng.choice((64, 128, 128)), kv, br, chain, kept, rng.randint(0, L), tree, rng.choice((16, 16, 64)))


def draw(rng):
    family = rng.choice((_draw_verify,) * 9 + (_draw_other_heads,) * 3 + (_draw_f32,) * 2 + (_draw_accept,) * 5 +
                        (_draw_commit,) * 2)
    while True:
        c = family(rng)
        if c["kind"] == "verify":
            bound = _MAX_FLOPS_F32 if c["q"] == "f32" else _MAX_FLOPS if c["D"] == 128 else _MAX_FLOPS_OTHER_HEADS
            if work(c)["flops"] <= bound:
                return c
        elif c["kind"] != "accept" or work(c)["bytes"] <= _MAX_LOGIT_BYTES:
            return c


# ------------------------------------------------------------------------------------------------ inputs

def _prefixes(case):
    return tuple(int(p) for p in case["prefix"].split(","))


def _attn_case(case, seed):
    return W.AttnCase("case", _prefixes(case), case["gamma"], case["L"], case["Hq"], case["Hkv"], case["D"], case["q"],
                      case["kv"], case["branch"], case["out"], block_size=case["block"], paged=case["paged"], seed=seed)


def _tree(case):
    """Parents of the nodes (level by level), and the nodes on the root path of each."""
    parents = [int(x) for x in W.tree_parents(case["width"], case["depth"])]
    paths = []
    for n, par in enumerate(parents):
        paths.append((paths[par] if par >= 0 else []) + [n])
    return parents, paths


def _visible(case):
    """Chain or pool tokens each branch sees."""
    g = case["gamma"]
    if case["form"] == "nested":
        return [(j * case["extra"]) // g for j in range(g)]
    if case["form"] == "tree":
        return [len(p) * case["extra"] for p in _branch_paths(case)]
    return [0] * g


def _branch_paths(case):
    """Branch 0 continues the bare prefix, branch 1 + n the path that ends in node n (wrapping around)."""
    _, paths = _tree(case)
    return [([] if j % (len(paths) + 1) == 0 else paths[j % (len(paths) + 1) - 1]) for j in range(case["gamma"])]


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _store(x, dtype, scale):
    """fp32 -> storage type; fp8 codes are the values divided by the per-head scale (heads: second last dimension)."""
    if dtype == "fp8_e4m3":
        x = (x / scale[:, None]).clamp_(-_FP8_MAX, _FP8_MAX)
    return x.to(_TORCH[dtype])


def _prepare_verify(case, seed):
    ac = _attn_case(case, seed)
    t = W.make_attention_inputs_device(ac)
    lens = list(ac.prefix_lens)
    desc = B.make_attn_desc(num_requests=ac.B, num_q_heads=ac.Hq, num_kv_heads=ac.Hkv, head_dim=ac.D, gamma=ac.gamma,
                            branch_len=ac.L, block_size=ac.block_size, max_blocks_per_request=ac.max_blocks,
                            q_dtype=ac.q_dtype, kv_dtype=ac.kv_dtype, branch_kv_dtype=ac.branch_kv_dtype,
                            out_dtype=ac.out_dtype, softmax_scale=ac.scale)
    ws_bytes = B.la_verify_attention_workspace(desc, lens)
    state = dict(t, case=case, desc=desc, lens=lens,
                 out=torch.empty((ac.B, ac.gamma, ac.L, ac.Hq, ac.D), dtype=_TORCH[ac.out_dtype], device="cuda"),
                 lse=torch.empty((ac.B, ac.gamma, ac.L, ac.Hq), dtype=torch.float32, device="cuda"),
                 workspace=torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda"))
    if case["form"] != "flat":
        gen = _generator(seed + 77)
        n = case["extra"] if case["form"] == "nested" else case["extra"] * len(_tree(case)[0])
        for which, scale in (("k", t["k_scale"]), ("v", t["v_scale"])):
            x = torch.randn((ac.B, n, ac.Hkv, ac.D), generator=gen, device="cuda")
            state[which + "_extra"] = _store(x, ac.branch_kv_dtype, scale)
        if case["form"] == "nested":
            vis = [_visible(case)] * ac.B
            state["vis"] = torch.tensor(vis, dtype=torch.int32, device="cuda")
            state["vis_host"] = vis
        else:
            seg = [[node for node in range(len(_tree(case)[0])) for _ in range(case["extra"])]] * ac.B
            mask = [[sum(1 << node for node in path) for path in _branch_paths(case)]] * ac.B
            state["seg"] = torch.tensor(seg, dtype=torch.int32, device="cuda")
            state["seg_host"] = seg
            state["mask"] = torch.tensor(mask, dtype=torch.int64, device="cuda")
    return state


def _prepare_accept(case, seed):
    nb, k, v = case["NB"], case["K"], case["V"]
    gen = _generator(seed)
    dtype = _TORCH[case["dtype"]]
    target = torch.randn((nb, k + 1, v), generator=gen, device="cuda") * case["target_std"]
    if case["lookup"]:   # tokens proposed by a lookup in the context: no draft logits, a target row peaked at them
        tokens = torch.randint(0, v, (nb, k), generator=gen, device="cuda")
        target[:, :k].scatter_add_(2, tokens[..., None], torch.full((nb, k, 1), case["peak"], device="cuda"))
        draft = None
    else:                # tokens sampled from the draft model's logits, which follow the target's
        draft = (target[:, :k] + torch.randn((nb, k, v), generator=gen, device="cuda")).to(dtype)
        tokens = torch.empty((nb, k), dtype=torch.int64, device="cuda")
        for b in range(nb):
            e = torch.empty((k, v), device="cuda").exponential_(generator=gen)
            tokens[b] = torch.argmax(draft[b].float() / case["T"] - e.log(), dim=-1)
    desc = B.make_accept_desc(num_branches=nb, num_draft=k, vocab=v, logits_dtype=case["dtype"],
                              temperature=case["T"], top_k=case["top_k"], top_p=case["top_p"])
    return {"case": case, "desc": desc, "target": target.to(dtype), "draft": draft, "tokens": tokens.to(torch.int32),
            "u_accept": torch.rand((nb, k), generator=gen, device="cuda"),
            "u_sample": torch.rand((nb,), generator=gen, device="cuda"),
            "accepted": torch.empty(nb, dtype=torch.int32, device="cuda"),
            "next": torch.empty(nb, dtype=torch.int32, device="cuda"),
            "ratio": torch.empty((nb, k), dtype=torch.float32, device="cuda"),
            "workspace": torch.empty(B.la_spec_accept_workspace(desc), dtype=torch.uint8, device="cuda")}


def _prepare_commit(case, seed):
    gen = _generator(seed)
    n, hkv, d, bs, c = case["layers"], case["Hkv"], case["D"], case["block"], case["chain"]
    blocks = -(-(case["prefix"] + c + case["L"]) // bs)

    def drawn(shape, dtype):   # storage codes of N(0, 1) values
        x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)
        if dtype == "fp8_e4m3":
            x = (x * 100.0).clamp_(-_FP8_MAX, _FP8_MAX)
        return x.to(_TORCH[dtype])

    state = {"case": case, "lens": [case["prefix"]], "new_lens": torch.empty(1, dtype=torch.int32, device="cuda"),
             "prefix_lens": torch.tensor([case["prefix"]], dtype=torch.int32, device="cuda"),
             "table": torch.randperm(blocks, generator=gen, device="cuda").to(torch.int32)[None].contiguous(),
             "k_scale": torch.full((n, hkv), 0.01, device="cuda"), "v_scale": torch.full((n, hkv), 0.0101, device="cuda"),
             "src": torch.tensor([seed % case["gamma"]], dtype=torch.int32, device="cuda"),
             "n_chain": torch.tensor([case["kept_chain"]], dtype=torch.int32, device="cuda"),
             "n_own": torch.tensor([case["kept_own"]], dtype=torch.int32, device="cuda")}
    for w in "kv":
        state[w + "_cache"] = drawn((n, blocks, hkv, bs, d), case["kv"])
        state[w + "_branch"] = drawn((n, 1, case["gamma"], case["L"], hkv, d), case["branch"])
        state[w + "_chain"] = drawn((n, 1, c, hkv, d), case["branch"]) if c else None
    if case["tree"]:
        seg = torch.arange(14, dtype=torch.int32, device="cuda").repeat_interleave(c // 14)
        state["seg"] = seg[None].contiguous()
        state["mask"] = torch.tensor([(1 << 0) | (1 << 2) | (1 << 6)], dtype=torch.int64, device="cuda")
    state["desc"] = B.make_attn_desc(
        num_requests=1, num_q_heads=hkv, num_kv_heads=hkv, head_dim=d, gamma=case["gamma"], branch_len=case["L"],
        block_size=bs, max_blocks_per_request=blocks, q_dtype="bf16", kv_dtype=case["kv"],
        branch_kv_dtype=case["branch"], out_dtype="bf16", softmax_scale=d ** -0.5)
    state["strides"] = B.la_layer_strides(n, blocks * hkv * bs * d, case["gamma"] * case["L"] * hkv * d, c * hkv * d, hkv)
    return state


def prepare(case, seed):
    return {"verify": _prepare_verify, "accept": _prepare_accept, "commit": _prepare_commit}[case["kind"]](case, seed)


# ------------------------------------------------------------------------------------------------ one pass

def run(state):
    s, case = state, state["case"]
    if case["kind"] == "verify":
        head = (s["desc"], s["q"], s["k_cache"], s["v_cache"], s["block_tables"], s["prefix_lens"], s["lens"],
                s["k_branch"], s["v_branch"])
        tail = (s["k_scale"], s["v_scale"], s["out"], s["lse"], s["workspace"])
        if case["form"] == "flat":
            B.la_verify_attention(*head, *tail)
        elif case["form"] == "nested":
            B.la_verify_attention_nested(*head, s["k_extra"], s["v_extra"], s["vis"], s["vis_host"], *tail)
        else:
            B.la_verify_attention_tree(*head, s["k_extra"], s["v_extra"], s["seg"], s["seg_host"], s["mask"], *tail)
        return {"out": s["out"], "lse": s["lse"]}
    if case["kind"] == "accept":
        B.la_spec_accept(s["desc"], s["target"], s["draft"], s["tokens"], s["u_accept"], s["u_sample"], s["accepted"],
                         s["next"], s["ratio"], s["workspace"])
        return {"accepted_len": s["accepted"], "next_token": s["next"], "ratio": s["ratio"]}
    head = (s["desc"], s["k_cache"], s["v_cache"], s["table"], s["prefix_lens"], s["lens"], s["k_branch"],
            s["v_branch"], s["k_chain"], s["v_chain"])
    tail = (s["k_scale"], s["v_scale"], s["new_lens"], s["strides"])
    if case["tree"]:
        B.la_kv_commit_tree(*head, s["seg"], s["mask"], s["src"], s["n_own"], *tail)
    else:
        B.la_kv_commit(*head, s["src"], s["n_chain"], s["n_own"], *tail)
    return {"k_cache": s["k_cache"], "v_cache": s["v_cache"], "new_prefix_lens": s["new_lens"]}


# ------------------------------------------------------------------------------------------------ what it takes

def work(case):
    if case["kind"] == "verify":
        ac = _attn_case(case, 0)
        vis = _visible(case)
        flops = ac.flops() + 4.0 * ac.B * ac.L * ac.Hq * ac.D * sum(vis)
        extra = 0
        if case["form"] == "nested":
            extra = max(vis)
        elif case["form"] == "tree":
            extra = case["extra"] * len({node for path in _branch_paths(case) for node in path})
        read = 2.0 * ac.B * extra * ac.Hkv * ac.D * _SIZE[case["branch"]]
        return {"bytes": ac.algorithmic_bytes() + read + 4.0 * ac.branch_tokens * ac.Hq, "flops": flops}
    if case["kind"] == "accept":
        rows = case["NB"] * ((case["K"] + 1) + (0 if case["lookup"] else case["K"]))
        # every logit: one exponential's argument and one addition
        return {"bytes": float(rows * case["V"] * _SIZE[case["dtype"]]), "flops": 2.0 * rows * case["V"]}
    tokens = case["kept_chain"] + case["kept_own"]
    per = 2.0 * case["layers"] * case["Hkv"] * case["D"]
    return {"bytes": max(16.0, per * tokens * (_SIZE[case["kv"]] + _SIZE[case["branch"]])), "flops": 0.0}


def tolerance(case):
    """About four times the distance of the outputs from the same computation in 64 bits."""
    if case["kind"] == "commit":
        return "exact"
    if case["kind"] == "accept":   # the p/q ratios are fp32 sums over the vocabulary; lengths and tokens do not differ
        return {"rel": 3e-6, "differ": 0.0}
    if case["out"] == "f32" and (case["q"] == "f32" or case["D"] != 128):   # fp32 arithmetic and results
        return {"rel": 4e-6}
    if case["D"] != 128:           # fp32 arithmetic, results rounded to bf16
        return {"rel": 7e-3}
    return {"rel": 1.2e-2}         # bf16 matrix operands
