"""The fp64 masses of bf16 logits by table: logits outside it (large, tiny, zero, masked), rows whose maximum is their unit,
temperatures on both sides of the table's limit, calls too small for one, and top-p rows of many and of few values."""
import numpy as np
import pytest

from paper_2506_19830_amd import workloads as W
from test_gpu_accept import check_inputs

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("accept_tables")]


def rows(kind, x, rng):
    """x: [NB, rows, V] normal logits of deviation 3."""
    if kind == "beyond":      # up to +-250: past the table's 64; |max| / T on both sides of 300 at T 0.6 ... 1.5
        return x * np.where(np.arange(x.shape[0]) % 2, 10.0, 18.0)[:, None, None]
    if kind == "tiny":        # below 2^-12, zeros of both signs among them
        x = x * 1e-4
        x[:, :, ::7] = 0.0
        x[:, :, 3::7] = -0.0
        return x
    if kind == "edges":       # around the table's first and last entries
        return np.sign(x) * np.exp2(rng.choice([-12.02, -12.0, -11.98, -3.0, 0.0, 2.0], x.shape)) * (1 + 0.01 * np.abs(x))
    if kind == "negative":    # far below zero
        return x - np.where(np.arange(x.shape[0]) % 2, 100.0, 400.0)[:, None, None]
    if kind == "masked":      # most of the vocabulary
        x[rng.random(x.shape) < 0.9] = -np.inf
        x[:, :, 5] = 1.0
        return x
    return x


def make(case, kind):
    inp = W.make_accept_inputs(case)
    rng = np.random.default_rng(case.seed)
    t = rows(kind, W._decode_for_sampling(inp["target_logits"], case.logits_dtype).astype(np.float64), rng)
    inp["target_logits"] = W.encode(t.astype(np.float32), case.logits_dtype)
    if inp["draft_logits"] is not None:
        d = t[:, :case.K] + rng.standard_normal(t[:, :case.K].shape) * 0.5 * (1e-4 if kind == "tiny" else 1.0)
        inp["draft_logits"] = W.encode(d.astype(np.float32), case.logits_dtype)
        # tokens a draft would propose from these rows (the accept test is fp32: masses of e^-100 have no quotient there)
        inp["draft_tokens"] = np.argsort(-d, axis=-1)[..., int(rng.integers(0, 3))].astype(np.int32)
    return inp


@pytest.mark.parametrize("V", [8200, 8201])     # 16-byte aligned rows, and not
@pytest.mark.parametrize("kind", ["plain", "beyond", "tiny", "edges", "negative", "masked"])
@pytest.mark.parametrize("temperature,top_k,top_p", [(1.0, 0, 1.0), (0.6, 0, 0.95), (0.11, 0, 1.0), (0.1, 0, 0.9),
                                                     (1.5, 30, 0.9)])
def test_masses(oracle, V, kind, temperature, top_k, top_p):
    """14 branches of five slices: a table; the last slice nearly empty."""
    for point_mass in (False, True):
        case = W.AcceptCase(f"tab_{kind}", 14, 2, V, "bf16", temperature=temperature, top_k=top_k, top_p=top_p,
                            point_mass=point_mass, peak=6.0, seed=700 + V % 2)
        inp = make(case, kind)
        if kind == "beyond" and temperature < 0.5 and not point_mass:
            # one token holds all but e^-100 of every row: what is left of a residual is rounding on every side.  So the
            # drafts are accepted and the draw is from the bonus row.
            t = W._decode_for_sampling(inp["target_logits"], "bf16")
            inp["draft_tokens"] = t[:, :2].argmax(-1).astype(np.int32)
            inp["u_accept"][:] = 0.0
        check_inputs(oracle, case, inp)


def has_table(case):
    from paper_2506_19830_amd import binding as B
    return B.la_selftest_accept_table(B.make_accept_desc(num_branches=case.NB, num_draft=case.K, vocab=case.V,
                                                         logits_dtype=case.logits_dtype, temperature=case.temperature,
                                                         top_k=case.top_k, top_p=case.top_p))[0]


COLDEST = float(np.float32(0.11))


@pytest.mark.parametrize("temperature,table", [(COLDEST, True), (float(np.nextafter(np.float32(0.11), np.float32(0))), False),
                                               (0.125, True)])
@pytest.mark.parametrize("kind", ["plain", "tiny", "edges", "negative", "masked"])
def test_coldest_table(oracle, accept_tables, kind, temperature, table):
    """Temperatures around the lowest one with a table: entries up to e^+-582, and rows whose maximum is 300 T or more, which
    keep it as their unit (8200 logits of deviation 3 reach 11, or 100 T; shifted by 100 and 400 they are beyond)."""
    for point_mass, top_p in ((False, 1.0), (True, 0.9)):
        case = W.AcceptCase(f"tab_cold_{kind}", 14, 2, 8200, "bf16", temperature=temperature, top_p=top_p,
                            point_mass=point_mass, peak=6.0, seed=710)
        assert has_table(case) == (table and accept_tables == "table")
        check_inputs(oracle, case, make(case, kind))


@pytest.mark.parametrize("NB,V", [(63, 2048), (64, 2048), (1, 131071), (1, 129023), (13, 10000), (2, 65535)])
def test_smallest_calls_with_a_table(oracle, accept_tables, NB, V):
    """64 slices in all, and one less; odd numbers of slices per branch."""
    for top_p in (1.0, 0.9):
        case = W.AcceptCase("tab_small", NB, 2, V, "bf16", temperature=0.7, top_p=top_p, seed=800 + NB)
        assert has_table(case) == (accept_tables == "table" and NB * ((V + 2047) // 2048) >= 64)
        check_inputs(oracle, case, make(case, "plain"))


@pytest.mark.parametrize("std,top_p", [(0.01, 0.5), (0.3, 0.9), (8.0, 0.999)])
def test_top_p_values(oracle, std, top_p):
    """Listed tokens of a few dozen values, and from the row maximum down to zero and below (more octaves than there are
    counts for)."""
    case = W.AcceptCase("tab_values", 12, 2, 16400, "bf16", target_std=3.0, temperature=1.0, top_p=top_p, point_mass=True,
                        peak=0.0, seed=820)
    inp = W.make_accept_inputs(case)
    x = W._decode_for_sampling(inp["target_logits"], "bf16") * (std / 3.0)
    x[1::2] *= np.where(np.arange(16400) % 3, 1.0, 1e-4)     # every other branch: values near zero among them
    inp["target_logits"] = W.encode(x.astype(np.float32), "bf16")
    check_inputs(oracle, case, inp)
