"""Causal attention of long prompts (k2_attn_prompt: 128 rows a work-group, two tiles of 32 tokens a round) against the CPU oracle:
rows that end inside a wave's 32, at and behind a work-group's 128, in an odd number of tiles; every head dimension; grouped heads and
a number of heads that is no multiple of 8; a second pass over the first one's cache of fewer and of more than 64 pages, and a second
pass that takes the kernel of 32 rows; the bf16 cache of a mixture of experts."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from plans import Plans

# Two bf16 pieces hold 16 bits of a factor: 2^-17 relative per factor and some hundred terms of mixed sign stay below 2^-13 of the
# largest logit, which is at most 4 in these models.  bf16 cache: the rounding of K and V can turn, 2^-9 of about one entry in a thousand.
BOUND = {"fp32": 4 * 2.0 ** -13, "bf16": 1e-3}


def _shape(base, heads, kv_heads, dh, **kw):
    return replace(synth.SHAPES[base], name=f"{base}-h{heads}x{dh}", n_layers=1, n_heads=heads, n_kv_heads=kv_heads, head_dim=dh, **kw)


# ..., rows, cache, page, and whether each pass of the prompt takes the kernel
CASES = [
    ("mini-gqa", 64, 8, 32, 256, "fp32", 64, (True,)), ("mini-gqa", 64, 64, 32, 257, "fp32", 64, (True,)), ("mini-gqa", 64, 8, 32, 383, "fp32", 32, (True,)),
    ("mini-gqa", 52, 4, 64, 385, "fp32", 64, (True,)), ("mini-gqa", 52, 52, 64, 511, "fp32", 64, (True,)), ("mini-gqa", 40, 8, 128, 448, "fp32", 128, (True,)),
    ("mini-gqa", 32, 4, 128, 513, "fp32", 64, (True,)), ("mini-gqa", 12, 4, 32, 2700, "fp32", 32, (True, False)),
    ("mini-gqa", 16, 4, 32, 2700, "fp32", 32, (True, True)), ("mini-gqa", 20, 4, 64, 2563, "fp32", 64, (True, True)),
    ("mini-moe", 64, 8, 64, 300, "bf16", 64, (True,)), ("mini-moe", 64, 8, 128, 290, "fp32", 64, (True,))]


def test_cases_take_the_kernel_that_they_name(tmp_path):
    plans, behind = Plans(str(tmp_path)), set()
    for base, heads, kv_heads, dh, rows, kv, page, want in CASES:
        passes = plans.prompt_attn(heads, rows, rows + 64)
        assert tuple(p[2] for p in passes) == want, (heads, rows, passes)
        behind |= {(at + n + page - 1) // page > 64 for at, n, takes in passes if takes and at}
    assert behind == {False, True}                               # passes over a cache, with the page numbers of one register and of more
    for heads, rows, want in ((64, 255, False), (64, 256, True), (63, 256, False), (16, 992, False), (16, 993, True)):
        assert plans.prompt_attn(heads, rows, rows)[-1][2] == want, (heads, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("base,heads,kv_heads,dh,rows,kv,page", [c[:-1] for c in CASES])
def test_prompt_attention(base, heads, kv_heads, dh, rows, kv, page):
    s = _shape(base, heads, kv_heads, dh)
    par, rk = synth.TREES["T8"]
    print(s.name, "prompt of", rows, kv, "pages of", page, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=rows + 64, kv_dtype=kv, page_tokens=page)
    eng.load_weights(synth.iter_weights(s, 71, synth.device_fmt(s)))
    orc = Oracle(s, synth.make_weights(s, 71, synth.oracle_fmt(s)), par, rk, max_seq=rows + 64, dtype=np.float32, kv_store="bf16" if kv == "bf16" else None)
    err = check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), BOUND[kv])
    st = Stats()
    lockstep_step(eng, orc, st, 2e-2)                            # the head's cache of every prompt row is what drafting reads
    print(f"max|dL| prompt {err:.2e} verify {st.max_logit_err:.2e}", flush=True)
    eng.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [64, 256, 300])
def test_rows_whose_scores_are_all_minus_infinity_attend_to_nothing(rows):
    """Queries and keys so large that every score of a row overflows to -inf (one token repeated, queries opposite to the keys, in the
    columns that the rotary embedding turns least: 1.8e-4 a position): such rows take nothing from the values, with either attention
    kernel (64 rows: 32 rows a work-group), as if the output projection were zero."""
    s = _shape("mini-gqa", 64, 8, 32)
    par, rk = synth.TREES["T8"]
    token, low = 5, s.head_dim // 2 - 1
    w = synth.make_weights(s, 72, synth.oracle_fmt(s))
    u = w["embed"][token] / np.linalg.norm(w["embed"][token])
    extreme = {}
    for name, sign in (("layers.0.wq", 1e19), ("layers.0.wk", -1e19)):
        m = np.zeros_like(w[name])
        m[low::s.head_dim] = sign * u
        extreme[name] = synth._bf16_round_bits(m)
    eng = pkg.Eagle(s, par, rk, max_seq=rows + 64)
    eng.load_weights((n, extreme.get(n, a)) for n, a in synth.iter_weights(s, 72, synth.device_fmt(s)))
    w["layers.0.wo"] = np.zeros_like(w["layers.0.wo"])
    orc = Oracle(s, w, par, rk, max_seq=rows + 64, dtype=np.float32)
    err = check_prefill(eng, orc, np.full(rows, token, np.int32), BOUND["fp32"])
    assert np.isfinite(err)
    eng.close()
