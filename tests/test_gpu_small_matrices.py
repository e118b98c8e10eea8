"""Passes of at most 32 rows whose matrices are small enough for a work-group per row block over all of K, and their neighbours that are
not: widths on both sides of the rule (csrc/plans.h, plan_is_whole_k), bf16 and fp32 weights, in lock-step with the oracle."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from plans import Plans
from test_gpu_parity import TOL

# shape, d_model, d_ffn, heads, key heads, head dimension, and whether QKV and gate/up (K = d), O (K = heads x dim), down (K = d_ffn) are whole-K
CASES = [("tiny", 64, 64, 2, 1, 32, (True, True, True)), ("tiny", 1024, 1056, 16, 4, 64, (True, True, True)), ("tiny", 1088, 1072, 16, 16, 64, (False, True, False)),
         ("mini-gqa", 2048, 2112, 32, 8, 64, (True, True, True)), ("mini-gqa", 2176, 2144, 32, 32, 64, (False, True, False)), ("mini-gqa", 64, 64, 1, 1, 64, (True, True, True)),
         ("mini-moe", 512, 2144, 8, 8, 64, (True, True, False))]


def _shape(base, d, ffn, heads, kv_heads, dh):
    return replace(synth.SHAPES[base], name=f"{base}-d{d}-f{ffn}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=heads, n_kv_heads=kv_heads, head_dim=dh)


def test_cases_lie_on_the_sides_of_the_rule_that_they_name(tmp_path):
    plans = Plans(str(tmp_path))
    for base, d, ffn, heads, kv_heads, dh, want in CASES:
        planes = 6 if synth.SHAPES[base].dtype == "fp32" else 3
        got = tuple(plans.whole_k((d + 31) // 32, k // 16, planes) for k in (d, heads * dh, ffn))
        assert got == want, (base, d, ffn, got)
    assert plans.whole_k(256, 64, 3) and not plans.whole_k(257, 64, 3)


@pytest.mark.gpu
@pytest.mark.parametrize("base,d,ffn,heads,kv_heads,dh,whole", CASES)
def test_small_matrices_lockstep(base, d, ffn, heads, kv_heads, dh, whole):
    s = _shape(base, d, ffn, heads, kv_heads, dh)
    par, rk = synth.TREES["T26"]
    print(s.name, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=160)
    eng.load_weights(synth.iter_weights(s, 47, synth.device_fmt(s)))
    orc = Oracle(s, synth.make_weights(s, 47, synth.oracle_fmt(s)), par, rk, max_seq=160, dtype=np.float32)
    tol = TOL[s.dtype]
    check_prefill(eng, orc, synth.prompt(47, 40, s.vocab), tol)
    st = Stats()
    for _ in range(3):
        lockstep_step(eng, orc, st, tol)
    print(f"max|dL| verify {st.max_logit_err:.2e} draft {st.max_draft_logit_err:.2e}", flush=True)
    eng.close()
