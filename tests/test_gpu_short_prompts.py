"""Prompts and last prompt passes around 32 rows, where the fused kernels of the decoding steps take over from the general path: every row's
features and the logits against the CPU oracle, and two steps behind them.  fp32 models take 128 rows a pass, and the general path whatever the
rows where d_model is no short K (plan_is_short_prompt)."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

# waves of the whole-K stream with no, one and a few k-steps: K 64 (4 of them for eight waves), 256, 384
SHAPES = {"tiny": synth.SHAPES["tiny"], "mini-gqa": synth.SHAPES["mini-gqa"], "mini-moe": synth.SHAPES["mini-moe"],
          "fp32-d64": replace(synth.SHAPES["tiny"], name="tiny-d64", d_model=64, n_heads=1, n_kv_heads=1, d_ffn=80),
          "fp32-d1024": replace(synth.SHAPES["tiny"], name="tiny-d1024", n_layers=1, d_model=1024, d_ffn=80), "fp32-d1088": replace(synth.SHAPES["tiny"], name="tiny-d1088", n_layers=1, d_model=1088, d_ffn=80),
          "bf16-d128": replace(synth.SHAPES["mini-gqa"], name="mini-d128", d_model=128, n_heads=4, n_kv_heads=2, d_ffn=192)}


@pytest.mark.parametrize("shape,kv", [("tiny", "fp32"), ("fp32-d64", "fp32"), ("fp32-d1024", "fp32"), ("fp32-d1088", "fp32"), ("mini-gqa", "fp32"), ("mini-gqa", "bf16"), ("bf16-d128", "fp32"), ("mini-moe", "fp32")])
@pytest.mark.parametrize("rows", [1, 2, 31, 32, 33, 129, 160])
def test_prompts_around_a_pass_of_32_rows(shape, kv, rows):
    s = SHAPES[shape]
    par, rk = synth.TREES["T10"]
    print(s.name, kv, rows, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=256, kv_dtype=kv)
    eng.load_weights(synth.iter_weights(s, 91, synth.device_fmt(s)))
    orc = Oracle(s, synth.make_weights(s, 91, synth.oracle_fmt(s)), par, rk, max_seq=256, dtype=np.float32, kv_store="bf16" if kv == "bf16" else None)
    tol = 2e-2 if kv == "bf16" else TOL[s.dtype]
    check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), tol)
    st = Stats()
    for _ in range(2):
        lockstep_step(eng, orc, st, tol)
    eng.close()
