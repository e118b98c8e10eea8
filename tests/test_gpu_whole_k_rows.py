"""Gate/up of 33 to 128 rows over all of K in a work-group (k_gemm_wk) against the fp32 oracle: every number of row tiles with its last
row at either end of a tile, two and three (three and four) row blocks a work-group, K ranges of a wave that are shorter than the
ring, end inside it, and fill it more than once; prompt passes, and verify passes of two to four sequences.  Tolerance: that of the other
bf16 models (make_pair's TOL)."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step, lockstep_step_batch
from oracle.eagle_oracle import Oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

# name -> (d_model, d_ffn, prompt rows): k-steps of a wave = d / 64, row blocks = d_ffn / 16 (256 CUs: 513..768 or
# 769..1024); every K a multiple of 64, as the large-M path asks
CASES = {"516-blocks-4-steps": (256, 516 * 16, (33, 64, 65, 96, 97, 128)),
         "600-blocks-13-steps": (832, 600 * 16, (40, 77, 126)),
         "768-blocks-21-steps": (1344, 768 * 16, (64, 96, 128)),
         "772-blocks-5-steps": (320, 772 * 16, (33, 64)),
         "1024-blocks-12-steps": (768, 1024 * 16, (50,))}


@pytest.mark.parametrize("name", CASES)
def test_gate_up_rows(name):
    d, ffn, rows = CASES[name]
    assert d % 64 == 0 and ffn % 64 == 0 and (512 < ffn // 16 <= 768 or max(rows) <= 64)
    shape = replace(synth.SHAPES["mini-gqa"], name=f"wk-{name}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=d // 64, n_kv_heads=d // 64, head_dim=64)
    par, rk = synth.TREES["T8"]
    W = synth.make_weights(shape, 71, synth.oracle_fmt(shape))
    eng = pkg.Eagle(shape, par, rk, max_seq=192)
    eng.load_weights(synth.iter_weights(shape, 71, synth.device_fmt(shape)))
    for n in rows:
        orc = Oracle(shape, W, par, rk, max_seq=192, dtype=np.float32)
        print(name, "prompt of", n, flush=True)
        eng.reset()
        err = check_prefill(eng, orc, synth.prompt(n, n, shape.vocab), TOL["bf16"])
        lockstep_step(eng, orc, Stats(), TOL["bf16"])
        print(f"max|dL| prompt {err:.2e}", flush=True)
    eng.close()


@pytest.mark.parametrize("name, batch, tree", [("516-blocks-4-steps", 4, "T26"), ("600-blocks-13-steps", 3, "T26"), ("772-blocks-5-steps", 2, "T26"), ("516-blocks-4-steps", 2, "B63")])
def test_gate_up_rows_of_batched_verify(name, batch, tree):
    """104, 78, 52 and 126 verify rows, sequences of different lengths."""
    d, ffn, _ = CASES[name]
    shape = replace(synth.SHAPES["mini-gqa"], name=f"wk-{name}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=d // 64, n_kv_heads=d // 64, head_dim=64)
    par, rk = synth.TREES[tree]
    W = synth.make_weights(shape, 71, synth.oracle_fmt(shape))
    eng = pkg.Eagle(shape, par, rk, max_batch=batch, max_seq=192)
    eng.load_weights(synth.iter_weights(shape, 71, synth.device_fmt(shape)))
    orcs = [Oracle(shape, W, par, rk, max_seq=192, dtype=np.float32, seq_id=b) for b in range(batch)]
    for b, orc in enumerate(orcs):
        check_prefill(eng, orc, synth.prompt(71 + b, 24 + 9 * b, shape.vocab), TOL["bf16"], seq=b)
    sts = [Stats() for _ in orcs]
    print(name, "verify of", batch * len(par), "rows", flush=True)
    for _ in range(2):
        lockstep_step_batch(eng, orcs, sts, TOL["bf16"])
    print(f"max|dL| {max(st.max_logit_err for st in sts):.2e}", flush=True)
    eng.close()
