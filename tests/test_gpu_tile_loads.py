"""Both ways in which the large-M GEMM brings its tiles (plain loads and buffer loads, plan_pf_plain_loads in csrc/plans.h), for every
tile of two and four waves that takes them, with and without SwiGLU in the epilogue, rows ending inside a tile and at its end, against
the CPU oracle.  test_plans.py says which launches the cases below get.  Tolerance: that of the other bf16 models."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

# (d_model, d_ffn, prompt rows)
CASES = [(256, 512, (33, 64, 72, 97, 105, 128, 161)), (1536, 8192, (33, 72)), (2048, 512, (300,)), (256, 14336, (161, 192))]


def shape_of(d, ffn):
    return replace(synth.SHAPES["mini-gqa"], name=f"loads-{d}-{ffn}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=d // 64, n_kv_heads=d // 64, head_dim=64)


@pytest.mark.parametrize("d, ffn, rows", CASES)
def test_prompt_rows(d, ffn, rows):
    shape = shape_of(d, ffn)
    par, rk = synth.TREES["T8"]
    W = synth.make_weights(shape, 91, synth.oracle_fmt(shape))
    eng = pkg.Eagle(shape, par, rk, max_seq=384)
    eng.load_weights(synth.iter_weights(shape, 91, synth.device_fmt(shape)))
    for n in rows:
        orc = Oracle(shape, W, par, rk, max_seq=384, dtype=np.float32)
        print(shape.name, "prompt of", n, flush=True)
        eng.reset()
        err = check_prefill(eng, orc, synth.prompt(n, n, shape.vocab), TOL["bf16"])
        lockstep_step(eng, orc, Stats(), TOL["bf16"])
        print(f"max|dL| prompt {err:.2e}", flush=True)
    eng.close()
