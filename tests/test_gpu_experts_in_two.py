"""Tree passes of wide mixtures of experts, whose experts run in two launches a layer (plan_experts_in_two in csrc/plans.h), in lock-step
with the fp32 oracle: one choice of three experts (most passes leave some unused), four of five, two of eight with a full tree, four of
forty; gate/up with two, three and four row blocks a work-group, down with two, three and four, in three and in seven to nine K slices.
test_plans.py says which kernels the cases get.  Tolerance: that of the other bf16 models."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu

# name -> (experts, choices, d_model, d_ffn, tree): at least 256 gate/up row blocks (d_ffn / 16), K too long for plan_is_whole_k
CASES = {"e3-top1": (3, 1, 2176, 4160, "T8"), "e5-top4": (5, 4, 2176, 4160, "chain5"), "e8-top2": (8, 2, 2176, 4160, "T26"), "e2-top1-long-k": (2, 1, 2176, 16384, "T8"),
         "e2-top2-three-slices": (2, 2, 2368, 4096, "T8"), "e2-top1-gate-up3": (2, 1, 2112, 8256, "T26"), "e2-top1-down3": (2, 1, 2752, 12288, "T8"),
         "e2-top1-down4": (2, 1, 3520, 16064, "T8"), "e40-top4": (40, 4, 2112, 4160, "T8")}


def shape_of(name):
    E, k, d, ffn, _ = CASES[name]
    return replace(synth.SHAPES["mini-moe"], name=f"moe-{name}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=d // 64, n_kv_heads=d // 64, head_dim=64,
                   n_experts=E, experts_per_tok=k, draft_moe=E <= 8)


@pytest.mark.parametrize("name", CASES)
def test_lockstep(name):
    shape, tree = shape_of(name), CASES[name][4]
    par, rk = synth.TREES[tree]
    W = synth.make_weights(shape, 83, synth.oracle_fmt(shape))
    eng = pkg.Eagle(shape, par, rk, max_seq=192)
    eng.load_weights(synth.iter_weights(shape, 83, synth.device_fmt(shape)))
    orc = Oracle(shape, W, par, rk, max_seq=192, dtype=np.float32)
    print(name, flush=True)
    check_prefill(eng, orc, synth.prompt(5, 20, shape.vocab), TOL["bf16"])
    st = Stats()
    for _ in range(3):
        lockstep_step(eng, orc, st, TOL["bf16"])
    print(f"{name}: verify max|dL| {st.max_logit_err:.2e} draft {st.max_draft_logit_err:.2e}", flush=True)
    eng.close()
