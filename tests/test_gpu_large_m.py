"""The large-M GEMM (k_gemm_pf) at the edges of its tiles: prompt passes whose rows end inside a 32-row tile, inside a work-group
tile (4 or 8 row tiles), at a window of 512 rows, and beyond one pass of 2048; rows grouped by expert;
4-bit weights; a loss pass of more than 1024 rows.  Against the
CPU oracle in fp64."""
import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from oracle.int4_weights import quantize_model
from test_gpu_head_loss import _check, _engine, _features, _lm_head
from test_gpu_parity import TOL, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [33, 64, 65, 97, 129, 257, 333, 512, 513, 600, 1100, 2049, 2200])
def test_prompt_rows_at_tile_edges(rows):
    s, eng, orc = make_pair("mini-gqa", "T8", seed=11, max_seq=2300)
    print("prompt of", rows, flush=True)
    check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), TOL["bf16"])
    lockstep_step(eng, orc, Stats(), TOL["bf16"])               # the head's cache of every prompt row is what drafting reads
    eng.close()


@pytest.mark.parametrize("rows", [1, 7, 33, 64, 131, 513, 1100])
def test_expert_rows_grouped(rows):
    """Experts with no row, a few rows, and several tiles of rows; the grouped MLP adds a row's experts in ascending order."""
    s, eng, orc = make_pair("mini-moe", "T8", seed=12, max_seq=1200)
    print("prompt of", rows, flush=True)
    check_prefill(eng, orc, synth.prompt(rows + 5, rows, s.vocab), TOL["bf16"])
    lockstep_step(eng, orc, Stats(), TOL["bf16"])
    eng.close()


@pytest.mark.parametrize("rows", [32, 33, 65, 128, 257, 600, 1100])
def test_int4_prompt_rows(rows):
    """4-bit weights: the fused kernels up to 32 rows, the large-M GEMM beyond (2 and 3 groups along K)."""
    s = synth.SHAPES["mini-gqa"].twin(2)
    par, rk = synth.TREES["T8"]
    eng = pkg.Eagle(s, par, rk, max_seq=1200, weight_bits=4)
    eng.load_weights(synth.iter_weights(s, 61, synth.device_fmt(s)))
    orc = Oracle(s, quantize_model(synth.make_weights(s, 61, synth.oracle_fmt(s))), par, rk, max_seq=1200, dtype=np.float64)
    print("prompt of", rows, flush=True)
    err = check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), TOL["bf16"])
    st = Stats()
    lockstep_step(eng, orc, st, TOL["bf16"])
    print(f"max|dL| prompt {err:.2e} verify {st.max_logit_err:.2e}", flush=True)
    eng.close()


def test_loss_of_two_large_passes():
    shape = synth.SHAPES["mini-gqa"]
    eng = _engine(shape, head_loss_rows=1100)
    Wdev, W64 = _lm_head(shape, 3)
    eng.load_named("lm_head", Wdev)
    f, fhat = _features(1100, shape.d_model, 9, 0.7)
    _check(eng, W64.astype(np.float64), f, fhat, 0.1, "mini-gqa")
    eng.close()
