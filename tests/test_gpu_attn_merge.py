"""Tree attention over contexts that several work-groups share (k2_attn): one to sixteen splits of the keys, merged by the last of them;
passes of 1 to 32 rows, so that a thread merges one row, two or four; every head dimension; cached lengths that the host hands over (up to
four sequences) and that the kernel reads; against the CPU oracle."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step
from oracle.eagle_oracle import Oracle
from plans import Plans

# Two bf16 pieces hold 16 bits of a factor: see test_gpu_attn_prompt.py; the steps' logits: the suite's bound for bf16 weights.
BOUND, STEP = {"fp32": 4 * 2.0 ** -13, "bf16": 1e-3}, 2e-2

# heads, key heads, head dimension, tree, prompt, cache, splits of a verify pass
CASES = [(4, 2, 128, "T26", 150, "fp32", 2), (4, 4, 128, "T26", 520, "fp32", 5), (4, 2, 128, "T10", 840, "fp32", 8), (4, 2, 128, "T15", 970, "fp32", 9),
         (4, 1, 128, "root", 400, "fp32", 4), (4, 2, 64, "T26", 1500, "fp32", 13), (4, 4, 64, "T10", 300, "fp32", 3), (8, 2, 32, "T26", 1960, "fp32", 16),
         (8, 2, 32, "chain5", 700, "bf16", 6), (4, 2, 128, "T26", 2300, "bf16", 16), (4, 2, 64, "T8", 860, "bf16", 8),
         (4, 2, 128, "T26", 100, "fp32", 1), (4, 2, 128, "T26", 790, "fp32", 7), (4, 4, 64, "T26", 1200, "fp32", 10), (4, 2, 128, "T15", 1330, "fp32", 11),
         (8, 2, 32, "T26", 1450, "bf16", 12), (4, 2, 64, "T10", 1710, "fp32", 14), (4, 1, 128, "T26", 1840, "fp32", 15)]


def _shape(heads, kv_heads, dh):
    return replace(synth.SHAPES["mini-gqa"], name=f"mini-h{heads}x{dh}", n_layers=1, n_heads=heads, n_kv_heads=kv_heads, head_dim=dh)


def test_cases_have_the_splits_that_they_name(tmp_path):
    plans = Plans(str(tmp_path))
    for heads, _, _, tree, prompt, kv, splits in CASES:
        assert plans.attn_splits(kv == "bf16", prompt + 64, heads) == splits, (tree, prompt)
    assert {c[-1] for c in CASES} == set(range(1, 17))


@pytest.mark.gpu
@pytest.mark.parametrize("heads,kv_heads,dh,tree,prompt,kv,splits", CASES)
def test_splits_merge(heads, kv_heads, dh, tree, prompt, kv, splits):
    s = _shape(heads, kv_heads, dh)
    par, rk = synth.TREES[tree]
    print(s.name, tree, "prompt of", prompt, kv, splits, "splits", flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=prompt + 96, kv_dtype=kv)
    eng.load_weights(synth.iter_weights(s, 83, synth.device_fmt(s)))
    orc = Oracle(s, synth.make_weights(s, 83, synth.oracle_fmt(s)), par, rk, max_seq=prompt + 96, dtype=np.float32, kv_store="bf16" if kv == "bf16" else None)
    check_prefill(eng, orc, synth.prompt(prompt, prompt, s.vocab), BOUND[kv])
    st = Stats()
    for _ in range(2):
        lockstep_step(eng, orc, st, STEP)
    assert st.max_logit_err < BOUND[kv], st.max_logit_err
    print(f"max|dL| verify {st.max_logit_err:.2e}", flush=True)
    eng.close()


@pytest.mark.gpu
@pytest.mark.parametrize("seqs", [4, 5])
def test_sequences_of_different_lengths(seqs):
    """The host hands the cached lengths of up to four sequences to the kernel; with five it reads them: the same logits either way as alone."""
    s = _shape(4, 2, 64)
    par, rk = synth.TREES["chain5"]
    lens = [300, 40, 129, 520, 64][:seqs]
    eng = pkg.Eagle(s, par, rk, max_batch=seqs, max_seq=640)
    eng.load_weights(synth.iter_weights(s, 84, synth.device_fmt(s)))
    one = pkg.Eagle(s, par, rk, max_seq=640)
    one.load_weights(synth.iter_weights(s, 84, synth.device_fmt(s)))
    for b, n in enumerate(lens):
        eng.prefill(b, synth.prompt(84, n, s.vocab, stream=b))
    eng.draft_tree()
    eng.verify()
    for b, n in enumerate(lens):
        one.reset()
        one.prefill(0, synth.prompt(84, n, s.vocab, stream=b))
        one.draft_tree()
        one.verify()
        got, want = eng.get_buffer(pkg.BUF_LOGITS, b), one.get_buffer(pkg.BUF_LOGITS, 0)
        assert np.abs(got - want).max() < BOUND["fp32"], (b, n, np.abs(got - want).max())
    eng.close()
    one.close()
