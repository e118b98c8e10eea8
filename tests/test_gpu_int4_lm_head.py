"""The LM head of 4-bit models over all of K with up to four row blocks of 32 tokens a CU (k2_logits_q4): vocabularies at the edges of its range
(more than 768 blocks, at most 1024; the kernels beside it take the others), ends inside a block and inside four tokens, K of one to twenty
groups for four K parts, one row and up to 32."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from oracle.int4_weights import dequantize, quantize
from plans import Plans

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 256, 768, 2560])
@pytest.mark.parametrize("vocab", [24576, 24577, 26003, 32000, 32766, 32768, 32769])
def test_logits_of_every_row(vocab, d):
    s = replace(synth.SHAPES["mini-gqa"], name=f"q4-v{vocab}-d{d}", n_layers=1, d_model=d, n_heads=4, n_kv_heads=2, d_ffn=128, vocab=vocab)
    par, rk = synth.TREES["chain5"]
    print(s.name, flush=True)
    B = 5                                                        # verify passes of 30 rows
    eng = pkg.Eagle(s, par, rk, max_batch=B, max_seq=64, weight_bits=4)
    W = synth.make_weights(s, 71, synth.oracle_fmt(s))
    eng.load_weights(synth.iter_weights(s, 71, synth.device_fmt(s)))
    q, sc = quantize(W["lm_head"])
    Wq = dequantize(q, sc).astype(np.float64)
    first = [eng.prefill(b, synth.prompt(71, 3 + 7 * b, vocab, stream=b)) for b in range(B)]
    assert first == [int(np.argmax(eng.get_buffer(pkg.BUF_VANILLA_LOGITS, b))) for b in range(B)]
    eng.draft_tree()
    eng.verify()
    for b in range(B):
        x = eng.get_buffer(pkg.BUF_FEATURES, b).astype(np.float64)
        got = eng.get_buffer(pkg.BUF_LOGITS, b).astype(np.float64)
        # x passes as two bf16 planes (2^-17 of it at most are left), products with 16 + code or 128 + code <= 143 are summed in fp32 over the 128
        # columns of a group (2^-24 times 2 x 128 terms, 2^-16), then scaled and added over at most 20 groups and 4 parts (32 x 2^-24, less)
        bound = 143 * 2.0 ** -15 * np.einsum("mg,ng->mn", np.abs(x).reshape(len(x), -1, 128).sum(2), sc.astype(np.float64))
        err = np.abs(got - x @ Wq.T)
        assert (err <= bound).all() and err.max() < 2e-3 * np.abs(got).max(), (b, err.max(), (err / bound).max())
    eng.close()


@pytest.mark.parametrize("d,slices", [(4096, 4), (4224, 5)])
def test_bf16_cache_keeps_the_order_of_sums(d, slices, tmp_path):
    """With a bf16 cache the order of sums depends on no choice of kernel: 32000 tokens and 32800 of which the first 32000 are the same (one row
    block more than k2_logits_q4 takes: the split-K kernel, with the K slices that it always had) give the same bits for those."""
    plans = Plans(str(tmp_path))
    assert plans.staged_q4(1000, d // 16) == plans.staged_q4(1025, d // 16) == (slices, 1) and not plans.logits_q4(1025, d // 16)
    s = replace(synth.SHAPES["mini-gqa"], name=f"q4-bf16-d{d}", n_layers=1, d_model=d, n_heads=4, n_kv_heads=2, d_ffn=128, vocab=32800)
    par, rk = synth.TREES["T26"]
    print(s.name, flush=True)
    W = synth.make_weights(s, 73, synth.device_fmt(s))
    W["lm_head"][32000:] = 0                                     # (logits of zero: never chosen)
    got = []
    for vocab in (32800, 32000):
        eng = pkg.Eagle(replace(s, vocab=vocab), par, rk, max_seq=96, weight_bits=4, kv_dtype="bf16")
        eng.load_weights({k: np.ascontiguousarray(w[:vocab]) if k in ("embed", "lm_head") else w for k, w in W.items()})
        first = eng.prefill(0, synth.prompt(73, 29, 32000))
        out = [eng.get_buffer(pkg.BUF_VANILLA_LOGITS)[:32000]]
        tree = eng.draft_tree()[0]
        eng.verify()
        out += [eng.get_buffer(pkg.BUF_DRAFT_LOGITS)[0, :32000], eng.get_buffer(pkg.BUF_LOGITS)[:, :32000]]
        got.append((first, list(tree), out))
        eng.close()
    assert got[0][:2] == got[1][:2]
    for a, b in zip(got[0][2], got[1][2]):
        assert np.array_equal(a, b), np.abs(a - b).max()
