"""The bf16 LM head of vocabularies so large that the work-groups' shares of it are no longer found by a multiplication (csrc/plans.h, share_of: up to
3248 row blocks of 32 tokens, then the longer shares stand in front): every logit of both sides of that line, ends inside a block and inside
four tokens."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [103930, 103936, 103937, 104003, 128256])
def test_logits_of_every_row(vocab):
    s = replace(synth.SHAPES["mini-gqa"], name=f"bf16-v{vocab}", n_layers=1, d_model=128, n_heads=2, n_kv_heads=1, head_dim=64, d_ffn=128, vocab=vocab)
    par, rk = synth.TREES["chain5"]
    print(s.name, flush=True)
    B = 5                                                        # verify passes of 30 rows
    eng = pkg.Eagle(s, par, rk, max_batch=B, max_seq=64)
    eng.load_weights(synth.iter_weights(s, 79, synth.device_fmt(s)))
    W = synth.gen_tensor(s, 79, synth.tensor_specs(s)[1], "bf16_f32").astype(np.float64)
    for b in range(B):
        first = eng.prefill(b, synth.prompt(79, 3 + 7 * b, vocab, stream=b))
        assert first == int(np.argmax(eng.get_buffer(pkg.BUF_VANILLA_LOGITS, b)))
    eng.draft_tree()
    eng.verify()
    for b in range(B):
        # x passes as two bf16 planes (2^-17 of it at most are left), 128 products each are summed in fp32 (2^-24 times 2 x 128 terms)
        for feat, logits, rows in ((pkg.BUF_FEATURES, pkg.BUF_LOGITS, 6), (pkg.BUF_DRAFT_FEATURES, pkg.BUF_DRAFT_LOGITS, 5)):
            x, got = eng.get_buffer(feat, b)[:rows].astype(np.float64), eng.get_buffer(logits, b)[:rows].astype(np.float64)
            err = np.abs(got - x @ W.T)
            assert (err <= 2.0 ** -15 * (np.abs(x) @ np.abs(W).T)).all(), (b, err.max())
    eng.close()
