"""The loss rows' kernel at its edges: whole and ragged blocks of 64 rows, vocabularies of a part of a thread's first chunk up to
all four chunks, more features than one round of the work-group, and caller's buffers that start at any float."""
from dataclasses import replace

import numpy as np
import pytest

import synth
from oracle import head_loss as hl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,d", [(64, 64, 256), (65, 8256, 256), (127, 8192, 256), (193, 512, 256), (3, 32768, 256), (66, 128, 4160)])
def test_rows_vocabularies_and_unaligned_buffers(rows, vocab, d):
    import torch
    import paper_2401_15077_amd as pkg
    shape = replace(synth.SHAPES["mini-gqa"], name="loss-rows", vocab=vocab, d_model=d)
    parent, rank = synth.TREES["T8"]
    eng = pkg.Eagle(shape, parent, rank, max_batch=1, max_seq=128, head_loss_rows=1)
    spec = [s for s in synth.tensor_specs(shape) if s[0] == "lm_head"][0]
    eng.load_named("lm_head", synth.gen_tensor(shape, 3, spec, synth.device_fmt(shape)))
    W64 = synth.gen_tensor(shape, 3, spec, synth.oracle_fmt(shape)).astype(np.float64)
    rng = np.random.default_rng(rows)
    f = rng.standard_normal((rows, d)).astype(np.float32)
    fhat = (f + 0.7 * rng.standard_normal((rows, d))).astype(np.float32)
    ref, gref = hl.head_loss(f, fhat, W64, 0.1), hl.head_loss_grad(f, fhat, W64, 0.1)

    def shifted(x):                                     # the same rows, one float behind an aligned start
        t = torch.zeros(x.size + 1, dtype=torch.float32, device=eng.device)
        t[1:] = torch.from_numpy(x).to(eng.device).reshape(-1)
        return t[1:].view(x.shape)

    tf, th, tg = shifted(f), shifted(fhat), shifted(np.zeros_like(f))
    guard = tg._base
    L, Lr, Lc = eng.head_loss_device(tf, th, tg, 0.1)
    g = tg.cpu().numpy()
    # logits carry the two-piece rounding of the activations (2^-16 relative), as do the logits' gradients; the sums are fp32
    assert abs(Lr - ref["L_reg"]) <= 2e-5 * abs(ref["L_reg"]) and abs(Lc - ref["L_cls"]) <= 2e-4 * abs(ref["L_cls"]) and abs(L - ref["L"]) <= 2e-4 * abs(ref["L"])
    assert np.abs(g - gref).max() <= 1e-4 * np.abs(gref).max()
    assert float(guard[0]) == 0.0                       # nothing is written in front of the buffer
    # the same bits as from aligned buffers
    (L2, Lr2, Lc2), g2 = eng.head_loss(f, fhat, 0.1)
    assert (L, Lr, Lc) == (L2, Lr2, Lc2)
    np.testing.assert_array_equal(g, g2)
    eng.close()
