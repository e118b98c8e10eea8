"""Dense models with a bf16 cache keep the order and the rounding of their sums: what the library returned for such a model before, it returns bit for
bit.  A model's checksums (prompt logits; draft logits, target logits and features of the last of four steps; logits of a plain step behind
them) stand here as they were taken; contexts of 1 to 16 key splits, prompts of one and of several passes, both weight formats, one to
four sequences.  (Two correct orders differ by 1e-6 at these sizes, and by more where the cache rounds a key the other way.)"""
import zlib
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from plans import Plans

# heads, key heads, head dimension, weight bits, tree, sequences, prompt, checksum
CASES = [(8, 8, 64, 16, "T15", 1, 20, 1858644574), (8, 2, 128, 16, "T26", 1, 90, 2641670117), (16, 4, 64, 4, "T26", 1, 31, 1099901717), (8, 2, 128, 16, "T10", 4, 300, 1270259743),
         (8, 2, 64, 16, "T26", 1, 950, 1738170599), (8, 2, 128, 16, "T26", 1, 1020, 1651703197), (8, 2, 64, 16, "T15", 1, 1150, 2551763012), (8, 4, 32, 16, "T26", 1, 1270, 3779072706),
         (8, 2, 128, 4, "T26", 1, 1400, 166373955), (8, 2, 128, 16, "chain5", 2, 1530, 793747279), (8, 8, 128, 16, "T26", 1, 1660, 1533529701), (8, 2, 64, 4, "chain5", 2, 1780, 1707420727),
         (8, 2, 32, 16, "B63", 1, 1900, 922800457), (4, 2, 128, 16, "T26", 4, 2050, 2579053517), (16, 16, 64, 16, "T26", 1, 2600, 82818660)]


def checksum(heads, kv_heads, dh, bits, tree, B, prompt):
    s = replace(synth.SHAPES["mini-gqa"], name=f"kept-h{heads}x{dh}", n_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_model=heads * dh, d_ffn=512, vocab=2000)
    par, rk = synth.TREES[tree]
    print(s.name, bits, tree, B, prompt, flush=True)
    eng = pkg.Eagle(s, par, rk, max_batch=B, max_seq=prompt + 96, weight_bits=bits, kv_dtype="bf16")
    eng.load_weights(synth.iter_weights(s, 83, synth.device_fmt(s)))
    out = []
    for b in range(B):
        eng.prefill(b, synth.prompt(83, prompt - 7 * b, s.vocab, stream=b))
        out.append(eng.get_buffer(pkg.BUF_VANILLA_LOGITS, b))
    for _ in range(4):
        tokens, lens, _ = eng.step()
        out += [tokens[b, :lens[b]] for b in range(B)]
    for b in range(B):
        out += [eng.get_buffer(pkg.BUF_DRAFT_LOGITS, b)[sorted({int(p) for p in par[1:]})], eng.get_buffer(pkg.BUF_LOGITS, b), eng.get_buffer(pkg.BUF_FEATURES, b)]
    eng.vanilla_step()
    out += [eng.get_buffer(pkg.BUF_VANILLA_LOGITS, b) for b in range(B)]
    eng.close()
    crc = 0
    for a in out:
        crc = zlib.crc32(np.ascontiguousarray(a).tobytes(), crc)
    return crc


def test_cases_span_all_numbers_of_splits(tmp_path):
    plans = Plans(str(tmp_path))
    got = {plans.attn_splits(True, prompt + 64, heads * B) for heads, _, _, _, _, B, prompt, _ in CASES}
    assert got >= {1, 2, 8, 9, 10, 11, 12, 13, 14, 15, 16}, got


@pytest.mark.gpu
@pytest.mark.parametrize("heads,kv_heads,dh,bits,tree,B,prompt,want", CASES)
def test_outputs_keep_their_bits(heads, kv_heads, dh, bits, tree, B, prompt, want):
    assert checksum(heads, kv_heads, dh, bits, tree, B, prompt) == want
