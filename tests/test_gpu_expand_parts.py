"""Child selection where a row's vocabulary is shared by several work-groups (k_expand: parts of about 2048 tokens, at most 16, then several
rounds of a part): vocabularies at the edges of parts and rounds, nodes with one to eight children, two sequences, ties that cross parts."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth

pytestmark = pytest.mark.gpu

# eight children of the root, of which the first four have 8, 3, 1 and 2
TREE = synth.tree_from_paths([str(i) for i in range(8)] + [f"0{i}" for i in range(8)] + [f"1{i}" for i in range(3)] + ["20", "30", "31", "000"])


@pytest.mark.parametrize("vocab", [9, 2047, 2048, 2049, 4096, 4097, 30720, 32768, 32785, 65536, 65553, 70001])
@pytest.mark.parametrize("kind", ["normal", "ties", "last"])
def test_children_of_shared_rows(vocab, kind):
    par, rk = TREE
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, d_ffn=64, vocab=vocab)
    M, B = len(par), 2
    print(s.name, kind, flush=True)
    eng = pkg.Eagle(s, par, rk, max_batch=B, max_seq=128)
    eng.load_weights(synth.iter_weights(s, 61, synth.device_fmt(s)))
    for b in range(B):
        eng.prefill(b, synth.prompt(61, 9, vocab, stream=b))
    eng.draft_tree()
    rng = np.random.default_rng(vocab)
    draft = rng.standard_normal((B, M, vocab)).astype(np.float32)
    if kind == "ties":                                           # a handful of values: the best entries are equal and all over the row
        draft = np.round(draft)
    elif kind == "last":                                         # the best entries side by side at a part's end, the row's end among them
        part = -(-vocab // max(1, min(16, -(-vocab // 2048))))
        for v in range(M):
            end = min(vocab, part * (1 + v % 16)) if part * (v % 16) < vocab else vocab
            draft[:, v, max(0, end - 5):end] += 50.0
    children = [[v for v in range(1, M) if par[v] == p] for p in range(M)]
    for b in range(B):
        eng.set_buffer(pkg.BUF_DRAFT_LOGITS, draft[b], b)
    for _ in range(2):                                           # (the second time over the counters that the first left)
        for level in [-1] + list(range(1, eng.D)):
            eng.expand_level(level)
        for b in range(B):
            tok = eng.get_buffer(pkg.BUF_TREE_TOKENS, b)
            for p in range(M):
                want = np.argsort(-draft[b, p], kind="stable")[:len(children[p])]
                got = [int(tok[v]) for v in sorted(children[p], key=lambda v: rk[v])]
                assert got == list(want), (b, p, got, list(want))
    eng.close()
