"""Commits that move rows (k_outcome / k_accept / k_force_commit, then k_commit): paths over late siblings in every sequence, with cached lengths that
the host hands over (up to four sequences) and that the kernel reads (more), pages of 32 tokens that a tree spans three of, paths of up to 16
rows.  The target's logits are set so that the path is known; moved rows keep their bits, and the oracle, led along the same path, checks the
next step's drafts (features kept at the commit) and target pass (moved cache rows)."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, _check_draft, _check_verify, check_prefill
from oracle.eagle_oracle import Oracle

# two chains of 15 side by side: the second one's nodes are 2, 4, ... 30
TREES = dict(synth.TREES, chains=synth.tree_from_paths(["0" * n for n in range(1, 16)] + ["1" + "0" * n for n in range(15)]))

# tree, sequences, tokens of a page, cache, vocabulary, temperature, prompt of the first sequence
CASES = [("T15", 1, 64, "fp32", 1024, 0.0, 20), ("T15", 4, 64, "fp32", 1024, 1.0, 40), ("T15", 5, 64, "fp32", 1024, 0.0, 50), ("T15", 8, 32, "fp32", 1024, 1.0, 45),
         ("T8", 16, 32, "bf16", 1024, 0.0, 60), ("T15", 6, 64, "fp32", 33000, 1.0, 30), ("B63", 1, 32, "fp32", 1024, 0.0, 29), ("B63", 2, 32, "fp32", 1024, 1.0, 62),
         ("B63", 2, 32, "bf16", 1024, 0.0, 31), ("B63", 2, 32, "fp32", 33000, 1.0, 30), ("chains", 4, 32, "fp32", 1024, 0.0, 33), ("chains", 1, 32, "fp32", 1024, 1.0, 50)]


def _lead(par, rng, last):
    """A path from the root; `last`: over the last child of every node, as far as it goes"""
    path = [0]
    while True:
        kids = [v for v in range(len(par)) if par[v] == path[-1]]
        if not kids or (not last and len(path) > 1 and rng.random() < 0.25):
            return path
        path.append(max(kids) if last else int(rng.choice(kids)))


def test_cases_span_pages_and_move_rows():
    assert len(_lead(TREES["chains"][0], None, True)) == 16
    three = 0
    for tree, B, page, _, _, _, n in CASES:
        path = _lead(TREES[tree][0], None, True)
        assert any(v != i for i, v in enumerate(path))
        three += (n + path[-1]) // page - n // page == 2
    assert three >= 4


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["accept", "static", "force"])
@pytest.mark.parametrize("tree,B,page,kv,vocab,temperature,prompt", CASES)
def test_rows_move(tree, B, page, kv, vocab, temperature, prompt, how):
    par, rk = TREES[tree]
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", vocab=vocab) if vocab == 1024 else \
        replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, d_model=64, n_heads=2, n_kv_heads=1, head_dim=32, d_ffn=64, vocab=vocab)
    M = len(par)
    tol = 2e-2 if kv == "bf16" else 1e-4
    print(s.name, tree, B, "sequences", kv, "temperature", temperature, how, flush=True)
    eng = pkg.Eagle(s, par, rk, max_batch=B, max_seq=192, page_tokens=page, kv_dtype=kv, temperature=temperature, seed=77)
    eng.load_weights(synth.iter_weights(s, 77, synth.device_fmt(s)))
    n_pages = B * eng.pages_per_slot
    eng.set_page_table(np.random.default_rng(n_pages).permutation(n_pages).astype(np.int32))
    W = synth.make_weights(s, 77, synth.oracle_fmt(s))
    orcs = [Oracle(s, W, par, rk, max_seq=192, seq_id=b, temperature=temperature, seed=77, dtype=np.float32, kv_store="bf16" if kv == "bf16" else None) for b in range(B)]
    for b in range(B):
        check_prefill(eng, orcs[b], synth.prompt(77, max(2, prompt - 3 * b), vocab, stream=b), tol, seq=b)
    rng = np.random.default_rng(B)
    sts = [Stats() for _ in range(B)]
    for step in range(3):
        trees = eng.draft_tree()
        for b in range(B):
            _check_draft(eng, orcs[b], sts[b], trees[b], tol, 2e-2, b)
        eng.verify()
        paths, bonus = [], []
        for b in range(B):
            _check_verify(eng, orcs[b], sts[b], tol, b)
            path = _lead(par, rng, (step + b) % 2 == 0)
            kids = {int(trees[b][v]) for v in range(M) if par[v] == path[-1]}
            token = next(t for t in rng.permutation(vocab) if int(t) not in kids)
            logits = np.zeros((M, vocab), np.float32)            # 60 above the rest: 1 - 1e-21 of the probability
            for v, t in zip(path, [int(trees[b][v]) for v in path[1:]] + [int(token)]):
                logits[v, t] = 60.0
            eng.set_buffer(pkg.BUF_LOGITS, logits, b)
            paths.append(path)
            bonus.append(int(token))
        ctx = [o.ctx for o in orcs]
        before = [[{v: eng.get_kv_row(b, l, ctx[b] + v) for v in set(paths[b]) | {-1}} for l in range(s.n_layers)] for b in range(B)]
        if how == "force":
            eng.force_accept(paths, [len(p) for p in paths], bonus)
        else:
            out, lens, got = eng.accept() if how == "accept" else eng.accept_static()
            for b in range(B):
                assert list(got[b][:lens[b]]) == paths[b], (step, b, list(got[b]), paths[b])
                assert list(out[b][:lens[b]]) == [int(trees[b][v]) for v in paths[b][1:]] + [bonus[b]]
        for b in range(B):
            for l in range(s.n_layers):
                for i, v in enumerate([-1] + paths[b]):
                    k, w = eng.get_kv_row(b, l, ctx[b] + i - 1)
                    assert np.array_equal(k, before[b][l][v][0]) and np.array_equal(w, before[b][l][v][1]), (step, b, l, i, v)
            orcs[b].commit(paths[b], bonus[b])
            assert list(eng.get_buffer(pkg.BUF_STATE, b)[:3]) == [len(orcs[b].x), orcs[b].ctx, len(paths[b])]
            assert list(eng.get_buffer(pkg.BUF_TOKENS, b)) == orcs[b].x
    trees = eng.draft_tree()                                     # what the last commit left
    for b in range(B):
        _check_draft(eng, orcs[b], sts[b], trees[b], tol, 2e-2, b)
    eng.close()
