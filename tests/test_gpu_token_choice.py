"""Child selection and acceptance at the edges of their vocabulary ranges (child selection: parts of 2048 entries, several rounds of sixteen beyond
32768; acceptance: a thread owns every 1024th entry, at most 32 of them in registers): the fp32 oracle's own logits, and integer logits full of ties."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import check_prefill
from oracle.eagle_oracle import Oracle
from test_gpu_parity import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [64, 1000, 1024, 1025, 4099, 31999, 32767, 32768, 32769])
@pytest.mark.parametrize("temperature", [0.0, 1.0])
def test_selection_and_acceptance_on_oracle_logits(vocab, temperature):
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, vocab=vocab)
    par, rk = synth.TREES["T26"]
    print(s.name, "temperature", temperature, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=128, temperature=temperature, seed=99)
    eng.load_weights(synth.iter_weights(s, 41, synth.device_fmt(s)))
    orc = Oracle(s, synth.make_weights(s, 41, synth.oracle_fmt(s)), par, rk, max_seq=128, temperature=temperature, seed=99, dtype=np.float32)
    check_prefill(eng, orc, synth.prompt(41, 20, vocab), TOL["fp32"], margin_thr=1e-4)
    for step in range(4):
        eng.draft_tree()
        orc.draft_tree()
        raw = np.zeros((len(par), vocab), np.float32)
        for v, lg in orc.node_logits.items():
            raw[v] = lg
        eng.set_buffer(pkg.BUF_DRAFT_LOGITS, raw)
        for level in [-1] + list(range(1, orc.tree.D)):
            eng.expand_level(level)
        assert list(eng.get_buffer(pkg.BUF_TREE_TOKENS)) == orc.tok, f"step {step}: tree tokens differ"
        eng.verify()
        _, L = orc.verify()
        eng.set_buffer(pkg.BUF_LOGITS, L.astype(np.float32))
        out, ln, path = eng.accept()
        r = orc.accept()
        n = int(ln[0])
        same = [int(v) for v in path[0][:n]] == r["path"] and [int(t) for t in out[0][:n]] == r["emitted"]
        # the same numbers in the same precision: only sums of probabilities are taken in another order (1e-6 relative)
        assert same or r["margin"] < 1e-5, f"step {step}: {path[0][:n]} {out[0][:n]} against {r['path']} {r['emitted']} (margin {r['margin']})"
        if not same:
            break
        orc.commit(r["path"], r["bonus"])
    eng.close()


@pytest.mark.parametrize("vocab", [64, 1025, 32768, 33000])
def test_ties_go_to_the_lowest_token(vocab):
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, vocab=vocab)
    par, rk = synth.TREES["T26"]
    M = len(par)
    eng = pkg.Eagle(s, par, rk, max_seq=128)
    eng.load_weights(synth.iter_weights(s, 43, synth.device_fmt(s)))
    rng = np.random.default_rng(vocab)
    levels = rng.integers(-3, 3, (2 * M, vocab)).astype(np.float32)
    levels[::3] = -np.inf                                        # rows with a handful of finite entries, zeros of both signs among them
    for row in levels[::3]:
        row[rng.choice(vocab, 9, replace=False)] = np.array([0.0, -0.0, 0.0, -0.0, -1.0, -1.0, 2.0, -np.inf, -5.0], np.float32)
    children = [[v for v in range(1, M) if par[v] == p] for p in range(M)]
    for start in range(2):
        eng.reset()
        eng.prefill(0, synth.prompt(43 + start, 12, vocab))
        eng.draft_tree()
        draft, target = np.roll(levels[:M], start, 0), np.roll(levels[M:], start, 0)
        eng.set_buffer(pkg.BUF_DRAFT_LOGITS, draft)
        for level in [-1] + list(range(1, eng.D)):
            eng.expand_level(level)
        tok = eng.get_buffer(pkg.BUF_TREE_TOKENS)
        for p in range(M):
            want = np.argsort(-draft[p], kind="stable")[:len(children[p])]
            got = [int(tok[v]) for v in sorted(children[p], key=lambda v: rk[v])]
            assert got == list(want), (p, got, list(want))
        eng.verify()
        eng.set_buffer(pkg.BUF_LOGITS, target)
        out, ln, path = eng.accept()
        cur, walk, emitted = 0, [0], []
        while True:
            best = int(np.argmax(target[cur]))
            nxt = [v for v in children[cur] if int(tok[v]) == best]
            emitted.append(best)
            if not nxt:
                break
            cur = nxt[0]
            walk.append(cur)
        n = int(ln[0])
        assert [int(v) for v in path[0][:n]] == walk and [int(t) for t in out[0][:n]] == emitted
    eng.close()


@pytest.mark.parametrize("vocab", [64, 1025, 32768, 33000])
@pytest.mark.parametrize("temperature", [0.0, 1.0])
def test_nan_logits_hide_no_other_token(vocab, temperature):
    """Children of rows with NaN among the head's logits are those of the same rows with -inf in their places: NaN in every thread's first
    entry, in the best one's neighbours, in nearly all."""
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, vocab=vocab)
    par, rk = synth.TREES["T26"]
    M = len(par)
    print(s.name, "temperature", temperature, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=128, temperature=temperature, seed=7)
    eng.load_weights(synth.iter_weights(s, 45, synth.device_fmt(s)))
    eng.prefill(0, synth.prompt(45, 12, vocab))
    eng.draft_tree()
    rng = np.random.default_rng(vocab)
    clean = rng.standard_normal((M, vocab)).astype(np.float32)
    dirty = rng.random((M, vocab)) < 0.3
    dirty[0::3, :min(1024, vocab - 16)] = True
    dirty[1::3] = True
    for row in dirty[1::3]:
        row[rng.choice(vocab, 16, replace=False)] = False
    children = [[v for v in range(1, M) if par[v] == p] for p in range(M)]
    assert (vocab - dirty.sum(1)).min() >= max(len(c) for c in children)

    def chosen(masked_with):
        eng.set_buffer(pkg.BUF_DRAFT_LOGITS, np.where(dirty, np.float32(masked_with), clean))
        for level in [-1] + list(range(1, eng.D)):
            eng.expand_level(level)
        return eng.get_buffer(pkg.BUF_TREE_TOKENS).copy()

    tok = chosen(np.nan)
    np.testing.assert_array_equal(tok, chosen(-np.inf))
    for p in range(M):
        got = [int(tok[v]) for v in sorted(children[p], key=lambda v: rk[v])]
        assert len(set(got)) == len(got) and not any(dirty[p][t] for t in got), (p, got)
        if temperature == 0.0:
            assert got == list(np.argsort(np.where(dirty[p], np.inf, -clean[p]), kind="stable")[:len(got)]), (p, got)
    eng.close()


@pytest.mark.parametrize("vocab", [2, 3, 32768, 33000])
@pytest.mark.parametrize("temperature", [0.0, 1.0])
def test_children_name_tokens_of_the_vocabulary(vocab, temperature):
    """Rows of NaN alone, rows with fewer numbers than children, vocabularies with fewer tokens than children."""
    s = replace(synth.SHAPES["tiny"], name=f"tiny-v{vocab}", n_layers=1, vocab=vocab)
    par, rk = synth.TREES["T26"]
    M = len(par)
    print(s.name, "temperature", temperature, flush=True)
    eng = pkg.Eagle(s, par, rk, max_seq=128, temperature=temperature, seed=7)
    eng.load_weights(synth.iter_weights(s, 46, synth.device_fmt(s)))
    eng.prefill(0, [1, 0, 1])
    eng.draft_tree()
    draft = np.full((M, vocab), np.nan, np.float32)
    draft[1::2, vocab // 2] = 1.0
    eng.set_buffer(pkg.BUF_DRAFT_LOGITS, draft)
    for level in [-1] + list(range(1, eng.D)):
        eng.expand_level(level)
    tok = eng.get_buffer(pkg.BUF_TREE_TOKENS)
    assert tok.min() >= 0 and tok.max() < vocab, tok
    for p in range(M):
        got = [int(tok[v]) for v in sorted((v for v in range(1, M) if par[v] == p), key=lambda v: rk[v])]
        if vocab > 4:                                            # the row's number first, then the lowest tokens
            assert got == ([vocab // 2, 0, 1, 2] if p % 2 else [0, 1, 2, 3])[:len(got)], (p, got)
    eng.verify()
    out, ln, path = eng.accept()
    n = int(ln[0])
    assert 1 <= n <= eng.D + 1 and path[0][0] == 0 and all(0 <= int(t) < vocab for t in out[0][:n])
    eng.close()
