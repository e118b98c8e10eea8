"""The large-M GEMM (k_gemm_pf) at the edges of its tiles, against the CPU oracle.  The small models (fp64 oracle): prompt passes whose
rows end inside a 32-row tile, inside a work-group tile (2 or 4 row tiles: all that the planner takes at these widths), at a window
of 512 rows, and beyond one pass of 2048; rows grouped by expert; 4-bit weights; a loss pass of more than 1024 rows; the same with a
bf16 cache.  Wider models (fp32 oracle): the tiles that real widths take, 8 row tiles with all of their waves at work among them;
test_plans.py says which tiles the cases below get."""
from dataclasses import replace

import numpy as np
import pytest

import paper_2401_15077_amd as pkg
import synth
from lockstep import Stats, check_prefill, lockstep_step, lockstep_step_batch
from oracle.eagle_oracle import Oracle, silu, softmax, topk_desc
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


# ----------------------------------------------------------------------------- wider models: the other tiles
def _wide(base, d, ffn, **kw):
    return replace(synth.SHAPES[base], name=f"{base}-d{d}", n_layers=1, d_model=d, d_ffn=ffn, n_heads=d // 64, n_kv_heads=d // 64, head_dim=64, **kw)


DENSE = {"7b-widths": (synth.SHAPES["llama2-7b"].twin(1), (50, 333, 1060)), "d1536": (_wide("mini-gqa", 1536, 4096), (1490,))}
EXPERTS = {"mixtral-widths": (synth.SHAPES["mixtral-8x7b"].twin(1), (300, 700), 31),
           "d256-e8": (replace(synth.SHAPES["mini-moe"], name="mini-moe-e8", n_experts=8, d_ffn=640), (1900,), 37),
           "d768-e4": (_wide("mini-moe", 768, 2048), (1500,), 33),
           # the most experts and choices a model may have (most of the columns hold a few rows), and one choice of an odd number
           "d256-e64-top4": (replace(synth.SHAPES["mini-moe"], name="mini-moe-e64", n_layers=1, n_experts=64, experts_per_tok=4), (3, 40, 150), 44),
           "d256-e3-top1": (replace(synth.SHAPES["mini-moe"], name="mini-moe-e3", n_experts=3, experts_per_tok=1), (1, 200, 900), 40)}
LOSS_ROWS = (300, 500, 1000)


class RowsByExpert(Oracle):
    """The oracle's mixture of experts for many rows: the same sums, an expert's rows multiplied together."""

    def _mlp(self, prefix, x, moe, stage_key):
        if not moe:
            return super()._mlp(prefix, x, moe, stage_key)
        logits = x @ self._lw(prefix, "router").T
        self.router_log[stage_key] = logits
        sel = np.stack([topk_desc(l, self.s.experts_per_tok) for l in logits])
        w = np.stack([softmax(l[e]) for l, e in zip(logits, sel)])
        out = np.zeros_like(x)
        for e in range(self.s.n_experts):
            r, j = np.nonzero(sel == e)
            if r.size:
                g, u = x[r] @ self._lw(prefix, "gate")[e].T, x[r] @ self._lw(prefix, "up")[e].T
                out[r] += w[r, j][:, None] * ((silu(g) * u) @ self._lw(prefix, "down")[e].T)
        return out


def _prompts(shape, rows, seed, oracle):
    par, rk = synth.TREES["T8"]
    print(shape.name, "weights", flush=True)
    W = synth.make_weights(shape, seed, synth.oracle_fmt(shape))
    eng = pkg.Eagle(shape, par, rk, max_seq=max(rows) + 64)
    eng.load_weights(synth.iter_weights(shape, seed, synth.device_fmt(shape)))
    for n in rows:
        orc = oracle(shape, W, par, rk, max_seq=max(rows) + 64, dtype=np.float32)
        print(shape.name, "prompt of", n, flush=True)
        eng.reset()
        err = check_prefill(eng, orc, synth.prompt(seed, n, shape.vocab), TOL["bf16"])
        for key, lg in orc.router_log.items():                  # the comparison says nothing about a row whose experts are a matter of rounding
            top = -np.sort(-lg, axis=1)
            gap = float((top[:, shape.experts_per_tok - 1] - top[:, shape.experts_per_tok]).min())
            assert gap > 1e-4, f"{key}: router gap {gap} in the oracle: take another seed"
        st = Stats()
        lockstep_step(eng, orc, st, TOL["bf16"])
        print(f"max|dL| prompt {err:.2e} verify {st.max_logit_err:.2e} draft {st.max_draft_logit_err:.2e}", flush=True)
    eng.close()


@pytest.mark.parametrize("name", DENSE)
def test_prompt_rows_wider_models(name):
    shape, rows = DENSE[name]
    _prompts(shape, rows, 21, Oracle)


@pytest.mark.parametrize("name", EXPERTS)
def test_expert_rows_wider_models(name):
    shape, rows, seed = EXPERTS[name]
    _prompts(shape, rows, seed, RowsByExpert)


def test_loss_rows_at_7b_widths():
    shape = synth.SHAPES["llama2-7b"].twin(1)
    eng = _engine(shape, head_loss_rows=max(LOSS_ROWS))
    Wdev, W64 = _lm_head(shape, 5)
    eng.load_named("lm_head", Wdev)
    W64 = W64.astype(np.float64)
    for rows in LOSS_ROWS:
        print("loss of", rows, flush=True)
        f, fhat = _features(rows, shape.d_model, rows, 0.6)
        _check(eng, W64, f, fhat, 0.1, "7B widths")
    eng.close()


@pytest.mark.parametrize("kv", ["fp32", "bf16"])
@pytest.mark.parametrize("batch,tree", [(2, "T26"), (4, "T26"), (2, "B63"), (40, "root")])
def test_batched_verify(batch, tree, kv):
    """52, 104, 126 and 40 verify rows of several sequences through the large-M GEMM, LM head over all rows included; then a vanilla step."""
    s = synth.SHAPES["mini-gqa"]
    par, rk = synth.TREES[tree]
    W = synth.make_weights(s, 15, synth.oracle_fmt(s))
    eng = pkg.Eagle(s, par, rk, max_batch=batch, max_seq=256, kv_dtype=kv)
    eng.load_weights(synth.iter_weights(s, 15, synth.device_fmt(s)))
    orcs = [Oracle(s, W, par, rk, max_seq=256, dtype=np.float64, kv_store="bf16" if kv == "bf16" else None, seq_id=b) for b in range(batch)]
    for b, orc in enumerate(orcs):
        check_prefill(eng, orc, synth.prompt(15 + b, 30 + (17 * b) % 70, s.vocab), TOL["bf16"], seq=b)
    sts = [Stats() for _ in orcs]
    for _ in range(3):
        lockstep_step_batch(eng, orcs, sts, TOL["bf16"])
    eng.vanilla_step()                                          # the target alone: the root's row of the next verify pass
    err = 0.0
    for b, orc in enumerate(orcs):
        orc.draft_tree()
        err = max(err, float(np.abs(eng.get_buffer(pkg.BUF_VANILLA_LOGITS, b) - orc.verify()[1][0]).max()))
    print(f"max|dL| {max(st.max_logit_err for st in sts):.2e} vanilla {err:.2e}", flush=True)
    assert err <= TOL["bf16"]
    eng.close()


# ----------------------------------------------------------------------------- a bf16 cache
# The oracle rounds K and V as the library does; an entry within rounding of a tie may go the other way on the two sides (one
# bf16 ulp of that entry), which the tolerance of the bf16 models covers at these widths (the fp32 model's test of the bf16 cache
# takes the same).
@pytest.mark.parametrize("rows", [33, 64, 65, 129, 513, 1100])
def test_prompt_rows_bf16_cache(rows):
    """bf16 weights with a bf16 cache: sums in one order, passes of 512 rows, k_gemm up to 64 rows."""
    s, eng, orc = make_pair("mini-gqa", "T8", seed=14, max_seq=1200, kv_dtype="bf16")
    print("prompt of", rows, flush=True)
    check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), TOL["bf16"])
    st = Stats()
    for _ in range(3):
        lockstep_step(eng, orc, st, TOL["bf16"])
    eng.close()


@pytest.mark.parametrize("rows", [7, 131, 600])
def test_expert_rows_bf16_cache(rows):
    s, eng, orc = make_pair("mini-moe", "T8", seed=16, max_seq=700, kv_dtype="bf16")
    print("prompt of", rows, flush=True)
    check_prefill(eng, orc, synth.prompt(rows + 5, rows, s.vocab), TOL["bf16"])
    lockstep_step(eng, orc, Stats(), TOL["bf16"])
    eng.close()


@pytest.mark.parametrize("rows", [20, 33, 70, 200])
def test_int4_prompt_rows_bf16_cache(rows):
    """4-bit weights with a bf16 cache: 32 rows at a time, codes that expand around 128."""
    s = synth.SHAPES["mini-gqa"].twin(2)
    par, rk = synth.TREES["T8"]
    eng = pkg.Eagle(s, par, rk, max_seq=300, weight_bits=4, kv_dtype="bf16")
    eng.load_weights(synth.iter_weights(s, 62, synth.device_fmt(s)))
    orc = Oracle(s, quantize_model(synth.make_weights(s, 62, synth.oracle_fmt(s))), par, rk, max_seq=300, dtype=np.float64, kv_store="bf16")
    print("prompt of", rows, flush=True)
    err = check_prefill(eng, orc, synth.prompt(rows, rows, s.vocab), TOL["bf16"])
    st = Stats()
    for _ in range(3):
        lockstep_step(eng, orc, st, TOL["bf16"])
    print(f"max|dL| prompt {err:.2e} verify {st.max_logit_err:.2e}", flush=True)
    eng.close()
