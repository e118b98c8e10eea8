"""The library's work-split planners (csrc/plans.h, host arithmetic only) compiled into a small shared object and called from
Python, so that tests can say which tile shape and how many K slices a matrix product gets."""
import ctypes
import os
import subprocess
from collections import namedtuple

import paper_2401_15077_amd as pkg

Plan = namedtuple("Plan", "S kps rbw mw")

_SHIM = r"""
#include "plans.h"
static void put(const GemmPlan& p, int* o) { o[0] = p.S; o[1] = p.ks_per_split; o[2] = p.rbw; o[3] = p.mw; }
extern "C" {
int shim_large_m(int MT, int big, int fixed, int q4) { return plan_is_large_m(MT, big != 0, fixed != 0, q4 != 0); }
void shim_pf(int NRB, int KS, int MT, int n_cu, int fused, int q4, int fixed, int* o) { put(plan_pf(NRB, KS, MT, n_cu, fused != 0, q4 != 0, fixed != 0), o); }
void shim_moe(const int* a, int* o) {
  const PlanMoe p = plan_moe(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]);
  put(p.gu, o); put(p.dn, o + 4); o[8] = p.cols;
}
int shim_whole_k(int NRB, int KS, int planes, int n_cu) { return plan_is_whole_k(NRB, KS, planes, n_cu); }
int shim_plain_loads(int NRB, int MT, int M, int n_cu, int S, int rbw, int mw) { GemmPlan p{}; p.S = S; p.rbw = rbw; p.mw = mw; return plan_pf_plain_loads(NRB, MT, M, n_cu, p); }
int shim_one_round(int NRB, int cols, int n_cu, int S, int rbw, int mw) { GemmPlan p{}; p.S = S; p.rbw = rbw; p.mw = mw; return plan_pf_one_round(NRB, cols, n_cu, p); }
int shim_wk(int NRB, int KS, int MT, int n_cu, int big, int fixed, int q4) { return plan_is_wk(NRB, KS, MT, n_cu, big != 0, fixed != 0, q4 != 0); }
// matrices: row blocks and k-steps of n of them, gate/up and down of an expert first; bf16 weights (one plane), two planes of activations
int shim_experts_in_two(const int* m, int n, int n_cu, int* o) {
  size_t pt = 0;
  for (int i = 0; i < n; ++i) pt = std::max(pt, plan2(m[2 * i], m[2 * i + 1], 2, 1, n_cu).S * (size_t)m[2 * i] * 32 * 32);
  const PlanXK dn = plan_streamed(m[2], m[3], 2, 1, n_cu, pt);
  const int grid = std::max(n_cu, (m[0] + 3) / 4);
  o[0] = (m[0] + grid - 1) / grid; o[1] = dn.S; o[2] = dn.nrmax;
  return plan_experts_in_two(m[0], m[1], m[2], m[3], 2, 1, n_cu, pt);
}
uint32_t shim_div(uint32_t x, uint32_t n) { return div_magic(x, magic_of(n)); }
int shim_div_holds(uint64_t x, uint32_t n) { return magic_holds(x, n); }
int shim_shares(uint32_t units, uint32_t n, uint32_t* o) {
  const Share s = share_of(units, n);
  for (uint32_t i = 0; i <= n; ++i) o[i] = share_begin(i, units, s.a, s.b);
  return s.b == SHARE_IN_TURN;
}
void shim_staged(int NRB, int KS, int planes, int n_cu, int q4, int* o) {
  const Plan2 p = plan2(NRB, KS, planes, 1, n_cu, q4 != 0);
  o[0] = p.S; o[1] = p.kparts;
}
int shim_logits_q4(int NRB, int KS, int n_cu, int fixed) { return plan_is_logits_q4(NRB, n_cu, plan2(NRB, KS, 2, 1, n_cu, true), fixed != 0); }
int shim_short_prompt(int rows, int d, int f32, int q4, int fixed, int experts) {
  return plan_is_short_prompt(rows, d, f32 ? 6 : 3, f32 != 0, q4 != 0, fixed != 0, experts);
}
int shim_attn_splits(int fixed, int tokens, int units, int n_cu) { return plan_attn_splits(fixed != 0, tokens, units, n_cu); }
int shim_prompt_attn(int rows, int heads, int n_cu) { return plan_is_prompt_attn(rows, heads, n_cu); }
int shim_q4_x_span(int planes, int KS) { return q4_x_span(planes, KS); }
int shim_q4_w_span(int nr, int KS) { return q4_w_span(nr, KS); }
int shim_moe_tiles(int M, int topk, int E) { return moe_tiles(M, topk, E); }
}
"""


class Plans:
    def __init__(self, folder):
        src, lib = os.path.join(folder, "shim.cpp"), os.path.join(folder, "shim.so")
        with open(src, "w") as f:
            f.write(_SHIM)
        inc = os.path.join(os.path.dirname(pkg.__file__), "csrc")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", inc, src, "-o", lib])
        self.lib = ctypes.CDLL(lib)
        self.lib.shim_div.argtypes = [ctypes.c_uint32, ctypes.c_uint32]
        self.lib.shim_div.restype = ctypes.c_uint32
        self.lib.shim_div_holds.argtypes = [ctypes.c_uint64, ctypes.c_uint32]

    def large_m(self, MT, big=True, fixed=False, q4=False):
        return bool(self.lib.shim_large_m(MT, big, fixed, q4))

    def pf(self, NRB, KS, MT, fused=False, q4=False, fixed=False, n_cu=256):
        o = (ctypes.c_int * 4)()
        self.lib.shim_pf(NRB, KS, MT, n_cu, fused, q4, fixed, o)
        return Plan(*o)

    def plain_loads(self, NRB, rows, p, n_cu=256):
        """Whether a launch of the large-M GEMM with plan `p` brings its tiles by plain loads (else by buffer loads)"""
        return bool(self.lib.shim_plain_loads(NRB, (rows + 31) // 32, rows, n_cu, p.S, p.rbw, p.mw))

    def experts_plain_loads(self, s, rows, n_cu=256):
        """The same of the grouped gate/up and down launches of a mixture: (gate/up, down)"""
        gu, dn, cols = self.moe(s.d_model, s.d_ffn, (rows + 31) // 32 * 32, s.experts_per_tok, s.n_experts, n_cu)
        cols = min(cols, rows * s.experts_per_tok)
        return tuple(bool(self.lib.shim_one_round(NRB, cols, n_cu, p.S, p.rbw, p.mw)) for NRB, p in ((2 * s.d_ffn // 32, gu), (s.d_model // 32, dn)))

    def moe(self, d, F, M, topk, E, n_cu=256):
        """-> (gate/up plan, down plan, columns) for M rows of a mixture of E experts with widths d and F"""
        a = (ctypes.c_int * 8)(2 * F // 32, d // 16, d // 32, F // 16, M, topk, E, n_cu)
        o = (ctypes.c_int * 9)()
        self.lib.shim_moe(a, o)
        return Plan(*o[:4]), Plan(*o[4:8]), o[8]

    def shares(self, units, n):
        """Where the n shares of `units` units begin (and the last one ends), and whether longer and shorter ones take turns"""
        o = (ctypes.c_uint32 * (n + 1))()
        in_turn = bool(self.lib.shim_shares(units, n, o))
        return list(o), in_turn

    def attn_splits(self, fixed, tokens, units, n_cu=256):
        """Work-groups that share the keys of `units` (head, sequence, row block) triples"""
        return self.lib.shim_attn_splits(fixed, tokens, units, n_cu)

    def short_prompt(self, s, rows, kv="fp32", bits=16):
        """Whether a prompt pass of `rows` rows takes the fused kernels of the decoding steps"""
        return bool(self.lib.shim_short_prompt(rows, s.d_model, s.dtype == "fp32", bits == 4, kv == "bf16" and s.n_experts == 0, s.n_experts))

    def staged_q4(self, NRB, KS, n_cu=256):
        """(K slices, parts of K in a work-group) of the split-K kernel that holds the activations in LDS, 4-bit weights"""
        o = (ctypes.c_int * 2)()
        self.lib.shim_staged(NRB, KS, 2, n_cu, 1, o)
        return tuple(o)

    def logits_q4(self, NRB, KS, fixed=False, n_cu=256):
        """Whether a 4-bit LM head of NRB row blocks runs over all of K in a work-group of four (k2_logits_q4)"""
        return bool(self.lib.shim_logits_q4(NRB, KS, n_cu, fixed))

    def whole_k(self, NRB, KS, planes, n_cu=256):
        return bool(self.lib.shim_whole_k(NRB, KS, planes, n_cu))

    def whole_k_rows(self, NRB, KS, rows, n_cu=256, big=True, fixed=False, q4=False):
        """Whether a gate/up product of `rows` rows runs over all of K in a work-group (k_gemm_wk)"""
        return bool(self.lib.shim_wk(NRB, KS, (rows + 31) // 32, n_cu, big, fixed, q4))

    def experts_in_two(self, s, n_cu=256):
        """Passes of up to 32 rows: (most gate/up row blocks of a work-group, K slices and most row blocks of down) where all experts share
        two launches a layer, else None"""
        a, d = s.n_heads * s.head_dim, s.d_model
        m = [(2 * s.d_ffn // 32, d // 16), (d // 32, s.d_ffn // 16), ((s.vocab + 31) // 32, d // 16), (d // 32, 2 * d // 16),
             ((a + 2 * s.n_kv_heads * s.head_dim) // 32, d // 16), (d // 32, a // 16)]
        o = (ctypes.c_int * 3)()
        two = self.lib.shim_experts_in_two((ctypes.c_int * 12)(*[x for r in m for x in r]), len(m), n_cu, o)
        return tuple(o) if two and s.n_experts > 1 else None

    def prompt_attn(self, heads, rows, max_seq, n_cu=256):
        """-> for every pass of a prompt of a bf16 model with an fp32 cache (eagle_prefill: whole windows of 512 rows, at most 2048, passes of
        about equal length): its first row, its rows and whether it takes the attention kernel of 128 rows a work-group"""
        chunk = min(2048, -(-max_seq // 512) * 512)
        n = -(-rows // chunk)
        each = -(-(-(-rows // n)) // 512) * 512
        return [(at, min(each, rows - at), bool(self.lib.shim_prompt_attn(min(each, rows - at), heads, n_cu))) for at in range(0, rows, each)]

    def q4_spans(self, planes, row_blocks, KS):
        return self.lib.shim_q4_x_span(planes, KS), self.lib.shim_q4_w_span(row_blocks, KS)

    def moe_tiles(self, M, topk, E):
        return self.lib.shim_moe_tiles(M, topk, E)

    def prompt(self, s, rows, kv="fp32", bits=16):
        """matrix -> plan of one prompt pass of `rows` rows of a bf16 model (matrices that do not take the large-M GEMM are left out, gate/up
        that runs over all of K in a work-group among them)"""
        MT, fixed = (rows + 31) // 32, kv == "bf16" and s.n_experts == 0
        d, a, q4, out = s.d_model, s.n_heads * s.head_dim, bits == 4, {}
        kw = dict(q4=q4, fixed=fixed)
        if self.large_m(MT, bits == 16, fixed, q4):
            out["qkv"] = self.pf((a + 2 * s.n_kv_heads * s.head_dim) // 32, d // 16, MT, **kw)
            out["o"], out["fc"] = self.pf(d // 32, a // 16, MT, **kw), self.pf(d // 32, 2 * d // 16, MT, **kw)
            if not s.n_experts:
                if not self.whole_k_rows(2 * s.d_ffn // 32, d // 16, rows, **kw):
                    out["gate_up"] = self.pf(2 * s.d_ffn // 32, d // 16, MT, fused=True, **kw)
                out["down"] = self.pf(d // 32, s.d_ffn // 16, MT, **kw)
        if s.n_experts:                         # experts are grouped whatever the rows
            out["gate_up"], out["down"], _ = self.moe(d, s.d_ffn, 32 * MT, s.experts_per_tok, s.n_experts)
        return out

    def loss(self, s, rows):
        """The two products of one loss pass of `rows` label rows: LM head over labels and predictions, and its transpose."""
        mt = (rows + 31) // 32
        return {"lm_head": self.pf((s.vocab + 31) // 32, s.d_model // 16, 2 * mt), "lm_head_T": self.pf(s.d_model // 32, s.vocab // 16, mt)}
