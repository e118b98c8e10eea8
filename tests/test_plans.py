"""The work splits of the matrix products (csrc/plans.h): every split covers K in whole units, every tile shape is one that the
library launches, grouped experts stay within the columns and tiles that the workspace holds."""
import random
from dataclasses import replace

import pytest

import synth
from plans import Plans
from test_gpu_experts_in_two import CASES as IN_TWO, shape_of as mixture_of
from test_gpu_large_m import DENSE, EXPERTS, LOSS_ROWS
from test_gpu_tile_loads import CASES as TILE_LOADS, shape_of
from test_gpu_whole_k_rows import CASES as WHOLE_K

SHAPES_16 = {(4, 1), (3, 1), (4, 2), (3, 2), (4, 4), (3, 4), (2, 4)}     # what gemm() launches
SHAPES_4 = {(2, 2)}
SHAPES_MOE = {(4, 2), (3, 2), (4, 4), (3, 4), (2, 4)}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return Plans(str(tmp_path_factory.mktemp("plans")))


def _sizes(rng, unit):
    """row blocks, k-steps (a multiple of `unit`), row tiles: spread over their logarithm"""
    return int(2 ** rng.uniform(1, 11)), unit * max(1, int(2 ** rng.uniform(0, 9))), int(2 ** rng.uniform(0, 6.01))


def test_splits_cover_k_in_whole_units_and_use_launched_tiles(plans):
    rng, seen = random.Random(1), {False: set(), True: set()}
    for _ in range(20000):
        q4, fixed = rng.random() < 0.3, rng.random() < 0.3
        NRB, KS, MT = _sizes(rng, 8 if q4 else 4)
        MT = MT if q4 else max(2, MT)
        p = plans.pf(NRB, KS, MT, fused=rng.random() < 0.5, q4=q4, fixed=fixed and not q4, n_cu=rng.choice([256, 256, 256, 64, 32]))
        assert 1 <= p.S <= 16 and p.kps % (8 if q4 else 4) == 0 and (p.S - 1) * p.kps < KS <= p.S * p.kps, (NRB, KS, MT, p)
        assert q4 or (p.mw == 1) == (MT <= 2), (NRB, KS, MT, p)
        seen[q4].add((p.rbw, p.mw))
    assert seen[False] == SHAPES_16 and seen[True] == SHAPES_4      # no shape is launched that no size takes


def test_fixed_sums_take_their_slices_whatever_tile_serves_them(plans):
    """Dense models with a bf16 cache: the K slices do not depend on whether the epilogue is fused."""
    rng = random.Random(2)
    for _ in range(3000):
        NRB, KS, MT = _sizes(rng, 4)
        a, b = (plans.pf(NRB, KS, max(2, MT), fused=f, fixed=True) for f in (False, True))
        assert (a.S, a.kps) == (b.S, b.kps)


def test_expert_columns_and_tiles_hold_any_routing(plans):
    rng, seen = random.Random(3), set()
    for _ in range(4000):
        E = rng.choice([2, 4, 8, 16, 64])
        k = rng.randint(1, min(4, E))
        M = 32 * int(2 ** rng.uniform(0, 6.01))
        d, F = 64 * int(2 ** rng.uniform(0, 7)), 64 * int(2 ** rng.uniform(0, 8))
        gu, dn, cols = plans.moe(d, F, M, k, E)
        assert gu.S == 1 and gu.mw == dn.mw and cols <= 256
        seen |= {(gu.rbw, gu.mw), (dn.rbw, dn.mw)}
        # rows per expert: even, one expert with all rows, random subsets
        rows = rng.randint(max(1, M - 31), M)
        counts = [0] * E
        bias = [rng.random() ** rng.choice([0, 1, 6]) for _ in range(E)]
        for _ in range(rows):
            for e in sorted(range(E), key=lambda e: rng.random() * bias[e])[-k:]:
                counts[e] += 1
        rt = 2 * gu.mw
        assert sum((c + 32 * rt - 1) // (32 * rt) for c in counts) <= cols
        assert sum((c + 31) // 32 for c in counts) <= plans.moe_tiles(M, k, E)
    assert seen == SHAPES_MOE


def test_expert_columns_are_not_wider_than_an_experts_rows(plans):
    """Columns of eight row tiles only where an expert has more than four on average: waves without a live tile multiply nothing."""
    for E, k in ((4, 2), (8, 2), (16, 1), (64, 4)):
        for M in range(32, 2049, 32):
            tiles = -(-M * k // (32 * min(E, M * k)))
            for d, F in ((256, 320), (4096, 14336), (2048, 1408)):
                gu, dn, _ = plans.moe(d, F, M, k, E)
                assert gu.mw == 2 or tiles > 4, (E, k, M, d, F, gu)


def test_oracle_cases_reach_every_tile(plans):
    """What the oracle tests of test_gpu_large_m.py run: every tile shape of the 16-bit kernels, with and without split K, the tiles of
    8 row tiles (mw 4) with all waves at work, a last column that is partly filled, and SwiGLU in the epilogue."""
    dense = [(m, p, rows) for s, lens in DENSE.values() for rows in lens for m, p in plans.prompt(s, rows).items()]
    tiles = {(p.rbw, p.mw) for _, p, _ in dense}
    assert tiles == SHAPES_16
    wide = [(m, p, rows) for m, p, rows in dense if (p.rbw, p.mw) == (4, 4)]
    assert any(p.S > 1 for _, p, _ in wide) and any(m == "gate_up" and p.S == 1 for m, p, _ in wide)
    assert any((rows + 31) // 32 > 8 and ((rows + 31) // 32) % 8 not in (0, 7) for _, _, rows in wide)
    # at LLaMA2-7B widths a prompt of some thousand rows takes the widest tile for every matrix
    s, lens = DENSE["7b-widths"]
    assert {(p.rbw, p.mw) for p in plans.prompt(s, lens[-1]).values()} == {(4, 4)}
    experts = [p for s, lens, _ in EXPERTS.values() for rows in lens for m, p in plans.prompt(s, rows).items() if m in ("gate_up", "down")]
    assert {(p.rbw, p.mw) for p in experts} >= {(4, 2), (4, 4), (3, 4), (2, 4)} and any(p.S > 1 and p.mw == 4 for p in experts)
    loss = [plans.loss(synth.SHAPES["llama2-7b"], rows) for rows in LOSS_ROWS]
    assert any(l["lm_head"].mw == 4 and l["lm_head"].S == 1 for l in loss) and any(l["lm_head_T"].mw == 4 and l["lm_head_T"].S > 1 for l in loss)
    # the small models of that file: tiles of two and four row tiles only
    small = [plans.prompt(synth.SHAPES["mini-gqa"], rows) for rows in range(33, 2049, 32)]
    assert {(p.rbw, p.mw) for l in small for p in l.values()} == {(3, 1), (3, 2)}


def _row_blocks(s):
    a = s.n_heads * s.head_dim
    return {"qkv": (a + 2 * s.n_kv_heads * s.head_dim) // 32, "o": s.d_model // 32, "fc": s.d_model // 32, "gate_up": 2 * s.d_ffn // 32, "down": s.d_model // 32}


def test_launches_that_bring_their_tiles_by_plain_loads(plans):
    """Two- and four-wave work-groups in a single round of them, but for one column of four tiles with 16 rows or more beyond the
    end; the cases of test_gpu_tile_loads.py take both ways with every such tile."""
    def ways(s, rows):
        blocks = _row_blocks(s)
        return {m: (p, plans.plain_loads(blocks[m], rows, p)) for m, p in plans.prompt(s, rows).items()}

    for name in ("llama2-7b", "llama2-13b"):
        for rows in (40, 64, 113, 128, 161, 192, 256):
            assert all(plain for p, plain in ways(synth.SHAPES[name], rows).values() if p.mw <= 2), (name, rows)
        for rows in (65, 72, 96, 104, 112):
            assert not any(plain for _, plain in ways(synth.SHAPES[name], rows).values()), (name, rows)
    for rows in (700, 1024):
        w = ways(synth.SHAPES["llama2-7b"], rows)
        assert w["o"][1] and not w["gate_up"][1]               # one round of O's work-groups, three of gate/up's
    assert not any(plain for p, plain in ways(synth.SHAPES["llama2-70b"], 2011).values() if p.mw == 4)
    seen = {(p.rbw, p.mw, m == "gate_up" and p.S == 1, plain) for d, ffn, lens in TILE_LOADS for rows in lens for m, (p, plain) in ways(shape_of(d, ffn), rows).items()}
    assert seen >= {(3, 1, False, True), (3, 1, True, True), (4, 1, False, True), (3, 2, False, True), (3, 2, True, True), (4, 2, False, True), (4, 2, True, True),
                    (3, 2, False, False), (3, 2, True, False), (4, 2, False, False)}, seen


def test_expert_launches_that_bring_their_tiles_by_plain_loads(plans):
    """A single round of work-groups, columns beyond rows x choices not counted; the oracle cases take both ways."""
    narrow, mixtral = EXPERTS["d256-e64-top4"][0], synth.SHAPES["mixtral-8x7b"]
    assert plans.experts_plain_loads(narrow, 3) == (True, True) and plans.experts_plain_loads(narrow, 150) == (False, False)
    assert plans.experts_plain_loads(mixtral, 1) == (True, True) and plans.experts_plain_loads(mixtral, 300) == (False, False)
    seen = {plain for s, lens, _ in EXPERTS.values() for rows in lens for plain in plans.experts_plain_loads(s, rows)}
    assert seen == {True, False}


WK_LAUNCHED = {(3, 2), (3, 3), (3, 4), (4, 2)}                           # (most row blocks of a work-group, row tiles) that gemm_wk() launches


@pytest.mark.parametrize("n_cu", [256, 64])
def test_whole_k_gate_up_gives_every_work_group_what_it_is_built_for(plans, n_cu):
    """Accepted sizes leave a work-group NRMAX - 1 or NRMAX row blocks, with a kernel for that NRMAX and the row tiles; everything else
    that the large-M GEMM serves is refused."""
    seen = set()
    for NRB in range(n_cu, 5 * n_cu + 2):
        for KS in (16, 64, 192, 196, 256, 320, 512, 640, 768, 1024):
            for rows in (1, 32, 33, 64, 65, 96, 97, 128, 129, 512):
                MT = (rows + 31) // 32
                if not plans.whole_k_rows(NRB, KS, rows, n_cu):
                    continue
                shares = {(w + 1) * NRB // n_cu - w * NRB // n_cu for w in range(n_cu)}
                most = -(-NRB // n_cu)
                assert max(shares) == most and min(shares) >= most - 1 and (most, MT) in WK_LAUNCHED, (NRB, KS, rows)
                seen.add((most, MT))
                assert not any(plans.whole_k_rows(NRB, KS, rows, n_cu, **kw) for kw in (dict(big=False), dict(fixed=True), dict(q4=True)))
    assert seen == WK_LAUNCHED


def test_whole_k_gate_up_only_where_it_is_the_faster_one(plans):
    """Four tiles of rows with a long K need nearly three row blocks on every CU, three tiles with a K beyond 10240 too."""
    for d, blocks, slower in ((4096, 516, (104, 128)), (4096, 536, (104, 128)), (7168, 672, (120, 128)), (8192, 516, (104, 128)), (8192, 640, (104, 128)),
                              (12288, 576, (80, 96, 104, 128)), (16384, 768, (128,))):
        assert not any(plans.whole_k_rows(blocks, d // 16, rows) for rows in slower), (d, blocks)
    for d, blocks, faster in ((1024, 516, (40, 64, 72, 96, 104, 128)), (4096, 516, (40, 64, 72)), (4096, 576, (104, 128)), (4096, 688, (40, 72, 104, 128)),
                              (8192, 516, (40, 64)), (8192, 704, (40, 72, 104, 128)), (5120, 864, (40, 64)), (16384, 1024, (40, 64))):
        assert all(plans.whole_k_rows(blocks, d // 16, rows) for rows in faster), (d, blocks)


def test_whole_k_gate_up_cases_take_it(plans):
    """Every row count of test_gpu_whole_k_rows.py; work-groups of two and three and of three and four blocks, every number of row tiles."""
    seen = set()
    for d, ffn, lens in WHOLE_K.values():
        for rows in lens:
            assert plans.whole_k_rows(ffn // 16, d // 16, rows), (d, ffn, rows)
            seen.add((-(-(ffn // 16) // 256), (rows + 31) // 32))
    assert seen == WK_LAUNCHED


def test_expert_cases_share_two_launches(plans):
    """All cases of test_gpu_experts_in_two.py, and between them every kernel that such a launch may take; not narrow experts (fewer gate/up row
    blocks than CUs, or as many with a short K) nor a single one."""
    two = {name: plans.experts_in_two(mixture_of(name)) for name in IN_TWO}
    assert all(two.values()), two
    assert {max(2, gu) for gu, _, _ in two.values()} == {2, 3, 4} == {max(2, dn) for _, _, dn in two.values()}
    assert min(S for _, S, _ in two.values()) <= 4 < max(S for _, S, _ in two.values())
    assert plans.experts_in_two(synth.SHAPES["mixtral-8x7b"]) == (4, 4, 2)
    wide = mixture_of("e3-top1")
    for other in (replace(wide, d_ffn=4032), replace(wide, d_ffn=4096, d_model=2048, n_heads=32, n_kv_heads=32), replace(wide, n_experts=1), synth.SHAPES["mini-moe"]):
        assert plans.experts_in_two(other) is None, other


@pytest.mark.parametrize("slices", [1, 3, 8])
def test_4bit_streams_keep_their_scalar_offsets_inside_the_buffers(plans, slices):
    """What the 4-bit stream with three row blocks (fk_stream_q4) requests while a wave works on group g of its run [gb, ge): the tiles
    of group g + 1, in the last round with the lanes out of range.  Tiles of both buffers, 8 k-steps a group: scalar offsets stay inside
    the resources, requests whose lanes are in range inside the tiles that exist."""
    planes, blocks = 2, 3
    for NG in (1, 2, 3, 7, 8, 9, 32, 86, 112):
        KS = 8 * NG
        x_span, w_span = plans.q4_spans(planes, blocks, KS)
        groups = []
        for s in range(slices):
            G0, G1 = s * NG // slices, (s + 1) * NG // slices
            for w in range(8):
                gb, ge = G0 + w * (G1 - G0) // 8, G0 + (w + 1) * (G1 - G0) // 8
                for g in range(gb, ge):
                    x, c = (planes - 1) * KS + 8 * (g + 1) + 7, (blocks - 1) * (KS // 4) + 2 * (g + 1) + 1
                    assert x < x_span and c < w_span, (NG, g)
                    assert g + 1 == ge or (x < planes * KS and c < blocks * (KS // 4)), (NG, g)
                    groups.append(g)
        assert groups == list(range(NG))


@pytest.mark.parametrize("n_cu", [64, 256, 304])
def test_whole_k_matrices_leave_no_more_partial_sums_of_squares_than_their_buffers_hold(plans, n_cu):
    for NRB in (1, 63, 64, 65, 255, 256, 257, 304, 305):
        assert plans.whole_k(NRB, 64, 3, n_cu) == (NRB <= min(n_cu, 256)), NRB


def test_divisions_by_a_multiplication_are_exact(plans):
    """Row groups (up to 256 of four row blocks) and K slices (up to 16 of any K) of k2_gemm_xk: every quotient it forms."""
    for n in list(range(1, 257)):
        for x in {0, 1, n - 1, n, n + 1, 4 * n * n - 1, 4 * n * n, *range(0, 4 * n * n, max(1, n * n // 50))}:
            assert plans.lib.shim_div_holds(x, n) and plans.lib.shim_div(x, n) == x // n, (x, n)
    for n in range(1, 17):
        for ks in (16, 250, 344, 688, 896, 1792, 5000, 8191):
            for s in range(n + 1):
                assert plans.lib.shim_div(s * ks, n) == s * ks // n, (s, ks, n)
    assert not plans.lib.shim_div_holds(1 << 31, 1) and plans.lib.shim_div((1 << 31) - 1, 1) == (1 << 31) - 1


@pytest.mark.parametrize("units,n,in_turn", [(688, 256, True), (768, 256, True), (1000, 256, True), (1792, 448, True), (8, 8, True), (32, 32, True), (1, 1, True), (257, 256, True),
                                             (4000, 1000, False), (8016, 2004, False), (3001, 751, True), (3248, 812, True), (3249, 813, False), (5, 256, True)])
def test_shares_cover_all_units_and_differ_by_one(plans, units, n, in_turn):
    begin, got = plans.shares(units, n)
    assert got == in_turn
    assert begin[0] == 0 and begin[-1] == units
    sizes = [b - a for a, b in zip(begin, begin[1:])]
    assert min(sizes) >= units // n and max(sizes) <= -(-units // n)
    if in_turn:
        assert begin == [i * units // n for i in range(n + 1)]


def test_4bit_lm_heads_over_all_of_k(plans):
    """Four row blocks a CU and no more; where sums keep their order, only with the split-K kernel's own parts of K (four slices)."""
    for KS in (8, 128, 256, 264, 320, 512):
        assert [NRB for NRB in range(700, 1100) if plans.logits_q4(NRB, KS)] == list(range(769, 1025)), KS
    for KS in range(8, 1025, 8):
        for NRB in (769, 1000, 1024):
            assert plans.logits_q4(NRB, KS, fixed=True) == (plans.staged_q4(NRB, KS) == (4, 1)), (NRB, KS)
    assert plans.logits_q4(1000, 256, fixed=True)                # d 4096
    assert not any(plans.logits_q4(1000, KS, fixed=True) for KS in (128, 264, 320, 512))   # 2048, 4224, 5120, 8192


def test_prompts_of_at_most_32_rows_take_the_fused_kernels_where_those_are_ahead(plans):
    for rows in (1, 2, 31, 32):
        for d in (64, 1024, 1088, 2048, 2560, 4096, 8192):
            fp32, bf16 = (replace(synth.SHAPES[base], d_model=d) for base in ("tiny", "llama2-7b"))
            assert plans.short_prompt(fp32, rows) == (d <= 1024)
            assert plans.short_prompt(bf16, rows) and plans.short_prompt(bf16, rows, bits=4) and plans.short_prompt(bf16, rows, kv="bf16", bits=4)
            assert not plans.short_prompt(bf16, rows, kv="bf16") and not plans.short_prompt(fp32, rows, kv="bf16")
        assert not plans.short_prompt(synth.SHAPES["mixtral-8x7b"], rows) and not plans.short_prompt(synth.SHAPES["mini-moe"], rows)
    for s in synth.SHAPES.values():
        assert not plans.short_prompt(s, 33) and not plans.short_prompt(s, 33, bits=4)
