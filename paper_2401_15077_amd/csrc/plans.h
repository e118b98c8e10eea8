// Work splits of the matrix products: which tile shape, how many K slices, how many work-groups.  Arithmetic on sizes only (no device
// code, no context), so that it can be built and tested without a GPU; the kernels call the constexpr functions too.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

constexpr int PLAN_MAX_SLICES = 16;   // most K slices any plan of the general path takes
constexpr int PLAN_MAX_NORM_GROUPS = 256;   // most work-groups whose partial sums of squares a norm adds up

// 1-KiB tiles that the buffer resources of the 4-bit stream (fk_stream_q4) span: those that exist -- activations [plane][k-step], codes
// [row block][4 k-steps] -- and one group of 8 k-steps behind them.  With three row blocks the last group of a wave requests the one
// behind it, with every lane's offset out of range so that nothing is read; the check compares that offset with the span minus the
// scalar offset, so the scalar offset has to lie inside the span.  (Held at the last group instead, it costs the kernel 4 spilled
// registers.)
constexpr int q4_x_span(int planes, int KS) { return planes * KS + 8; }
constexpr int q4_w_span(int row_blocks, int KS) { return row_blocks * (KS / 4) + 2; }

// Shares of a launch's work without a division on the GPU, where one stands in front of a work-group's first request (forty instructions,
// 0.2 us).  div_magic(x, magic_of(n)) = floor(x / n) for x * n < 2^31.
static inline uint32_t magic_of(uint32_t n) { return (uint32_t)((1ull << 31) / n + 1); }
static inline bool magic_holds(uint64_t x_max, uint32_t n) { return n > 0 && x_max * n < (1ull << 31); }
constexpr uint32_t div_magic(uint32_t x, uint32_t magic) { return (uint32_t)((uint64_t)(2 * x) * magic >> 32); }
// Where share i of `units` in n shares begins: floor(i * units / n), longer and shorter shares in turn (7B, us with the longer ones in front: LM
// head 46.0, gate/up 32.8; in turn 45.1 and 32.5); beyond the magic's range the longer ones in front: LM heads of more than 3248 row blocks, 103936
// tokens, on a quarter as many work-groups.
constexpr uint32_t SHARE_IN_TURN = 0xFFFFFFFFu;
struct Share { uint32_t a, b; };
static inline Share share_of(uint32_t units, uint32_t n) {
  return magic_holds((uint64_t)units * n, n) ? Share{magic_of(n), SHARE_IN_TURN} : Share{units / n, units % n};
}
constexpr uint32_t share_begin(uint32_t i, uint32_t units, uint32_t a, uint32_t b) { return b == SHARE_IN_TURN ? div_magic(i * units, a) : i * a + (i < b ? i : b); }

// Work-groups that share a row's vocabulary in the choice of its children: 2048 tokens each, what a work-group takes in one round, at most
// EXPAND_PARTS_MAX of them.  Smaller parts cost the exchange (2 us) where one part would do, larger ones a round each.  us a launch (root with four
// children, greedy / with noise), parts of 1024, 2048, 4096: 2048 tokens 6.4 / 7.5, 4.3 / 6.2, 4.3 / 6.5; 4096 6.3 / 7.9, 6.2 / 7.3, 6.7 / 9.2; 8192 6.4 / 8.2, 6.4 / 7.6, 8.4 / 11.1;
// 32000 (16 parts, 16, 8) 6.4 / 8.1, 6.4 / 7.9, 8.9 / 11.6; beyond 32768 more rounds of 16 parts: 65536 9.3 / 12.0, 128256 14.5 / 19.3.
constexpr int EXPAND_PARTS_MAX = 16;
static inline int plan_expand_parts(int vocab) { return std::max(1, std::min(EXPAND_PARTS_MAX, (vocab + 2047) / 2048)); }

struct GemmPlan { int S, ks_per_split, chunk, rbw, mw; };   // rbw, mw: tile shape of the large-M GEMM (0: k_gemm)

static inline GemmPlan plan_gemm(int NRB, int KS, int NXP, int MT) {
  GemmPlan p{};
  int wg_n = (NRB + 3) / 4;
  int S = std::max(1, std::min(PLAN_MAX_SLICES, 512 / std::max(1, wg_n)));
  S = std::min(S, std::max(1, KS / 8));
  p.ks_per_split = (KS + S - 1) / S;
  p.S = (KS + p.ks_per_split - 1) / p.ks_per_split;
  p.chunk = std::max(1, 64 / (NXP * MT));
  return p;
}

// Which passes of the general path take the large-M GEMM: every pass of more than 128 rows (only prompts, and only where the
// kernel exists), and shorter ones of the models it covers: prompts and batched tree passes of 33..128 rows (33..64 rows, us a
// matrix against k_gemm: 7B QKV 27 / 34, O 12.3 / 17.3, gate/up 40 / 59, down 24 / 33; LM head 58 / 71), 65..128 where the sums
// keep their order (fixed_sums); with 4-bit weights all.
static inline bool plan_is_large_m(int MT, bool big_gemm, bool fixed_sums, bool q4) { return MT > 4 || (MT >= (fixed_sums ? 3 : 2) && big_gemm) || q4; }

// Which gate/up products of 33 to 128 rows run over all of K in a work-group (k_gemm_wk; plan_pf otherwise): dense bf16 models whose
// sums are not fixed, with three row blocks on the busiest CU, or four and at most 64 rows.  (With fewer the activations that every
// work-group fetches outweigh what the K slices cost; with four and more rows the CUs that have three idle for a quarter of the time.)
// The same two things bound it below three: the work-groups with two blocks idle, and with four tiles of rows what each fetches grows
// with K, while the K slices' partial sums do not.  Hence the least number of row blocks a CU for four tiles, and for three with a K
// beyond 10240.  Whole prompts at 20 to 61 sizes of each K, time with all of K over time with slices, rows 40 to 64 / 72 to 96 / 104 to 128:
//   K 1024 to 3072, 2.02 to 3 blocks   0.89 to 0.96 / 0.90 to 0.97 / 0.93 to 1.00
//   K 4096          2.02               0.98 to 0.99 / 0.99 to 1.00 / 1.01 to 1.02,  2.12  0.97 / 0.98 to 0.99 / 0.99 to 1.01,  2.25 to 2.62  0.94 to 0.96 / 0.96 to 0.97 / 0.97 to 1.00
//   K 5120, 6144    2.02 to 2.62       0.95 to 0.98 / 0.96 to 0.99 / 0.98 to 1.02
//   K 7168 to 10240 2.02 to 2.62       0.95 to 0.99 / 0.97 to 1.01 / 0.99 to 1.03
//   K 12288, 16384  2.02 to 2.62       0.98 to 1.01 / 0.99 to 1.02 / 1.01 to 1.04
//   K 4096 to 10240 2.75 to 3          0.92 to 0.95 / 0.93 to 0.97 / 0.96 to 0.99
//   K 12288         2.75 to 3          0.95 to 0.97 / 0.97 to 0.98 / 0.99 to 1.00
//   K 16384         2.75 to 3          0.97 to 0.98 / 0.98 to 0.99 / 1.00 to 1.01
//   K 1024 to 16384 3.02 to 4          0.86 to 1.00
static inline bool plan_is_wk(int NRB, int KS, int MT, int n_cu, bool big_gemm, bool fixed_sums, bool q4) {
  if (!big_gemm || fixed_sums || q4 || MT < 2 || MT > 4 || NRB <= 2 * n_cu || NRB > (MT == 2 ? 4 : 3) * n_cu) return false;
  const int least = MT == 4 ? (KS <= 192 ? 32 : KS <= 256 ? 34 : KS <= 768 ? 43 : 64) : MT == 3 && KS > 640 ? 43 : 32;   // sixteenths of a row block a CU
  return 16 * NRB >= least * n_cu;
}

// Which prompt passes take the attention kernel of 128 rows a work-group (k2_attn_prompt) instead of the one of 32 (k2_attn): those
// whose small work-groups would go through the chip at least twice.  (Where they all fit at once, the run of tiles of one work-group
// is what counts, and with few rows most of a 128-row block is padding.)  us a launch, 32 / 128 rows: 32 heads, 256 rows 16 / 22, 384
// rows 29 / 31, 512 rows 40 / 38, 1024 rows 108 / 67; 40 heads, 300 rows 27 / 26, 1024 rows 140 / 69; 64 heads (8 of keys), 300
// rows 40 / 27, 2011 rows 690 / 290.
static inline bool plan_is_prompt_attn(int rows, int heads, int n_cu) { return rows >= 256 && heads * ((rows + 31) / 32) >= 2 * n_cu; }

// KV splits of the attention kernel for `tokens` keys and `units` (head, sequence, row block) triples: one 32-token
// block per wave (128 tokens per work-group) while that keeps the grid within one work-group per CU -- the kernel's
// registers allow no more, and a second round of work-groups costs more than a wave walking a few blocks in turn.  Up to 192
// tokens stay in one work-group: a second block in two of its waves costs less than the exchange between two work-groups (a
// tiny model's launch 8.9 -> 5.1 us; 7B with 139 tokens: a request of 8 layers 22.6 -> 22.3 ms).
static inline int plan_attn_splits(bool fixed_sums, int tokens, int units, int n_cu) {
  const int by_tokens = !fixed_sums && tokens <= 192 ? 1 : (tokens + 127) / 128, by_cus = std::max(1, n_cu / std::max(1, units));
  return std::max(1, std::min(16, std::min(by_tokens, by_cus)));
}

// Tile shape and work split of the large-M GEMM (k_gemm_pf): the (row blocks per wave, wave columns, K slices) that is cheapest
// in a model of two terms, in us.  What the busiest CU multiplies: rounds x (32 x 32 tiles of a work-group) x k-steps of a slice
// x the shape's measured time per tile and k-step.  Groups of work-groups that share a weight tile go round the 8 XCDs, so a
// round is full when the XCD with one group more than the others is (LM-head transpose, 10 row tiles, 3 slices of 27 x 3
// tiles: 243 work-groups, but 33 on the 32 CUs of one XCD: 355 us against 197 for 240 of the next shape).  And what the partial
// sums cost that all but the fused epilogue write and read back, at 4.5 TB/s.
// 4-bit weights (k_gemm_pf_q4): one shape, two row blocks per wave and two wave columns; K slices of whole groups of 8 k-steps.
static inline int plan_slices(int NRB, int KS, int MT, int n_cu) {     // fixed_sums: K slices of a matrix and a number of row tiles, whatever tile serves them
  const int wgs = ((NRB + 7) / 8) * ((MT + 3) / 4);
  int S = wgs * 2 > n_cu ? 1 : std::min(MT <= 4 ? PLAN_MAX_SLICES : KS >= 1024 ? 8 : 4, n_cu / std::max(1, wgs));
  return std::max(1, std::min(S, KS / (MT <= 4 ? 16 : 32)));
}
static inline GemmPlan plan_pf(int NRB, int KS, int MT, int n_cu, bool fused_epilogue, bool q4, bool fixed_sums) {
  GemmPlan best{};
  double best_us = -1;
  static const struct { int rbw, mw; double ns; } shapes[8] = {{4, 1, 20.0}, {3, 1, 22.0}, {4, 2, 13.3}, {3, 2, 15.0}, {4, 4, 12.0}, {3, 4, 13.3}, {2, 4, 15.0}, {2, 2, 17.0}};
  const int xcds = 8, cu_x = std::max(1, n_cu / xcds);
  for (int i = q4 ? 7 : 0; i < (q4 ? 8 : 7); ++i) {
    const auto& sh = shapes[i];
    const int wt = 2 * sh.rbw, rt = 2 * sh.mw, mq = (MT + rt - 1) / rt, nt = (NRB + wt - 1) / wt;
    if (MT <= 4 && sh.mw > 2) continue;                        // half of the work-group would idle
    if (!q4 && (MT <= 2) != (sh.mw == 1)) continue;            // two tiles of rows: work-groups of two waves, bound by the weight stream
    const int S_fix = fixed_sums ? plan_slices(NRB, KS, MT, n_cu) : 0;
    // no split can beat all CUs at work all the time: shapes and slices whose price is above the best one already are not looked at
    const double least = 1e-3 * sh.ns * NRB * MT * KS / (xcds * cu_x), slice_us = MT * NRB * 8192.0 / 4.5e6;
    if (!fixed_sums && best_us >= 0 && least > best_us) continue;
    for (int S = fixed_sums ? S_fix : 1; S <= (fixed_sums ? S_fix : PLAN_MAX_SLICES); ++S) {
      if (!fixed_sums && S > 1 && (KS / S < 16 || least + S * slice_us > best_us)) break;
      const int unit = q4 ? 8 : 4, kps = ((KS + S - 1) / S + unit - 1) / unit * unit, s_real = (KS + kps - 1) / kps;
      const int rounds = ((nt * s_real + xcds - 1) / xcds * mq + cu_x - 1) / cu_x;
      double us = 1e-3 * sh.ns * rounds * wt * rt * kps + 4.0;
      if (!(fused_epilogue && s_real == 1)) us += s_real * slice_us;
      if (fused_epilogue && s_real > 1) us += 10.0;             // the SwiGLU kernel behind it
      if (best_us < 0 || us < best_us) { best_us = us; best.S = s_real; best.ks_per_split = kps; best.chunk = 4; best.rbw = sh.rbw; best.mw = sh.mw; }
    }
  }
  return best;
}

// Work-groups of the large-M GEMM: weight-row tiles x K slices, rounded up to whole rounds over the 8 XCDs, x columns of row tiles.
static inline int pf_cols(int MT, const GemmPlan& p) { return (MT + 2 * p.mw - 1) / (2 * p.mw); }
static inline int pf_grid(int NRB, int cols, const GemmPlan& p) { return ((NRB + 2 * p.rbw - 1) / (2 * p.rbw) * p.S + 7) / 8 * 8 * cols; }
// Which of its launches bring their tiles by plain loads, an address a lane, instead of buffer loads: those of two- and four-wave
// work-groups in a single round (a work-group a CU, hence a wave a SIMD or less).  us a launch, buffer / plain loads, on each of two
// cards: 192 rows at 7B widths, gate/up 75.9 / 70.8 and 79.0 / 76.5, QKV 42.4 / 40.5 and 43.7 / 42.6, down 37.0 / 35.5 and 38.7 / 38.4;
// 512 rows, down 73.5 / 71.9 and 79.4 / 79.3; 700 rows, O 48.5 / 45.9 and 55.2 / 49.0; 512 rows at 13B widths, down 118.7 / 116.5 and
// 127.2 / 125.6.  (Fewer scalar instructions a k-step do not change it.)  Everywhere else buffer loads are the faster ones: two
// work-groups a CU (700 rows at 7B widths, QKV in 768 work-groups 115.8 / 123.4 and 123.6 / 130.9; 1024 rows, gate/up in 704 273 / 306
// and 293 / 325), eight waves (512 rows at 7B widths, gate/up 140 / 148 and 154 / 161; 2011 rows at 70B widths 2589 / 2882 and 2750 /
// 3016), and a single column of four tiles with 16 rows or more beyond the end, which buffer loads leave out and the waves would
// multiply (72 rows at 7B widths, down 25.4 / 26.6 and 25.9 / 27.5; 104 rows 30.0 / 31.1 and 30.2 / 31.2; whole prompts of 80 and 96
// rows 3.7 and 2.5 % slower with plain loads, 112 rows 1.3, 120 even, 128 rows 0.2 to 1.5 % faster).
// Grouped experts (`cols` columns, each with rows of its own) take the same line without the last exception: 5 rows at d 1024, ffn 2048, two
// experts, 48 and 96 work-groups, 22.4 / 20.7 and 7.3 / 6.8; 200 rows at Mixtral widths with two experts, down in 240 76.5 / 73.9, gate/up in 336
// 184 / 197; 64 rows at d 1024, ffn 2816, eight experts, 288 each, 35.3 / 39.5 and 20.7 / 22.5.
static inline bool plan_pf_one_round(int NRB, int cols, int n_cu, const GemmPlan& p) { return p.mw <= 2 && pf_grid(NRB, cols, p) <= n_cu; }
static inline bool plan_pf_plain_loads(int NRB, int MT, int M, int n_cu, const GemmPlan& p) {
  return plan_pf_one_round(NRB, pf_cols(MT, p), n_cu, p) && !(p.mw == 2 && M <= 112);
}

// The same model for the grouped GEMMs of a mixture of experts: M rows x topk experts each, padded per expert to columns of
// 2 * mw tiles.  Routing is uneven, so half a column more per expert and half a round more at the end are counted.  Both GEMMs of
// the MLP share the column width; gate/up keeps one K slice (SwiGLU in its epilogue).
// Columns of eight tiles only where an expert has more than four on average: in the others half of the work-group or more has no
// live tile, moves 24 KiB a k-step whatever is live and leaves room for one work-group per CU.  Prompt of a model with two
// Mixtral layers and an expert head, ms with columns of eight / four tiles: 8 rows 2.25 / 1.97, 32 rows 2.33 / 2.08, 50 to 256
// rows the same, 300 rows 3.25 / 3.01, 450 rows 3.56 / 3.32, 512 rows 4.01 / 3.94.
struct PlanMoe { GemmPlan gu, dn; int cols; };
static inline int moe_tiles(int M, int topk, int E) { return (M * topk + 31) / 32 + std::min(E, M * topk); }
static inline PlanMoe plan_moe(int gu_NRB, int gu_KS, int dn_NRB, int dn_KS, int M, int topk, int E, int n_cu) {
  PlanMoe best{};
  double best_us = -1;
  static const struct { int rbw, mw; double ns; } shapes[5] = {{4, 2, 13.3}, {3, 2, 15.0}, {4, 4, 12.0}, {3, 4, 13.3}, {2, 4, 15.0}};
  const int used = std::min(E, M * topk), te = (M * topk + 32 * used - 1) / (32 * used), cu_x = std::max(1, n_cu / 8);
  for (int mw = 2; mw <= 4; mw += 2) {
    const int rt = 2 * mw;
    if (mw > 2 && te <= 4) continue;
    const double cols = used * std::max(1.0, (double)te / rt + 0.5);
    GemmPlan q[2] = {};
    double us[2] = {-1, -1};
    for (auto& sh : shapes) {
      if (sh.mw != mw) continue;
      for (int m = 0; m < 2; ++m) {
        const int wt = 2 * sh.rbw, KS = m ? dn_KS : gu_KS, NRB = m ? dn_NRB : gu_NRB, nt = (NRB + wt - 1) / wt;
        for (int S = 1; S <= (m ? PLAN_MAX_SLICES : 1); ++S) {
          if (S > 1 && KS / S < 16) break;
          const int kps = ((KS + S - 1) / S + 3) / 4 * 4, s_real = (KS + kps - 1) / kps;
          const double full = (nt * s_real + 7) / 8 * cols / cu_x, rounds = full <= 1.0 ? 1.0 : full + 0.5;
          const double t = 1e-3 * sh.ns * rounds * wt * std::min(rt, te) * kps + 4.0 + (m ? (double)s_real * used * te * NRB * 8192.0 / 4.5e6 : 0.0);
          if (us[m] < 0 || t < us[m]) { us[m] = t; q[m].S = s_real; q[m].ks_per_split = kps; q[m].chunk = 4; q[m].rbw = sh.rbw; q[m].mw = mw; }
        }
      }
    }
    if (best_us < 0 || us[0] + us[1] < best_us) {
      best_us = us[0] + us[1]; best.gu = q[0]; best.dn = q[1];
      best.cols = std::min(M * topk, E + M * topk / (32 * rt));  // most columns any routing gives
    }
  }
  return best;
}

// Small matrices of the fast path: a work-group per row block over all of K (k2_gemm_fk) instead of K slices whose partial sums cross
// work-groups.  K x planes is what a work-group then fetches, in KiB per 16 columns: 400 of them take about what the exchange does
// (store, acknowledge, count, read back: 5 us).  Whole requests, ms, sliced / whole: fp32, d 256 (96 KiB) 8.8 / 7.6; bf16, d 1024 (192)
// 9.7 / 8.9; d 2048 (384) 12.5 / 12.0; matrices of 528 KiB 8.8 / 9.3.  A matrix that feeds a norm leaves partial sums of squares per
// work-group, of which there may be PLAN_MAX_NORM_GROUPS, however many CUs the device has.
static inline bool plan_is_short_k(int KS, int planes) { return (long)KS * planes <= 400; }
static inline bool plan_is_whole_k(int NRB, int KS, int planes, int n_cu) { return NRB <= std::min(n_cu, PLAN_MAX_NORM_GROUPS) && plan_is_short_k(KS, planes); }

// Which prompt passes of at most 32 rows take the fused kernels of the decoding steps: those of dense models, in fp32 only where d_model is a short K, and
// not where sums keep the order of the general path (fixed_sums); with 4-bit weights all.  (Two such passes for 33 rows would be 1.6 times the general one.)
// A prompt of 2 / 22 / 32 tokens, us, general / fused: 7B widths, 16 layers 2243 / 1636, 2301 / 1758, 2339 / 1838; 13B, 8 layers 1675 / 1337, 1711 / 1429, 1746 /
// 1494; 70B, 4 layers 2092 / 1723, 2108 / 1839, 2117 / 1914; tiny fp32 191 / 145, 205 / 142, 207 / 148.
// bf16, two layers, 21 shapes with d 64 to 8192 (ffn of 1.5 d to 11 d, attention of d / 4 to 4 d), general over fused for 1 to 32 rows: 1.10 to 1.38.
// fp32, four layers, general over fused for 1 to 32 rows: d 64 to 768 1.17 to 1.47, 1024 1.11 to 1.19 (attention of 4 d 1.02 to 1.06, ffn of 16 d 1.04 to 1.07, of 32 d 0.97 to 1.00).  Beyond, where
// the fused products are k2_gemm's with three planes of weights, neither is ahead: d 1088 to 1280 1.02 to 1.09, 1408 0.97, 1536 to 1792 1.02 to 1.06, 1984 and 2048
// 0.92, 2304 and 2560 1.04, 3072 0.99, 3584 and 4096 0.95, 5120 0.85, and with longer ffn 0.92 to 0.98 from d 1280 on.
// Mixtures gain or lose with their widths and stay on the general path, which groups the rows by expert: 2 / 22 / 32 tokens, Mixtral widths, 6 layers, 2742 / 1785,
// 4273 / 3797, 4285 / 4033; eight experts at d 2176, ffn 4160, 4 layers, 771 / 618, 975 / 1052, 980 / 1130; four at d 256 224 / 215, 232 / 229, 232 / 230.
static inline bool plan_is_short_prompt(int rows, int d, int planes, bool f32, bool q4, bool fixed_sums, int experts) {
  return rows <= 32 && (q4 || (!fixed_sums && experts == 0 && (!f32 || plan_is_short_k(d / 16, planes))));
}

// Work split of the split-K kernel with streamed activations: S slices x groups of at most 4 row blocks, chosen by a
// fetch model in KiB per work-group (weights + the live part of the X slice + twice the partials the last work-group
// of a row group reads back, which sit on the critical path of one CU).  Depends on the matrix shape only.
struct PlanXK { int S, groups, nrmax; long cost; };
static inline PlanXK plan_xk(int NRB, int KS, int NXP, int n_cu, size_t pt_floats_per_slice, size_t pt_floats) {
  PlanXK best; best.S = 0; best.groups = 0; best.nrmax = 0; best.cost = -1;
  for (int S = 1; S <= 16; ++S) {
    const int groups = std::min(NRB, n_cu / S);
    if (groups < 1) break;
    const int nrm = (NRB + groups - 1) / groups, kt = (KS + S - 1) / S;
    if (nrm > 4 || kt < 16 || (size_t)S * pt_floats_per_slice > pt_floats) continue;
    const long cost = (long)nrm * kt + (long)NXP * kt * 4 / 5 + 2L * S * nrm * 4;
    if (best.cost < 0 || cost < best.cost) { best.S = S; best.groups = groups; best.nrmax = nrm; best.cost = cost; }
  }
  return best;
}

// Work split of the LDS-staged split-K kernel: S K-slices x `groups` row groups = one work-group each; inside a
// work-group `lanes` x `kparts` waves (product 8): a wave owns every lanes-th row block of the group over one k-part.
struct Plan2 { int S, groups, lanes, kparts, RW, kt_max; size_t lds; };
static inline Plan2 plan2(int NRB, int KS, int NXP, int NWP, int n_cu, bool q4 = false) {
  Plan2 p;
  const int x_cap_kb = 128;                                   // LDS given to the X slice / the wave reduction
  int S = 1;
  // fewest K slices whose X slice fits (fewer partials to exchange); 4-bit weights: slices are whole groups of 8 k-steps
  auto slice_ks = [&](int S_) { return q4 ? 8 * ((KS / 8 + S_ - 1) / S_) : (KS + S_ - 1) / S_; };
  while (NXP * slice_ks(S) > x_cap_kb) ++S;
  int groups = std::max(1, std::min(NRB, n_cu / S));
  // few row blocks: split K further (slices of at least 4 k-steps) until the grid fills the chip
  while (!q4 && groups * S * 2 <= n_cu && (KS + 2 * S - 1) / (2 * S) >= 4) S *= 2;
  // many row blocks (wide matrices with a long K): more work-groups than CUs rather than more than 3 row blocks per wave
  const int r_cap = 24;
  if ((NRB + groups - 1) / groups > r_cap) groups = (NRB + r_cap - 1) / r_cap;
  const int R = (NRB + groups - 1) / groups, kt = slice_ks(S);
  long best = -1; int bl = 8, bk = 1;
  const int cand[4][2] = {{8, 1}, {4, 2}, {2, 4}, {1, 8}};
  for (auto& cd : cand) {
    int rw = (R + cd[0] - 1) / cd[0];
    if (rw > 3) continue;
    if ((size_t)cd[0] * (cd[1] - 1) * rw * 4 > (size_t)x_cap_kb) continue;
    long cost = (long)rw * ((kt + cd[1] - 1) / cd[1]);
    if (best < 0 || cost < best) { best = cost; bl = cd[0]; bk = cd[1]; }
  }
  p.S = S; p.groups = groups; p.lanes = bl; p.kparts = bk;
  int rw = (R + bl - 1) / bl;
  p.RW = rw <= 1 ? 1 : rw <= 2 ? 2 : 3;
  p.kt_max = kt;
  size_t xs = (size_t)NXP * kt * 1024, red = (size_t)bl * (bk - 1) * p.RW * 4096;
  p.lds = std::max(xs, red);
  return p;
}

// LM heads of 4-bit models that run over all of K in work-groups of four row blocks, K in four parts (k2_logits_q4): one round of them.  (Fewer blocks fit
// three a work-group of k2_gemm_fk.  More are a second round, which is dearer at first: 26 rows, K 4096, us a launch, split-K in LDS / this in several
// rounds: 32769 tokens 35 / 39, 40000 37 / 40, 49152 43 / 41, 65536 72 / 46, 128256 123 / 102; K 8192 87 / 86, 128 / 99 at 65536, 264 / 190 at 128256;
// K 1024 17 / 17, 20 / 19, 30 / 32.  The largest vocabularies stay as they are, with that to gain.)  us a launch at the ends of the range, split-K in LDS / this,
// K 4096: 26 rows, 24608 tokens 29 / 23, 32768 32.5 / 24.5; 1 to 4 rows 24 / 17.5 and 27 / 19.  Where sums keep their order (fixed_sums) only if `staged`, the split-K plan, cuts K into the
// same four parts and adds them in the same order: K of 3200 to 4096.  (The others, 26 rows: K 2048 20 / 15.5, 5120 38 / 29, 8192 80 / 50.)
constexpr int LQ4_BLOCKS = 4, LQ4_PARTS = 4;
static inline bool plan_is_logits_q4(int NRB, int n_cu, const Plan2& staged, bool fixed_sums) {
  return NRB > 3 * n_cu && NRB <= LQ4_BLOCKS * n_cu && (!fixed_sums || (staged.S == LQ4_PARTS && staged.kparts == 1));
}

// Split-K plan of a matrix with streamed activations; S = 0 where the fetch model prices the LDS-staged kernel (plan2) lower.
static inline PlanXK plan_streamed(int NRB, int KS, int NXP, int NWP, int n_cu, size_t pt_floats, bool q4 = false) {
  const Plan2 p = plan2(NRB, KS, NXP, NWP, n_cu, q4);
  PlanXK px = plan_xk(NRB, KS, NXP, n_cu, (size_t)NRB * 32 * 32, pt_floats);
  const int R = (NRB + p.groups - 1) / p.groups, kt_s = (KS + p.S - 1) / p.S;
  const long staged = (long)R * kt_s + (long)NXP * kt_s + 2L * p.S * R * 4 + 40;
  if (px.S > 0 && px.cost >= staged) px.S = 0;
  return px;
}

// Passes of up to 32 rows of a mixture: all experts' gate/up in one launch and all their downs in another, where those are the whole-K and
// the streamed split-K kernel (wide matrices).  Two launches an expert are sixteen a layer with eight experts, each with its own first
// tiles, drain and (down) exchange, and many of them for nothing in the head's passes of a few rows.  In two, a row is fetched only for
// the experts it selected.  Two layers and the head, 26-node tree, us a step, launches an expert / two: Mixtral widths, 8 experts, 2 choices 3376 / 3098,
// 2 and 1 1498 / 1459, 16 and 4 6341 / 5714; d 6144, ffn 16384, 8 and 2 5176 / 4885; d 2176, ffn 4160, 8 and 2 1574 / 1311, 64 and 1
// 4138 / 2077.  (Slices of down are planned for one expert.)
static inline bool plan_experts_in_two(int gu_NRB, int gu_KS, int dn_NRB, int dn_KS, int NXP, int NWP, int n_cu, size_t pt_floats) {
  return gu_NRB >= n_cu && !plan_is_whole_k(gu_NRB, gu_KS, NWP + NXP, n_cu) && !plan_is_whole_k(dn_NRB, dn_KS, NWP + NXP, n_cu) &&
         plan_streamed(dn_NRB, dn_KS, NXP, NWP, n_cu, pt_floats).S > 0;
}
