// Device kernels of libeagle (gfx950).  One speculative step = drafting (Sec. 3.1, App. A.1 of the paper),
// tree-masked verification (Sec. 3.3) and acceptance (Sec. 2, App. A.2 Alg. 1) + commit.
#pragma once
#include "common.h"
#include "plans.h"

// ============================================================================ device-side model state
struct TreeDev {
  int M, D;
  int parent[EAGLE_MAX_NODES], depth[EAGLE_MAX_NODES], nchild[EAGLE_MAX_NODES];
  int child[EAGLE_MAX_NODES][EAGLE_MAX_CHILD];           // children in rank order
  unsigned long long anc[EAGLE_MAX_NODES];               // bit u set <=> u is v or an ancestor of v
  int n_level_rows[EAGLE_MAX_DEPTH + 1];                 // level d: depth-d nodes that have children
  int level_rows[EAGLE_MAX_DEPTH + 1][EAGLE_MAX_NODES];
};

struct SeqState {          // all device pointers, one entry per sequence slot
  int* ctx_len;            // positions held by the target KV cache
  int* n_pend;             // target features waiting for the head's first pass (1..D+1)
  int* n_tok;              // committed tokens (= ctx_len + 1 between steps)
  int* step_no;            // draw counter for the generator
  int* commit_base;        // ctx_len before the last commit (read by the commit kernel)
  int* tokens;             // [max_batch][tok_stride]
  int tok_stride;
};

enum { PASS_VERIFY = 0, PASS_VANILLA, PASS_DRAFT_PENDING, PASS_DRAFT_LEVEL, PASS_PREFILL_T, PASS_PREFILL_D };
struct Pass {
  int kind, rows_per_seq, n_seq, seq0, level, chunk_start, chunk_n;
  // cached target positions of sequences seq0..seq0+3 as the host knows them at launch (it mirrors the device value
  // between calls); saves every kernel a dependent load at its start.  ctx_known = 0: read st.ctx_len instead.
  int ctx_known, ctx0, ctx1, ctx2, ctx3;
};
struct RowInfo {
  int seq, valid, pos, slot, base, rel, node, causal;
  unsigned long long mask;
};

// level_node: the row's node in a level pass, where the caller knows it.
__device__ inline RowInfo row_info(const Pass& p, const TreeDev* t, const SeqState& st, int r, int level_node = -1) {
  RowInfo o;
  int i = r % p.rows_per_seq;
  o.seq = p.seq0 + r / p.rows_per_seq;
  o.valid = 1; o.causal = 0; o.node = -1; o.mask = 0;
  int ctx;
  if (p.ctx_known) { const int j = o.seq - p.seq0; ctx = j == 0 ? p.ctx0 : j == 1 ? p.ctx1 : j == 2 ? p.ctx2 : p.ctx3; }
  else ctx = st.ctx_len[o.seq];
  switch (p.kind) {
    case PASS_VERIFY:
      o.node = i; o.base = ctx; o.rel = i; o.pos = ctx + t->depth[i]; o.slot = ctx + i; o.mask = t->anc[i];
      break;
    case PASS_VANILLA:
      o.base = ctx; o.rel = 0; o.pos = ctx; o.slot = ctx; o.mask = 1ull;
      break;
    case PASS_DRAFT_PENDING: {
      int np = st.n_pend[o.seq];
      o.valid = i < np;
      o.base = ctx - np; o.rel = o.valid ? i : 0; o.pos = o.base + o.rel; o.slot = o.pos; o.causal = 1;
      o.node = (i == np - 1) ? 0 : -1;
      break;
    }
    case PASS_DRAFT_LEVEL: {
      const int v = level_node >= 0 ? level_node : t->level_rows[p.level][i];
      o.node = v; o.base = ctx - 1; o.rel = v; o.pos = ctx - 1 + t->depth[v]; o.slot = ctx - 1 + v; o.mask = t->anc[v];
      break;
    }
    default:  // PASS_PREFILL_T / PASS_PREFILL_D
      o.valid = i < p.chunk_n;
      o.base = p.chunk_start; o.rel = o.valid ? i : 0; o.pos = o.base + o.rel; o.slot = o.pos; o.causal = 1;
      break;
  }
  return o;
}

// What every kernel of a pass needs to know about a row, written once by the pass's first kernel (token embedding / FC
// input).  The kernels behind it fetch it with one independent 16-byte load per half instead of walking tree, state and page
// table again: that walk is a chain of three to four dependent loads, 1 us or more each, in front of every weight stream.
struct alignas(16) RowFact {
  int pos;                       // RoPE position
  int kv_row;                    // (page * kv_heads << page_shift) | slot in page: row of the paged cache for kv head 0; -1: none
  int out_row;                   // row of the pass's logits buffer, -1: no logits for this row
  int seq;
  int base, rel;                 // attention: keys [0, base) are visible; the row's own index among the new keys
  uint32_t mask_lo, mask_hi;     // tree passes: visible new keys
};

struct KVCache {
  void* k; void* v;              // this layer's pages: [phys_page][kv_head][slot_in_page][head_dim]
  const int* page_table;         // [max_batch][pages_per_seq] -> physical page
  int pages_per_seq, page_shift, n_kv_heads, head_dim;
};
__device__ inline size_t kv_offset(const KVCache& c, int seq, int pos, int kvh) {
  int phys = c.page_table[seq * c.pages_per_seq + (pos >> c.page_shift)];
  return (((size_t)phys * c.n_kv_heads + kvh) << c.page_shift | (size_t)(pos & ((1 << c.page_shift) - 1))) * c.head_dim;
}

// The logits buffer of a pass: per tree node in drafting and verification, per sequence in vanilla passes and for a prompt's
// last row.
__device__ inline RowFact row_fact(const Pass& p, const TreeDev* t, const RowInfo& ri, const KVCache& c) {
  RowFact f;
  f.pos = ri.pos; f.seq = ri.seq; f.base = ri.base; f.rel = ri.rel;
  f.mask_lo = (uint32_t)ri.mask; f.mask_hi = (uint32_t)(ri.mask >> 32);
  f.kv_row = -1; f.out_row = -1;
  if (ri.valid) {
    const int phys = c.page_table[ri.seq * c.pages_per_seq + (ri.slot >> c.page_shift)];
    f.kv_row = (phys * c.n_kv_heads << c.page_shift) | (ri.slot & ((1 << c.page_shift) - 1));
    if (p.kind == PASS_VANILLA) f.out_row = ri.seq;
    else if (p.kind == PASS_PREFILL_T) f.out_row = ri.rel == p.chunk_n - 1 ? ri.seq : -1;
    else if (p.kind != PASS_PREFILL_D && ri.node >= 0) f.out_row = ri.seq * t->M + ri.node;
  }
  return f;
}

__device__ inline float cache_load(const float* p) { return *p; }
__device__ inline float cache_load(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ inline void cache_store(float* p, float v) { *p = v; }
__device__ inline void cache_store(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// Ints between two arrival counters: a 256-byte piece of memory each.  (Side by side, the arrivals of a launch were 256 atomic additions to two
// cache lines: O 11.7 -> 11.4 us, the head's O 10.6 -> 10.2, fc 17.4 -> 17.2 at 7B widths.)
constexpr int COUNTER_STRIDE = 64;

// Before a work-group announces its coherent stores through an arrival counter, every wave waits until its own
// vector-memory stores have been acknowledged.  A work-group-scope release fence alone does not do that on this
// target (waves of one work-group share a CU, so the compiler emits no vector-memory wait for it), and the stores
// go to other L2 channels than the counter: without the wait the counter can be seen before the data.
// s_waitcnt 0x0F70 = vmcnt(0), expcnt and lgkmcnt left alone.
__device__ __forceinline__ void publish_wait() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0x0F70);
}

// A value that nothing writes while the kernel runs, at an address that is the same for the whole wave: fetched into a scalar register.
template <typename T>
__device__ __forceinline__ T read_only(const T* p) { return *(const __attribute__((address_space(4))) T*)p; }

// ============================================================================ block reductions
__device__ inline float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// Sum over the block in a fixed order (wave partials added in wave order): deterministic.
__device__ inline float block_sum(float v, float* sh /*>= 16 floats*/) {
  v = wave_sum(v);
  int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += sh[i];
  return t;
}
__device__ inline float block_max(float v, float* sh) {
  v = wave_max(v);
  int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = sh[0];
  for (int i = 1; i < nw; ++i) t = fmaxf(t, sh[i]);
  return t;
}
// (value, index) with the larger value winning and, on equal values, the LOWER index.
__device__ inline void better(float& v, int& i, float v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
}
// The pair as one number: larger value first, then lower index; -0 and +0 are equal, a NaN counts as -inf.  0 is below every pair.
__device__ inline unsigned long long arg_key(float v, int i) {
  uint32_t b = __builtin_bit_cast(uint32_t, v == v ? v + 0.0f : -INFINITY);
  b ^= (uint32_t)((int)b >> 31) | 0x80000000u;
  return (unsigned long long)b << 32 | (uint32_t)~i;
}
__device__ inline int arg_index(unsigned long long key) { return (int)~(uint32_t)key; }
template <int CTRL, int ROWS>
__device__ inline unsigned long long key_max_dpp(unsigned long long k) {   // lanes without a source lane take 0
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)k, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(k >> 32), CTRL, ROWS, 0xf, false);
  const unsigned long long o = (unsigned long long)hi << 32 | lo;
  return o > k ? o : k;
}
__device__ inline unsigned long long key_of_lane(unsigned long long k, int lane) {
  return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(k >> 32), lane) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k, lane);
}
// Largest key of the wave.
__device__ inline unsigned long long wave_max_key(unsigned long long k) {
  k = key_max_dpp<0x111, 0xf>(k); k = key_max_dpp<0x112, 0xf>(k); k = key_max_dpp<0x114, 0xf>(k); k = key_max_dpp<0x118, 0xf>(k);   // row_shr 1, 2, 4, 8
  k = key_max_dpp<0x142, 0xa>(k); k = key_max_dpp<0x143, 0xc>(k);                                                                  // row_bcast 15, 31
  return key_of_lane(k, 63);
}
// The n largest of a wave's keys, N of them a lane, no two alike but for 0 (none): lane r returns the r-th.
template <int N>
__device__ inline unsigned long long wave_top_keys(const unsigned long long* keys, int n) {
  unsigned long long mine = 0, res = 0;
#pragma unroll
  for (int u = 0; u < N; ++u) mine = keys[u] > mine ? keys[u] : mine;
  for (int r = 0; r < n; ++r) {
    const unsigned long long top = wave_max_key(mine);
    if ((int)(threadIdx.x & 63) == r) res = top;
    if (mine == top && r + 1 < n) {                              // its owner: the next of its own
      mine = 0;
#pragma unroll
      for (int u = 0; u < N; ++u) mine = keys[u] < top && keys[u] > mine ? keys[u] : mine;
    }
  }
  return res;
}
// Largest key of the block (at most 16 waves); sh: 16 entries.  Lane moves inside the vector unit (row shifts, row broadcasts) instead of
// exchanges through the LDS unit (child selection at 1024 entries, two to four rounds: 12.3 -> 8.6 us a launch).
__device__ inline unsigned long long block_max_key(unsigned long long k, unsigned long long* sh) {
  k = wave_max_key(k);
  const int nw = (blockDim.x + 63) >> 6, l = threadIdx.x & 15;
  __syncthreads();                                               // (sh may still be read from the call before)
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = k;
  __syncthreads();
  k = l < nw ? sh[l] : 0;
  k = key_max_dpp<0x111, 0xf>(k); k = key_max_dpp<0x112, 0xf>(k); k = key_max_dpp<0x114, 0xf>(k); k = key_max_dpp<0x118, 0xf>(k);
  return key_of_lane(k, 15);
}

// ============================================================================ weight packing
// src: row-major [N][K] (float or bf16).  dst: nplanes packed planes (see wpack_index) of a matrix with KS k-steps;
// plane p starts at dst + p*plane_stride.  Source row n lands in packed row row_offset + map(n):
//   PACK_PLAIN  map(n) = n
//   PACK_ROPE   rows of a head are interleaved so that the two members of a rotate-half pair (i, i + dh/2) become
//               neighbours: head*dh + i + half*dh/2  ->  head*dh + 2i + half
//   PACK_GATE / PACK_UP  fused gate/up matrix: every 32-row block holds gate rows 16j..16j+15 then up rows
//               16j..16j+15, so SwiGLU partners sit in the same block
// One thread builds one 16-byte lane chunk (8 elements along k) of every plane.
enum { PACK_PLAIN = 0, PACK_ROPE = 1, PACK_GATE = 2, PACK_UP = 3 };
__host__ __device__ inline int pack_row_map(int mode, int n, int dh) {
  if (mode == PACK_ROPE) {
    int head = n / dh, r = n % dh, half = dh >> 1;
    return head * dh + 2 * (r % half) + r / half;
  }
  if (mode == PACK_GATE) return (n >> 4) * 32 + (n & 15);
  if (mode == PACK_UP) return (n >> 4) * 32 + 16 + (n & 15);
  return n;
}
template <typename SrcT>
__global__ __launch_bounds__(256) void k_pack_weight(const SrcT* __restrict__ src, bf16_t* __restrict__ dst, int N, int K,
                                                     int row_offset, int KS, int nplanes, size_t plane_stride, int mode, int dh,
                                                     size_t ldn = 0 /*source stride between rows n (0 = K)*/, size_t ldk = 1 /*between columns k*/) {
  if (ldn == 0) ldn = (size_t)K;
  size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  int nrb = (N + 31) >> 5;
  size_t total = (size_t)nrb * KS * 64;
  if (gid >= total) return;
  int lane = gid & 63;
  size_t tile = gid >> 6;
  int ks = tile % KS;
  int rb = tile / KS;
  int n = rb * 32 + (lane & 31);
  int k0 = ks * 16 + (lane >> 5) * 8;
  if (n >= N && mode != PACK_PLAIN) return;               // only the plain map pads its last block with zero rows
  bf16_t out[3][8];
  for (int t = 0; t < 8; ++t) {
    float x = 0.f;
    if (n < N && k0 + t < K) {
      if constexpr (sizeof(SrcT) == 4) x = ((const float*)src)[(size_t)n * ldn + (size_t)(k0 + t) * ldk];
      else x = bf16_to_f32(((const bf16_t*)src)[(size_t)n * ldn + (size_t)(k0 + t) * ldk]);
    }
    bf16_t p[3];
    split_bf16(x, p, nplanes);
    for (int q = 0; q < nplanes; ++q) out[q][t] = p[q];
  }
  size_t o = wpack_index(row_offset + pack_row_map(mode, n, dh), k0, KS);
  for (int q = 0; q < nplanes; ++q) {
    u32x4 v;
    v.x = out[q][0] | ((uint32_t)out[q][1] << 16); v.y = out[q][2] | ((uint32_t)out[q][3] << 16);
    v.z = out[q][4] | ((uint32_t)out[q][5] << 16); v.w = out[q][6] | ((uint32_t)out[q][7] << 16);
    *(u32x4*)(dst + q * plane_stride + o) = v;
  }
}

// ---- 4-bit weights (Sec. 4.2: the int4 case study) ---------------------------------------------------------------------
// Weight-only, symmetric, groups of 128 input columns: s = bf16(max|w| / 7), code = clip(rint(w / s), -8, 7) + 8, value
// s * (code - 8).  Layout: "super-tiles" of 32 rows x 64 k = 1 KiB, tile (rb, T) at ((rb*KT + T) * 64) 16-byte lane
// chunks (KT = K / 64); lane l (row l%32, k-half l/32) holds four 32-bit words, word j = the 8 codes of k-step j of
// the super-tile, k = 64T + 16j + 8(l/32) + e, with code e at bit 4*(e/2) + 16*(e%2), the word then rotated left by 3:
// ((word rotated right by 4p) & 0x00780078) | 0x41804180 is then the bf16 pair (16 + code 2p, 16 + code 2p+1), i.e. the MFMA A
// operand of the k-step comes out of one shift and one and-or per pair (16 + c is exact in bf16; the offset 24 = 16 + 8 is
// taken off per group: the smallest that leaves room for four bits, so that as little as possible cancels).  Not rotated, the
// same takes 0x000F000F and 0x43004300 to pairs of 128 + code (offset 136).
// Scales: bf16 [rb][group][lane-half][16] in accumulator-register order: entry (hh, r) belongs to row
// 8*(r/4) + 4*hh + r%4 of the block, so a lane reads the scales of its 16 accumulator rows as 32 contiguous bytes.
#define EAGLE_Q4_GROUP 128
struct Q4Format { uint32_t keep, bias; float offset; };        // bits of the codes, what they are or-ed into, what that adds to a code's value
constexpr int Q4_ROT_LARGE_M = 3;                               // the packing that k_gemm_pf_q4 and k_group_sums are built for
__host__ __device__ constexpr Q4Format q4_format(int rot) { return rot ? Q4Format{0x00780078u, 0x41804180u, 24.0f} : Q4Format{0x000F000Fu, 0x43004300u, 136.0f}; }
// An instruction reads one scalar register or constant at most: with `bias` in a vector register the mask and the bias are one instruction
// (v_and_or_b32), with both constants scalar two; seven instead of eleven instructions for the eight codes.  7B in 4 bits, us a launch before / after: QKV 15.75 / 15.55, gate/up
// 19.9 / 19.5, down 13.9 / 13.7, LM head of a draft level 21.3 / 20.5, prompt of 512 tokens 18.3 / 17.9 ms; the same bits.
__device__ __forceinline__ Q4Format q4_pin(Q4Format f) {
  asm volatile("" : "+s"(f.keep), "+v"(f.bias));
  return f;
}
__device__ __forceinline__ u32x4 q4_expand(uint32_t wd, const Q4Format& f) {
  u32x4 v;
  v.x = (wd & f.keep) | f.bias;
  v.y = ((wd >> 4) & f.keep) | f.bias;
  v.z = ((wd >> 8) & f.keep) | f.bias;
  v.w = (__builtin_amdgcn_alignbit(wd, wd, 12) & f.keep) | f.bias;   // (rotated, the last high code straddles the word's end)
  return v;
}
template <typename SrcT>
__global__ __launch_bounds__(256) void k_pack_weight_q4(const SrcT* __restrict__ src, uint32_t* __restrict__ dst, bf16_t* __restrict__ sc,
                                                        int N, int K, int row_offset, int mode, int dh, int rot) {
  const int NG = K / EAGLE_Q4_GROUP, KT = K / 64;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int nrows = mode == PACK_PLAIN ? (N + 31) / 32 * 32 : N;          // only the plain map pads its last block
  if (gid >= (size_t)nrows * NG) return;
  const int n = (int)(gid / NG), g = (int)(gid % NG);
  float w[EAGLE_Q4_GROUP];
  float mx = 0.f;
  for (int t = 0; t < EAGLE_Q4_GROUP; ++t) {
    float x = 0.f;
    if (n < N) {
      if constexpr (sizeof(SrcT) == 4) x = ((const float*)src)[(size_t)n * K + g * EAGLE_Q4_GROUP + t];
      else x = bf16_to_f32(((const bf16_t*)src)[(size_t)n * K + g * EAGLE_Q4_GROUP + t]);
    }
    w[t] = x;
    mx = fmaxf(mx, fabsf(x));
  }
  const bf16_t sb = f32_to_bf16(mx / 7.0f);
  const float s = bf16_to_f32(sb), safe = s > 0.f ? s : 1.0f;
  const int prow = row_offset + pack_row_map(mode, n, dh);
  const int rb = prow >> 5, rho = prow & 31, hh = (rho >> 2) & 1, r = 4 * (rho >> 3) + (rho & 3);
  sc[(((size_t)rb * NG + g) * 2 + hh) * 16 + r] = sb;
  for (int st = 0; st < 2; ++st) {                                        // the group's two super-tiles
    const int T = 2 * g + st;
    for (int kh = 0; kh < 2; ++kh) {
      uint32_t words[4];
      for (int j = 0; j < 4; ++j) {
        uint32_t wd = 0;
        for (int e = 0; e < 8; ++e) {
          const float q = fminf(fmaxf(rintf(w[64 * st + 16 * j + 8 * kh + e] / safe), -8.f), 7.f);
          wd |= (uint32_t)((int)q + 8) << (4 * (e >> 1) + 16 * (e & 1));
        }
        words[j] = __builtin_amdgcn_alignbit(wd, wd, (32 - rot) & 31);   // rotated left
      }
      u32x4 v; v.x = words[0]; v.y = words[1]; v.z = words[2]; v.w = words[3];
      *(u32x4*)(dst + (((size_t)rb * KT + T) * 64 + rho + 32 * kh) * 4) = v;
    }
  }
}

// ============================================================================ skinny weight-streaming GEMM
// PT[s][m][n] = sum over the split's k range of W[n][k] * X[m][k];  W packed (NWP bf16 planes), X in XF layout
// (NXP bf16 planes, MT 32-row tiles).  A block is 4 waves; wave w owns row-block blockIdx.x*4+w (32 rows of W)
// and streams it once: every tile is one coalesced 1 KiB load that goes straight into the MFMA A operand.  The
// block's X slice passes through LDS (already in B-operand order) in chunks of CH k-steps.  While a chunk is being
// multiplied, the next chunk's weight tiles AND activation tiles are already on their way into registers, so neither
// HBM nor L2 latency is exposed between chunks.  Products kept: plane pairs (p, q) with p + q < max(NWP, NXP);
// pieces beyond that are below fp32 resolution of the sum.
template <int NXP> struct GemmChunk { static constexpr int CH = NXP == 2 ? 8 : 4; };   // k-steps per LDS stage
template <int NWP, int NXP, int MT>
__global__ __launch_bounds__(256) void k_gemm(const bf16_t* __restrict__ Wp, size_t w_plane_stride,
                                              const bf16_t* __restrict__ XF, float* __restrict__ PT, int NRB, int KS,
                                              int ks_per_split, int Npad) {
  constexpr int CH = GemmChunk<NXP>::CH;
  constexpr int XT = NXP * MT * CH;                             // activation tiles (1 KiB each) per chunk
  constexpr int XR = (XT * 64 + 255) / 256;                     // 16-byte pieces of them per thread
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* xs = (u32x4*)smem;                                     // [NXP*MT][CH][64] 16-byte lane chunks
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rb = min(blockIdx.x * 4 + wave, NRB - 1);           // waves past the end repeat the last block, store nothing
  const bool live = blockIdx.x * 4 + wave < NRB;
  const int s = blockIdx.y;
  const int k_begin = s * ks_per_split;
  const int k_end = min(KS, k_begin + ks_per_split);
  constexpr int PMAX = NWP > NXP ? NWP : NXP;
  f32x16 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
  if (k_end <= k_begin) return;
  const int klast = k_end - 1;
  const u32x4* wbase = (const u32x4*)(Wp + (size_t)rb * KS * 512) + lane;

  u32x4 xr[XR], ar[CH][NWP];
  // piece i of a chunk: tile pm = i / (CH*64), k-step kk = (i / 64) % CH, lane-chunk i % 64 (the LDS order)
  auto load_x = [&](int c0) {
#pragma unroll
    for (int u = 0; u < XR; ++u) {
      const int i = min(u * 256 + (int)threadIdx.x, XT * 64 - 1);
      const int pm = i / (CH * 64), kk = (i / 64) % CH, l = i & 63;
      xr[u] = *((const u32x4*)(XF + ((size_t)pm * KS + min(c0 + kk, klast)) * 512) + l);
    }
  };
  auto load_a = [&](int c0) {
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
      for (int p = 0; p < NWP; ++p)
        ar[u][p] = *(const u32x4*)((const bf16_t*)(wbase + (size_t)min(c0 + u, klast) * 64) + p * w_plane_stride);
  };
  auto store_x = [&]() {
#pragma unroll
    for (int u = 0; u < XR; ++u) {
      const int i = u * 256 + (int)threadIdx.x;
      if (i < XT * 64) xs[i] = xr[u];
    }
  };
  load_x(k_begin);
  load_a(k_begin);
  store_x();
  __syncthreads();
  for (int c0 = k_begin; c0 < k_end; c0 += CH) {
    const int nk = min(CH, k_end - c0);
    const bool more = c0 + CH < k_end;
    u32x4 a[CH][NWP];
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
      for (int p = 0; p < NWP; ++p) a[u][p] = ar[u][p];
    if (more) { load_x(c0 + CH); load_a(c0 + CH); }            // in flight while this chunk is multiplied
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      if (u < nk) {
#pragma unroll
        for (int q = 0; q < NXP; ++q)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            const u32x4 b = xs[((size_t)(q * MT + mt) * CH + u) * 64 + lane];
#pragma unroll
            for (int p = 0; p < NWP; ++p)
              if (p + q < PMAX)
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u][p]),
                                                                  __builtin_bit_cast(bf16x8, b), acc[mt], 0, 0, 0);
          }
      }
    }
    __syncthreads();                                            // every wave is done with this chunk's LDS
    if (more) { store_x(); __syncthreads(); }
  }
  if (live) {
    // accumulator register r of lane l holds W-row 8*(r/4) + 4*(l/32) + r%4, X-row l%32; partials are stored
    // PT[s][m][n] (n fastest, which is how every epilogue kernel walks them): registers 4i..4i+3 are 16 contiguous bytes
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float* out = PT + ((size_t)s * (MT * 32) + mt * 32 + (lane & 31)) * Npad + (size_t)rb * 32 + 4 * (lane >> 5);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 v; v.x = acc[mt][4 * i]; v.y = acc[mt][4 * i + 1]; v.z = acc[mt][4 * i + 2]; v.w = acc[mt][4 * i + 3];
        *(f32x4*)(out + 8 * i) = v;
      }
    }
  }
}

// ============================================================================ large-M GEMM (prompt passes, batched tree passes, the loss)
// Same operands and the same PT[s][m][n] result as k_gemm, for passes whose rows fill several 32-row tiles: here the
// MFMA pipes, not the weight stream, are the bound (Sec. 3.1: the head consumes the whole prompt's features, so the
// prompt runs through the target and the head once, as one large matrix product per weight matrix).
//   work-group tile  2 * RBW row blocks of weights x 2 * MW tiles of 32 activation rows; 2 x MW waves
//   wave (wn, wm)    RBW row blocks x 2 activation tiles, both activation planes: 4 * RBW MFMAs per k-step
//   LDS              a ring of four k-steps of BOTH operands (20 to 24 KiB each for MW = 4, 14 to 16 for MW = 2, 10 to 12 for MW = 1), filled by
//                    direct global -> LDS loads (both operands lie in memory in fragment order: one load = one 1 KiB tile)
// At the barrier of k-step k every wave holds that step's fragments in registers, so its slot is refilled with step k + 4 at
// once, step k + 1 is read from LDS behind the barrier, and both travel while the 4 * RBW MFMAs run: neither memory nor LDS
// latency is waited for, and no registers are spent on data in flight (four separate arrays, so that the compiler can
// tell the slot being filled from the slot being read and adds no wait of its own).
// (Rings of 6 and 8 k-steps measured the same or slower, a K order rotated per work-group the same.)
// Which tile: the host (plan_pf) takes the shape whose work-groups fill the CUs of every XCD in the fewest, fullest rounds.
// Bound: the matrix pipes at the clock the card holds under them; the library's own 8192-cubed bf16 product reaches 1.2 PFLOP/s on
// this card.  Issued work of both planes: 512 rows at 7B widths 1.0 to 1.07 PFLOP/s (QKV 102, O and down 64 on average, gate/up 173 us; the
// kernel before, tiles of 8 x 4 with the activations through registers, 125, 67 and 217), 1024 rows at 13B widths 1.20 (gate/up 481
// us), 2011 rows at 70B widths 1.33 (gate/up 2837 us).  With N(0, 0.02) weights the clock is higher: 95, 59 and 159 us at 7B.  Pipes
// busy: 63 to 74 % at 512 rows, 77 to 78 % from 1024 on.
// Work-groups that share a weight tile (the activation-row tiles of one weight-row tile) get ids 8 apart, i.e. the same
// XCD under round-robin dispatch, next to each other in dispatch order: the tile comes from HBM once and from that
// XCD's L2 afterwards.
// Every K range is a multiple of 4 k-steps (host).
__device__ inline void xf_store8(bf16_t* XF, int m, int k8, int MT, int KS, int nplanes, const float* x);   // defined with the row producers below
// What both large-M GEMMs do with a wave's accumulators (row blocks rb0.., tiles mt0, mt0 + 1 below tile_end, rows below row_end).
// SWIGLU (only with S = 1, gate/up matrices): silu(gate) * up as the next GEMM's input (XF layout, `act`, rows beyond the end as
// zeros).  A row block of the fused matrix holds 16 gate rows and the 16 up rows of the same features, and accumulator registers
// r and r + 8 of a lane are such a pair; the two lanes of an activation row swap four values so that each holds 8 consecutive
// features = its 16 bytes of the output tile.
constexpr int PF_STAGE_LD = 36;      // row stride of the staged tile in words
template <int RBW, bool SWIGLU>
__device__ __forceinline__ void pf_store(f32x16 (&acc)[RBW][2], float* __restrict__ PT, int s, int NRB, int Npad, int MT, bf16_t* act, int rb0, int mt0, int tile_end, int row_end,
                                         float* stage) {
  constexpr int NXP = 2;
  const int lane = threadIdx.x & 63;
  // accumulator register r of lane l: weight row 8*(r/4) + 4*(l/32) + r%4, activation row l%32; PT[s][m][n], n fastest
  if constexpr (SWIGLU) {
    const int hh = lane >> 5;
#pragma unroll
    for (int j = 0; j < RBW; ++j) {
      const int rb = rb0 + j;
      if (rb >= NRB) continue;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int mt = mt0 + t;
        if (mt >= tile_end) continue;
        const int m = mt * 32 + (lane & 31);
        float v[8];                                             // features 4hh + {0..3} and 8 + 4hh + {0..3} of the block
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float gs = acc[j][t][r], us = acc[j][t][r + 8];
          v[r] = m < row_end ? gs / (1.0f + __expf(-gs)) * us : 0.f;
        }
        float x[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float got = __shfl_xor(hh ? v[i] : v[4 + i], 32, 64);   // the partner's features 4..7 (for hh = 0) or 8..11 (for hh = 1)
          x[i] = hh ? got : v[i];
          x[4 + i] = hh ? v[4 + i] : got;
        }
        xf_store8(act, m, 16 * rb + 8 * hh, MT, NRB, NXP, x);
      }
    }
    return;
  }
  // A 32 x 32 tile of sums passes through this wave's own piece of LDS, so that a store instruction writes eight whole 128-byte lines
  // of PT.  (Straight from the accumulators it touched 32 lines with 32 bytes each, four times over.  us before / after: 104 rows at
  // 7B widths, gate/up 53.5 / 52.2, QKV 37.4 / 36.2, O and down on average 25.4 / 24.0; 300 rows 41.5 / 38.9; 1024 rows at 13B widths
  // 197 / 193.)  The LDS operations of a wave stay in order; the stride of PF_STAGE_LD words spreads rows over the banks.
  const int Mpad = MT * 32;
#pragma unroll
  for (int j = 0; j < RBW; ++j) {
    const int rb = rb0 + j;
    if (rb >= NRB) continue;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int mt = mt0 + t;
      if (mt >= tile_end) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 v; v.x = acc[j][t][4 * i]; v.y = acc[j][t][4 * i + 1]; v.z = acc[j][t][4 * i + 2]; v.w = acc[j][t][4 * i + 3];
        *(f32x4*)(stage + (lane & 31) * PF_STAGE_LD + 8 * i + 4 * (lane >> 5)) = v;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      float* out = PT + ((size_t)s * Mpad + mt * 32 + (lane >> 3)) * Npad + (size_t)rb * 32 + 4 * (lane & 7);
#pragma unroll
      for (int i = 0; i < 4; ++i) *(f32x4*)(out + (size_t)(8 * i) * Npad) = *(const f32x4*)(stage + (8 * i + (lane >> 3)) * PF_STAGE_LD + 4 * (lane & 7));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

struct BufferRsrc { __amdgpu_buffer_rsrc_t rs; };
// 16 bytes a lane straight into LDS (at `l` + 16 * lane).
__device__ __forceinline__ void buffer_to_lds16(__amdgpu_buffer_rsrc_t rs, void* l, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)l, 16, lane_off, off, 0, 0);
}
// GROUPED (mixture of experts): the activation tiles are the experts' rows gathered one expert after the other (k_moe_gather),
// every work-group column of RT tiles belongs to one expert (k_moe_plan), whose matrix starts `expert_stride` elements behind
// the previous one's; columns beyond the last expert's end leave at once.
constexpr int MOE_MAX_COLS = 256;
struct MoePlan { int n_cols, pad[3]; int expert[MOE_MAX_COLS], tile0[MOE_MAX_COLS], rows[MOE_MAX_COLS]; };   // per column: expert, first tile, rows
template <int RBW, int MW, bool SWIGLU = false, bool GROUPED = false, bool PLAIN = false>
__global__ __launch_bounds__(128 * MW, 2) void k_gemm_pf(const bf16_t* __restrict__ Wp, const bf16_t* __restrict__ XF,
                                                         float* __restrict__ PT, int NRB, int KS, int ks_per_split, int S, int Npad,
                                                         int MT /*32-row tiles of the pass*/, bf16_t* act, int M,
                                                         const MoePlan* moe = nullptr, size_t expert_stride = 0, int MQ_grid = 0) {
  constexpr int NXP = 2, WT = 2 * RBW, RT = 2 * MW, NTILE = WT + NXP * RT, NW = 2 * MW, LPW = (NTILE + NW - 1) / NW;
  constexpr int SLOT = NTILE * 64;
  __shared__ u32x4 s0[SLOT];                                    // per k-step: WT weight tiles, then NXP planes of RT activation tiles
  __shared__ u32x4 s1[SLOT];
  __shared__ u32x4 s2[SLOT];
  __shared__ u32x4 s3[SLOT];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wn = w & 1, wm = w >> 1;
  // id -> (group = (weight-row tile, split), activation-row tile)
  const int MQ = GROUPED ? MQ_grid : (MT + RT - 1) / RT, NT = (NRB + WT - 1) / WT, G = NT * S;
  const int L = blockIdx.x, blk = L / (8 * MQ), rem = L % (8 * MQ), mq = rem >> 3, g = blk * 8 + (rem & 7);
  if (g >= G) return;
  // this column's tiles [tile0, tile_end) and rows [.., row_end)
  int tile0 = mq * RT, tile_end = min(MT, tile0 + RT), row_end = M;
  if constexpr (GROUPED) {
    if (mq >= moe->n_cols) return;
    tile0 = moe->tile0[mq];
    row_end = tile0 * 32 + moe->rows[mq];
    tile_end = (row_end + 31) >> 5;
    Wp += (size_t)moe->expert[mq] * expert_stride;
  }
  const int nt = g / S, s = g % S;
  const int k_begin = s * ks_per_split, k_end = min(KS, k_begin + ks_per_split);
  if (k_end <= k_begin) return;
  const int klast = k_end - 1;
  const int rb0 = nt * WT + wn * RBW, mt0 = tile0 + wm * 2;
  // a wave whose activation tiles or row blocks all lie beyond the end moves data and keeps the barriers, but multiplies nothing
  const bool busy = mt0 < tile_end && rb0 < NRB;
  // The tiles this wave loads, the same number in every wave (the last tile is loaded more than once where they do not divide).  Buffer
  // loads: a tile's base in a resource, the k-step in the scalar offset, no address arithmetic in the vector unit, and lanes of rows or
  // blocks beyond the end out of range, which move nothing and leave zeros (zeros also cost the matrix pipes less power).  PLAIN:
  // loads of an address a lane, tiles beyond the end as the last one there is.  (Which launches take which, and what both measured:
  // plan_pf_plain_loads.  Grouped experts of a 1000-row prompt at Mixtral widths, us, buffer / plain loads on each of two cards: gate/up 931 / 970 and 865 /
  // 1013, down 474 / 460 and 444 / 491; of a 104-row one 381 / 386 and 381 / 389, 255 / 272 and 257 / 283.)
  BufferRsrc src[LPW];
  const bf16_t* ptr[LPW];
  uint32_t vo[LPW];
  int dst[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int i = min(w + u * NW, NTILE - 1), t = tile0 + (i - WT) % RT;
    ptr[u] = i < WT ? Wp + (size_t)min(nt * WT + i, NRB - 1) * KS * 512 : XF + (size_t)((i - WT) / RT * MT + min(t, tile_end - 1)) * KS * 512;
    src[u].rs = __builtin_amdgcn_make_buffer_rsrc((void*)ptr[u], 0, KS * 1024, 0x00020000);
    vo[u] = (i < WT ? nt * WT + i < NRB : t * 32 + (lane & 31) < row_end) ? lane * 16u : 0x80000000u;
    dst[u] = i * 64;
  }
  // (k-steps beyond the end are clamped, so that the number of loads in flight is the same on every path)
  auto dma = [&](u32x4* slot, int k) {
    const uint32_t kk = (uint32_t)min(k, klast);
#pragma unroll
    for (int u = 0; u < LPW; ++u) {
      if constexpr (PLAIN) __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(ptr[u] + (size_t)kk * 512 + lane * 8), (__attribute__((address_space(3))) void*)(slot + dst[u]), 16, 0, 0);
      else buffer_to_lds16(src[u].rs, slot + dst[u], vo[u], kk * 1024u);
    }
  };
  f32x16 acc[RBW][2];
#pragma unroll
  for (int j = 0; j < RBW; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.f;
  u32x4 fa[2][RBW], fb[2][NXP * 2];
  auto frags = [&](const u32x4* slot, int b) {
#pragma unroll
    for (int j = 0; j < RBW; ++j) fa[b][j] = slot[(wn * RBW + j) * 64 + lane];
#pragma unroll
    for (int q = 0; q < NXP; ++q)
#pragma unroll
      for (int t = 0; t < 2; ++t) fb[b][q * 2 + t] = slot[(WT + q * RT + wm * 2 + t) * 64 + lane];
  };
  auto mul = [&](int b) {
#pragma unroll
    for (int q = 0; q < NXP; ++q)
#pragma unroll
      for (int j = 0; j < RBW; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[b][j]), __builtin_bit_cast(bf16x8, fb[b][q * 2 + t]), acc[j][t], 0, 0, 0);
  };
  dma(s0, k_begin); dma(s1, k_begin + 1); dma(s2, k_begin + 2); dma(s3, k_begin + 3);
  // vmcnt(n), the other counters left alone; a bare barrier: __syncthreads() would drain every load in flight
#define PF_WAITV(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define PF_BAR() do { asm volatile("" ::: "memory"); __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); } while (0)
  PF_WAITV(3 * LPW);
  PF_BAR();
  frags(s0, 0);
  // all fragments of step k are in registers and this wave's loads of step k + 1 have landed -> barrier -> so have everyone's
#define PF_STEP(i, cur, nxt)                                                        \
  {                                                                                 \
    __builtin_amdgcn_s_waitcnt(0xC07F);                    /* lgkmcnt(0) */         \
    PF_WAITV(2 * LPW);                                                              \
    PF_BAR();                                                                       \
    frags(nxt, ((i) & 1) ^ 1);                                                      \
    dma(cur, k + (i) + 4);                                                          \
    if (busy) mul((i) & 1);                                                         \
    __builtin_amdgcn_sched_barrier(0);                                              \
  }
  for (int k = k_begin; k < k_end; k += 4) {
    PF_STEP(0, s0, s1)
    PF_STEP(1, s1, s2)
    PF_STEP(2, s2, s3)
    PF_STEP(3, s3, s0)
  }
  PF_WAITV(0);                                                  // no load may be on its way into LDS when the work-group ends,
  PF_BAR();                                                     // nor into the piece of it that a wave stages its sums in
#undef PF_STEP
#undef PF_WAITV
#undef PF_BAR
  if (!busy) return;
  static_assert(SLOT * 16 / (NW > 4 ? 2 : 1) >= 32 * PF_STAGE_LD * 4 && NW <= 8, "a wave's piece of a slot holds a staged tile");
  u32x4* const slot = w & 2 ? (w & 1 ? s3 : s2) : (w & 1 ? s1 : s0);
  pf_store<RBW, SWIGLU>(acc, PT, s, NRB, Npad, MT, act, rb0, mt0, tile_end, row_end, (float*)(slot + (w >> 2) * (SLOT / 2)));
}

// ---- the same over 4-bit weights (layout: k_pack_weight_q4) -----------------------------------------------------------------
// A wave owns 2 row blocks x 2 activation tiles.  Per group of 8 k-steps the MFMAs sum (16 + code) x into `part` (the codes become
// bf16 with one shift and one and-or per pair, beside the MFMAs), and the group is folded into the result in fp32:
// acc += scale * (part - 24 * sum of x).  The activations pass through the four-slot ring of k_gemm_pf; the codes of four k-steps (one
// 1 KiB tile per row block) through two slots; the group's scales and its sums of x (-24 times them: k_group_sums) through one
// slot each, requested at the group's first step and read behind its last.  Loads in flight are counted: step i waits for all
// but the loads of the two steps before it.  K ranges are whole groups (host).
// Bound: the matrix pipes; 8 MFMAs a k-step and wave, 16 more registers of sums than k_gemm_pf's 8-MFMA shape allow no more.
// (The prompt used to walk through the decoding kernels 32 rows at a time, every pass streaming all codes: 3.2 ms per 32 rows
// at 7B widths.)
template <bool SWIGLU>
__global__ __launch_bounds__(256, 2) void k_gemm_pf_q4(const u32x4* __restrict__ Wq, const bf16_t* __restrict__ SC, const bf16_t* __restrict__ XF,
                                                            const float* __restrict__ SX, float* __restrict__ PT, int NRB, int KS, int groups_per_split,
                                                            int S, int Npad, int MT, bf16_t* act, int M) {
  constexpr int RBW = 2, NXP = 2, WT = 2 * RBW, RT = 4, NW = 4, XT = NXP * RT, LPW = XT / NW;
  __shared__ u32x4 s0[XT * 64];
  __shared__ u32x4 s1[XT * 64];
  __shared__ u32x4 s2[XT * 64];
  __shared__ u32x4 s3[XT * 64];
  __shared__ u32x4 c0[WT * 64];                                 // codes of the group's first / second four k-steps
  __shared__ u32x4 c1[WT * 64];
  __shared__ u32x4 scl[64];                                     // the group's scales: [WT row blocks][2 lane halves][16] bf16
  __shared__ u32x4 sxs[64];                                     // -24 * sum of x over the group: [RT * 32 rows] fp32
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wn = w & 1, wm = w >> 1, hh = lane >> 5;
  const int MQ = (MT + RT - 1) / RT, NT = (NRB + WT - 1) / WT, G = NT * S, NG = KS / 8, KT = KS / 4;
  const int L = blockIdx.x, blk = L / (8 * MQ), rem = L % (8 * MQ), mq = rem >> 3, g = blk * 8 + (rem & 7);
  if (g >= G) return;
  const int nt = g / S, s = g % S;
  const int g_begin = s * groups_per_split, g_end = min(NG, g_begin + groups_per_split);
  if (g_end <= g_begin) return;
  const int klast = g_end * 8 - 1, Tlast = g_end * 2 - 1;
  const int tile0 = mq * RT, tile_end = min(MT, tile0 + RT);
  const int rb0 = nt * WT + wn * RBW, mt0 = tile0 + wm * 2;
  const bool busy = mt0 < tile_end && rb0 < NRB;
  BufferRsrc src[LPW];                                          // (as in k_gemm_pf: rows beyond the end out of range)
  uint32_t vo[LPW];
  int dst[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int i = w + u * NW, t = tile0 + i % RT;
    src[u].rs = __builtin_amdgcn_make_buffer_rsrc((void*)(XF + (size_t)(i / RT * MT + min(t, tile_end - 1)) * KS * 512), 0, KS * 1024, 0x00020000);
    vo[u] = t * 32 + (lane & 31) < M ? lane * 16u : 0x80000000u;
    dst[u] = i * 64;
  }
  auto dma = [&](u32x4* slot, int k) {
    const uint32_t ko = (uint32_t)min(k, klast) * 1024u;
#pragma unroll
    for (int u = 0; u < LPW; ++u) buffer_to_lds16(src[u].rs, slot + dst[u], vo[u], ko);
  };
  // One code tile per wave: w % WT is w.  (Written as w the same loop comes out one instruction earlier, and a 500-token request at 7B
  // widths measured 0.7 to 0.9 % slower in two builds' comparisons, against 0.2 to 0.3 % between identical kernels; so it stays.)
  BufferRsrc csrc, ssrc, xsrc;
  csrc.rs = __builtin_amdgcn_make_buffer_rsrc((void*)(Wq + (size_t)min(nt * WT + w % WT, NRB - 1) * KT * 64), 0, KT * 1024, 0x00020000);
  auto dma_codes = [&](u32x4* slot, int T) { buffer_to_lds16(csrc.rs, slot + (w % WT) * 64, lane * 16u, (uint32_t)min(T, Tlast) * 1024u); };
  // lane l brings 16 bytes of the scales of row block l / 4 (lanes beyond the tile repeat the last ones) and of the sums of x
  ssrc.rs = __builtin_amdgcn_make_buffer_rsrc((void*)(SC + (size_t)nt * WT * NG * 32), 0, min(WT, NRB - nt * WT) * NG * 64, 0x00020000);
  const uint32_t s_lane = (uint32_t)(min(min(lane >> 2, WT - 1), NRB - 1 - nt * WT) * NG * 32 + (lane & 3) * 8) * 2u;
  xsrc.rs = __builtin_amdgcn_make_buffer_rsrc((void*)SX, 0, NG * MT * 128, 0x00020000);
  const uint32_t x_lane = (uint32_t)(tile0 * 32 + (lane & (RT * 8 - 1)) * 4) * 4u;
  f32x16 acc[RBW][2], part[RBW][2];
#pragma unroll
  for (int j = 0; j < RBW; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.f;
  u32x4 fb[2][NXP * 2], cd[2][RBW];
  const Q4Format fmt = q4_pin(q4_format(Q4_ROT_LARGE_M));
  auto frags = [&](const u32x4* slot, int b) {
#pragma unroll
    for (int q = 0; q < NXP; ++q)
#pragma unroll
      for (int t = 0; t < 2; ++t) fb[b][q * 2 + t] = slot[(q * RT + wm * 2 + t) * 64 + lane];
  };
  auto codes = [&](const u32x4* slot, int b) {
#pragma unroll
    for (int j = 0; j < RBW; ++j) cd[b][j] = slot[(wn * RBW + j) * 64 + lane];
  };
  auto mul = [&](int i) {                                       // k-step i of the group
    const int b = i & 1;
    u32x4 av[RBW];
#pragma unroll
    for (int j = 0; j < RBW; ++j) {
      const uint32_t wd = cd[(i >> 2) & 1][j][i & 3];
      av[j] = q4_expand(wd, fmt);
    }
#pragma unroll
    for (int q = 0; q < NXP; ++q)
#pragma unroll
      for (int j = 0; j < RBW; ++j)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f32x16 z;
#pragma unroll
          for (int r = 0; r < 16; ++r) z[r] = 0.f;
          part[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[j]), __builtin_bit_cast(bf16x8, fb[b][q * 2 + t]),
                                                               i == 0 && q == 0 ? z : part[j][t], 0, 0, 0);
        }
  };
#define PF_WAITV(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define PF_BAR() do { asm volatile("" ::: "memory"); __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); } while (0)
  dma_codes(c0, 2 * g_begin);
  dma(s0, 8 * g_begin); dma(s1, 8 * g_begin + 1); dma(s2, 8 * g_begin + 2); dma(s3, 8 * g_begin + 3);
  PF_WAITV(3 * LPW);
  PF_BAR();
  frags(s0, 0);
  codes(c0, 0);
  // extra loads: 3 in a group's step 0 (codes, scales, sums of x), 1 in its step 4 (codes)
#define PF_STEP(i, cur, nxt)                                                                            \
  {                                                                                                     \
    __builtin_amdgcn_s_waitcnt(0xC07F);                    /* lgkmcnt(0) */                             \
    PF_WAITV(2 * LPW + ((i) == 1 || (i) == 2 ? 3 : (i) == 5 || (i) == 6 ? 1 : 0));                      \
    PF_BAR();                                                                                           \
    if ((i) == 0) {                                                                                     \
      buffer_to_lds16(ssrc.rs, scl, s_lane, (uint32_t)gi * 64u);                                        \
      buffer_to_lds16(xsrc.rs, sxs, x_lane, (uint32_t)(gi * MT) * 128u);                                \
      dma_codes(c1, 2 * gi + 1);                                                                        \
    }                                                                                                   \
    if ((i) == 4) dma_codes(c0, 2 * gi + 2);                                                            \
    frags(nxt, ((i) & 1) ^ 1);                                                                          \
    if ((i) == 3) codes(c1, 1);                                                                         \
    if ((i) == 7) codes(c0, 0);                                                                         \
    dma(cur, 8 * gi + (i) + 4);                                                                         \
    if (busy) mul(i);                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
  }
  for (int gi = g_begin; gi < g_end; ++gi) {
    PF_STEP(0, s0, s1)
    PF_STEP(1, s1, s2)
    PF_STEP(2, s2, s3)
    PF_STEP(3, s3, s0)
    PF_STEP(4, s0, s1)
    PF_STEP(5, s1, s2)
    PF_STEP(6, s2, s3)
    PF_STEP(7, s3, s0)
    if (busy) {
#pragma unroll
      for (int j = 0; j < RBW; ++j) {
        const u32x4 sa = scl[(wn * RBW + j) * 4 + 2 * hh], sb = scl[(wn * RBW + j) * 4 + 2 * hh + 1];
        const uint32_t sw[8] = {sa.x, sa.y, sa.z, sa.w, sb.x, sb.y, sb.z, sb.w};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const float sx = ((const float*)sxs)[(wm * 2 + t) * 32 + (lane & 31)];
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float sv = __builtin_bit_cast(float, (r & 1) ? (sw[r >> 1] & 0xFFFF0000u) : (sw[r >> 1] << 16));
            acc[j][t][r] += sv * (part[j][t][r] + sx);
          }
        }
      }
    }
  }
  PF_WAITV(0);                                                  // no load may be on its way into LDS when the work-group ends,
  PF_BAR();                                                     // nor into the piece of it that a wave stages its sums in
#undef PF_STEP
#undef PF_WAITV
#undef PF_BAR
  if (!busy) return;
  static_assert(XT * 1024 >= 32 * PF_STAGE_LD * 4 && NW == 4, "a slot holds a staged tile");
  pf_store<RBW, SWIGLU>(acc, PT, s, NRB, Npad, MT, act, rb0, mt0, tile_end, M, (float*)(w & 2 ? (w & 1 ? s3 : s2) : (w & 1 ? s1 : s0)));
}

// SX[group][row] = -24 * sum of x over the group's 128 columns (x = the sum of its planes), for k_gemm_pf_q4.  A wave per (32-row tile, group).
__global__ __launch_bounds__(256) void k_group_sums(const bf16_t* __restrict__ XF, float* __restrict__ SX, int MT, int KS, int nplanes) {
  const int lane = threadIdx.x & 63, g = blockIdx.y * 4 + (threadIdx.x >> 6), t = blockIdx.x;
  if (g * 8 >= KS) return;
  u32x4 v[8][2];
#pragma unroll
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int q = 0; q < 2; ++q) v[u][q] = *(const u32x4*)(XF + (((size_t)min(q, nplanes - 1) * MT + t) * KS + 8 * g + u) * 512 + lane * 8);
  float a = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (q < nplanes) a += __builtin_bit_cast(float, v[u][q][j] << 16) + __builtin_bit_cast(float, v[u][q][j] & 0xFFFF0000u);
  a += __shfl_xor(a, 32, 64);
  if (lane < 32) SX[(size_t)g * MT * 32 + t * 32 + lane] = -q4_format(Q4_ROT_LARGE_M).offset * a;
}

// ============================================================================ row producers
// Row facts of a pass of at most 64 rows whose first kernel does not write them.
__global__ __launch_bounds__(64) void k_row_facts(Pass pass, const TreeDev* tree, SeqState st, int M, KVCache kv, RowFact* facts) {
  if ((int)threadIdx.x < M) facts[threadIdx.x] = row_fact(pass, tree, row_info(pass, tree, st, threadIdx.x), kv);
}
// h[r][:] = embedding of row r's token (fp32).  EmbT = float or bf16_t.
template <typename EmbT>
__global__ __launch_bounds__(256) void k_embed(Pass pass, const TreeDev* tree, SeqState st, const int* tree_tok,
                                               const EmbT* __restrict__ embed, float* __restrict__ h, int d, int vocab, KVCache kv, RowFact* facts) {
  int r = blockIdx.x;
  RowInfo ri = row_info(pass, tree, st, r);
  if (threadIdx.x == 0) facts[r] = row_fact(pass, tree, ri, kv);
  int tok = 0;
  if (ri.valid) {
    if (pass.kind == PASS_VERIFY) tok = tree_tok[ri.seq * tree->M + ri.node];
    else tok = st.tokens[(size_t)ri.seq * st.tok_stride + ri.pos];
  }
  tok = min(max(tok, 0), vocab - 1);
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    float v;
    if constexpr (sizeof(EmbT) == 4) v = ((const float*)embed)[(size_t)tok * d + k];
    else v = bf16_to_f32(((const bf16_t*)embed)[(size_t)tok * d + k]);
    h[(size_t)r * d + k] = ri.valid ? v : 0.f;
  }
}

// Eight consecutive numbers of a row.
__device__ __forceinline__ void embed8(const float* p, float* x) {
  const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
__device__ __forceinline__ void embed8(const bf16_t* p, float* x) {
  const u32x4 r = *(const u32x4*)p;
#pragma unroll
  for (int t = 0; t < 4; ++t) { x[2 * t] = __builtin_bit_cast(float, r[t] << 16); x[2 * t + 1] = __builtin_bit_cast(float, r[t] & 0xFFFF0000u); }
}
__device__ inline void xf_store8(bf16_t* XF, int m, int k8, int MT, int KS, int nplanes, const float* x) {
  // plane q holds bf16(x - planes 0..q-1), as split_bf16 defines it; written plane by plane so that nothing is indexed
  // by a run-time value (an array indexed by the plane number would live on the stack)
  float r[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) r[t] = x[t];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q < nplanes) {
      u32x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = split_pair(r[2 * t], r[2 * t + 1]);
      *(u32x4*)(XF + xf_index(m, k8, q, MT, KS)) = v;
    }
  }
}

// Row of a work-group in kernels that make one row of a GEMM input each.  A 128-byte line of that input holds 16 bytes of eight
// rows (xf_index), and work-groups go to the eight XCDs in turn: with row = work-group number every line was written in eight pieces
// by eight L2s.  Here eight neighbouring rows are the work-groups of one XCD, whose L2 puts the line together; the rows behind the
// last whole block of 64 are taken as they come, so passes of a few rows still spread over the XCDs.  k_rows_to_xf, 1024 rows of 4096:
// 20.3 -> 10.9 us; k_resnorm, 1024 rows of 5120: 33 -> 27, 2011 rows of 8192: 84 -> 66.
__device__ inline int xcd_row() {
  const int b = blockIdx.x;
  return b < ((int)gridDim.x & ~63) ? (b & ~63) | (b & 7) << 3 | (b >> 3 & 7) : b;
}

// Input of the head's FC layer: concat(feature, embedding of the token one step ahead)  (Sec. 3.1).
//   pending pass : feature = target feature kept at the last commit, token = committed token at pos+1
//   level pass   : feature = the head's output at the node's parent, token = the node's drafted token
//   draft prefill: feature = target feature of the prompt position, token = the next prompt token
struct LevelParents { int M, D1; uint8_t node[EAGLE_MAX_NODES], parent[EAGLE_MAX_NODES]; };   // nodes of the tree, its depth + 1, a level's nodes and their parents by row
template <typename EmbT>
__global__ __launch_bounds__(256) void k_fc_input(Pass pass, const TreeDev* tree, SeqState st, const int* tree_tok,
                                                  const float* pend_f /*[seq][D+1][d]*/, const float* node_f /*[seq][M][d]*/,
                                                  const float* chunk_f /*[chunk][d]*/, const EmbT* __restrict__ embed,
                                                  bf16_t* XF, int d, int vocab, int MT, int nplanes, KVCache kv, RowFact* facts, LevelParents lp) {
  const int r = xcd_row();
  const bool level = pass.kind == PASS_DRAFT_LEVEL;
  const int i = level ? r % pass.rows_per_seq : 0;
  RowInfo ri = row_info(pass, tree, st, r, level ? lp.node[i] : -1);
  if (blockIdx.y == 0 && threadIdx.x == 0) facts[r] = row_fact(pass, tree, ri, kv);
  const int KS = 2 * d / 16;
  const float* f = nullptr;
  int tok = 0;
  if (ri.valid) {
    if (pass.kind == PASS_DRAFT_PENDING) {
      f = pend_f + ((size_t)ri.seq * lp.D1 + ri.rel) * d;
      tok = st.tokens[(size_t)ri.seq * st.tok_stride + ri.pos + 1];
    } else if (pass.kind == PASS_DRAFT_LEVEL) {
      f = node_f + ((size_t)ri.seq * lp.M + lp.parent[i]) * d;
      tok = tree_tok[ri.seq * lp.M + ri.node];
    } else {
      f = chunk_f + (size_t)ri.rel * d;
      tok = st.tokens[(size_t)ri.seq * st.tok_stride + ri.pos + 1];
    }
  }
  tok = min(max(tok, 0), vocab - 1);
  // blockIdx.y splits the 2d columns so that a pass of a few rows still spreads over many CUs
  for (int k8 = (blockIdx.y * blockDim.x + threadIdx.x) * 8; k8 < 2 * d; k8 += gridDim.y * blockDim.x * 8) {
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (ri.valid) {
      if (k8 < d) embed8(f + k8, x);
      else embed8(embed + (size_t)tok * d + (k8 - d), x);
    }
    xf_store8(XF, r, k8, MT, KS, nplanes, x);
  }
}

// h_out[r] = h_in[r] + sum_s PT[s][:, r] + bias ;  x = gain ? rmsnorm(h_out[r]) * gain : h_out[r]
// x goes out in XF layout (GEMM input) and, optionally, as fp32 rows (features).  One block per row; a thread owns chunks of 8
// consecutive columns, the first RESNORM_KEEP of which (rows of up to 8192 columns) stay in registers between the two phases.
// Bound by memory latency for passes of some hundred rows: everything a chunk needs -- residual, up to eight splits, bias and the
// next norm's gain -- is requested together as 16-byte loads before anything is stored (h_out may be h_in: with element-wise
// loads and stores in turn, each load waited for the store before it: 16.1 us a call at 104 rows and d = 4096, now 8.8).
// MOE: the pass's experts ran grouped (k_moe_plan); the row's result is sum over its experts, ascending, of weight * sum_s PT[s][slot].
constexpr int RESNORM_THREADS = 512, RESNORM_KEEP = 2;
template <bool MOE = false>
__global__ __launch_bounds__(RESNORM_THREADS) void k_resnorm(const float* h_in, const float* __restrict__ PT, int S, int Npad, int Mpad,
                                                             const float* __restrict__ bias, float* h_out, const float* __restrict__ gain, float eps,
                                                             bf16_t* __restrict__ XF, int MT, int nplanes, float* __restrict__ xout, int d, const float* __restrict__ row_w,
                                                             const float* __restrict__ moe_w, const int* __restrict__ moe_slot, int moe_stride, int E) {
  __shared__ float sh[16];
  __shared__ float pick_w[4];                    // MOE: weight and gathered row of each expert of this row, ascending
  __shared__ int pick_s[4], n_pick;
  const int r = xcd_row();
  if constexpr (MOE) {
    if (threadIdx.x < 64) {                      // one wave looks at (at most 64) experts
      const int e = threadIdx.x;
      const int slot = e < E ? moe_slot[(size_t)e * moe_stride + r] : -1;
      const unsigned long long sel = __ballot(slot >= 0);
      if (slot >= 0) {
        const int at = __popcll(sel & ((1ull << e) - 1ull));
        pick_s[at] = slot; pick_w[at] = moe_w[(size_t)e * moe_stride + r];
      }
      if (e == 0) n_pick = __popcll(sel);
    }
    __syncthreads();
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f}, one = {1.f, 1.f, 1.f, 1.f};
  struct Chunk { f32x4 lo, hi, glo, ghi; };      // the residual's new values and the gain
  Chunk keep[RESNORM_KEEP];
  float ss = 0.f;
  const float rw = row_w ? row_w[r] : 1.0f;      // every expert over all rows: this expert's routing weight (0 = not routed here)
  auto add_splits = [&](int row, int k8, f32x4& alo, f32x4& ahi) {   // added in split order, eight splits' worth of loads in flight
    for (int s0 = 0; s0 < S; s0 += 8) {
      f32x4 lo[8], hi[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* src = PT + ((size_t)min(s0 + u, S - 1) * Mpad + row) * Npad + k8;
        lo[u] = *(const f32x4*)src; hi[u] = *(const f32x4*)(src + 4);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < S) { alo += lo[u]; ahi += hi[u]; }
    }
  };
  auto phase1 = [&](int k8, Chunk& c) {
    const float* hp = h_in + (size_t)r * d + k8;
    c.lo = h_in ? *(const f32x4*)hp : zero; c.hi = h_in ? *(const f32x4*)(hp + 4) : zero;
    c.glo = gain ? *(const f32x4*)(gain + k8) : one; c.ghi = gain ? *(const f32x4*)(gain + k8 + 4) : one;
    const f32x4 blo = bias ? *(const f32x4*)(bias + k8) : zero, bhi = bias ? *(const f32x4*)(bias + k8 + 4) : zero;
    if constexpr (MOE) {
      for (int j = 0; j < n_pick; ++j) {
        f32x4 alo = zero, ahi = zero;
        add_splits(pick_s[j], k8, alo, ahi);
        c.lo += pick_w[j] * alo; c.hi += pick_w[j] * ahi;
      }
    } else if (PT) {
      f32x4 alo = zero, ahi = zero;
      add_splits(r, k8, alo, ahi);
      if (row_w) { alo *= rw; ahi *= rw; }
      c.lo += alo; c.hi += ahi;
    }
    if (bias) { c.lo += blo; c.hi += bhi; }
    float* out = h_out + (size_t)r * d + k8;
    *(f32x4*)out = c.lo; *(f32x4*)(out + 4) = c.hi;
#pragma unroll
    for (int t = 0; t < 4; ++t) ss += c.lo[t] * c.lo[t];
#pragma unroll
    for (int t = 0; t < 4; ++t) ss += c.hi[t] * c.hi[t];
  };
#pragma unroll
  for (int it = 0; it < RESNORM_KEEP; ++it) {
    const int k8 = (it * RESNORM_THREADS + (int)threadIdx.x) * 8;
    if (k8 < d) phase1(k8, keep[it]);
  }
  for (int k8 = (RESNORM_KEEP * RESNORM_THREADS + (int)threadIdx.x) * 8; k8 < d; k8 += RESNORM_THREADS * 8) { Chunk c; phase1(k8, c); }
  if (!XF && !xout) return;
  ss = block_sum(ss, sh);
  const float rstd = gain ? 1.0f / sqrtf(ss / (float)d + eps) : 1.0f;
  const int KS = d / 16;
  auto phase2 = [&](int k8, const Chunk& c) {
    f32x4 lo = c.lo, hi = c.hi;
    if (gain) { lo = lo * rstd * c.glo; hi = hi * rstd * c.ghi; }
    if (xout) { *(f32x4*)(xout + (size_t)r * d + k8) = lo; *(f32x4*)(xout + (size_t)r * d + k8 + 4) = hi; }
    const float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    if (XF) xf_store8(XF, r, k8, MT, KS, nplanes, x);
  };
#pragma unroll
  for (int it = 0; it < RESNORM_KEEP; ++it) {
    const int k8 = (it * RESNORM_THREADS + (int)threadIdx.x) * 8;
    if (k8 < d) phase2(k8, keep[it]);
  }
  for (int k8 = (RESNORM_KEEP * RESNORM_THREADS + (int)threadIdx.x) * 8; k8 < d; k8 += RESNORM_THREADS * 8) {
    Chunk c;
    const float* hp = h_out + (size_t)r * d + k8;
    c.lo = *(const f32x4*)hp; c.hi = *(const f32x4*)(hp + 4);
    c.glo = gain ? *(const f32x4*)(gain + k8) : one; c.ghi = gain ? *(const f32x4*)(gain + k8 + 4) : one;
    phase2(k8, c);
  }
}

// The same for dense models with a bf16 cache, which keep the sums of 256 threads a row (with 512 a row's sum of squares rounds
// differently in one row of some hundred, and the cache then rounds some K and V the other way): element by element, 16.1 us at 104
// rows.
__global__ __launch_bounds__(256) void k_resnorm_fixed(const float* h_in, const float* __restrict__ PT, int S, int Npad, int Mpad,
                                                 const float* bias, float* h_out, const float* gain, float eps,
                                                 bf16_t* XF, int MT, int nplanes, float* xout, int d) {
  __shared__ float sh[16];
  const int r = xcd_row();
  float ss = 0.f;
  // each thread owns chunks of 8 consecutive k; the first four chunks (rows of up to 8192 columns) stay in registers
  // for the second phase, further ones are read back from h_out
  constexpr int KEEP = 4;
  float keep[KEEP][8];
  auto phase1 = [&](int k8, float* v) {
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (PT) {
      for (int s0 = 0; s0 < S; s0 += 8) {        // eight splits' worth of loads in flight, added in split order
        f32x4 lo[8], hi[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float* src = PT + ((size_t)min(s0 + u, S - 1) * Mpad + r) * Npad + k8;
          lo[u] = *(const f32x4*)src; hi[u] = *(const f32x4*)(src + 4);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u < S) {
            a[0] += lo[u].x; a[1] += lo[u].y; a[2] += lo[u].z; a[3] += lo[u].w;
            a[4] += hi[u].x; a[5] += hi[u].y; a[6] += hi[u].z; a[7] += hi[u].w;
          }
      }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      int k = k8 + t;
      float x = h_in ? h_in[(size_t)r * d + k] : 0.f;
      if (PT) x += a[t];
      if (bias) x += bias[k];
      h_out[(size_t)r * d + k] = x;
      ss += x * x;
      v[t] = x;
    }
  };
#pragma unroll
  for (int it = 0; it < KEEP; ++it) {
    const int k8 = (it * (int)blockDim.x + (int)threadIdx.x) * 8;
    if (k8 < d) phase1(k8, keep[it]);
  }
  for (int k8 = (KEEP * blockDim.x + threadIdx.x) * 8; k8 < d; k8 += blockDim.x * 8) { float v[8]; phase1(k8, v); }
  ss = block_sum(ss, sh);
  float rstd = gain ? 1.0f / sqrtf(ss / (float)d + eps) : 1.0f;
  const int KS = d / 16;
  auto phase2 = [&](int k8, const float* v) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      x[t] = gain ? v[t] * rstd * gain[k8 + t] : v[t];
      if (xout) xout[(size_t)r * d + k8 + t] = x[t];
    }
    if (XF) xf_store8(XF, r, k8, MT, KS, nplanes, x);
  };
  if (!XF && !xout) return;
#pragma unroll
  for (int it = 0; it < KEEP; ++it) {
    const int k8 = (it * (int)blockDim.x + (int)threadIdx.x) * 8;
    if (k8 < d) phase2(k8, keep[it]);
  }
  for (int k8 = (KEEP * blockDim.x + threadIdx.x) * 8; k8 < d; k8 += blockDim.x * 8) {
    float v[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) v[t] = h_out[(size_t)r * d + k8 + t];
    phase2(k8, v);
  }
}

// q, k, v = rows of PT (the fused QKV projection); rotate-half RoPE on q and k with the row's position id;
// q -> Q[r][head][dh] fp32, k and v -> this layer's paged cache at the row's slot.
// A thread owns four consecutive rows of the fused matrix: two rotate-half pairs of a q or k head (packed with partners adjacent,
// PACK_ROPE), or four columns of a v head; the splits are read 16 bytes at a time, four in flight.  Where the row goes comes
// from the pass's row facts, one load.  (A wave per head with element-wise loads, page-table walk included: 8.1 us a call at 104
// rows, now 6.3.)  Grid (rows, columns / 1024).
template <typename CT>
__global__ __launch_bounds__(256) void k_qkv_rope_store(const RowFact* __restrict__ facts, const float* __restrict__ PT, int S, int N, int Npad, int Mpad,
                                                        const float* __restrict__ rope_cos, const float* __restrict__ rope_sin,
                                                        float* __restrict__ Q, KVCache kv, int H) {
  const int r = blockIdx.x, n = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (n >= N) return;                                           // N is a multiple of 32
  const int pos = facts[r].pos, kv_row = facts[r].kv_row;
  const int dh = kv.head_dim, half = dh >> 1, KVH = kv.n_kv_heads, hd = n / dh, pr = n % dh;
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < S; s0 += 4) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *(const f32x4*)(PT + ((size_t)min(s0 + u, S - 1) * Mpad + r) * Npad + n);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < S) a += v[u];
  }
  if (hd >= H + KVH) {                                          // v head
    if (kv_row < 0) return;
    CT* base = (CT*)kv.v + ((size_t)kv_row + ((size_t)(hd - H - KVH) << kv.page_shift)) * dh + pr;
#pragma unroll
    for (int t = 0; t < 4; ++t) cache_store(base + t, a[t]);
    return;
  }
  const int i = pr >> 1;                                        // pairs i, i + 1
  float x1[2], x2[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float c = rope_cos[(size_t)pos * half + i + p], sn = rope_sin[(size_t)pos * half + i + p];
    x1[p] = a[2 * p] * c - a[2 * p + 1] * sn;
    x2[p] = a[2 * p + 1] * c + a[2 * p] * sn;
  }
  if (hd < H) {
    float* q = Q + ((size_t)r * H + hd) * dh + i;
#pragma unroll
    for (int p = 0; p < 2; ++p) { q[p] = x1[p]; q[half + p] = x2[p]; }
  } else if (kv_row >= 0) {
    CT* base = (CT*)kv.k + ((size_t)kv_row + ((size_t)(hd - H) << kv.page_shift)) * dh + i;
#pragma unroll
    for (int p = 0; p < 2; ++p) { cache_store(base + p, x1[p]); cache_store(base + half + p, x2[p]); }
  }
}

// (Tree-masked paged attention for both paths is k2_attn, in kernels2.h.)

// ============================================================================ SwiGLU and logits epilogues
// act[r][k] = silu(gate) * up with the fused matrix's row order (PACK_GATE / PACK_UP)   (F = d_ffn)
// A wave owns one tile of the output (32 rows x one k-step of 16 features): lane = (row, half of the k-step), which is
// the tile's own lane order, so the wave writes 1 KiB contiguous per plane; the lane's 8 gate and 8 up values are
// 32 bytes each in the row's 128-byte line of the fused block, so the two lanes of a row read that line exactly once.
// Grid (k-steps / 4, 32-row tiles); rows beyond M are written as zeros.
__global__ __launch_bounds__(256) void k_swiglu(const float* __restrict__ PT, int S, int Npad, int Mpad, int F, int M,
                                                bf16_t* XF, int MT, int nplanes) {
  const int lane = threadIdx.x & 63, ks = blockIdx.x * 4 + (threadIdx.x >> 6), KSF = F / 16;
  if (ks >= KSF) return;
  const int r = blockIdx.y * 32 + (lane & 31), half = lane >> 5;
  const int ng = 32 * ks + 8 * half;                 // this lane's 8 gate rows of the fused matrix; the up rows sit 16 further
  float gs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, us[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (r < M) {
    for (int s0 = 0; s0 < S; s0 += 4) {              // four splits' worth of loads in flight, added in split order
      f32x4 g0[4], g1[4], u0[4], u1[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float* src = PT + ((size_t)min(s0 + q, S - 1) * Mpad + r) * Npad + ng;
        g0[q] = *(const f32x4*)src; g1[q] = *(const f32x4*)(src + 4);
        u0[q] = *(const f32x4*)(src + 16); u1[q] = *(const f32x4*)(src + 20);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (s0 + q < S) {
          gs[0] += g0[q].x; gs[1] += g0[q].y; gs[2] += g0[q].z; gs[3] += g0[q].w;
          gs[4] += g1[q].x; gs[5] += g1[q].y; gs[6] += g1[q].z; gs[7] += g1[q].w;
          us[0] += u0[q].x; us[1] += u0[q].y; us[2] += u0[q].z; us[3] += u0[q].w;
          us[4] += u1[q].x; us[5] += u1[q].y; us[6] += u1[q].z; us[7] += u1[q].w;
        }
    }
  }
  float x[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) x[t] = r < M ? gs[t] / (1.0f + __expf(-gs[t])) * us[t] : 0.f;
  xf_store8(XF, r, 16 * ks + 8 * half, MT, KSF, nplanes, x);
}

// logits[dst_row(r)][v] = sum_s PT[s][v][r].  Where a pass's row maps to no output (padding rows, pending rows
// other than the root pair) nothing is written.  out_kind 0: per-node buffer [seq][M][V]; 1: per-seq [seq][V].
__global__ __launch_bounds__(256) void k_logits(Pass pass, const TreeDev* tree, SeqState st, const float* __restrict__ PT,
                                                int S, int Npad, int Mpad, float* out, int out_kind, int V, int only_last_row) {
  int r = blockIdx.y;
  RowInfo ri = row_info(pass, tree, st, r);
  if (!ri.valid) return;
  size_t dst;
  if (out_kind == 0) {
    if (ri.node < 0) return;
    dst = ((size_t)ri.seq * tree->M + ri.node) * V;
  } else {
    if (only_last_row && ri.rel != pass.chunk_n - 1 && pass.kind != PASS_VANILLA) return;
    dst = (size_t)ri.seq * V;
  }
  int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= V) return;
  float a = 0.f;
  for (int s = 0; s < S; ++s) a += PT[((size_t)s * Mpad + r) * Npad + v];
  out[dst + v] = a;
}

// Where row r of a pass keeps its feature (nullptr: nowhere): tree nodes [seq][M][d], pending rows [seq][D+1][d], prompt rows [chunk][d].
__device__ inline float* feature_row(const Pass& pass, const TreeDev* tree, const SeqState& st, int r, float* node_dst, float* pend_dst, float* chunk_dst, int d) {
  RowInfo ri = row_info(pass, tree, st, r);
  if (!ri.valid) return nullptr;
  if (pass.kind == PASS_VERIFY || pass.kind == PASS_DRAFT_LEVEL) return node_dst + ((size_t)ri.seq * tree->M + ri.node) * d;
  if (pass.kind == PASS_DRAFT_PENDING) return ri.node == 0 ? node_dst + ((size_t)ri.seq * tree->M) * d : nullptr;
  if (pass.kind == PASS_PREFILL_T) return chunk_dst + (size_t)ri.rel * d;
  if (pass.kind == PASS_VANILLA) return pend_dst + (size_t)ri.seq * (tree->D + 1) * d;
  return nullptr;
}
// copy rows (features): feature_row(r) = src[r]
__global__ __launch_bounds__(256) void k_store_rows(Pass pass, const TreeDev* tree, SeqState st, const float* __restrict__ src,
                                                    float* __restrict__ node_dst, float* __restrict__ pend_dst, float* __restrict__ chunk_dst, int d) {
  const int r = blockIdx.x;
  float* dst = feature_row(pass, tree, st, r, node_dst, pend_dst, chunk_dst, d);
  if (!dst) return;
  for (int k = 4 * threadIdx.x; k < d; k += 1024) *(f32x4*)(dst + k) = *(const f32x4*)(src + (size_t)r * d + k);
}

// ============================================================================ training loss of the head (Sec. 3.2)
// Rows of fp32 features -> rows [row0, row0 + rows) of a GEMM input of MT 32-row tiles (XF layout).  Grid (rows, parts).
__global__ __launch_bounds__(256) void k_rows_to_xf(const float* __restrict__ src, int row0, bf16_t* XF, int MT, int nplanes, int d) {
  const int r = xcd_row();
  for (int k8 = (blockIdx.y * blockDim.x + threadIdx.x) * 8; k8 < d; k8 += gridDim.y * blockDim.x * 8) {
    float x[8];
    const f32x4 a = *(const f32x4*)(src + (size_t)r * d + k8), b = *(const f32x4*)(src + (size_t)r * d + k8 + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    xf_store8(XF, row0 + r, k8, MT, d / 16, nplanes, x);
  }
}

// One row of the loss (block = row r of the pass).  Z holds the LM head's logits of the pass as S split-K partials
// PT[s][m][n]: row r = logits of the label feature f, row zh_row0 + r = logits of the prediction fhat.
//   p = softmax(z), q = softmax(zh);  cross entropy of the row = lse(zh) - sum_v p_v zh_v
//   dZ[r][v] = (q_v - p_v) * cls_scale            (cls_scale = w_cls / rows of the whole call), written as GEMM input
//   Smooth L1 of the row over d columns (threshold 1), its derivative clip(x, -1, 1) * reg_scale -> grad[r][:]
// row_loss[r] = (sum of the row's smooth-L1 terms, the row's cross entropy); means are taken by the caller.
// NCH > 0: a thread keeps its NCH chunks of 8 logits of both rows in registers (V <= 8192 * NCH), so the logits are
// read once; NCH = 0: any V, three passes over the logits.
// Bound by what one work-group has in flight (one of 1024 threads fits a CU): the features, and the first partial of every chunk, are
// requested together before anything is added, the reductions of a phase share two barriers, and rows go to XCDs as xcd_row says.
// 1024 rows of 32000: 193 us with two loads in flight a thread, now 127 (393 MB read and written, 3.1 TB/s); 300 rows: 93, now 64.
template <int NCH>
__global__ __launch_bounds__(1024) void k_head_loss_row(const float* __restrict__ Z, int S, int Mpad, int Npad, int zh_row0, int V,
                                                        const float* __restrict__ f, const float* __restrict__ fhat, int d,
                                                        float cls_scale, float reg_scale, bf16_t* DZ, int MT, int nplanes,
                                                        float* grad /*[rows][d] or null*/, float* row_loss /*[rows][2]*/) {
  __shared__ float sh[4 * 16];
  const int r = xcd_row(), tid = threadIdx.x;
  f += (size_t)r * d; fhat += (size_t)r * d;
  if (grad) grad += (size_t)r * d;
  const float* zrow = Z + (size_t)r * Npad;
  const float* hrow = Z + (size_t)(zh_row0 + r) * Npad;
  struct Eight { f32x4 lo, hi; };
  auto at = [](const Eight& e, int t) { return t < 4 ? e.lo[t] : e.hi[t - 4]; };
  auto first8 = [&](const float* row, int v8) { return Eight{*(const f32x4*)(row + v8), *(const f32x4*)(row + v8 + 4)}; };
  auto more8 = [&](const float* row, int v8, Eight& e) {            // the other partials, in split order
    for (int s = 1; s < S; ++s) {
      const float* src = row + (size_t)s * Mpad * Npad + v8;
      e.lo += *(const f32x4*)src; e.hi += *(const f32x4*)(src + 4);
    }
  };
  auto load8 = [&](const float* row, int v8) { Eight e = first8(row, v8); more8(row, v8, e); return e; };
  // one reduction over the block for up to four values: waves' results in sh[value][wave], combined in wave order
  auto to_sh = [&](int i, float v) { if ((tid & 63) == 0) sh[i * 16 + (tid >> 6)] = v; };
  auto sum16 = [&](int i) { float t = 0.f; for (int w = 0; w < 16; ++w) t += sh[i * 16 + w]; return t; };
  auto max16 = [&](int i) { float t = sh[i * 16]; for (int w = 1; w < 16; ++w) t = fmaxf(t, sh[i * 16 + w]); return t; };

  const int k0 = min(4 * tid, d - 4);                               // this thread's first four features
  typedef f32x4 __attribute__((aligned(4))) caller4;                // the caller's rows may start at any float
  const f32x4 f0 = *(const caller4*)(f + k0), p0 = *(const caller4*)(fhat + k0);
  constexpr int NR = NCH > 0 ? NCH : 1;
  Eight zr[NR], hr[NR];
  float mz = -INFINITY, mh = -INFINITY;
  auto max8 = [&](const Eight& z, const Eight& h) {
#pragma unroll
    for (int t = 0; t < 8; ++t) { mz = fmaxf(mz, at(z, t)); mh = fmaxf(mh, at(h, t)); }
  };
  if constexpr (NCH > 0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {                                 // (behind the row's end: its last chunk again, not used)
      const int v8 = min((c * 1024 + tid) * 8, V - 8);
      zr[c] = first8(zrow, v8); hr[c] = first8(hrow, v8);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  float reg = 0.f;
  auto reg4 = [&](int k, f32x4 a, f32x4 b) {
    f32x4 g;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float x = b[t] - a[t], ax = fabsf(x);
      reg += ax < 1.0f ? 0.5f * x * x : ax - 0.5f;
      g[t] = fminf(fmaxf(x, -1.0f), 1.0f) * reg_scale;
    }
    if (grad) *(caller4*)(grad + k) = g;
  };
  if (4 * tid < d) reg4(4 * tid, f0, p0);
  for (int k = 4 * (tid + 1024); k < d; k += 4096) reg4(k, *(const caller4*)(f + k), *(const caller4*)(fhat + k));
  if constexpr (NCH > 0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int v8 = (c * 1024 + tid) * 8;
      if (v8 < V) { more8(zrow, v8, zr[c]); more8(hrow, v8, hr[c]); max8(zr[c], hr[c]); }
    }
  } else {
    for (int v8 = tid * 8; v8 < V; v8 += 8192) max8(load8(zrow, v8), load8(hrow, v8));
  }
  to_sh(0, wave_max(mz)); to_sh(1, wave_max(mh));
  __syncthreads();
  mz = max16(0); mh = max16(1);
  __syncthreads();
  float sz = 0.f, shh = 0.f, dot = 0.f;
  auto sums8 = [&](Eight& z, Eight& zh) {                           // the logits become exp(z - max) for the gradient
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float h = at(zh, t) - mh, e = __expf(at(z, t) - mz), eh = __expf(h);
      sz += e; shh += eh; dot += e * h;
      if (t < 4) { z.lo[t] = e; zh.lo[t] = eh; } else { z.hi[t - 4] = e; zh.hi[t - 4] = eh; }
    }
  };
  if constexpr (NCH > 0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if ((c * 1024 + tid) * 8 < V) sums8(zr[c], hr[c]);
  } else {
    for (int v8 = tid * 8; v8 < V; v8 += 8192) { zr[0] = load8(zrow, v8); hr[0] = load8(hrow, v8); sums8(zr[0], hr[0]); }
  }
  to_sh(0, wave_sum(sz)); to_sh(1, wave_sum(shh)); to_sh(2, wave_sum(dot)); to_sh(3, wave_sum(reg));
  __syncthreads();
  sz = sum16(0); shh = sum16(1); dot = sum16(2);
  const float isz = 1.0f / sz, ish = 1.0f / shh;
  auto store8 = [&](int v8, const Eight& e, const Eight& eh) {
    float x[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = (at(eh, t) * ish - at(e, t) * isz) * cls_scale;
    xf_store8(DZ, r, v8, MT, V / 16, nplanes, x);
  };
  if constexpr (NCH > 0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int v8 = (c * 1024 + tid) * 8;
      if (v8 < V) store8(v8, zr[c], hr[c]);
    }
  } else {
    for (int v8 = tid * 8; v8 < V; v8 += 8192) {
      Eight e = load8(zrow, v8), eh = load8(hrow, v8);
      e.lo -= mz; e.hi -= mz; eh.lo -= mh; eh.hi -= mh;
#pragma unroll
      for (int t = 0; t < 4; ++t) { e.lo[t] = __expf(e.lo[t]); e.hi[t] = __expf(e.hi[t]); eh.lo[t] = __expf(eh.lo[t]); eh.hi[t] = __expf(eh.hi[t]); }
      store8(v8, e, eh);
    }
  }
  if (tid == 0) { row_loss[2 * r] = sum16(3); row_loss[2 * r + 1] = logf(shh) - dot / sz; }   // lse(zh) - sum_v p_v zh_v, both relative to mh
}

// grad[r][k] += sum over the S split-K partials of (dZ W)[r][k]   (the classification part of the gradient)
__global__ __launch_bounds__(256) void k_head_loss_grad_finish(const float* __restrict__ PT, int S, int Mpad, int Npad, float* grad, int d) {
  const int r = blockIdx.y, k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d) return;
  float a = 0.f;
  for (int s = 0; s < S; ++s) a += PT[((size_t)s * Mpad + r) * Npad + k];
  grad[(size_t)r * d + k] += a;
}

// acc[0] += sum of the rows' smooth-L1 sums, acc[1] += sum of the rows' cross entropies, in fp64 and in a fixed order:
// lane l of one wave adds rows l, l + 64, ...; lane 0 then adds the 64 lane sums in lane order.
__global__ __launch_bounds__(64) void k_head_loss_accumulate(const float* row_loss, int rows, double* acc) {
  __shared__ double sa[64], sb[64];
  double a = 0.0, b = 0.0;
  for (int r = threadIdx.x; r < rows; r += 64) { a += (double)row_loss[2 * r]; b += (double)row_loss[2 * r + 1]; }
  sa[threadIdx.x] = a; sb[threadIdx.x] = b;
  __syncthreads();
  if (threadIdx.x == 0) {
    double ta = acc[0], tb = acc[1];
    for (int l = 0; l < 64; ++l) { ta += sa[l]; tb += sb[l]; }
    acc[0] = ta; acc[1] = tb;
  }
}

// out = in + amplitude * n, n = the odd multiple of 2^-24 in (-1, 1) that the counter-based generator draws for
// (row, column); the product and the sum are rounded separately (no fused multiply-add), so the result is the same
// bits wherever it is computed.
__global__ __launch_bounds__(256) void k_feature_noise(const float* in, float* out, int rows, int d, float amplitude, unsigned long long prefix) {
#pragma clang fp contract(off)
  const size_t n = (size_t)rows * d;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const uint32_t r = (uint32_t)(i / d), k = (uint32_t)(i % d);
    const int k24 = (int)rng_u24(prefix, r >> 16, r & 0xFFFFu, k);
    const float u = (float)(2 * (k24 - (1 << 23)) + 1) * 5.9604644775390625e-8f;
    const float prod = amplitude * u;
    out[i] = in[i] + prod;
  }
}

// ============================================================================ token choice
struct HintDev {
  const int* future;     // [max_batch][stride]
  int stride;
  const int* n;          // [max_batch] tokens known (0 = off)
  const float* alpha;    // [max_batch]
  const float* bias;
  const unsigned long long* seed;
};

// Children of one tree node = the top-k entries of its (knob-adjusted, Gumbel-perturbed when non-greedy) head
// logits, rank r = (r+1)-th largest, equal scores -> lower token id (App. A.1).  Block = (parent row, seq).
struct LevelNodes { uint8_t node[EAGLE_MAX_NODES]; };            // a level's parent nodes, by row of its pass (kernel argument: no load in front)
// A row's vocabulary is shared by `parts` work-groups of four waves (plan_expand_parts), eight tokens a thread at a time: each wave keeps its best
// children without a barrier, one wave the work-group's, and the row's last work-group to arrive the row's (the exchange of k2_gemm: store,
// acknowledge, count, read back).  Bound: a work-group's chain of latencies.  One work-group of sixteen waves for a row took two barriers a child
// and all of a row's noise: us a launch, one row with four children of 32000 tokens 22.7 / now 7.7; four rows 16.2 / 6.2; one row with
// noise 22.6 / 6.4; 1024 tokens (one part) 8.6 / 3.7.  (With the next level's FC input made here as well -- the features beside the choice, the embeddings by the
// last work-group -- a launch grew by the 4 to 8 us that k_fc_input takes.)
constexpr int EXPAND_THREADS = 256, EXPAND_KEYS = 8;             // tokens a thread takes at a time
__global__ __launch_bounds__(EXPAND_THREADS) void k_expand(int level /*-1 = root*/, LevelNodes nodes, const TreeDev* tree, int M, SeqState st,
                                                           float* draft_logits /*[seq][M][V]*/, int* tree_tok, int* on_path, HintDev hint,
                                                           int V, int parts, int per /*tokens of a part*/, int rows, float temperature, unsigned long long rng_seed,
                                                           unsigned long long* part_keys /*[seq][row][parts][8]*/, int* arrivals /*[seq][row]*/,
                                                           const float* __restrict__ feat_src /*[pass rows][d] or null*/, float* node_f /*[seq][M][d]*/,
                                                           int d, int src_rows_per_seq) {
  __shared__ unsigned long long list[4 * EAGLE_MAX_CHILD];
  const int part = blockIdx.x, row = blockIdx.y, seq = blockIdx.z;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int v = nodes.node[row];
  float* lg = draft_logits + ((size_t)seq * M + v) * V;
  const int begin = part * per, end = min(V, begin + per);
  // the first tokens' logits are on their way before any fact about the row is known
  float x[EXPAND_KEYS];
  auto request = [&](int at) {
#pragma unroll
    for (int u = 0; u < EXPAND_KEYS; ++u) x[u] = lg[min(at + u * EXPAND_THREADS + (int)threadIdx.x, V - 1)];
  };
  request(begin);
  const int n = read_only(st.n_tok + seq), hn = read_only(hint.n + seq), nk = read_only(tree->nchild + v);
  const int child = tree->child[v][min(lane, EAGLE_MAX_CHILD - 1)];
  // acceptance knob of the synthetic workload
  int hinted = -1, on = 0;
  float adj = 0.f;
  if (hn > 0) {
    const int pos_child = n + read_only(tree->depth + v), last = max(n - 1, 0);
    const int* future = hint.future + (size_t)seq * hint.stride;
    on = v ? on_path[seq * M + v] : hn > n - 1 && read_only(future + min(last, hint.stride - 1)) == read_only(st.tokens + (size_t)seq * st.tok_stride + last);
    if (on && pos_child < hn) {
      hinted = read_only(future + min(pos_child, hint.stride - 1));
      const uint32_t k24 = rng_u24(rng_prefix(read_only(hint.seed + seq), PURPOSE_HINT, 0), (uint32_t)seq, 0, (uint32_t)pos_child);
      adj = ((float)k24 * 5.9604644775390625e-8f < read_only(hint.alpha + seq)) ? read_only(hint.bias + seq) : -read_only(hint.bias + seq);
    }
  }
  const bool gumbel = temperature > 0.f;
  unsigned long long pre = 0ull;
  if (gumbel) pre = rng_prefix(rng_seed, PURPOSE_GUMBEL, (unsigned long long)read_only(st.step_no + seq));
  // The node's own head feature (the row of the pass that produced these logits) goes to node_f when the caller asks for it, which saves a
  // separate copy kernel per pass.  Row of the pass: a level pass lists the level's parent nodes in order; in a pending pass the root is the
  // sequence's last pending row.
  if (feat_src) {
    const float* src = feat_src + (size_t)(seq * src_rows_per_seq + (level < 0 ? max(read_only(st.n_pend + seq) - 1, 0) : row)) * d;
    float* dst = node_f + ((size_t)seq * M + v) * d;
    for (int k = 4 * (part * EXPAND_THREADS + (int)threadIdx.x); k < d; k += 4 * parts * EXPAND_THREADS) *(f32x4*)(dst + k) = *(const f32x4*)(src + k);
  }
  unsigned long long best = 0;                                 // wave 0: lane r has the work-group's r-th best so far
  for (int at = begin; at < end; at += EXPAND_KEYS * EXPAND_THREADS) {
    if (at > begin) request(at);
    unsigned long long keys[EXPAND_KEYS];
#pragma unroll
    for (int u = 0; u < EXPAND_KEYS; ++u) {
      const int j = at + u * EXPAND_THREADS + (int)threadIdx.x;
      float sc = x[u];
      if (j == hinted && j < end) { sc += adj; lg[j] = sc; }     // later phases read the adjusted logits
      if (gumbel) {
        const float un = ((float)rng_u24(pre, (uint32_t)seq, (uint32_t)v, (uint32_t)min(j, V - 1)) + 0.5f) * 5.9604644775390625e-8f;
        sc = sc / temperature - logf(-logf(un));
      }
      keys[u] = j < end ? arg_key(sc, j) : 0ull;               // (a NaN is no better than -inf, but it has a token)
    }
    const unsigned long long wave_best = wave_top_keys<EXPAND_KEYS>(keys, nk);
    if (at > begin) __syncthreads();                           // (wave 0 has read the last ones)
    if (lane < EAGLE_MAX_CHILD) list[w * EAGLE_MAX_CHILD + lane] = wave_best;
    __syncthreads();
    if (w == 0) {
      const unsigned long long both[2] = {lane < 4 * EAGLE_MAX_CHILD ? list[min(lane, 4 * EAGLE_MAX_CHILD - 1)] : 0ull, best};
      best = wave_top_keys<2>(both, nk);
    }
  }
  if (w) return;
  if (parts > 1) {
    const int slot = seq * rows + row;
    unsigned long long* keys = part_keys + (size_t)slot * parts * EAGLE_MAX_CHILD;
    int* cnt = arrivals + slot * COUNTER_STRIDE;
    if (lane < EAGLE_MAX_CHILD) __hip_atomic_store(keys + part * EAGLE_MAX_CHILD + lane, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    publish_wait();
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(old) != parts - 1) return;
    if (lane == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    unsigned long long all[EXPAND_PARTS_MAX * EAGLE_MAX_CHILD / 64];
#pragma unroll
    for (int u = 0; u < EXPAND_PARTS_MAX * EAGLE_MAX_CHILD / 64; ++u) {
      const int i = u * 64 + lane;
      all[u] = __hip_atomic_load(keys + min(i, parts * EAGLE_MAX_CHILD - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (i >= parts * EAGLE_MAX_CHILD) all[u] = 0ull;
    }
    best = wave_top_keys<EXPAND_PARTS_MAX * EAGLE_MAX_CHILD / 64>(all, nk);
  }
  if (lane < nk) {
    // (fewer tokens in the vocabulary than children: nothing is left to pick, and acceptance indexes its vectors with the token)
    const int pick = best ? arg_index(best) : -1;
    tree_tok[seq * M + child] = min(max(pick, 0), V - 1);
    on_path[seq * M + child] = hinted >= 0 && pick == hinted;
  }
  if (v == 0 && lane == 0) {
    tree_tok[seq * M] = read_only(st.tokens + (size_t)seq * st.tok_stride + max(n - 1, 0));
    on_path[seq * M] = on;
  }
}

// softmax(x / T) over V entries into p (block-wide), returns nothing; sh >= 16 floats
__device__ inline void block_softmax(const float* x, float* p, int V, float invT, float* sh) {
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < V; j += blockDim.x) mx = fmaxf(mx, x[j] * invT);
  mx = block_max(mx, sh);
  float sm = 0.f;
  for (int j = threadIdx.x; j < V; j += blockDim.x) { float e = expf(x[j] * invT - mx); p[j] = e; sm += e; }
  sm = block_sum(sm, sh);
  for (int j = threadIdx.x; j < V; j += blockDim.x) p[j] = p[j] / sm;
  __syncthreads();
}

// smallest x with cumsum(p)[x] > u * sum(p); block-wide, result broadcast through *res (shared).  The running sum is
// carried in fp64: with 32000 entries a bin is ~3e-5 wide, which an fp32 running sum cannot resolve -- the draw would
// depend on the order of the additions instead of on p.  (Thread chunks, then a prefix over the chunk sums, then a
// sequential walk of the one chunk that holds the target: fixed order.)
__device__ inline int block_inverse_cdf(const float* p, int V, float u, double* sh_d /*>= blockDim.x + 1*/, int* res) {
  const int nt = blockDim.x;
  const int per = (V + nt - 1) / nt;
  const int j0 = threadIdx.x * per, j1 = min(V, j0 + per);
  double s = 0.0;
  for (int j = j0; j < j1; ++j) s += (double)p[j];
  sh_d[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int i = 0; i < nt; ++i) { double t = sh_d[i]; sh_d[i] = tot; tot += t; }   // exclusive prefix, fixed order
    sh_d[nt] = tot;
    *res = V - 1;
  }
  __syncthreads();
  const double target = (double)u * sh_d[nt];
  double c = sh_d[threadIdx.x];
  const double nxt = threadIdx.x + 1 < nt ? sh_d[threadIdx.x + 1] : sh_d[nt];
  __syncthreads();
  if (j0 < j1 && c <= target && (target < nxt || threadIdx.x + 1 == nt || j1 == V)) {
    int found = -1, last_pos = -1;
    for (int j = j0; j < j1; ++j) {
      if (p[j] > 0.f) last_pos = j;
      c += (double)p[j];
      if (c > target) { found = j; break; }
    }
    if (found < 0) found = last_pos;            // rounding left the running sum just short of the target
    if (found >= 0) atomicMin(res, found);
  }
  __syncthreads();
  return *res;
}

// The same two for at most 32768 entries, which a block of 1024 threads holds in registers: thread t owns entries t, t + 1024, ...
// (the order in which block_softmax adds them).  Through memory every pass over a row was 128 KB of one CU's fetches (32000 entries,
// two sequences, T26: acceptance 293 -> 122 us a launch, a sampled token of a vanilla step 60 -> 20).
constexpr int VPT = 32;
__device__ inline void reg_softmax(const float* __restrict__ x, float (&p)[VPT], int V, float invT, float* sh) {
  const int tid = threadIdx.x;
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    p[u] = -INFINITY;
    if (tid < V - u * 1024) p[u] = (x + u * 1024)[tid];          // (a scalar base: per-thread addresses would be kept, and spilled)
  }
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    p[u] = tid < V - u * 1024 ? p[u] * invT : -INFINITY;
    mx = fmaxf(mx, p[u]);
  }
  mx = block_max(mx, sh);
  float sm = 0.f;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const float e = tid < V - u * 1024 ? expf(p[u] - mx) : 0.f;
    p[u] = e;
    sm += e;
    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);           // (interleaved over all entries the temporaries spill)
  }
  sm = block_sum(sm, sh);
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    p[u] /= sm;
    if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
}
// As block_inverse_cdf; ps: 33 * 1024 floats of LDS, in which the entries are laid out in order (a gap after every 32: the threads
// then read their runs without bank conflicts).  The prefix over the threads' sums is a scan per wave and then over the waves.
__device__ inline int reg_inverse_cdf(const float (&p)[VPT], int V, float u, float* ps, double* sh_d /*>= 1025 + 16*/, int* res) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                                  // (its LDS addresses are not worth registers before this point)
  const int lane = tid & 63, w = tid >> 6;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int j = i * 1024 + tid;
    if (j < V) ps[j + (j >> 5)] = p[i];
  }
  if (tid == 0) *res = V - 1;
  __syncthreads();
  const int per = (V + 1023) / 1024, j0 = tid * per, j1 = min(V, j0 + per);
  double s = 0.0;
  for (int j = j0; j < j1; ++j) s += (double)ps[j + (j >> 5)];
  double inc = s;
  for (int o = 1; o < 64; o <<= 1) {
    const double v = __shfl_up(inc, o, 64);
    if (lane >= o) inc += v;
  }
  double* wave_tot = sh_d + 1025;
  if (lane == 63) wave_tot[w] = inc;
  const double before = __shfl_up(inc, 1, 64);
  __syncthreads();
  double base = 0.0;
  for (int i = 0; i < w; ++i) base += wave_tot[i];
  sh_d[tid] = lane == 0 ? base : base + before;
  if (tid == 1023) sh_d[1024] = base + inc;
  __syncthreads();
  const double target = (double)u * sh_d[1024];
  double c = sh_d[tid];
  const double nxt = sh_d[tid + 1];
  if (j0 < j1 && c <= target && (target < nxt || tid == 1023 || j1 == V)) {
    int found = -1, last_pos = -1;
    for (int j = j0; j < j1; ++j) {
      const float pj = ps[j + (j >> 5)];
      if (pj > 0.f) last_pos = j;
      c += (double)pj;
      if (c > target) { found = j; break; }
    }
    if (found < 0) found = last_pos;            // rounding left the running sum just short of the target
    if (found >= 0) atomicMin(res, found);
  }
  __syncthreads();
  return *res;
}
constexpr size_t CDF_LDS = (size_t)33 * 1024 * 4;              // dynamic LDS of the sampling kernels for at most 32768 entries

// Index of the largest of V values (lowest among equals) for a block of 1024 threads, 16 loads of a thread in flight.
__device__ inline int row_argmax(const float* __restrict__ lg, int V, unsigned long long* shk) {
  const int tid = threadIdx.x;
  float bv = -INFINITY; int bi = 0x7fffffff;
  for (int j0 = 0; j0 < V; j0 += 16 * 1024) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      v[u] = -INFINITY;
      if (tid < V - j0 - u * 1024) v[u] = (lg + j0 + u * 1024)[tid];
    }
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (tid < V - j0 - u * 1024) better(bv, bi, v[u], j0 + u * 1024 + tid);
  }
  return arg_index(block_max_key(arg_key(bv, bi), shk));
}

// Pick the next token of every sequence from logits[seq][V] (prefill's first token, vanilla decoding):
// argmax when greedy, else one inverse-CDF draw from softmax(logits / T).  Also advances the sequence state.
template <bool BIGV>   // BIGV: more than 32768 vocabulary entries
__global__ __launch_bounds__(1024) void k_choose(SeqState st, int seq0, const float* logits, int V, float temperature,
                                                 unsigned long long rng_seed, float* pbuf /*[seq][V]*/, int is_prefill,
                                                 int prefill_n, int max_pend) {
  __shared__ float shv[16];
  __shared__ unsigned long long shk[16];
  __shared__ double sh_f[1025 + 16];
  __shared__ int res;
  extern __shared__ __attribute__((aligned(16))) float ps[];
  const int seq = seq0 + blockIdx.x;
  const float* lg = logits + (size_t)seq * V;
  int tok;
  if (temperature <= 0.f) {
    tok = row_argmax(lg, V, shk);
  } else {
    int step = is_prefill ? 0 : st.step_no[seq];
    float u = (float)rng_u24(rng_prefix(rng_seed, PURPOSE_FINAL, (unsigned long long)step), (uint32_t)seq, 0, 0) * 5.9604644775390625e-8f;
    if constexpr (BIGV) {
      float* p = pbuf + (size_t)seq * V;
      block_softmax(lg, p, V, 1.0f / temperature, shv);
      tok = block_inverse_cdf(p, V, u, sh_f, &res);
    } else {
      float p[VPT];
      reg_softmax(lg, p, V, 1.0f / temperature, shv);
      tok = reg_inverse_cdf(p, V, u, ps, sh_f, &res);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (is_prefill) {
      st.tokens[(size_t)seq * st.tok_stride + prefill_n] = tok;
      st.n_tok[seq] = prefill_n + 1; st.ctx_len[seq] = prefill_n; st.n_pend[seq] = 1; st.step_no[seq] = 1;
    } else {
      int n = st.n_tok[seq];
      st.tokens[(size_t)seq * st.tok_stride + n] = tok;
      st.n_tok[seq] = n + 1; st.ctx_len[seq] += 1; st.n_pend[seq] = max_pend + 1 /* head is stale after vanilla */;
      st.step_no[seq] += 1;
    }
  }
}

// Acceptance (Sec. 2; App. A.2, Alg. 1 applied recursively at every node).
//   greedy : follow the child whose token equals argmax of the target logits at the current node
//   T > 0  : children in rank order, accept child i when r * q_i(t_i) < p(t_i); on rejection
//            p <- norm(max(0, p - q_i)) and q_{i+1} = q_i without t_i, renormalised (children were drawn
//            without replacement); when nothing is accepted draw the bonus token from what is left of p.
// What happens at a node depends on the node alone (its rows, its children, random numbers named after the nodes), not on how the walk came
// there.  So every node's outcome -- the child that is accepted or -1, and the token that follows the path if it ends there -- is found at once,
// a work-group a node, and the walk is a few look-ups (k_commit).
enum { ACCEPT_GREEDY, ACCEPT_SAMPLED };
struct AcceptShared { float v[16]; double f[1025 + 16]; int res, next; float pt, qt; };
// T > 0 at one node, target and proposal in registers (see reg_softmax); the child that is accepted, else -1 and the bonus token.
__device__ inline int sample_node(const TreeDev* tree, const float* L, const float* draft_logits, const int* tree_tok, int V, float temperature, unsigned long long rng_seed,
                                  int step, int seq, int M, int cur, float* ps, AcceptShared& sh, int* bonus) {
  const float* lg = L + ((size_t)seq * M + cur) * V;
  const int nk = tree->nchild[cur];
  const int tid = threadIdx.x;
  const float invT = 1.0f / temperature;
  float p[VPT], q[VPT];
  reg_softmax(lg, p, V, invT, sh.v);
  if (nk > 0) reg_softmax(draft_logits + ((size_t)seq * M + cur) * V, q, V, invT, sh.v);
  if (tid == 0) sh.next = -1;
  for (int r = 0; r < nk; ++r) {
    const int c = tree->child[cur][r];
    const int t = __builtin_amdgcn_readfirstlane(tree_tok[seq * M + c]);
    const float rr = (float)rng_u24(rng_prefix(rng_seed, PURPOSE_ACCEPT, (unsigned long long)step), (uint32_t)seq, (uint32_t)c, 0) * 5.9604644775390625e-8f;
    float sm = 0.f, qs = 0.f;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      if (u * 1024 >= V) continue;
      if (tid == t - u * 1024) { sh.pt = p[u]; sh.qt = q[u]; }
      sm += fmaxf(p[u] - q[u], 0.f);
    }
    __syncthreads();
    if (rr * sh.qt < sh.pt) { if (tid == 0) sh.next = c; break; }
    // residual target, proposal without t
    sm = block_sum(sm, sh.v);
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      if (u * 1024 >= V) continue;
      if (sm > 1e-20f) p[u] = fmaxf(p[u] - q[u], 0.f) / sm;
      if (tid == t - u * 1024) q[u] = 0.f;
      qs += q[u];
      if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    qs = block_sum(qs, sh.v);
    if (qs > 0.f)
#pragma unroll
      for (int u = 0; u < VPT; ++u) {
        q[u] /= qs;
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    __syncthreads();                                            // (sh.pt, sh.qt and sh.v are written again)
  }
  __syncthreads();
  const int next = sh.next;
  if (next < 0) {
    const float u = (float)rng_u24(rng_prefix(rng_seed, PURPOSE_FINAL, (unsigned long long)step), (uint32_t)seq, (uint32_t)cur, 0) * 5.9604644775390625e-8f;
    *bonus = reg_inverse_cdf(p, V, u, ps, sh.f, &sh.res);
  }
  return next;
}

// The outcome of every node (block = node, sequence; at most 128 of them), and where the commit begins.  Sampled, us a launch at 32000 entries: a chain
// of six nodes 60 along the walk / 35, 26 nodes 117 / 38.
template <int KIND>
__global__ __launch_bounds__(1024) void k_outcome(const TreeDev* tree, int M, SeqState st, const float* L /*[seq][M][V]*/, const float* draft_logits, const int* tree_tok, int V,
                                                  float temperature, unsigned long long rng_seed, int2* outcome /*[seq][M]: next node or -1, token*/) {
  const int node = blockIdx.x, seq = blockIdx.y;
  if (node == 0 && threadIdx.x == 0) st.commit_base[seq] = st.ctx_len[seq];
  int2 o;
  if constexpr (KIND == ACCEPT_GREEDY) {
    __shared__ unsigned long long shk[16];
    const int lane = threadIdx.x & 63, nk = read_only(tree->nchild + node);
    const int child = tree->child[node][min(lane, EAGLE_MAX_CHILD - 1)];
    const int tok = lane < nk ? tree_tok[seq * M + child] : -1;
    o.y = row_argmax(L + ((size_t)seq * M + node) * V, V, shk);   // (every thread has it)
    const unsigned long long hit = __ballot(tok == o.y);
    o.x = hit ? __builtin_amdgcn_readlane(child, __ffsll((long long)hit) - 1) : -1;
  } else {
    __shared__ AcceptShared sh;
    extern __shared__ __attribute__((aligned(16))) float ps[];
    o.y = 0;
    o.x = sample_node(tree, L, draft_logits, tree_tok, V, temperature, rng_seed, st.step_no[seq], seq, M, node, ps, sh, &o.y);
  }
  if (threadIdx.x == 0) outcome[seq * M + node] = o;
}

// T > 0, vocabularies beyond 32768 entries: the walk of one sequence by one block, node after node, over two vectors in memory.
__global__ __launch_bounds__(1024) void k_accept(const TreeDev* tree, SeqState st, const float* L /*[seq][M][V]*/,
                                                 const float* draft_logits, const int* tree_tok, int V, float temperature,
                                                 unsigned long long rng_seed, float* pbuf, float* qbuf,
                                                 int* path_out /*[seq][D+1]*/, int* tok_out, int* len_out) {
  __shared__ AcceptShared sh;
  float* shv = sh.v;
  double* sh_f = sh.f;
  int &res = sh.res, &s_next = sh.next;
  const int seq = blockIdx.x, M = tree->M, D1 = tree->D + 1;
  int cur = 0, len = 1, bonus = 0;
  if (threadIdx.x == 0) path_out[seq * D1] = 0;
  const int step = st.step_no[seq];
  while (true) {
    const float* lg = L + ((size_t)seq * M + cur) * V;
    const int nk = tree->nchild[cur];
    float* p = pbuf + (size_t)seq * V;
    float* q = qbuf + (size_t)seq * V;
    const float invT = 1.0f / temperature;
    block_softmax(lg, p, V, invT, shv);
    if (nk > 0) block_softmax(draft_logits + ((size_t)seq * M + cur) * V, q, V, invT, shv);
    if (threadIdx.x == 0) s_next = -1;
    __syncthreads();
    for (int r = 0; r < nk; ++r) {
      const int c = tree->child[cur][r];
      const int t = tree_tok[seq * M + c];
      float rr = (float)rng_u24(rng_prefix(rng_seed, PURPOSE_ACCEPT, (unsigned long long)step), (uint32_t)seq, (uint32_t)c, 0) * 5.9604644775390625e-8f;
      bool ok = rr * q[t] < p[t];
      __syncthreads();
      if (ok) { if (threadIdx.x == 0) s_next = c; break; }
      // residual target, proposal without t
      float sm = 0.f;
      for (int j = threadIdx.x; j < V; j += blockDim.x) { float d = fmaxf(p[j] - q[j], 0.f); sm += d; }
      sm = block_sum(sm, shv);
      if (sm > 1e-20f)
        for (int j = threadIdx.x; j < V; j += blockDim.x) p[j] = fmaxf(p[j] - q[j], 0.f) / sm;
      __syncthreads();
      if (threadIdx.x == 0) q[t] = 0.f;
      __syncthreads();
      float qs = 0.f;
      for (int j = threadIdx.x; j < V; j += blockDim.x) qs += q[j];
      qs = block_sum(qs, shv);
      if (qs > 0.f)
        for (int j = threadIdx.x; j < V; j += blockDim.x) q[j] = q[j] / qs;
      __syncthreads();
    }
    __syncthreads();
    if (s_next < 0) {
      float u = (float)rng_u24(rng_prefix(rng_seed, PURPOSE_FINAL, (unsigned long long)step), (uint32_t)seq, (uint32_t)cur, 0) * 5.9604644775390625e-8f;
      bonus = block_inverse_cdf(p, V, u, sh_f, &res);
      break;
    }
    cur = s_next;
    if (threadIdx.x == 0) path_out[seq * D1 + len] = cur;
    ++len;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int n = st.n_tok[seq];
    for (int i = 1; i < len; ++i) {
      int t = tree_tok[seq * M + path_out[seq * D1 + i]];
      tok_out[seq * D1 + i - 1] = t;
      st.tokens[(size_t)seq * st.tok_stride + n + i - 1] = t;
    }
    tok_out[seq * D1 + len - 1] = bonus;
    st.tokens[(size_t)seq * st.tok_stride + n + len - 1] = bonus;
    len_out[seq] = len;
    st.commit_base[seq] = st.ctx_len[seq];
    st.n_tok[seq] = n + len; st.ctx_len[seq] += len; st.n_pend[seq] = len; st.step_no[seq] = step + 1;
  }
}

// Commit (Sec. 3.3: accepted tokens and their features are kept): for every layer, KV rows of the accepted
// nodes move from slot base+path[i] to base+i, and the accepted nodes' target features become the pending
// features of the next drafting phase.  ONE launch: blockIdx.y = layer (last y = the feature rows).
// A thread owns one 16-byte column of a row and moves i = 1..len-1 in increasing order, four at a time; since path[i] >= i and
// path is increasing, a destination is never a source that is still to be read.
// WALK: the path is not there yet; every block finds it from the nodes' outcomes, and the block of the features writes it and the sequence's new
// state, which no other block reads (they begin at commit_base).  us a step, 26 nodes, 7B: arg-max 6.7, walk 7.3 and
// this 10.4 / now outcomes 7.7 and this 10.6.  (132 blocks of 256 threads instead of a block a layer: 14.3; each first reads the same few lines, and the XCDs
// get those one after the other.)  Blocks a layer (1, 2, 4), five or six rows a sequence, us: 7B 9.3, 9.9, 13.5; 16 layers of it with four sequences 13.4, 15.3,
// 21.1, with sixteen 24.3, 24.5, 30.0; 13B, 10 layers, 8.0, 7.7, 8.5, with four 13.6, 13.5, 17.4; 70B, 8 layers, 7.0, 6.3, 7.7, with four 10.8, 12.1, 15.9; two tiny layers 5.2, 6.0,
// 5.6, with eight 7.5, 8.6, 11.5.
template <typename CT, bool WALK>
__global__ __launch_bounds__(1024) void k_commit(int M, int D1, Pass pass /*cached lengths, where the host knows them*/, SeqState st, const int2* __restrict__ outcome, const int* __restrict__ tree_tok, int* path, int* len_p, int* tok_out,
                                                void* kcache, void* vcache, size_t layer_stride_elems, int n_layers, KVCache kv,
                                                const float* __restrict__ F /*[seq][M][d]*/, float* __restrict__ pend_f, int d) {
  __shared__ int2 s_out[EAGLE_MAX_NODES];
  __shared__ int s_path[EAGLE_MAX_DEPTH + 1], s_len, s_bonus;
  const int seq = blockIdx.z, layer = blockIdx.y, tid = threadIdx.x;
  int base;
  if (pass.ctx_known) base = seq == 0 ? pass.ctx0 : seq == 1 ? pass.ctx1 : seq == 2 ? pass.ctx2 : pass.ctx3;
  else base = __builtin_amdgcn_readfirstlane(st.commit_base[seq]);
  if (WALK) {
    if (tid < M) s_out[tid] = outcome[seq * M + tid];
  } else if (tid < D1) s_path[tid] = path[seq * D1 + tid];
  // pages of the new rows (at most 64 of them, in pages of at least 32 tokens)
  const int p0 = base >> kv.page_shift;
  int page[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) page[i] = kv.page_table[seq * kv.pages_per_seq + min(p0 + i, kv.pages_per_seq - 1)];
  if (!WALK && tid == 0) s_len = len_p[seq];
  __syncthreads();
  if (WALK) {
    if (tid == 0) {
      int cur = 0, len = 1;
      s_path[0] = 0;
      for (int2 o = s_out[0]; o.x >= 0 && len < D1; o = s_out[cur]) { cur = o.x; s_path[len++] = cur; }
      s_len = len; s_bonus = s_out[cur].y;
    }
    __syncthreads();
  }
  const int len = s_len;
  if (layer == n_layers) {
    const int step = 4 * (int)(gridDim.x * blockDim.x);
    for (int i0 = 0; i0 < len; i0 += 4)
      for (int k = 4 * (int)(blockIdx.x * blockDim.x + tid); k < d; k += step) {
        f32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const f32x4*)(F + ((size_t)seq * M + s_path[min(i0 + i, len - 1)]) * d + k);
#pragma unroll
        for (int i = 0; i < 4; ++i) if (i0 + i < len) *(f32x4*)(pend_f + ((size_t)seq * D1 + i0 + i) * d + k) = v[i];
      }
    if (WALK && blockIdx.x == 0 && tid < len) {                // (len <= 16: lanes of the first wave)
      const int n = st.n_tok[seq], steps = st.step_no[seq];
      const int t = tid + 1 < len ? tree_tok[seq * M + s_path[tid + 1]] : s_bonus;
      path[seq * D1 + tid] = s_path[tid];
      tok_out[seq * D1 + tid] = t;
      st.tokens[(size_t)seq * st.tok_stride + n + tid] = t;
      if (tid == 0) {
        len_p[seq] = len;
        st.n_tok[seq] = n + len; st.ctx_len[seq] = base + len; st.n_pend[seq] = len; st.step_no[seq] = steps + 1;
      }
    }
    return;
  }
  int first = 1;                                               // rows up to the first that moves stay (behind it all move)
  while (first < len && s_path[first] == first) ++first;
  constexpr int EPC = 16 / sizeof(CT);                        // elements per 16-byte column
  const int cols = kv.n_kv_heads * kv.head_dim / EPC, dh_shift = 31 - __builtin_clz(kv.head_dim);
  const uint32_t mask = (1u << kv.page_shift) - 1;
  for (int c = blockIdx.x * blockDim.x + tid; c < 2 * cols; c += gridDim.x * blockDim.x) {
    const int cc = c >= cols ? c - cols : c;
    const int kvh = cc * EPC >> dh_shift, off = cc * EPC & (kv.head_dim - 1);
    CT* cache = (CT*)(c >= cols ? vcache : kcache) + (size_t)layer * layer_stride_elems + off;
    auto row_at = [&](int i) {
      const int pos = base + i, k = (pos >> kv.page_shift) - p0;
      const int phys = k == 0 ? page[0] : k == 1 ? page[1] : page[2];
      return (u32x4*)(cache + (((((size_t)phys * kv.n_kv_heads + kvh) << kv.page_shift) + (pos & mask)) << dh_shift));
    };
    for (int i0 = first; i0 < len; i0 += 4) {
      u32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *row_at(s_path[min(i0 + i, len - 1)]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i0 + i < len) *row_at(i0 + i) = v[i];
    }
  }
}

// Commit of paths handed in by the caller instead of found by acceptance (lock-step tests drive the engine along the
// oracle's choices with it): the bookkeeping at the end of a step, for every sequence.  bonus[seq] = the token that
// follows the accepted drafts.  k_commit runs afterwards along the given path.
__global__ void k_force_commit(const TreeDev* tree, SeqState st, const int* path /*[seq][D+1]*/, const int* len_p,
                               const int* bonus, const int* tree_tok, int* tok_out, int n_seq) {
  const int seq = blockIdx.x * blockDim.x + threadIdx.x;
  if (seq >= n_seq) return;
  const int M = tree->M, D1 = tree->D + 1, len = len_p[seq], n = st.n_tok[seq];
  for (int i = 1; i < len; ++i) {
    const int t = tree_tok[seq * M + path[seq * D1 + i]];
    tok_out[seq * D1 + i - 1] = t;
    st.tokens[(size_t)seq * st.tok_stride + n + i - 1] = t;
  }
  tok_out[seq * D1 + len - 1] = bonus[seq];
  st.tokens[(size_t)seq * st.tok_stride + n + len - 1] = bonus[seq];
  st.commit_base[seq] = st.ctx_len[seq];
  st.n_tok[seq] = n + len; st.ctx_len[seq] += len; st.n_pend[seq] = len; st.step_no[seq] += 1;
}

// ============================================================================ MoE router
// Row r: x = the normalised MLP input (given, or h * rstd * gain), router logits in fp32, top-k experts (equal
// logits -> lower expert id), softmax over the selected logits.  Writes the dense routing weights
// moe_w[e][row_stride] (0 where the row does not use expert e) and expert_used[e].  Block = one row.
__global__ __launch_bounds__(256) void k_router(const float* xnorm, const float* h, const float* ssq, int ssq_groups, float inv_d,
                                                float eps, const float* gain, const float* __restrict__ router, int E, int topk,
                                                int d, int M, float* moe_w, int row_stride, int* expert_used) {
  __shared__ float sh[16];
  __shared__ float lg[64], lgw[4][64];           // 256 threads: four waves
  const int r = blockIdx.x;
  float rstd = 1.f;
  if (!xnorm) {                                  // same class order as every other consumer of these partial sums
    if (threadIdx.x < 16) {
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int g = (int)threadIdx.x + 16 * i;
        v[i] = g < ssq_groups ? ssq[g * 32 + r] : 0.f;
      }
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) a += v[i];
      sh[threadIdx.x] = a;
    }
    __syncthreads();
    float tot = 0.f;
    for (int c = 0; c < 16; ++c) tot += sh[c];
    rstd = 1.0f / sqrtf(tot * inv_d + eps);
    __syncthreads();                             // sh is reused by block_sum below
  }
  // a thread walks its columns once for eight experts at a time (the row and eight router rows in flight together); the
  // waves' sums meet in LDS once for all of them.  (One expert after the other, each with a block-wide sum of its own: 62 us a
  // call at 8 experts and 4096 columns.)
  for (int e0 = 0; e0 < E; e0 += 8) {
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {   // d is a multiple of 64
      f32x4 x;
      if (xnorm) x = *(const f32x4*)(xnorm + (size_t)r * d + k);
      else { x = *(const f32x4*)(h + (size_t)r * d + k) * rstd; x *= *(const f32x4*)(gain + k); }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const f32x4 w = *(const f32x4*)(router + (size_t)min(e0 + j, E - 1) * d + k);
        a[j] += x.x * w.x + x.y * w.y + x.z * w.z + x.w * w.w;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      for (int o = 32; o > 0; o >>= 1) a[j] += __shfl_xor(a[j], o, 64);
      if ((threadIdx.x & 63) == 0 && e0 + j < E) lgw[threadIdx.x >> 6][e0 + j] = a[j];
    }
  }
  __syncthreads();
  if (threadIdx.x < 64) lg[threadIdx.x] = (lgw[0][threadIdx.x] + lgw[1][threadIdx.x]) + (lgw[2][threadIdx.x] + lgw[3][threadIdx.x]);
  __syncthreads();
  if (threadIdx.x == 0) {
    int sel[4];
    float sv[4];
    for (int j = 0; j < topk; ++j) {
      float bv = -INFINITY; int bi = -1;           // (the first free expert where no logit compares: a row of NaN stays one)
      for (int e = 0; e < E; ++e) {
        bool taken = false;
        for (int q = 0; q < j; ++q) taken |= (sel[q] == e);
        if (taken) continue;
        if (bi < 0) { bv = lg[e]; bi = e; }
        else better(bv, bi, lg[e], e);
      }
      sel[j] = bi; sv[j] = bv;
    }
    float mx = sv[0], den = 0.f, p[4];
    for (int j = 0; j < topk; ++j) { p[j] = expf(sv[j] - mx); den += p[j]; }
    for (int e = 0; e < E; ++e) moe_w[(size_t)e * row_stride + r] = 0.f;
    for (int j = 0; j < topk; ++j) {
      moe_w[(size_t)sel[j] * row_stride + r] = p[j] / den;
      if (r < M) atomicOr(expert_used + sel[j], 1);
    }
  }
}

// Groups the rows of a pass by expert for the grouped GEMMs: expert e's rows, ascending, take consecutive slots from the first
// free tile on, whole columns of `rt` 32-row tiles each.  slot_of[e][row] = slot or -1, row_of[slot] = row or -1 (the rest of an
// expert's last tile).  One work-group; a wave per expert, 64 rows at a time.
__global__ __launch_bounds__(1024) void k_moe_plan(const float* __restrict__ moe_w, int row_stride, int E, int M, int rt, MoePlan* plan, int* slot_of, int* row_of) {
  __shared__ int cnt[64], first[64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int e = w; e < E; e += 16) {
    int n = 0;
    for (int r0 = 0; r0 < M; r0 += 64) n += __popcll(__ballot(r0 + lane < M && moe_w[(size_t)e * row_stride + r0 + lane] != 0.f));
    if (lane == 0) cnt[e] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int tile = 0, cols = 0;
    for (int e = 0; e < E; ++e) {
      first[e] = tile * 32;
      for (int r = 0; r < cnt[e]; r += 32 * rt, ++cols) {
        plan->expert[cols] = e; plan->tile0[cols] = tile; plan->rows[cols] = min(cnt[e] - r, 32 * rt);
        tile += min(rt, (cnt[e] - r + 31) / 32);
      }
    }
    plan->n_cols = cols;
  }
  __syncthreads();
  for (int e = w; e < E; e += 16) {
    int at = first[e];
    for (int r0 = 0; r0 < M; r0 += 64) {
      const int r = r0 + lane;
      const bool mine = r < M && moe_w[(size_t)e * row_stride + r] != 0.f;
      const unsigned long long m = __ballot(mine);
      const int slot = at + __popcll(m & ((1ull << lane) - 1ull));
      if (r < M) slot_of[(size_t)e * row_stride + r] = mine ? slot : -1;
      if (mine) row_of[slot] = r;
      at += __popcll(m);
    }
    for (int q = at + lane; q < (at + 31) / 32 * 32; q += 64) row_of[q] = -1;
  }
}

// The experts' rows as one GEMM input: tile t of the output (32 slots) holds rows row_of[32 t ..] of XF; slots without a row are
// zero.  A wave copies four k-steps of a tile, both planes (16 bytes a lane and k-step).  Grid (tiles, k-steps / 16).
__global__ __launch_bounds__(256) void k_moe_gather(const MoePlan* __restrict__ plan, const int* __restrict__ row_of, const bf16_t* __restrict__ XF, int MT,
                                                    bf16_t* __restrict__ out, int MT_out, int KS, int nplanes) {
  const int last = plan->n_cols - 1, t = blockIdx.x;
  if (last < 0 || t >= plan->tile0[last] + (plan->rows[last] + 31) / 32) return;
  const int lane = threadIdx.x & 63, ks0 = blockIdx.y * 16 + (threadIdx.x >> 6) * 4;
  const int row = row_of[t * 32 + (lane & 31)];
  for (int q = 0; q < nplanes; ++q) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[u] = u32x4{0u, 0u, 0u, 0u};
      if (row >= 0 && ks0 + u < KS) v[u] = *(const u32x4*)(XF + xf_index(row, 16 * (ks0 + u) + 8 * (lane >> 5), q, MT, KS));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ks0 + u < KS) *(u32x4*)(out + (((size_t)q * MT_out + t) * KS + ks0 + u) * 512 + lane * 8) = v[u];
  }
}

// ============================================================================ debug / test access
template <typename CT>
__global__ void k_read_kv_row(KVCache kv, int seq, int pos, float* kout, float* vout) {
  int n = kv.n_kv_heads * kv.head_dim;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    int kvh = i / kv.head_dim, d = i % kv.head_dim;
    size_t o = kv_offset(kv, seq, pos, kvh) + d;
    kout[i] = cache_load((const CT*)kv.k + o);
    vout[i] = cache_load((const CT*)kv.v + o);
  }
}

// Profiling: adds the number of experts at least one row selected (flags set by k_router) to a running total.
__global__ void k_count_used(const int* expert_used, int E, int* total) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    int n = 0;
    for (int e = 0; e < E; ++e) n += expert_used[e] != 0;
    *total += n;
  }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
