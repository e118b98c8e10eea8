// Fast path for passes of at most 32 rows (tree verification at batch 1, the head's tree levels, vanilla
// decoding): weight-streaming GEMM with the reduction and the layer's element-wise work fused into it.
//
//   * A work-group owns (a group of 32-row weight blocks) x (one K slice).  Its K slice of the activations sits
//     in LDS in MFMA B-operand order; every wave streams its own weight tiles straight from HBM into the MFMA
//     A operand (one coalesced 1 KiB load per tile, many tiles in flight).
//   * Waves that share a weight block but split K are summed through LDS in a fixed order; work-groups that
//     split K write partials and the LAST one to arrive (an atomic counter, no waiting) sums them in split
//     order and runs the epilogue -- so results do not depend on timing.
//   * RMSNorm is folded around the GEMM: the producer writes h*gain (not normalised) plus per-row partial sums
//     of squares; the consumer multiplies its outputs by 1/rms, which commutes with the matrix product.
#pragma once
#include "kernels.h"
#include "plans.h"

#define V2_THREADS 512

// Data that one work-group writes and another reads INSIDE one kernel (split-K partials, attention partials) goes
// through agent-scope accesses: such stores are written through to the device-coherent level and such
// loads never hit a stale line of another XCD's L2, so no cache write-back / invalidate is needed around the
// arrival counter -- a work-group-scope fence (a wait for the stores to be acknowledged) is enough.
// Buffer instructions carry the scope bit (aux 16 = sc1); byte offsets below 2 GiB.
__device__ inline __amdgpu_buffer_rsrc_t coh_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 0x7FFFFFFF, 0x00020000);
}
__device__ inline f32x4 coh_load16(const void* base, uint32_t byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(coh_rsrc(base), byte_off, 0, 16));
}
__device__ inline void coh_store16(void* base, uint32_t byte_off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), coh_rsrc(base), byte_off, 0, 16);
}
// Split-K partials PT[s][n][m]: four consecutive weight rows n of one token m are adjacent (16 bytes), which is what
// one lane of the MFMA accumulator holds (registers 4i..4i+3) and what an epilogue thread consumes.
__device__ inline uint32_t pt_quad_bytes(int s, int Npad, int n4 /*multiple of 4*/, int m) {
  return (uint32_t)((((size_t)s * Npad + n4) * 32 + (size_t)m * 4) * 4);
}

// The wave's number as a scalar: everything derived from it (K range, tile addresses, buffer offsets) then stays in scalar
// registers.  Left to the compiler it is a per-lane value, and every buffer load whose offset depends on it becomes a loop
// over the lanes' distinct offsets.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

constexpr uint32_t OUT_OF_RANGE = 0x80000000u;   // lane offset beyond every buffer resource: a load returns zeros without a memory access (its scalar offset inside the resource)
struct RowScale {            // 1/rms of the rows that produced the GEMM input; groups == 0 -> 1
  const float* ssq;          // [groups <= 256][32] partial sums of squares
  int groups;
  float inv_d, eps;
};
// 1/rms of row m from the per-group partial sums of squares: 16 strided classes of groups, classes added in order
// (one fixed order for every caller).  The block shares the loads: threads 0..15 each own a class (at most 16 groups,
// all loads in flight), thread 0 adds the classes.  tmp: 17 floats of LDS.  Every thread of the block must call it.
__device__ inline float block_row_rstd(const float* ssq, int groups, float inv_d, float eps, int m, float* tmp) {
  if (!ssq) return 1.0f;
  if (threadIdx.x < 16) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int g = (int)threadIdx.x + 16 * i;
      v[i] = g < groups ? ssq[g * 32 + m] : 0.f;
    }
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) a += v[i];
    tmp[threadIdx.x] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float tot = 0.f;
    for (int c = 0; c < 16; ++c) tot += tmp[c];
    tmp[16] = 1.0f / sqrtf(tot * inv_d + eps);
  }
  __syncthreads();
  return tmp[16];
}
// The same value for all 32 rows at once, computed by a 512-thread block: thread (m, class c) requests the first four of its class's
// groups and its row's facts beside the weight stream's first requests without using them, so that no load of the stream waits for
// them; the classes are combined through LDS when the epilogue needs the result.  ssq always points at 256 * 32 floats.  (Read and summed in front of the stream, with the row's facts
// found by walking tree and page table, these were 4 to 5 dependent memory round trips before the first weight load; without
// them: QKV 26.9 -> 25.4, gate/up 38.1 -> 36.5, down 26.2 -> 25.4 us at 7B widths, 4-bit gate/up 30.0 -> 22.3 us.)
struct EarlyLoads { float ssq[4]; int pos, kv_row, out_row; };
__device__ __forceinline__ void early_issue(const float* ssq, const RowFact* facts, EarlyLoads& e) {
  const float* p = ssq + threadIdx.x;
  const RowFact* f = facts + (threadIdx.x & 31);
  e.pos = f->pos; e.kv_row = f->kv_row; e.out_row = f->out_row;
#pragma unroll
  for (int i = 0; i < 4; ++i) e.ssq[i] = p[(size_t)i * 512];   // (no branch: behind one, the wait for the first weight tile would be a wait for all requests)
}
__device__ inline float early_ssq(const RowScale& rs, EarlyLoads& e) {
  float a = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(e.ssq[i]));    // the sum stays here: hoisted, it would wait in front of the stream
#pragma unroll
  for (int i = 0; i < 4; ++i) a += (int)(threadIdx.x >> 5) + 16 * i < rs.groups ? e.ssq[i] : 0.f;
  if (rs.groups > 64) {
    const float* p = rs.ssq + threadIdx.x;
    float v[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) v[i] = p[(size_t)(i + 4) * 512];
#pragma unroll
    for (int i = 0; i < 12; ++i) a += (int)(threadIdx.x >> 5) + 16 * (i + 4) < rs.groups ? v[i] : 0.f;
  }
  return a;
}
// The classes' sums left in tmp[16][32] and, a barrier later, 1/rms of row m from them.
__device__ __forceinline__ void block_rstd_park(const RowScale& rs, float part, float* tmp) {
  if (rs.groups > 0) tmp[threadIdx.x] = part;
}
__device__ __forceinline__ float block_rstd(const RowScale& rs, const float* tmp, int m) {
  if (rs.groups == 0) return 1.0f;
  float v[16], tot = 0.f;
#pragma unroll
  for (int cc = 0; cc < 16; ++cc) v[cc] = tmp[cc * 32 + m];
#pragma unroll
  for (int cc = 0; cc < 16; ++cc) tot += v[cc];
  return 1.0f / sqrtf(tot * rs.inv_d + rs.eps);
}
__device__ inline void block_rstd_finish(const RowScale& rs, float part, float* out, float* tmp) {
  if (rs.groups == 0) {
    if (threadIdx.x < 32) out[threadIdx.x] = 1.0f;
    __syncthreads();
    return;
  }
  tmp[(threadIdx.x >> 5) * 32 + (threadIdx.x & 31)] = part;
  __syncthreads();
  if (threadIdx.x < 32) {
    float tot = 0.f;
    for (int cc = 0; cc < 16; ++cc) tot += tmp[cc * 32 + threadIdx.x];
    out[threadIdx.x] = 1.0f / sqrtf(tot * rs.inv_d + rs.eps);
  }
  __syncthreads();
}

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

struct Gemm2 {
  // what the start of a weight stream needs, side by side: one fetch of arguments before the first request
  const bf16_t* W; const bf16_t* XF;      // XF: NXP planes of KS tiles (one 32-row tile per k-step)
  int NRB, KS, M, groups;                 // groups: row groups = work-groups of a K slice
  uint32_t share_a, share_b, S_magic;     // the row groups' shares of the row blocks (share_begin; k2_gemm_xk: div_magic of groups) and div_magic of S
  int S, NG;                              // 4-bit weights: NG groups along K
  const int* skip_flag;                   // MoE: an expert's work is a no-op when its flag is 0 (no row uses it); [experts] with EXPERTS
  const RowFact* facts;                   // [32] rows of the pass
  RowScale in_scale;
  size_t wps; int Npad, N;
  int lanes, kparts;
  float* PT; int* counters;
  int epi;
  // EPI_QKV
  KVCache kv; int kv_f32; float* Q; const float* rope_cos; const float* rope_sin; int H;
  // EPI_RESID / EPI_SWIGLU
  const float* h_in; float* h_out; const float* bias; const float* gain_next; bf16_t* xf_out; int xf_KS; float* ssq_out; int d;
  // EPI_LOGITS
  float* logits; int V;
  Q4Format q4;                            // 4-bit weights: how a code becomes a bf16 value
  const bf16_t* SC;                       // 4-bit weights: scales [NRB][NG][2][16] (W then holds codes)
  const float* row_w;                     // MoE: per-row routing weight applied to this GEMM's result (nullptr = 1)
  // EXPERTS (all experts of a layer in one launch): elements between their matrices, inputs and outputs, and between their routing weights
  size_t w_stride, x_stride, out_stride; int row_w_stride;
  unsigned long long* trace;              // profiling builds (-DEAGLE_TRACE) only: [work-group][8] time stamps of this launch
};

// out[0..3] = sum over the K splits of rows nA..nA+3, out[4..7] the same for rows nB..nB+3 (nA, nB multiples of 4,
// below Npad), token m.  All loads of a batch of splits are in flight together; splits are added in order.
template <int B>
__device__ inline void pt_sum8_b(const float* __restrict__ PT, int S, int Npad, int nA, int nB, int m, float* out) {
  for (int s0 = 0; s0 < S; s0 += B) {
    f32x4 va[B], vb[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int s = min(s0 + u, S - 1);
      va[u] = coh_load16(PT, pt_quad_bytes(s, Npad, nA, m));
      vb[u] = coh_load16(PT, pt_quad_bytes(s, Npad, nB, m));
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (s0 + u < S) {
        out[0] += va[u].x; out[1] += va[u].y; out[2] += va[u].z; out[3] += va[u].w;
        out[4] += vb[u].x; out[5] += vb[u].y; out[6] += vb[u].z; out[7] += vb[u].w;
      }
  }
}
__device__ inline void pt_sum8(const float* __restrict__ PT, int S, int Npad, int nA, int nB, int m, float* out) {
#pragma unroll
  for (int t = 0; t < 8; ++t) out[t] = 0.f;
  // the batch size closest above S: loads beyond S would be wasted traffic in an epilogue that one CU's bandwidth bounds
  if (S <= 4) pt_sum8_b<4>(PT, S, Npad, nA, nB, m, out);
  else if (S <= 8) pt_sum8_b<8>(PT, S, Npad, nA, nB, m, out);
  else if (S <= 12) pt_sum8_b<12>(PT, S, Npad, nA, nB, m, out);
  else pt_sum8_b<16>(PT, S, Npad, nA, nB, m, out);
}

// four quads at once, S <= 4: 16 loads in flight; issue and summation are separate so that a caller can put the
// loads of several items in flight before it consumes the first
struct PtQuads4 { f32x4 v[4][4]; };
__device__ inline void pt_issue16(PtQuads4& b, const float* __restrict__ PT, int S, int Npad, int nA, int nB, int nC, int nD, int m) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int sp = min(u, S - 1);
    b.v[u][0] = coh_load16(PT, pt_quad_bytes(sp, Npad, nA, m));
    b.v[u][1] = coh_load16(PT, pt_quad_bytes(sp, Npad, nB, m));
    b.v[u][2] = coh_load16(PT, pt_quad_bytes(sp, Npad, nC, m));
    b.v[u][3] = coh_load16(PT, pt_quad_bytes(sp, Npad, nD, m));
  }
}
__device__ inline void pt_finish16(const PtQuads4& b, int S, float* outAB, float* outCD) {
#pragma unroll
  for (int t = 0; t < 8; ++t) { outAB[t] = 0.f; outCD[t] = 0.f; }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < S) {
      outAB[0] += b.v[u][0].x; outAB[1] += b.v[u][0].y; outAB[2] += b.v[u][0].z; outAB[3] += b.v[u][0].w;
      outAB[4] += b.v[u][1].x; outAB[5] += b.v[u][1].y; outAB[6] += b.v[u][1].z; outAB[7] += b.v[u][1].w;
      outCD[0] += b.v[u][2].x; outCD[1] += b.v[u][2].y; outCD[2] += b.v[u][2].z; outCD[3] += b.v[u][2].w;
      outCD[4] += b.v[u][3].x; outCD[5] += b.v[u][3].y; outCD[6] += b.v[u][3].z; outCD[7] += b.v[u][3].w;
    }
}
// the same for any S (more than 4 splits: two rounds of two quads)
__device__ inline void pt_sum16(const float* __restrict__ PT, int S, int Npad, int nA, int nB, int nC, int nD, int m, float* outAB, float* outCD) {
  if (S > 4) { pt_sum8(PT, S, Npad, nA, nB, m, outAB); pt_sum8(PT, S, Npad, nC, nD, m, outCD); return; }
  PtQuads4 b;
  pt_issue16(b, PT, S, Npad, nA, nB, nC, nD, m);
  pt_finish16(b, S, outAB, outCD);
}

// Kernel arguments that the start of a weight stream needs, fetched together: the arguments come from memory, and a wait
// between two groups of them costs another round trip in front of the first weight tile.
__device__ __forceinline__ void pin_args(const Gemm2& g) {
  asm volatile("" ::"s"(g.W), "s"(g.XF), "s"(g.NRB), "s"(g.KS), "s"(g.M), "s"(g.groups), "s"(g.share_a), "s"(g.share_b), "s"(g.S_magic), "s"(g.S), "s"(g.NG), "s"(g.skip_flag), "s"(g.facts), "s"(g.in_scale.ssq));
}

// The arguments again, for the epilogue: fetched where this stands (behind a stream's first requests) and not before it.  Left to the compiler,
// theirs is a second fetch, and a wait for it, in front of the first request.
__device__ __forceinline__ Gemm2 late_args() {
  const __attribute__((address_space(4))) Gemm2* p = (const __attribute__((address_space(4))) Gemm2*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p)::"memory");
  return *(const Gemm2*)p;
}

// Four consecutive values of row m, columns k.. (k a multiple of 4), as GEMM input (8 bytes per plane).
__device__ inline void xf_store4(bf16_t* XF, int m, int k, int MT, int KS, int nplanes, f32x4 x) {
  float r[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (q < nplanes) {
      uint2 v; v.x = split_pair(r[0], r[1]); v.y = split_pair(r[2], r[3]);
      *(uint2*)(XF + xf_index(m, k, q, MT, KS)) = v;
    }
}

// Rows n..n+3 (a multiple of 4) of the fused QKV matrix for token m: two rotate-half pairs of a query or key head, or four dimensions of a
// value head, where they belong.
__device__ __forceinline__ void qkv_store(const Gemm2& g, int n, int m, int dh_shift, f32x4 sum, float rs, float2 cs, float2 sn, int kv_row, int H, int KVH) {
  const int dh = 1 << dh_shift, hd = n >> dh_shift, pr = n & (dh - 1);
  const f32x4 v = {sum.x * rs, sum.y * rs, sum.z * rs, sum.w * rs};
  const int i = pr >> 1, half = dh >> 1;
  float2 lo, hi;                                                // dimensions i, i + 1 and half + i, half + i + 1
  { const float a = v.x, b = v.y; lo.x = a * cs.x - b * sn.x; hi.x = b * cs.x + a * sn.x; }
  { const float a = v.z, b = v.w; lo.y = a * cs.y - b * sn.y; hi.y = b * cs.y + a * sn.y; }
  if (hd < H) {
    float* q = g.Q + ((size_t)m * H + hd) * dh;
    *(float2*)(q + i) = lo; *(float2*)(q + half + i) = hi;
  } else if (kv_row >= 0) {
    const bool key = hd < H + KVH;
    const int kvh = hd - H - (key ? 0 : KVH);
    const size_t off = ((size_t)kv_row + ((size_t)kvh << g.kv.page_shift)) * dh;
    if (g.kv_f32) {
      float* p = (float*)(key ? g.kv.k : g.kv.v) + off;
      if (key) { *(float2*)(p + i) = lo; *(float2*)(p + half + i) = hi; }
      else *(f32x4*)(p + pr) = v;
    } else {
      bf16_t* p = (bf16_t*)(key ? g.kv.k : g.kv.v) + off;
      auto pack = [](float a, float b) { return (uint32_t)f32_to_bf16(a) | (uint32_t)f32_to_bf16(b) << 16; };
      if (key) { *(uint32_t*)(p + i) = pack(lo.x, lo.y); *(uint32_t*)(p + half + i) = pack(hi.x, hi.y); }
      else { uint2 u; u.x = pack(v.x, v.y); u.y = pack(v.z, v.w); *(uint2*)(p + pr) = u; }
    }
  }
}

template <int NXP>
__device__ inline void epilogue_qkv(const Gemm2& g, int n0, int n1, const float* rstd_s, const EarlyLoads& rp) {
  const int m = threadIdx.x & 31, slot = threadIdx.x >> 5;
  const int dh = g.kv.head_dim, half = dh >> 1, KVH = g.kv.n_kv_heads, H = g.H;
  const bool live = m < g.M;
  const float rs = live ? rstd_s[m] : 0.f;
  const int nquads = (n1 - n0) >> 2;                          // n0, n1 are multiples of 32 here (whole heads)
  constexpr int SL = V2_THREADS / 32;
  for (int q0 = slot; q0 < nquads; q0 += 4 * SL) {           // four quads = eight rotate-half pairs per batch of loads
    int nq[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) nq[c] = n0 + 4 * min(q0 + c * SL, nquads - 1);
    float cs[8], sn[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int n = nq[u >> 1] + 2 * (u & 1);
      const int i = (n % dh) >> 1;                            // rotation angle index (unused for v heads)
      cs[u] = g.rope_cos[(size_t)rp.pos * half + i];
      sn[u] = g.rope_sin[(size_t)rp.pos * half + i];
    }
    float val[16];
    pt_sum16(g.PT, g.S, g.Npad, nq[0], nq[1], nq[2], nq[3], m, val, val + 8);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (q0 + (u >> 1) * SL >= nquads || !live) continue;
      const int n = nq[u >> 1] + 2 * (u & 1), hd = n / dh, pr = n % dh;
      float a = val[2 * u] * rs, b = val[2 * u + 1] * rs;
      int d1, d2;
      if (hd < H + KVH) {        // q or k head: the two rows are a rotate-half pair
        const int i = pr >> 1;
        const float a2 = a * cs[u] - b * sn[u], b2 = b * cs[u] + a * sn[u];
        a = a2; b = b2; d1 = i; d2 = i + half;
      } else { d1 = pr; d2 = pr + 1; }
      if (hd < H) {
        float* q = g.Q + ((size_t)m * H + hd) * dh;
        q[d1] = a; q[d2] = b;
      } else if (rp.kv_row >= 0) {
        const int kvh = (hd - H) % KVH;
        const size_t off = ((size_t)rp.kv_row + ((size_t)kvh << g.kv.page_shift)) * dh;
        void* base = hd < H + KVH ? g.kv.k : g.kv.v;
        if (g.kv_f32) { ((float*)base)[off + d1] = a; ((float*)base)[off + d2] = b; }
        else { ((bf16_t*)base)[off + d1] = f32_to_bf16(a); ((bf16_t*)base)[off + d2] = f32_to_bf16(b); }
      }
    }
  }
}

// What a lane of the residual epilogue adds and multiplies in the chunk of 8 output rows from n8 on.
struct ResidItem { f32x4 h, bias, gain; };
__device__ __forceinline__ ResidItem resid_item(const Gemm2& g, int n8, bool on) {
  const int m = threadIdx.x & 31, n = n8 + 4 * ((threadIdx.x >> 5) & 1);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  ResidItem r;
  r.h = on && g.h_in && m < g.M ? *(const f32x4*)(g.h_in + (size_t)m * g.d + n) : zero;
  r.bias = on && g.bias ? *(const f32x4*)(g.bias + n) : zero;
  r.gain = on && g.gain_next ? *(const f32x4*)(g.gain_next + n) : zero;
  return r;
}
// A wave owns chunks of 8 output rows (n), a lane four of them: lanes 0..31 the first four of tokens 0..31, lanes 32..63 the other
// four; residual, bias, gain and the partials come as 16-byte loads, all in flight together.  (A lane per chunk and token, row by
// row, used half of the threads and touched 64 lines with each of its 16 four-byte accesses.)  A token's squares are added
// chunk by chunk in row order, chunks c, c + 16, ... in one chain: the lower lanes begin a chunk's part, the upper ones go on.
// EXPERTS: the partials of every expert in `used` (g.S slices each), added per row in expert order with the routing weights, as one
// launch per expert behind the other would.
// The items of the first ITEMS chunks of a wave (c = w, w + 8, ...) come with the call; ITEMS = 0: none, and any number of chunks.
template <int NXP, bool EXPERTS = false, int ITEMS = 0>
__device__ inline void epilogue_resid(const Gemm2& g, int grp, int n0, int n1, float* sh /*>= 16*32 floats*/, const ResidItem* ri = nullptr, unsigned long long used = 1) {
  const int lane = threadIdx.x & 63, m = lane & 31, hh = lane >> 5, w = threadIdx.x >> 6;
  const bool live = m < g.M;
  const int nchunks = (n1 - n0) >> 3;                        // n0 and n1 are multiples of 32 (d_model is one of 64)
  const float rw = !EXPERTS && g.row_w ? g.row_w[m] : 1.0f;
  float ss[2] = {0.f, 0.f};                                  // chains w and w + 8
  const uint32_t slice = (uint32_t)g.Npad * 128u;            // bytes of a slice's partials
  auto chunk = [&](int c, int turn, const ResidItem& r) {
    const int n = n0 + 8 * c + 4 * hh;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const uint32_t at = pt_quad_bytes(0, g.Npad, n, m);
    f32x4 v = zero;
    if constexpr (EXPERTS) {
      v = r.h;
      for (unsigned long long left = used; left; ) {           // four experts' first four slices in flight at once
        int ex[4], cnt = 0;
        f32x4 p[4][4];
        float re[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          ex[b] = __ffsll((long long)(left ? left : used)) - 1;
          cnt += left != 0;
          left &= left - 1;
          re[b] = g.row_w[(size_t)ex[b] * g.row_w_stride + m];
#pragma unroll
          for (int u = 0; u < 4; ++u) p[b][u] = coh_load16(g.PT, pt_quad_bytes(ex[b] * g.S + min(u, g.S - 1), g.Npad, n, m));
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (b >= cnt) continue;
          f32x4 sum = zero;
#pragma unroll
          for (int u = 0; u < 4; ++u) if (u < g.S) sum += p[b][u];
          for (int u = 4; u < g.S; ++u) sum += coh_load16(g.PT, pt_quad_bytes(ex[b] * g.S + u, g.Npad, n, m));
          sum *= re[b];
          v = sum + v;
        }
      }
    } else {
      const __amdgpu_buffer_rsrc_t pt = coh_rsrc(g.PT);
      for (int s0 = 0; s0 < g.S; s0 += 8) {                  // added in split order
        f32x4 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (u < 4 || g.S > 4) p[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(pt, at, (uint32_t)min(s0 + u, g.S - 1) * slice, 16));
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u < g.S) v += p[u];
      }
      if (g.row_w) v *= rw;
      if (g.bias) v += r.bias;
      if (g.h_in && live) v += r.h;
    }
    if (live) *(f32x4*)(g.h_out + (size_t)m * g.d + n) = v;
    float a = turn ? ss[1] : ss[0];
    float up = a;
#pragma unroll
    for (int t = 0; t < 4; ++t) up = fmaf(v[t], v[t], up);   // (upper lanes: not used)
    a = __shfl(up, m, 64);                                   // what the lower lanes have reached
#pragma unroll
    for (int t = 0; t < 4; ++t) a = fmaf(v[t], v[t], a);     // (lower lanes: not used)
    a = __shfl(a, m + 32, 64);
    if (turn) ss[1] = a; else ss[0] = a;
    f32x4 x = v;
    if (g.gain_next) x = v * r.gain;
    if (live) xf_store4(g.xf_out, m, n, 1, g.xf_KS, NXP, x);
  };
  if constexpr (ITEMS > 0) {
#pragma unroll
    for (int t = 0; t < ITEMS; ++t)
      if (w + 8 * t < nchunks) chunk(w + 8 * t, t & 1, ri[t]);
  } else {
    int turn = 0;
    for (int c = w; c < nchunks; c += V2_THREADS / 64, turn ^= 1) chunk(c, turn, resid_item(g, n0 + 8 * c, true));
  }
  if (!g.ssq_out) return;                                    // (uniform)
  __syncthreads();
  if (hh == 0) { sh[w * 32 + m] = ss[0]; sh[(w + 8) * 32 + m] = ss[1]; }
  __syncthreads();
  if (threadIdx.x < 32) {
    float v[V2_THREADS / 32], a = 0.f;
#pragma unroll
    for (int i = 0; i < V2_THREADS / 32; ++i) v[i] = sh[i * 32 + threadIdx.x];
#pragma unroll
    for (int i = 0; i < V2_THREADS / 32; ++i) a += v[i];
    g.ssq_out[grp * 32 + threadIdx.x] = a;
  }
}

__device__ inline void swiglu8(const float* gv, const float* uv, float rs, float* x) {
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const float gg = gv[t] * rs, uu = uv[t] * rs;
    x[t] = gg / (1.0f + __expf(-gg)) * uu;
  }
}
template <int NXP>
__device__ inline void epilogue_swiglu(const Gemm2& g, int n0, int n1, const float* rstd_s) {
  const int m = threadIdx.x & 31, slot = threadIdx.x >> 5;
  const bool live = m < g.M;
  const float rs = live ? rstd_s[m] : 0.f;
  const int items = ((n1 - n0) >> 5) * 2;                    // 8 outputs each: gate rows nb..nb+7, up rows 16 further
  constexpr int SL = V2_THREADS / 32;
  if (g.S <= 4) {
    for (int it = slot; it < items; it += 2 * SL) {          // two items = 32 loads in flight
      const int it2 = min(it + SL, items - 1);
      const int nbA = n0 + (it >> 1) * 32 + 8 * (it & 1), nbB = n0 + (it2 >> 1) * 32 + 8 * (it2 & 1);
      PtQuads4 qa, qb;
      pt_issue16(qa, g.PT, g.S, g.Npad, nbA, nbA + 4, nbA + 16, nbA + 20, m);
      pt_issue16(qb, g.PT, g.S, g.Npad, nbB, nbB + 4, nbB + 16, nbB + 20, m);
      float x[8], gv[8], uv[8];
      pt_finish16(qa, g.S, gv, uv);
      swiglu8(gv, uv, rs, x);
      if (live) xf_store8(g.xf_out, m, ((n0 >> 5) + (it >> 1)) * 16 + 8 * (it & 1), 1, g.xf_KS, NXP, x);
      pt_finish16(qb, g.S, gv, uv);
      swiglu8(gv, uv, rs, x);
      if (live && it + SL < items) xf_store8(g.xf_out, m, ((n0 >> 5) + (it2 >> 1)) * 16 + 8 * (it2 & 1), 1, g.xf_KS, NXP, x);
    }
    return;
  }
  for (int it = slot; it < items; it += SL) {
    const int rb = it >> 1, c2 = it & 1;
    const int nb = n0 + rb * 32 + 8 * c2;
    const int f = ((n0 >> 5) + rb) * 16 + 8 * c2;
    float x[8], gv[8], uv[8];
    pt_sum16(g.PT, g.S, g.Npad, nb, nb + 4, nb + 16, nb + 20, m, gv, uv);
    swiglu8(gv, uv, rs, x);
    if (live) xf_store8(g.xf_out, m, f, 1, g.xf_KS, NXP, x);
  }
}

__device__ inline void epilogue_logits(const Gemm2& g, int n0, int n1, const float* rstd_s, const EarlyLoads& rp) {
  const int m = threadIdx.x & 31, b = threadIdx.x >> 5;        // token m, quad b (and b + 16) of each 128-row batch
  const float rs = m < g.M ? rstd_s[m] : 0.f;
  const long dst = m < g.M && rp.out_row >= 0 ? (long)rp.out_row * g.V : -1;   // where token m's logits row starts, or -1
  const int nend = min(n1, g.V);
  const bool vec = (g.V & 3) == 0;                             // rows of the output are 16-byte aligned
  for (int nb0 = n0; nb0 < n1; nb0 += 128) {
    const int nA = nb0 + 4 * b, nB = nb0 + 64 + 4 * b;
    float val[8];
    pt_sum8(g.PT, g.S, g.Npad, min(nA, g.Npad - 4), min(nB, g.Npad - 4), m, val);
    if (dst < 0) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = h ? nB : nA;
      if (n >= nend) continue;
      if (vec && n + 4 <= nend) {
        f32x4 o; o.x = val[4 * h] * rs; o.y = val[4 * h + 1] * rs; o.z = val[4 * h + 2] * rs; o.w = val[4 * h + 3] * rs;
        *(f32x4*)(g.logits + dst + n) = o;
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) if (n + t < nend) g.logits[dst + n + t] = val[4 * h + t] * rs;
      }
    }
  }
}

// The streaming loop of one wave: NR weight blocks over k-steps [kb, ke), DEPTH k-steps (DEPTH*NR tiles of 1 KiB)
// in flight.  Loads are issued unconditionally (indices clamped to the last step) so that the number in flight is
// static and the compiler waits for exactly the tile it needs.  The first DEPTH steps are requested by
// k2_prologue BEFORE the block stages its X slice, so HBM is already busy while LDS is being filled.
// Tile registers: pre[(dd*NR + j)*NWP + p].
template <int NWP, int NR, int DEPTH>
__device__ __forceinline__ void k2_prologue(int kb, int ke, const u32x4* const* wp, size_t wps, u32x4* pre) {
  if (ke <= kb) return;
  const int klast = ke - 1;
#pragma unroll
  for (int dd = 0; dd < DEPTH; ++dd) {
    const int kk = min(kb + dd, klast);
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int p = 0; p < NWP; ++p) pre[(dd * NR + j) * NWP + p] = *(const u32x4*)((const bf16_t*)(wp[j] + (size_t)kk * 64) + p * wps);
  }
}

template <int NWP, int NXP, int NR, int DEPTH>
__device__ __forceinline__ void k2_stream(const u32x4* __restrict__ xs, int kt, int kb, int ke, const u32x4* const* wp,
                                          size_t wps, f32x16* acc, int lane, u32x4* pre) {
  constexpr int PMAX = NWP > NXP ? NWP : NXP;
  if (ke <= kb) return;
  const int klast = ke - 1;
  int k = kb;
  for (; k + DEPTH < ke; k += DEPTH) {
#pragma unroll
    for (int dd = 0; dd < DEPTH; ++dd) {
      const int kk = k + dd;
      u32x4 bq[NXP];
#pragma unroll
      for (int q = 0; q < NXP; ++q) bq[q] = xs[((size_t)q * kt + kk) * 64 + lane];
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int p = 0; p < NWP; ++p)
#pragma unroll
          for (int q = 0; q < NXP; ++q)
            if (p + q < PMAX)
              acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pre[(dd * NR + j) * NWP + p]),
                                                                __builtin_bit_cast(bf16x8, bq[q]), acc[j], 0, 0, 0);
      const int kn = min(kk + DEPTH, klast);
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int p = 0; p < NWP; ++p) pre[(dd * NR + j) * NWP + p] = *(const u32x4*)((const bf16_t*)(wp[j] + (size_t)kn * 64) + p * wps);
      __builtin_amdgcn_sched_barrier(0);          // keep "use a slot, refill that slot" in program order
    }
  }
#pragma unroll
  for (int dd = 0; dd < DEPTH; ++dd) {
    const int kk = k + dd;
    if (kk < ke) {
      u32x4 bq[NXP];
#pragma unroll
      for (int q = 0; q < NXP; ++q) bq[q] = xs[((size_t)q * kt + kk) * 64 + lane];
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int p = 0; p < NWP; ++p)
#pragma unroll
          for (int q = 0; q < NXP; ++q)
            if (p + q < PMAX)
              acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pre[(dd * NR + j) * NWP + p]),
                                                                __builtin_bit_cast(bf16x8, bq[q]), acc[j], 0, 0, 0);
    }
  }
}

// The sum of x over a k-step comes from a matrix instruction too, one of half the size: the activation fragment of a 32x32x16 product (lane l:
// row l % 32, eight k from 8 * (l / 32) on), read as the B operand of a 16x16x32 one, holds rows 0..15 in its quarters of k 0 and 2 and rows
// 16..31 in 1 and 3.  With this A (lane l: row l % 16, quarter l / 16) the four results of lane l are all the sum of activation row l % 32.
// A row's sum then passes over the row 16 beside it as a product with zero, which is not zero if that row holds an infinity or a NaN.  A wave
// that ends with NaN goes over its groups again and makes such sums with the other rows left out (APART: q4_row_sums), so that no row depends
// on another.  (A second pass: with the branch, or with a flag alone, in the first one's loop half of the gain below was lost.)
// (A 32x32x16 product with ones gave the same bits for twice the matrix time and twelve more registers: two of six products a k-step with two
// row blocks.  Request of a 500-token prompt and 16 steps at 7B widths: 70.4 ms, now 68.0.)
__device__ __forceinline__ u32x4 q4_ones(int lane) {
  const uint32_t o = (((lane & 15) >> 2) ^ (lane >> 4)) & 1 ? 0u : 0x3F803F80u;
  return u32x4{o, o, o, o};
}
// The sums of a group again, rows 0..15 and 16..31 apart.  fetch(i, on): fragment i of the group, zeros where not `on`.
template <int N, class F>
__device__ __forceinline__ float q4_row_sums(const u32x4& ones, int lane, F&& fetch) {
  const bool upper = lane & 16;
  float sum = 0.f;
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    const bool on = upper == (half != 0);
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int i = 0; i < N; ++i) t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, fetch(i, on)), t, 0, 0, 0);
    if (on) sum = t[0];
  }
  return sum;
}

// ---- 4-bit weights against an activation slice in LDS (layout and arithmetic: see k_pack_weight_q4 / fk_stream_q4) ------
// A wave owns NR row blocks over the groups [gb, ge) of the work-group's K slice (slice-relative group indices; the
// slice starts at group g0 of the matrix).  With a quarter of the weight bytes the activation fragments are what a CU
// fetches most of, so here they are fetched ONCE per work-group (into LDS) and every wave reads them from there.
template <int NXP, int NR, bool APART>
__device__ __forceinline__ bool k2_stream_q4(const Q4Format format, const u32x4* __restrict__ xs, int kt, int g0, int gb, int ge, const u32x4* const* wq,
                                             const u32x4* const* sq, f32x16* acc, int lane) {
  if (ge <= gb) return false;
  const Q4Format fmt = q4_pin(format);
  const int glast = ge - 1;
  u32x4 a4[2][NR];
  const u32x4 ones = q4_ones(lane);
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int j = 0; j < NR; ++j) a4[st][j] = wq[j][(size_t)(2 * (g0 + gb) + st) * 64];
  for (int g = gb; g < ge; ++g) {
    f32x16 part[NR];
    f32x4 sx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[j][r] = 0.f;
    u32x4 sraw[NR][2];
#pragma unroll
    for (int j = 0; j < NR; ++j) { sraw[j][0] = sq[j][(size_t)(g0 + g) * 4]; sraw[j][1] = sq[j][(size_t)(g0 + g) * 4 + 1]; }
    const int gn = min(g + 1, glast);
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int kk = 8 * g + 4 * st + ks;                    // k-step inside the slice
        u32x4 bq[NXP];
#pragma unroll
        for (int q = 0; q < NXP; ++q) bq[q] = xs[((size_t)q * kt + kk) * 64 + lane];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
          const uint32_t wd = ks == 0 ? a4[st][j].x : ks == 1 ? a4[st][j].y : ks == 2 ? a4[st][j].z : a4[st][j].w;
          const u32x4 av = q4_expand(wd, fmt);
#pragma unroll
          for (int q = 0; q < NXP; ++q)
            part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bq[q]), part[j], 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < NXP; ++q)
          sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, bq[q]), sx, 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < NR; ++j) a4[st][j] = wq[j][(size_t)(2 * (g0 + gn) + st) * 64];
      __builtin_amdgcn_sched_barrier(0);
    }
    if (APART && __any(sx[0] != sx[0]))
      sx[0] = q4_row_sums<8 * NXP>(ones, lane, [&](int i, bool on) {
        const u32x4 v = xs[((size_t)(i % NXP) * kt + 8 * g + i / NXP) * 64 + lane], none = {0u, 0u, 0u, 0u};
        return on ? v : none;
      });
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const uint32_t sw[8] = {sraw[j][0].x, sraw[j][0].y, sraw[j][0].z, sraw[j][0].w, sraw[j][1].x, sraw[j][1].y, sraw[j][1].z, sraw[j][1].w};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float sv = __builtin_bit_cast(float, (r & 1) ? (sw[r >> 1] & 0xFFFF0000u) : (sw[r >> 1] << 16));
        acc[j][r] += sv * (part[j][r] - fmt.offset * sx[0]);
      }
    }
  }
  return acc[0][0] != acc[0][0];                               // (a sum of NaN in any group stays in every result of its row)
}
template <int NXP, int RW, int NR>
__device__ __forceinline__ void k2_stream_q4_dispatch(int nr, const Q4Format fmt, const u32x4* xs, int kt, int g0, int gb, int ge, const u32x4* const* wq,
                                                      const u32x4* const* sq, f32x16* acc, int lane) {
  if (nr == NR) {
    if (!__any(k2_stream_q4<NXP, NR, false>(fmt, xs, kt, g0, gb, ge, wq, sq, acc, lane))) return;
#pragma unroll
    for (int j = 0; j < NR; ++j) acc[j] = f32x16{};
    k2_stream_q4<NXP, NR, true>(fmt, xs, kt, g0, gb, ge, wq, sq, acc, lane);
  } else if constexpr (NR > 1) k2_stream_q4_dispatch<NXP, RW, NR - 1>(nr, fmt, xs, kt, g0, gb, ge, wq, sq, acc, lane);
}

template <int NWP, int NXP, int RW, int NR, int DEPTH>
__device__ __forceinline__ void k2_prologue_dispatch(int nr, int kb, int ke, const u32x4* const* wp, size_t wps, u32x4* pre) {
  if (nr == NR) k2_prologue<NWP, NR, (DEPTH * RW) / NR>(kb, ke, wp, wps, pre);
  else if constexpr (NR > 1) k2_prologue_dispatch<NWP, NXP, RW, NR - 1, DEPTH>(nr, kb, ke, wp, wps, pre);
}
template <int NWP, int NXP, int RW, int NR, int DEPTH>
__device__ __forceinline__ void k2_stream_dispatch(int nr, const u32x4* xs, int kt, int kb, int ke, const u32x4* const* wp,
                                                   size_t wps, f32x16* acc, int lane, u32x4* pre) {
  if (nr == NR) k2_stream<NWP, NXP, NR, (DEPTH * RW) / NR>(xs, kt, kb, ke, wp, wps, acc, lane, pre);
  else if constexpr (NR > 1) k2_stream_dispatch<NWP, NXP, RW, NR - 1, DEPTH>(nr, xs, kt, kb, ke, wp, wps, acc, lane, pre);
}

template <int NWP, int NXP, int RW, int DEPTH, bool Q4 = false>
__global__ __launch_bounds__(V2_THREADS) void k2_gemm(Gemm2 g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float sh_small[16 * 33];
  __shared__ int s_last;
  pin_args(g);
  EarlyLoads el;                                                // used by the epilogue, much later
  early_issue(g.in_scale.ssq, g.facts, el);
  if (g.skip_flag && *g.skip_flag == 0) return;               // uniform over the whole grid
  u32x4* xs = (u32x4*)smem;
  const int lane = threadIdx.x & 63, w = wave_id();
  // the work split in 32-bit arithmetic: every product stays far below 2^31 (<= 1024 groups x a few thousand row blocks)
  const unsigned uS = g.S, ugroups = g.groups, uNRB = g.NRB, uKS = g.KS, ulanes = g.lanes, ukparts = g.kparts;
  const int s = blockIdx.x % uS, grp = blockIdx.x / uS;
  const int rb0 = (unsigned)grp * uNRB / ugroups, rb1 = (unsigned)(grp + 1) * uNRB / ugroups;
  // K slice of the work-group and K part of the wave: in k-steps, or (4-bit weights) in whole groups of 8 k-steps
  const int gs0 = Q4 ? (int)((unsigned)s * (unsigned)g.NG / uS) : 0, gs1 = Q4 ? (int)((unsigned)(s + 1) * (unsigned)g.NG / uS) : 0;
  const int ks0 = Q4 ? 8 * gs0 : (int)((unsigned)s * uKS / uS), ks1 = Q4 ? 8 * gs1 : (int)((unsigned)(s + 1) * uKS / uS), kt = ks1 - ks0;
  const int la = (unsigned)w % ulanes, kb_i = (unsigned)w / ulanes;
  const int qgb = (unsigned)kb_i * (unsigned)(gs1 - gs0) / ukparts, qge = (unsigned)(kb_i + 1) * (unsigned)(gs1 - gs0) / ukparts;
  const int kb = Q4 ? 8 * qgb : (int)((unsigned)kb_i * (unsigned)kt / ukparts), ke = Q4 ? 8 * qge : (int)((unsigned)(kb_i + 1) * (unsigned)kt / ukparts);
  unsigned long long* tr = TRACE_PTR((g.trace && threadIdx.x == 0) ? g.trace + (size_t)blockIdx.x * 8 : nullptr);
  TRACE_STAMP(tr, 0);
  int nr = 0;
  for (int j = 0; j < RW; ++j) nr += (rb0 + la + j * g.lanes < rb1) ? 1 : 0;
  nr = __builtin_amdgcn_readfirstlane(nr);

  const u32x4* wp[RW];
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    int rb = rb0 + la + j * g.lanes;
    if (rb >= rb1) rb = rb0;                                  // never dereferenced: only the first nr entries are used
    wp[j] = (const u32x4*)(g.W + ((size_t)rb * g.KS + ks0) * 512) + lane;
  }
  // the first weight tiles are requested before anything else (a wave with fewer row blocks keeps more k-steps in flight)
  u32x4 pre[DEPTH * RW * NWP];
  if constexpr (!Q4) k2_prologue_dispatch<NWP, NXP, RW, RW, DEPTH>(nr, kb, ke, wp, g.wps, pre);

  // stage this work-group's K slice of X: per plane a contiguous run of kt tiles (8 loads in flight per thread).  4-bit weights: rows beyond
  // the pass are staged as zeros, since what an earlier pass left there, a NaN say, would send the waves over their groups again (k2_stream_q4).
  const bool live = !Q4 || (int)(threadIdx.x & 31) < g.M;     // every element that a thread moves is of one row
  for (int p = 0; p < NXP; ++p) {
    const u32x4* src = (const u32x4*)(g.XF + ((size_t)p * g.KS + ks0) * 512);
    u32x4* dst = xs + (size_t)p * kt * 64;
    const int n = kt * 64;
    for (int i0 = 0; i0 < n; i0 += V2_THREADS * 8) {
      u32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = u32x4{0u, 0u, 0u, 0u};
      if (live) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[min(i0 + u * V2_THREADS + (int)threadIdx.x, n - 1)];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u * V2_THREADS + (int)threadIdx.x;
        if (i < n) dst[i] = v[u];
      }
    }
  }
  f32x16 acc[RW];
#pragma unroll
  for (int j = 0; j < RW; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  __syncthreads();
  TRACE_STAMP(tr, 1);
  if constexpr (Q4) {
    const u32x4* wq[RW];
    const u32x4* sq[RW];
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      int rb = rb0 + la + j * g.lanes;
      if (rb >= rb1) rb = rb0;
      wq[j] = (const u32x4*)g.W + (size_t)rb * (size_t)(g.KS / 4) * 64 + lane;
      sq[j] = (const u32x4*)g.SC + (size_t)rb * (size_t)g.NG * 4 + 2 * (lane >> 5);
    }
    k2_stream_q4_dispatch<NXP, RW, RW>(nr, g.q4, xs, kt, gs0, qgb, qge, wq, sq, acc, lane);
  } else
  k2_stream_dispatch<NWP, NXP, RW, RW, DEPTH>(nr, xs, kt, kb, ke, wp, g.wps, acc, lane, pre);
  TRACE_STAMP(tr, 2);
  // waves that split K inside the work-group: sum through LDS in k-part order
  if (g.kparts > 1) {
    __syncthreads();                                          // the X slice is no longer needed
    float* red = (float*)smem;
    if (kb_i > 0) {
#pragma unroll
      for (int j = 0; j < RW; ++j)
        if (j < nr)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            red[((((size_t)la * (g.kparts - 1) + (kb_i - 1)) * RW + j) * 16 + r) * 64 + lane] = acc[j][r];
    }
    __syncthreads();
    if (kb_i == 0) {
      for (int b = 1; b < g.kparts; ++b)
#pragma unroll
        for (int j = 0; j < RW; ++j)
          if (j < nr)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              acc[j][r] += red[((((size_t)la * (g.kparts - 1) + (b - 1)) * RW + j) * 16 + r) * 64 + lane];
    }
  }
  if (kb_i == 0) {
#pragma unroll
    for (int j = 0; j < RW; ++j)
      if (j < nr) {
        const int rb = rb0 + la + j * g.lanes;
#pragma unroll
        for (int i = 0; i < 4; ++i) {                           // accumulator registers 4i..4i+3 = rows 8i + 4(lane/32) + 0..3
          f32x4 v; v.x = acc[j][4 * i]; v.y = acc[j][4 * i + 1]; v.z = acc[j][4 * i + 2]; v.w = acc[j][4 * i + 3];
          coh_store16(g.PT, pt_quad_bytes(s, g.Npad, rb * 32 + 8 * i + 4 * (lane >> 5), lane & 31), v);
        }
      }
  }
  // publish the partials; the last work-group of this row group to arrive finishes the job
  publish_wait();                                               // every coherent store above has been acknowledged
  __syncthreads();
  if (threadIdx.x == 0) {
    int old = __hip_atomic_fetch_add(g.counters + grp * COUNTER_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (old == g.S - 1);
    if (s_last) __hip_atomic_store(g.counters + grp * COUNTER_STRIDE, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
  }
  __syncthreads();
  TRACE_STAMP(tr, 3);
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const int n0 = rb0 * 32, n1 = min(rb1 * 32, g.N);
  if (n1 <= n0) return;
  __shared__ float rstd_s[32];
  if (g.epi != EPI_RESID) block_rstd_finish(g.in_scale, early_ssq(g.in_scale, el), rstd_s, sh_small);
  switch (g.epi) {
    case EPI_QKV: epilogue_qkv<NXP>(g, n0, n1, rstd_s, el); break;
    case EPI_RESID: epilogue_resid<NXP>(g, grp, n0, n1, sh_small); break;
    case EPI_SWIGLU: epilogue_swiglu<NXP>(g, n0, n1, rstd_s); break;
    default: epilogue_logits(g, n0, n1, rstd_s, el); break;
  }
  TRACE_STAMP(tr, 4);
}

// ---- full-K variant for wide matrices (QKV, gate/up, LM head) and small ones ----------------------------------------------------------
// A work-group owns up to 4 whole row blocks over ALL of K: no partial sums leave the chip, no arrival counter, no
// last work-group.  The eight waves split K eight ways; a wave streams, per k-step, the weight tiles of the group's
// row blocks from HBM AND the activation fragments of that k-step straight from L2 (every work-group reads the whole
// X, 512 KB at d = 4096, which the 32 work-groups of an XCD share through its L2) -- no LDS staging, no barrier until
// the end.  The waves' sums meet in LDS (k-part order) and the epilogue runs on them in place.  Costs more bytes per
// CU than the split-K kernel and saves its publish / arrive / read-back round trips; pays off for matrices with at
// least as many row blocks as there are CUs, and for those whose K is short (plan_is_whole_k; one row block a work-group).
// The activation fragments come through buffer loads: a lane whose row (lane % 32) is not a live row of the pass gets
// an offset beyond the buffer, which the hardware answers with zeros WITHOUT touching memory -- a pass of M rows moves
// M/32 of the fragment bytes (26/32 in a 26-node verify, 1/8 and less in the head's passes).
// The weights come through buffer loads as well: a resource per plane over the work-group's row blocks, tile (j, k) at (j * KS + k) KiB,
// vo[j] the lane's byte offset inside a tile of block j -- out of range for lanes whose weight row is not this work-group's (half
// blocks).
template <int NWP>
struct FkWeights { __amdgpu_buffer_rsrc_t rs[NWP]; uint32_t vo[4]; };
template <int NWP>
__device__ __forceinline__ FkWeights<NWP> fk_weights(const bf16_t* W, size_t wps, int rb0, int nr, int KS, int lane, int row_lo = 0, int row_hi = 32) {
  FkWeights<NWP> f;
#pragma unroll
  for (int p = 0; p < NWP; ++p) f.rs[p] = __builtin_amdgcn_make_buffer_rsrc((void*)(W + p * wps + (size_t)rb0 * KS * 512), 0, nr * KS * 1024, 0x00020000);
  const int row = lane & 31;
#pragma unroll
  for (int j = 0; j < 4; ++j) f.vo[j] = j < nr && row >= (j == 0 ? row_lo : 0) && row < (j == nr - 1 ? row_hi : 32) ? (uint32_t)lane * 16u : OUT_OF_RANGE;
  return f;
}

// Zero sums, made here and not in front of the first requests.
template <int NR>
__device__ __forceinline__ void fk_zero(f32x16* acc) {
  float zero = 0.f;
  asm volatile("" : "+v"(zero));
#pragma unroll
  for (int j = 0; j < NR; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = zero;
}
// behind(): what else the kernel requests, behind the stream's first requests.
template <int NWP, int NXP, int NR, int DEPTH, class F>
__device__ __forceinline__ void fk_stream(const bf16_t* __restrict__ XF, int KS, bool row, int kb, int ke, const FkWeights<NWP>& fw, f32x16* acc, int lane, F&& behind) {
  constexpr int PMAX = NWP > NXP ? NWP : NXP;
  const int klast = max(ke - 1, kb);                            // (a wave without a k-step requests one that it does not use)
  u32x4 ta[DEPTH][NR][NWP], tb[DEPTH][NXP];
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)XF, 0, NXP * KS * 1024, 0x00020000);
  const uint32_t xlane = row ? (uint32_t)lane * 16u : OUT_OF_RANGE;   // row: this lane's activation row is wanted
  // Weights non-temporal: a weight byte is used once per pass and a pass's weights exceed every cache, so keeping them out leaves the L2s
  // to the activations (7B, LLaMA shapes, us before / after: gate/up 36.5 / 34.5, LM head 49.0 / 45.0, QKV 25.4 / 23.9; a bare
  // read of 2 GB runs at 6.9 TB/s with the hint and 6.25 without).  The 4-bit and fp32 streams keep plain loads: their head fits
  // the 256 MB memory-side cache, from which the drafting passes then re-read it (4-bit LM head 32.7 us plain, 35.6 with the hint).
  auto load = [&](int dd, int k) {
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int p = 0; p < NWP; ++p)
        ta[dd][j][p] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(fw.rs[p], fw.vo[j], (uint32_t)(j * KS + k) * 1024u, NWP == 1 ? 2 : 0));
#pragma unroll
    for (int q = 0; q < NXP; ++q)
      tb[dd][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrs, xlane, (uint32_t)(q * KS + k) * 1024u, 0));
  };
  auto mul = [&](int dd) {
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int p = 0; p < NWP; ++p)
#pragma unroll
        for (int q = 0; q < NXP; ++q)
          if (p + q < PMAX)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ta[dd][j][p]), __builtin_bit_cast(bf16x8, tb[dd][q]), acc[j], 0, 0, 0);
  };
#pragma unroll
  for (int dd = 0; dd < DEPTH; ++dd) load(dd, min(kb + dd, klast));
  __builtin_amdgcn_sched_barrier(0);
  behind();
  fk_zero<NR>(acc);
  int k = kb;
  // A round that has all of the next one to request; then the rounds that do not.  (With the k-steps behind the end clamped to the
  // last one, a wave's 32 came as 35 or 36 at K = 4096 and O's 8 as 12, on the L2 -> CU path that binds these kernels; requested out
  // of range they move nothing and still cost more than a branch.  26 rows at 7B, us clamped / out of range / branch: QKV 25.3 /
  // 25.9 / 24.7, gate/up 35.4 / 36.0 / 34.7, O 13.6 / 13.3 / 12.5, down 24.0 / 23.5 / 23.5.  Four row blocks, whose depth divides
  // the usual K: LM head 44.8 / 45.9 / 45.5, so they keep one loop.  A wave with fewer k-steps than DEPTH still fills its
  // ring with the last one above, but for one row block and at most half of the ring: fk_stream_dispatch.)
  constexpr bool EXACT = NR < 4;
  for (; k + (EXACT ? 2 * DEPTH - 1 : DEPTH) < ke; k += DEPTH) {
#pragma unroll
    for (int dd = 0; dd < DEPTH; ++dd) {
      mul(dd);
      load(dd, EXACT ? k + dd + DEPTH : min(k + dd + DEPTH, ke - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (EXACT && k + DEPTH < ke) {
#pragma unroll
    for (int dd = 0; dd < DEPTH; ++dd) {
      mul(dd);
      if (k + dd + DEPTH < ke) load(dd, k + dd + DEPTH);
      __builtin_amdgcn_sched_barrier(0);
    }
    k += DEPTH;
  }
#pragma unroll
  for (int dd = 0; dd < DEPTH; ++dd)
    if (k + dd < ke) mul(dd);
}
template <int NWP, int NXP, int NR, class F>
__device__ __forceinline__ void fk_stream_dispatch(int nr, const bf16_t* XF, int KS, bool row, int kb, int ke, const FkWeights<NWP>& fw, f32x16* acc, int lane, F&& behind) {
  constexpr int DEPTH = NWP == 1 ? (NR == 1 ? 8 : NR == 2 ? 6 : NR == 3 ? 5 : 4) : NR == 1 ? 4 : 2;   // ~24 KiB in flight per wave; deeper measured the same
  if (nr == NR) {
    // (small matrices: a ring of no more k-steps than the wave has.  Clamped to the last one, a launch at d 256 in fp32 fetched every tile twice: tiny request
    // 5.82 -> 5.37 ms)
    if constexpr (NR == 1)
      if (ke - kb <= DEPTH / 2) return fk_stream<NWP, NXP, NR, DEPTH / 2>(XF, KS, row, kb, ke, fw, acc, lane, behind);
    fk_stream<NWP, NXP, NR, DEPTH>(XF, KS, row, kb, ke, fw, acc, lane, behind);
  } else if constexpr (NR > 1) fk_stream_dispatch<NWP, NXP, NR - 1>(nr, XF, KS, row, kb, ke, fw, acc, lane, behind);
  else behind();                                               // (no row block: nothing to multiply)
}

// ---- the same stream over 4-bit weights (see k_pack_weight_q4 for the layout) -------------------------------------------
// A wave owns the groups [gb, ge) of 128 k.  Per group: two 16-byte loads per row block bring the codes of its 8 k-steps;
// a k-step's A operand is 16 + code (128 + code in the unrotated format) (exact in bf16) -- two ALU operations per pair of codes, which run beside the MFMAs
// -- so the group's partial sums come out as sum_k x_k (16 + c_k); a smaller MFMA (q4_ones) gives sum_k x_k of
// the same k-steps, and the group is folded into the result as  acc += s_row * (partial - 24 * sum_x)  in fp32.
// Activation fragments are streamed from L2 as in fk_stream, one group (8 k-steps) ahead; the next group's codes are
// requested as soon as a super-tile's registers are free.
// PIN: q4_pin.  (Not for QKV with three row blocks, which has no register left for it: four spilled.)
template <int NXP, int NR, bool APART, bool PIN, class F>
__device__ __forceinline__ bool fk_stream_q4(const Q4Format format, const bf16_t* __restrict__ XF, int KS, int M, int gb, int ge, __amdgpu_buffer_rsrc_t wrs /*codes from block 0 on*/,
                                             const u32x4* const* sq /*scales of (block j, group 0), this lane's half*/, int NG,
                                             f32x16* acc, int lane, F&& behind) {
  if (ge <= gb) {
    behind();
#pragma unroll
    for (int j = 0; j < NR; ++j) acc[j] = f32x16{};
    return false;
  }
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)XF, 0, q4_x_span(NXP, KS) * 1024, 0x00020000);
  const uint32_t xlane = (lane & 31) < M ? (uint32_t)lane * 16u : OUT_OF_RANGE;   // dead rows: zeros
#define Q4_XLOAD(q, kk, past) __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrs, xlane | (past), (uint32_t)(((q) * KS + (kk)) * 1024), 0))
#define Q4_WLOAD(j, T, past) __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wrs, (uint32_t)lane * 16u | (past), (uint32_t)((j) * (KS / 4) + (T)) * 1024u, 0))
  u32x4 a4[2][NR], tb[8][NXP];                                 // codes of a group; activation fragments one group ahead
  const u32x4 ones = q4_ones(lane);
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int j = 0; j < NR; ++j) a4[st][j] = Q4_WLOAD(j, 2 * gb + st, 0u);
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < NXP; ++q) tb[i][q] = Q4_XLOAD(q, 8 * gb + i, 0u);
  __builtin_amdgcn_sched_barrier(0);
  behind();
  const Q4Format fmt = PIN ? q4_pin(format) : format;
  fk_zero<NR>(acc);
  // The last group, a copy of the loop's body, requests nothing: clamped to itself it fetched its activations and codes twice, one
  // group in four at K = 4096 and the only one in O's slices.  (Three row blocks, for which a second body spills, request out of range.)
  constexpr bool COPY = NR < 3;
#pragma unroll
  for (int last = COPY ? 0 : 1; last < 2; ++last)
  for (int g = COPY && last ? ge - 1 : gb; g < (last ? ge : ge - 1); ++g) {
    const uint32_t past = COPY || g + 1 < ge ? 0u : OUT_OF_RANGE;
    f32x16 part[NR];
    f32x4 sx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[j][r] = 0.f;
    u32x4 sraw[NR][2];                                          // this group's scales: needed after its 8 k-steps
#pragma unroll
    for (int j = 0; j < NR; ++j) { sraw[j][0] = sq[j][(size_t)g * 4]; sraw[j][1] = sq[j][(size_t)g * 4 + 1]; }
    const int gn = g + 1;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int kk = 8 * g + 4 * st + ks;
        auto expand = [&](int j) {
          const uint32_t wd = ks == 0 ? a4[st][j].x : ks == 1 ? a4[st][j].y : ks == 2 ? a4[st][j].z : a4[st][j].w;
          return q4_expand(wd, fmt);
        };
        if constexpr (NR <= 2) {
          // plane by plane, so that consecutive MFMAs write different accumulators (measured: QKV 20.4 -> 19.3 us, down
          // 19.0 -> 17.8 us); with three row blocks the expanded operands held across the planes spill, so they keep the
          // block-by-block order
          u32x4 av[NR];
#pragma unroll
          for (int j = 0; j < NR; ++j) av[j] = expand(j);
#pragma unroll
          for (int q = 0; q < NXP; ++q) {
#pragma unroll
            for (int j = 0; j < NR; ++j)
              part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[j]), __builtin_bit_cast(bf16x8, tb[4 * st + ks][q]), part[j], 0, 0, 0);
            sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, tb[4 * st + ks][q]), sx, 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int j = 0; j < NR; ++j) {
            const u32x4 av = expand(j);
#pragma unroll
            for (int q = 0; q < NXP; ++q)
              part[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, tb[4 * st + ks][q]), part[j], 0, 0, 0);
          }
#pragma unroll
          for (int q = 0; q < NXP; ++q)
            sx = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, tb[4 * st + ks][q]), sx, 0, 0, 0);
        }
        // use a slot, refill that slot: the same k-step of the next group
        (void)kk;
#pragma unroll
        for (int q = 0; q < NXP; ++q) if (!(COPY && last)) tb[4 * st + ks][q] = Q4_XLOAD(q, 8 * gn + 4 * st + ks, past);
      }
      // the super-tile's code registers are free: request the next group's
#pragma unroll
      for (int j = 0; j < NR; ++j) if (!(COPY && last)) a4[st][j] = Q4_WLOAD(j, 2 * gn + st, past);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (APART && __any(sx[0] != sx[0]))
      sx[0] = q4_row_sums<8 * NXP>(ones, lane, [&](int i, bool on) { return Q4_XLOAD(i % NXP, 8 * g + i / NXP, on ? 0u : OUT_OF_RANGE); });
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const uint32_t sw[8] = {sraw[j][0].x, sraw[j][0].y, sraw[j][0].z, sraw[j][0].w, sraw[j][1].x, sraw[j][1].y, sraw[j][1].z, sraw[j][1].w};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float sv = __builtin_bit_cast(float, (r & 1) ? (sw[r >> 1] & 0xFFFF0000u) : (sw[r >> 1] << 16));
        acc[j][r] += sv * (part[j][r] - fmt.offset * sx[0]);
      }
    }
  }
#undef Q4_XLOAD
#undef Q4_WLOAD
  return acc[0][0] != acc[0][0];                               // (a sum of NaN in any group stays in every result of its row)
}
template <int NXP, int NR, bool PIN = true, class F>
__device__ __forceinline__ void fk_stream_q4_dispatch(int nr, const Q4Format fmt, const bf16_t* XF, int KS, int M, int gb, int ge, __amdgpu_buffer_rsrc_t wrs,
                                                      const u32x4* const* sq, int NG, f32x16* acc, int lane, F&& behind) {
  if (nr == NR) {
    if (!__any(fk_stream_q4<NXP, NR, false, PIN>(fmt, XF, KS, M, gb, ge, wrs, sq, NG, acc, lane, behind))) return;
    fk_stream_q4<NXP, NR, true, PIN>(fmt, XF, KS, M, gb, ge, wrs, sq, NG, acc, lane, [] {});
  } else if constexpr (NR > 1) fk_stream_q4_dispatch<NXP, NR - 1, PIN>(nr, fmt, XF, KS, M, gb, ge, wrs, sq, NG, acc, lane, behind);
  else behind();
}
// The codes of nr row blocks from rb0 on.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t q4_codes(const bf16_t* W, int rb0, int nr, int KS) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)W + (size_t)rb0 * KS * 256), 0, q4_w_span(nr, KS) * 1024, 0x00020000);
}

// The waves' accumulators parked in LDS as red[w][j][i][lane], 16 bytes each = registers 4i..4i+3 (MFMA layout: rows 8i + 4*(lane/32)
// + 0..3 of row block j, token lane%32).  Sum over the waves, in order, of the four rows 4*qd.. of block j, token m.
__device__ __forceinline__ void fk_park(float* red, int nrmax, int w, int j, int lane, const f32x16& acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f32x4 v; v.x = acc[4 * i]; v.y = acc[4 * i + 1]; v.z = acc[4 * i + 2]; v.w = acc[4 * i + 3];
    *(f32x4*)(red + ((((size_t)w * nrmax + j) * 4 + i) * 64 + lane) * 4) = v;
  }
}
template <int NW = 8>
__device__ __forceinline__ f32x4 fk_sum4(const float* red, int nrmax, int j, int qd, int m) {
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) a += *(const f32x4*)(red + ((((size_t)w * nrmax + j) * 4 + (qd >> 1)) * 64 + m + 32 * (qd & 1)) * 4);
  return a;
}
// HALF: the unit of the work split is half a row block (16 weight rows) instead of a whole one, for matrices whose
// row blocks do not divide evenly over the CUs (QKV at d = 4096: 384 blocks over 256 CUs = 1 or 2 each, but 3 halves
// each).  A work-group then owns a run of halves; of a block it shares with a neighbour it loads and finishes only its own
// 16 rows (the other lanes of the tile load nothing and multiply zeros).  Rotate-half pairs are adjacent rows, so a half
// holds whole pairs.  Epilogue: QKV.
// What a decoding step spends beside its streams is instructions on one chain, from a work-group's entry to its first request and from its
// last tile to its last store (a wave issues one in four to eight cycles): so the arguments come in one fetch, the shares without a
// division, everything else behind the first requests, what the epilogue reads on its way before the sums, and the epilogue is a template
// argument.  7B, us a launch before / after, here and in k2_gemm_xk: 26 rows, QKV 23.0 / 21.8, gate/up 32.9 / 32.5, O 11.4 / 10.7, down 23.0 /
// 22.3; the head's passes of a few rows, QKV 18.6 / 17.9, gate/up 32.0 / 31.1, O 10.2 / 9.3, down 19.9 / 19.3, fc 17.3 / 16.2.
template <int EPI, int NWP, int NXP, int NRMAX, bool HALF = false, bool Q4 = false, bool EXPERTS = false>
__global__ __launch_bounds__(V2_THREADS) void k2_gemm_fk(Gemm2 g) {
  static_assert(!Q4 || (!HALF && NWP == 1), "4-bit weights: whole row blocks, one plane");
  static_assert((!HALF || EPI == EPI_QKV) && (!EXPERTS || EPI == EPI_SWIGLU) && (EPI != EPI_RESID || NRMAX <= 2), "forms that exist");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float sh_small[16 * 32];
  float* red = (float*)smem;                                    // [8][NRMAX][16][64]
  pin_args(g);
  if (g.skip_flag && g.skip_flag[EXPERTS ? blockIdx.y : 0] == 0) return;   // MoE: no row selected this expert (uniform over its work-groups)
  const bf16_t* W = g.W;
  if constexpr (EXPERTS) W += blockIdx.y * g.w_stride;
  const int lane = threadIdx.x & 63, w = wave_id();
  bool row = (lane & 31) < g.M;                                 // dead rows (and, here, rows that did not select the expert) are not fetched
  if constexpr (EXPERTS) row = row && g.row_w[(size_t)blockIdx.y * g.row_w_stride + (lane & 31)] != 0.f;
  unsigned long long* tr = TRACE_PTR((g.trace && threadIdx.x == 0) ? g.trace + (size_t)blockIdx.x * 8 : nullptr);
  TRACE_STAMP(tr, 0);
  const uint32_t U = HALF ? 2u * (uint32_t)g.NRB : (uint32_t)g.NRB;
  const uint32_t u0 = share_begin(blockIdx.x, U, g.share_a, g.share_b), u1 = share_begin(blockIdx.x + 1, U, g.share_a, g.share_b);
  const int rb0 = HALF ? u0 >> 1 : u0, rb1 = HALF ? (u1 + 1) >> 1 : u1;
  const int row_lo = HALF && (u0 & 1) ? 16 : 0, row_hi = HALF && (u1 & 1) ? 16 : 32;   // rows [row_lo, 32) of the first block, [0, row_hi) of the last
  const int nr = rb1 - rb0;                                     // <= NRMAX (host)
  EarlyLoads el;                                                // used by the epilogue, much later
  constexpr bool LATE = Q4 && NRMAX == 3;                       // no registers to hold them through the 4-bit stream (12 to 15 spilled)
  Gemm2 e;                                                      // the arguments as the epilogue reads them
  auto early = [&] {
    e = late_args();
    if constexpr (!LATE) early_issue(g.in_scale.ssq, g.facts, el);
  };
  f32x16 acc[NRMAX];
  if constexpr (Q4) {
    // K is split over the waves by groups of 128; pointers to the codes / scales of each row block
    const int gb = (unsigned)w * (unsigned)g.NG / 8u, ge = (unsigned)(w + 1) * (unsigned)g.NG / 8u;
    const u32x4* sq[NRMAX];
#pragma unroll
    for (int j = 0; j < NRMAX; ++j) sq[j] = (const u32x4*)g.SC + (size_t)min(rb0 + j, g.NRB - 1) * (size_t)g.NG * 4 + 2 * (lane >> 5);
    fk_stream_q4_dispatch<NXP, NRMAX, !(NRMAX == 3 && EPI == EPI_QKV)>(nr, g.q4, g.XF, g.KS, g.M, gb, ge, q4_codes(W, rb0, nr, g.KS), sq, g.NG, acc, lane, early);
    if constexpr (LATE) early_issue(e.in_scale.ssq, e.facts, el);
  } else {
    const int kb = (unsigned)w * (unsigned)g.KS / 8u, ke = (unsigned)(w + 1) * (unsigned)g.KS / 8u;
    fk_stream_dispatch<NWP, NXP, NRMAX>(nr, g.XF, g.KS, row, kb, ke, fk_weights<NWP>(W, g.wps, rb0, nr, g.KS, lane, row_lo, row_hi), acc, lane, early);
  }
  TRACE_STAMP_AFTER(tr, 2, acc[0][0]);
  if constexpr (EXPERTS) e.xf_out += blockIdx.y * e.out_stride;
  const int m = threadIdx.x & 31, slot = threadIdx.x >> 5;     // 16 slots of 32 tokens
  const bool live = m < e.M;
  // what the first item of a thread needs from memory is requested before the sums
  f32x4 rh = {0.f, 0.f, 0.f, 0.f}, rbias = rh, rgain = rh;     // residual epilogue: what an item adds and multiplies
  auto load_resid = [&](int n) {
    if (e.h_in && live) rh = *(const f32x4*)(e.h_in + (size_t)m * e.d + n);
    if (e.bias) rbias = *(const f32x4*)(e.bias + n);
    if (e.gain_next) rgain = *(const f32x4*)(e.gain_next + n);
  };
  const int dh_shift = 31 - __builtin_clz(e.kv.head_dim), half = e.kv.head_dim >> 1;   // QKV (32, 64 or 128 dimensions)
  float2 rcs = {0.f, 0.f}, rsn = {0.f, 0.f};                    // ... the angles of an item's two pairs
  auto load_angles = [&](int n) {
    if (!live) return;                                          // (no position of its own)
    const size_t at = (size_t)el.pos * half + ((n & (2 * half - 1)) >> 1);
    rcs = *(const float2*)(e.rope_cos + at); rsn = *(const float2*)(e.rope_sin + at);
  };
  const int first = (rb0 + (slot >> 3)) * 32 + 4 * (slot & 7);
  if (EPI == EPI_RESID && (slot >> 3) < nr && first < e.N) load_resid(first);
  if (EPI == EPI_QKV && (slot >> 3) < nr && first < e.N) load_angles(first);
  // park every wave's sums in LDS
#pragma unroll
  for (int j = 0; j < NRMAX; ++j)
    if (j < nr) fk_park(red, NRMAX, w, j, lane, acc[j]);
  if constexpr (EPI != EPI_RESID) block_rstd_park(e.in_scale, early_ssq(e.in_scale, el), sh_small);
  __syncthreads();
  const float rs = EPI != EPI_RESID && live ? block_rstd(e.in_scale, sh_small, m) : 0.f;
  if constexpr (EPI == EPI_SWIGLU) {
    // item = (row block j, quarter qt): outputs f = rb*16 + 4*qt .. +3 from gate rows 4*qt.. and up rows 16 + 4*qt..
    for (int it = slot; it < nr * 4; it += 16) {
      const int j = it >> 2, qt = it & 3;
      const f32x4 gq = fk_sum4(red, NRMAX, j, qt, m), uq = fk_sum4(red, NRMAX, j, 4 + qt, m);
      f32x4 x;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float gg = gq[t] * rs, uu = uq[t] * rs;
        x[t] = gg / (1.0f + __expf(-gg)) * uu;
      }
      if (live) xf_store4(e.xf_out, m, (rb0 + j) * 16 + 4 * qt, 1, e.xf_KS, NXP, x);
    }
  } else if constexpr (EPI == EPI_QKV) {
    const int KVH = e.kv.n_kv_heads, H = e.H;
    // item = (row block j, quad qd of 8): rows 4qd.. of the block, two rotate-half pairs
    for (int it = slot; it < nr * 8; it += 16) {
      const int j = it >> 3, qd = it & 7;
      if (HALF && (4 * qd < (j == 0 ? row_lo : 0) || 4 * qd >= (j == nr - 1 ? row_hi : 32))) continue;   // the neighbour's rows
      const int n = (rb0 + j) * 32 + 4 * qd;
      if (n >= e.N) continue;                                   // (N is a multiple of 32)
      if (it != slot) load_angles(n);
      const f32x4 sum = fk_sum4(red, NRMAX, j, qd, m);
      if (!live) continue;
      qkv_store(e, n, m, dh_shift, sum, rs, rcs, rsn, el.kv_row, H, KVH);
    }
  } else if constexpr (EPI == EPI_RESID) {
    // h_out = h_in + (routing weight *) W x + bias; per-token partial sums of squares for the consumer's RMSNorm; x * gain of the
    // next norm as GEMM input.  item = (row block j, quad of 4 rows), the residual, bias and gain of the first on their way already
    const float rw = e.row_w ? e.row_w[m] : 1.0f;
    float ss = 0.f;
    for (int it = slot; it < nr * 8; it += 16) {
      const int j = it >> 3, qd = it & 7;
      const int n = (rb0 + j) * 32 + 4 * qd;
      if (n >= e.N) continue;                                   // (N is a multiple of 64)
      if (it != slot) load_resid(n);
      f32x4 v = fk_sum4(red, NRMAX, j, qd, m);
      if (e.row_w) v *= rw;
      if (e.bias) v += rbias;
      if (e.h_in && live) v += rh;
      if (live) *(f32x4*)(e.h_out + (size_t)m * e.d + n) = v;
#pragma unroll
      for (int t = 0; t < 4; ++t) ss = fmaf(v[t], v[t], ss);
      if (live) xf_store4(e.xf_out, m, n, 1, e.xf_KS, NXP, e.gain_next ? v * rgain : v);
    }
    if (e.ssq_out) {                                            // (uniform)
      sh_small[slot * 32 + m] = ss;
      __syncthreads();
      if (threadIdx.x < 32) {
        float a = 0.f;
        for (int i = 0; i < 16; ++i) a += sh_small[i * 32 + threadIdx.x];
        e.ssq_out[blockIdx.x * 32 + threadIdx.x] = a;
      }
    }
  } else {                                                      // EPI_LOGITS
    const int nend = min(e.N, e.V);
    const bool vec = (e.V & 3) == 0;
    const long dst = live && el.out_row >= 0 ? (long)el.out_row * e.V : -1;
    for (int it = slot; it < nr * 8; it += 16) {                // item = (row block j, quad of 4 rows)
      const int j = it >> 3, qd = it & 7;
      const int n = (rb0 + j) * 32 + 4 * qd;
      if (dst < 0 || n >= nend) continue;
      const f32x4 v = fk_sum4(red, NRMAX, j, qd, m) * rs;
      if (vec && n + 4 <= nend) *(f32x4*)(e.logits + dst + n) = v;
      else {
#pragma unroll
        for (int t = 0; t < 4; ++t) if (n + t < nend) e.logits[dst + n + t] = v[t];
      }
    }
  }
  TRACE_STAMP(tr, 4);
}

// ---- whole-K LM head over 4-bit weights -----------------------------------------------------------------------------------------
// Up to four row blocks a work-group, their sums scaled into logits in place: more than three blocks do not fit k2_gemm_fk's waves, so the
// LM head ran split over K with the activations in LDS (k2_gemm), and every K slice wrote and read back its sums of the whole vocabulary.
// Here wave w takes blocks 2 (w % 2) and on over K part w / 2, two waves a SIMD; the two waves of a part ask for the same activations one
// after the other.  us a launch, k2_gemm / here, 32000 tokens, 26 rows and 1 to 4: 4096 columns 32 / 24.1 and 26.6 / 18.2, 5120 38 / 28.8 and 32 /
// 21.4, 8192 80 / 50 and 64 / 43, 2048 20 / 15.4 and 16.8 / 12, 256 10.8 / 7.8 and 8.0 / 5.3.  Four waves of four blocks each (360 registers), a request's
// mean: 23.7 for 22.8.  Bound: instructions (expanding codes and folding groups beside the MFMAs) and 32 KB of codes
// in flight a CU; the codes' 65 MB take 11 us at 6 TB/s.
__global__ __launch_bounds__(V2_THREADS) void k2_logits_q4(Gemm2 g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float sh_small[16 * 32];
  float* red = (float*)smem;                                    // [LQ4_PARTS][LQ4_BLOCKS][16][64]
  pin_args(g);
  const int lane = threadIdx.x & 63, w = wave_id();
  const uint32_t NRB = g.NRB;
  const int rb0 = share_begin(blockIdx.x, NRB, g.share_a, g.share_b), rb1 = share_begin(blockIdx.x + 1, NRB, g.share_a, g.share_b), nr = rb1 - rb0;   // <= LQ4_BLOCKS (host)
  const int pair = w & 1, part = w >> 1, mine = min(max(nr - 2 * pair, 0), 2), first = min(rb0 + 2 * pair, g.NRB - 1);
  EarlyLoads el;
  Gemm2 e;                                                      // the arguments as the epilogue reads them
  auto early = [&] {
    e = late_args();
    early_issue(g.in_scale.ssq, g.facts, el);
  };
  f32x16 acc[2];
  const int gb = (unsigned)part * (unsigned)g.NG / LQ4_PARTS, ge = (unsigned)(part + 1) * (unsigned)g.NG / LQ4_PARTS;
  const u32x4* sq[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) sq[j] = (const u32x4*)g.SC + (size_t)min(first + j, g.NRB - 1) * (size_t)g.NG * 4 + 2 * (lane >> 5);
  fk_stream_q4_dispatch<2, 2>(mine, g.q4, g.XF, g.KS, g.M, gb, ge, q4_codes(g.W, first, mine, g.KS), sq, g.NG, acc, lane, early);
  const int m = threadIdx.x & 31, slot = threadIdx.x >> 5;      // 16 slots of 32 tokens
  const bool live = m < e.M;
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (j < mine) fk_park(red, LQ4_BLOCKS, part, 2 * pair + j, lane, acc[j]);
  block_rstd_park(e.in_scale, early_ssq(e.in_scale, el), sh_small);
  __syncthreads();
  const float rs = live ? block_rstd(e.in_scale, sh_small, m) : 0.f;
  const int nend = min(e.N, e.V);
  const bool vec = (e.V & 3) == 0;
  const long dst = live && el.out_row >= 0 ? (long)el.out_row * e.V : -1;
  for (int it = slot; it < nr * 8; it += 16) {                  // item = (row block j, quad of 4 rows)
    const int j = it >> 3, qd = it & 7;
    const int n = (rb0 + j) * 32 + 4 * qd;
    if (dst < 0 || n >= nend) continue;
    const f32x4 v = fk_sum4<LQ4_PARTS>(red, LQ4_BLOCKS, j, qd, m) * rs;
    if (vec && n + 4 <= nend) *(f32x4*)(e.logits + dst + n) = v;
    else {
#pragma unroll
      for (int t = 0; t < 4; ++t) if (n + t < nend) e.logits[dst + n + t] = v[t];
    }
  }
}

// ---- whole-K gate/up of passes of 33 to 128 rows --------------------------------------------------------------------------------
// The structure of k2_gemm_fk with MT 32-row tiles of activations: a work-group owns up to NRMAX row blocks over all of K, its four
// waves (one a SIMD: the sums of NRMAX x MT tiles take up to 192 registers) split K, weights HBM -> VGPR -> MFMA, activation fragments
// straight from L2, sums through LDS, SwiGLU on them.  No partial sums in memory and no SwiGLU launch behind it.
// A CU fetches weights from HBM and activations from L2 through one queue of about 38 KB in request order, so that a short L2 access
// waits behind the long HBM access in front of it: 48 B/ns a CU with the two interleaved by the tile, 66 in segments of 32 KB and
// 64 KB.  Hence the order here: the weights of four k-steps in one burst, all waves at once (the barrier), then activations only.
// 104 rows at 7B widths, us: k_gemm_pf with two K slices and k_swiglu 51.4 + 8.4; this 56.3 with weights and activations requested
// step by step, 54.0 in bursts; 55 rows 44.1 + 6.1 / 42.3 / 40.5.  Bound: the same queue (0.7 + 1.4 MB a CU) beside 25 to 30 us of MFMA.
// QKV (1.5 row blocks a CU) measured no better this way than k_gemm_pf and k_qkv_rope_store.
struct GemmWK { const bf16_t *W, *XF; int NRB, KS, M; bf16_t* act /*[plane][tile][NRB k-steps]*/; };
template <int NR, int MT, int NRMAX>
__device__ __forceinline__ void wk_stream(const GemmWK& g, int kb, int ke, const FkWeights<1>& fw, f32x16 (&acc)[NRMAX][MT], int lane) {
  constexpr int XD = 4;                                         // k-steps of activations in flight
  const int KS = g.KS;
  u32x4 ta[2][4][NR], tb[XD][2][MT];
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void*)g.XF, 0, 2 * MT * KS * 1024, 0x00020000);
  const uint32_t xlane = (uint32_t)lane * 16u, xlast = 32 * (MT - 1) + (lane & 31) < g.M ? xlane : OUT_OF_RANGE;   // dead rows of the last tile
  auto load_w = [&](int b, int k) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < NR; ++j) ta[b][i][j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(fw.rs[0], fw.vo[j], (uint32_t)(j * KS + min(k + i, ke - 1)) * 1024u, 2));
  };
  auto load_x = [&](int s, int k) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int t = 0; t < MT; ++t) tb[s][q][t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xrs, t == MT - 1 ? xlast : xlane, (uint32_t)((q * MT + t) * KS + k) * 1024u, 0));
  };
  auto mul = [&](int b, int i, int s) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ta[b][i][j]), __builtin_bit_cast(bf16x8, tb[s][q][t]), acc[j][t], 0, 0, 0);
  };
  load_w(0, kb);
#pragma unroll
  for (int i = 0; i < XD; ++i) load_x(i, min(kb + i, ke - 1));
  int k = kb;
  for (; k + 8 + XD <= ke; k += 8) {                            // (as often in every wave: the four K ranges are equally long)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      load_w(b ^ 1, k + 4 * b + 4);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mul(b, i, (4 * b + i) % XD);
        load_x((4 * b + i) % XD, k + 4 * b + i + XD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  for (; k < ke; k += 8) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (k + 4 * b + 4 < ke) load_w(b ^ 1, k + 4 * b + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k + 4 * b + i < ke) mul(b, i, (4 * b + i) % XD);
        if (k + 4 * b + i + XD < ke) load_x((4 * b + i) % XD, k + 4 * b + i + XD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}
template <int NRMAX, int MT>
__global__ __launch_bounds__(256, 1) void k_gemm_wk(GemmWK g) {
  constexpr int UNITS = NRMAX * MT, ROUNDS = (UNITS + 3) / 4;
  extern __shared__ __attribute__((aligned(16))) float wk_red[];    // [2][4 units][4 waves][4][64 lanes][4]
  const int lane = threadIdx.x & 63, w = wave_id(), hh = lane >> 5;
  const unsigned G = gridDim.x;
  const int rb0 = (unsigned)blockIdx.x * (unsigned)g.NRB / G, rb1 = (unsigned)(blockIdx.x + 1) * (unsigned)g.NRB / G, nr = rb1 - rb0;   // NRMAX - 1 or NRMAX (host)
  const int kq = g.KS / 4, kb = w * kq, ke = kb + kq;           // KS: a multiple of 4 (host)
  f32x16 acc[NRMAX][MT];
#pragma unroll
  for (int j = 0; j < NRMAX; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.f;
  const FkWeights<1> fw = fk_weights<1>(g.W, 0, rb0, nr, g.KS, lane);
  if (nr == NRMAX) wk_stream<NRMAX, MT>(g, kb, ke, fw, acc, lane);
  else wk_stream<NRMAX - 1, MT>(g, kb, ke, fw, acc, lane);
  // Four units (row block, row tile) at a time: every wave parks its sums of them, wave v adds unit v's in wave order and finishes it.
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    float* buf = wk_red + (r & 1) * 16384;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int u = 4 * r + v;
      if (u >= UNITS) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = acc[u / MT][u % MT][4 * i + e];
        *(f32x4*)(buf + ((size_t)((v * 4 + w) * 4 + i) * 64 + lane) * 4) = x;
      }
    }
    __syncthreads();                                            // (the other half of wk_red is free: its readers came through here)
    const int u = 4 * r + w, j = u / MT, t = u % MT, rb = rb0 + j;
    if (u >= UNITS || j >= nr) continue;
    const float* mine = buf + w * 4096;
    float x[16];                                                // register 4i + e: weight row 8i + 4hh + e of the block, token lane % 32 of the tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 a = *(const f32x4*)(mine + ((size_t)i * 64 + lane) * 4);
#pragma unroll
      for (int ww = 1; ww < 4; ++ww) a += *(const f32x4*)(mine + ((size_t)(ww * 4 + i) * 64 + lane) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * i + e] = a[e];
    }
    // registers e and e + 8 are gate and up of one feature; the two lanes of a row swap four values so that each holds 8 in a row
    const int m = 32 * t + (lane & 31);
    float v[8], y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = m < g.M ? x[e] / (1.0f + __expf(-x[e])) * x[e + 8] : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float got = __shfl_xor(hh ? v[e] : v[4 + e], 32, 64);
      y[e] = hh ? got : v[e];
      y[4 + e] = hh ? v[4 + e] : got;
    }
    xf_store8(g.act, m, 16 * rb + 8 * hh, MT, g.NRB, 2, y);
  }
}

// ---- split-K with streamed activations (narrow matrices with a long K: O, down) ------------------------------------------
// The split-K kernel above keeps its X slice in LDS, so a long K forces many slices (11 at K = 11008) and the last
// work-group of a row group reads that many partials on one CU.  Here the slice is streamed from L2 like in the
// whole-K kernel (8 waves split the slice's k-steps, sums meet in LDS), so S is free: a few slices of a few row
// blocks each.  The work-group then costs its weights plus M/32 of its X slice in fetches, but exchanges only
// S x (row blocks) x 4 KiB per row group, and nothing waits for an LDS fill before the weight stream starts.
// Partials, arrival counter and epilogues are those of k2_gemm.
// Q4: 4-bit codes (k_pack_weight_q4); the slices are then whole groups of 128 columns (host: at least 8 groups a slice).
// Grid: K slices, row groups, experts.  RESID: the residual epilogue, else whichever g.epi names.
template <bool RESID, int NXP, int NRMAX, bool Q4 = false, bool EXPERTS = false>
__global__ __launch_bounds__(V2_THREADS) void k2_gemm_xk(Gemm2 g) {
  static_assert(!EXPERTS || (RESID && !Q4), "forms that exist");
  constexpr int ITEMS = (NRMAX + 1) / 2;                        // (row block, register quad) items of a wave
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float sh_small[16 * 33];
  __shared__ float rstd_s[32];
  __shared__ int s_last;
  float* red = (float*)smem;                                    // [8][NRMAX][16][64]
  pin_args(g);
  if (g.skip_flag && g.skip_flag[EXPERTS ? blockIdx.z : 0] == 0) return;   // uniform over the expert's work-groups
  const bf16_t *W = g.W, *XF = g.XF;
  unsigned long long used = 1;                                  // the experts of this launch that some row selected
  if constexpr (EXPERTS) {
    used = __ballot((threadIdx.x & 63) < gridDim.z && g.skip_flag[min(threadIdx.x & 63, gridDim.z - 1)] != 0);
    W += blockIdx.z * g.w_stride; XF += blockIdx.z * g.x_stride;
  }
  const int lane = threadIdx.x & 63, w = wave_id();
  bool row = (lane & 31) < g.M;                                 // dead rows (and, here, rows that did not select the expert) are not fetched
  if constexpr (EXPERTS) row = row && g.row_w[(size_t)blockIdx.z * g.row_w_stride + (lane & 31)] != 0.f;
  unsigned long long* tr = TRACE_PTR((g.trace && threadIdx.x == 0) ? g.trace + (size_t)(blockIdx.x + g.S * blockIdx.y) * 8 : nullptr);
  TRACE_STAMP(tr, 0);
  const uint32_t uS = g.S, uNRB = g.NRB, uKS = g.KS, s = blockIdx.x, grp = blockIdx.y;
  const int rb0 = div_magic(grp * uNRB, g.share_a), rb1 = div_magic(grp * uNRB + uNRB, g.share_a);
  const int nr = rb1 - rb0;                                     // <= NRMAX (host)
  EarlyLoads el;                                                // used by the epilogue, much later
  constexpr bool LATE = Q4 && NRMAX == 3;                       // no registers to hold them through the 4-bit stream (12 to 15 spilled)
  Gemm2 e;                                                      // the arguments as the epilogue reads them
  auto early = [&] {
    e = late_args();
    if constexpr (!LATE && !RESID) early_issue(g.in_scale.ssq, g.facts, el);
  };
  f32x16 acc[NRMAX];
  if constexpr (Q4) {
    const uint32_t uNG = g.NG;
    const int G0 = div_magic(s * uNG, g.S_magic), G1 = div_magic(s * uNG + uNG, g.S_magic), gt = G1 - G0;
    const int gb = G0 + (unsigned)w * (unsigned)gt / 8u, ge = G0 + (unsigned)(w + 1) * (unsigned)gt / 8u;
    const u32x4* sq[NRMAX];
#pragma unroll
    for (int j = 0; j < NRMAX; ++j) sq[j] = (const u32x4*)g.SC + (size_t)min(rb0 + j, g.NRB - 1) * (size_t)g.NG * 4 + 2 * (lane >> 5);
    fk_stream_q4_dispatch<NXP, NRMAX>(nr, g.q4, XF, g.KS, g.M, gb, ge, q4_codes(W, rb0, nr, g.KS), sq, g.NG, acc, lane, early);
    if constexpr (LATE && !RESID) early_issue(e.in_scale.ssq, e.facts, el);
  } else {
    const int ks0 = div_magic(s * uKS, g.S_magic), ks1 = div_magic(s * uKS + uKS, g.S_magic), kt = ks1 - ks0;
    const int kb = ks0 + (unsigned)w * (unsigned)kt / 8u, ke = ks0 + (unsigned)(w + 1) * (unsigned)kt / 8u;
    fk_stream_dispatch<1, NXP, NRMAX>(nr, XF, g.KS, row, kb, ke, fk_weights<1>(W, g.wps, rb0, nr, g.KS, lane), acc, lane, early);
  }
  TRACE_STAMP_AFTER(tr, 2, acc[0][0]);
  // what the residual epilogue adds and multiplies, if this turns out to be the work-group that runs it: on its way during the sums
  ResidItem ri[ITEMS];
  if constexpr (RESID) {
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) ri[t] = resid_item(e, rb0 * 32 + 8 * (w + 8 * t), w + 8 * t < nr * 4);
  }
#pragma unroll
  for (int j = 0; j < NRMAX; ++j)
    if (j < nr) fk_park(red, NRMAX, w, j, lane, acc[j]);
  __syncthreads();
  // the waves share the sum and the publication: item = (row block j, register quad i) -> rows 8i + 4(lane/32) + 0..3
#pragma unroll
  for (int t = 0; t < ITEMS; ++t) {
    const int it = w + 8 * t, j = it >> 2, i = it & 3;
    if (it >= nr * 4) break;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < 8; ++ww) o += *(const f32x4*)(red + ((((size_t)ww * NRMAX + j) * 4 + i) * 64 + lane) * 4);
    coh_store16(e.PT, pt_quad_bytes(EXPERTS ? (int)(blockIdx.z * uS + s) : s, e.Npad, (rb0 + j) * 32 + 8 * i + 4 * (lane >> 5), lane & 31), o);
  }
  TRACE_STAMP(tr, 3);
  publish_wait();
  __syncthreads();
  if (threadIdx.x == 0) {
    int* cnt = e.counters + grp * COUNTER_STRIDE;
    int old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (old == (EXPERTS ? e.S * __popcll(used) : e.S) - 1);
    if (s_last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const int n0 = rb0 * 32, n1 = min(rb1 * 32, e.N);
  if (n1 <= n0) return;
  if constexpr (RESID) epilogue_resid<NXP, EXPERTS, ITEMS>(e, grp, n0, n1, sh_small, ri, used);
  else {
    block_rstd_finish(e.in_scale, early_ssq(e.in_scale, el), rstd_s, sh_small);
    switch (e.epi) {
      case EPI_QKV: epilogue_qkv<NXP>(e, n0, n1, rstd_s, el); break;
      case EPI_SWIGLU: epilogue_swiglu<NXP>(e, n0, n1, rstd_s); break;
      default: epilogue_logits(e, n0, n1, rstd_s, el); break;
    }
  }
  TRACE_STAMP(tr, 4);
}

// Rows of a pass that need no GEMM in front: h = embedding of the row's token.  Writes h, XF(h * gain) and the
// partial sums of squares, one column slab per block (the same outputs a residual epilogue produces).
template <typename EmbT, int NXP>
__global__ __launch_bounds__(256) void k2_embed(Pass pass, const TreeDev* tree, SeqState st, const int* tree_tok,
                                                const EmbT* __restrict__ embed, int vocab, int M, int nodes /*of the tree*/, int d, float* h,
                                                const float* __restrict__ gain, bf16_t* xf_out, float* ssq_out, KVCache kv, RowFact* facts) {
  __shared__ float sh[8 * 32];
  const int m = threadIdx.x & 31, slot = threadIdx.x >> 5;          // 8 slots
  const int grp = blockIdx.x, groups = gridDim.x;
  const int c0 = (int)((long)grp * (d / 8) / groups), c1 = (int)((long)(grp + 1) * (d / 8) / groups);
  const bool live = m < M;
  int tok = 0;
  if (live) {
    RowInfo ri = row_info(pass, tree, st, m);
    if (pass.kind == PASS_VERIFY) tok = tree_tok[ri.seq * nodes + ri.node];
    else tok = st.tokens[(size_t)ri.seq * st.tok_stride + ri.pos];
    tok = min(max(tok, 0), vocab - 1);
    if (blockIdx.x == 0 && slot == 0) facts[m] = row_fact(pass, tree, ri, kv);
  }
  float ss = 0.f;
  for (int c = c0 + slot; c < c1; c += 8) {
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, gn[8];
    embed8(gain + 8 * c, gn);
    if (live) {
      embed8(embed + (size_t)tok * d + 8 * c, x);
      *(f32x4*)(h + (size_t)m * d + 8 * c) = f32x4{x[0], x[1], x[2], x[3]};
      *(f32x4*)(h + (size_t)m * d + 8 * c + 4) = f32x4{x[4], x[5], x[6], x[7]};
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      ss += x[t] * x[t];
      x[t] *= gn[t];
    }
    if (live) xf_store8(xf_out, m, 8 * c, 1, d / 16, NXP, x);
  }
  sh[slot * 32 + m] = ss;
  __syncthreads();
  if (threadIdx.x < 32) {
    float a = 0.f;
    for (int i = 0; i < 8; ++i) a += sh[i * 32 + threadIdx.x];
    ssq_out[grp * 32 + threadIdx.x] = a;
  }
}

// The target's final RMSNorm (Sec. 2: f is what the LM head reads): h[m][k] * rstd[m] * gain[k], straight to where the pass keeps its
// rows' features (see k_store_rows).
__global__ __launch_bounds__(256) void k2_features(Pass pass, const TreeDev* tree, SeqState st, const float* __restrict__ h, RowScale rs, const float* __restrict__ gain,
                                                   int d, float* __restrict__ node_dst, float* __restrict__ pend_dst, float* __restrict__ chunk_dst) {
  __shared__ float tmp[17];
  const int m = blockIdx.x;
  constexpr int AHEAD = 4;                                      // chunks requested before the row's scale is known
  f32x4 hv[AHEAD], gv[AHEAD];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) {
    const int k = min(4 * (int)threadIdx.x + 1024 * i, d - 4);
    hv[i] = *(const f32x4*)(h + (size_t)m * d + k); gv[i] = *(const f32x4*)(gain + k);
  }
  float* dst = feature_row(pass, tree, st, m, node_dst, pend_dst, chunk_dst, d);
  const float r = block_row_rstd(rs.ssq, rs.groups, rs.inv_d, rs.eps, m, tmp);
  if (!dst) return;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) {
    const int k = 4 * (int)threadIdx.x + 1024 * i;
    if (k < d) *(f32x4*)(dst + k) = hv[i] * r * gv[i];
  }
  for (int k = 4 * (int)threadIdx.x + 1024 * AHEAD; k < d; k += 1024) *(f32x4*)(dst + k) = *(const f32x4*)(h + (size_t)m * d + k) * r * *(const f32x4*)(gain + k);
}

// ============================================================================ tree-masked paged attention, <= 32 rows per sequence
// Block = (kv split, query head, sequence), 4 waves.  Each wave runs flash attention on its own 32-token blocks
// entirely in registers on the MFMA units:
//   S^T[tok][q] = K[tok][:] . Q[q][:]      A = K block (32 tokens x 16 dims per step), B = Q fragments (kept in VGPRs)
//   O^T[d][q]  += V[tok][d] * P[q][tok]    A = V^T (gathered so that the token order matches the S^T accumulator
//                                          layout), B = P straight out of the accumulator registers
// fp32 cache values and probabilities are split into bf16 hi + lo on the fly (hi*hi + hi*lo + lo*hi), so the
// result keeps ~16 mantissa bits.  A lane always owns one query (column l%32): running max / sum and the rescale
// of O^T are lane-local, the only cross-lane traffic is one xor-32 shuffle per reduction.  Keys: cache slots
// [0, base) are visible to every row; slot base+j is visible iff bit j of the row's ancestor mask is set (tree
// passes) or j <= the row's own relative index (causal passes).  Waves are merged through LDS, splits through
// coherent partials and the last split to arrive, which writes XF layout for the output projection.
__device__ inline void split8(const float* x, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    hi[i] = (__bf16)x[i];
    lo[i] = (__bf16)(x[i] - (float)hi[i]);
  }
}
__device__ inline void load8(const float* p, float* x) {
  const f32x4 a = *(const f32x4*)p, b = *(const f32x4*)(p + 4);
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
__device__ inline void load8(const bf16_t* p, float* x) {
  const u32x4 r = *(const u32x4*)p;
  x[0] = __builtin_bit_cast(float, r.x << 16); x[1] = __builtin_bit_cast(float, r.x & 0xFFFF0000u);
  x[2] = __builtin_bit_cast(float, r.y << 16); x[3] = __builtin_bit_cast(float, r.y & 0xFFFF0000u);
  x[4] = __builtin_bit_cast(float, r.z << 16); x[5] = __builtin_bit_cast(float, r.z & 0xFFFF0000u);
  x[6] = __builtin_bit_cast(float, r.w << 16); x[7] = __builtin_bit_cast(float, r.w & 0xFFFF0000u);
}

// Folds NS splits of one (row, head) into the running (max, denominator, outputs) of IT items (rows, `row_o` / `row_ml` bytes apart in the two
// buffers) at once: every load of the chunk is in flight before the first use.  oo[i], om[i]: a lane's byte offsets of the first split's outputs
// and (max, sum) pairs.  FIRST: nothing to rescale.
// What a merge takes is instructions on one chain, not bytes (a wave alone on its SIMD issues one in four to eight cycles): so the addresses are
// 32-bit offsets with the split in the instruction, two pairs come with one load, and a thread merges all its rows at once.  From the last
// arrival to the end of a launch at 7B (26 rows, five splits), by time stamps: 3.6 us with 64-bit addresses, a load per number and two rows at a
// time, 2.5 us now; the loads' own round trip is 0.5.
template <int DH, int IT, int NS, bool FIRST>
__device__ __forceinline__ void attn_merge_chunk(__amdgpu_buffer_rsrc_t po, __amdgpu_buffer_rsrc_t pm, const uint32_t* oo, const uint32_t* om, uint32_t row_o, uint32_t row_ml,
                                                 float* mx, float* den, f32x4* x) {
  u32x4 ml[IT][(NS + 1) / 2];
  f32x4 ov[IT][NS];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
#pragma unroll
    for (int u = 0; u + 1 < NS; u += 2) ml[i][u / 2] = __builtin_amdgcn_raw_buffer_load_b128(pm, om[i] + u * 8, i * row_ml, 16);
    if (NS & 1) {
      const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(pm, om[i] + (NS - 1) * 8, i * row_ml, 16));
      ml[i][NS / 2].x = v.x; ml[i][NS / 2].y = v.y;
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) ov[i][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(po, oo[i] + u * (DH * 4), i * row_o, 16));
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    float msv[NS], lsv[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      msv[u] = __builtin_bit_cast(float, u & 1 ? ml[i][u / 2].z : ml[i][u / 2].x);
      lsv[u] = __builtin_bit_cast(float, u & 1 ? ml[i][u / 2].w : ml[i][u / 2].y);
    }
    float cmx = mx[i];
#pragma unroll
    for (int u = 0; u < NS; ++u) cmx = fmaxf(cmx, msv[u]);
    const float resc = FIRST || mx[i] == -INFINITY ? 0.f : __expf(mx[i] - cmx);
    mx[i] = cmx;
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const float wv = (msv[u] != -INFINITY) ? __expf(msv[u] - cmx) : 0.f;
      if (!FIRST && u == 0) {
        // A fused multiply-add rounds one of its two products by itself; which one is written out.  (Left to the compiler it changed with the code around
        // it, and with a bf16 cache logits moved by up to 1e-5.)
        const f32x4 r4 = {resc, resc, resc, resc}, w4 = {wv, wv, wv, wv};
        den[i] = NS == 1 ? __builtin_fmaf(wv, lsv[u], den[i] * resc) : __builtin_fmaf(den[i], resc, wv * lsv[u]);
        x[i] = NS == 1 ? __builtin_elementwise_fma(w4, ov[i][u], x[i] * r4) : __builtin_elementwise_fma(x[i], r4, ov[i][u] * w4);
        continue;
      }
      den[i] += wv * lsv[u];
      x[i] += wv * ov[i][u];
    }
  }
}

struct AttnArgs {
  int rows_per_seq, causal;                // rows of a sequence in the pass; pending rows and prompts see their own rows causally
  const RowFact* facts; KVCache kv; const float* Q; float* part_o; float* part_ml;
  int H, n_splits, n_new; float scale; int* counters; bf16_t* xf_out; int nplanes, MT, rblocks;   // MT = 32-row tiles of the XF output
  // positions in front of the new ones in the first four sequences as the host knows them, and the first sequence's slot (-1: the row facts hold both)
  int slot0, ctx[4];
  unsigned long long* trace;               // profiling builds only
};

// Four consecutive columns of attention output, as input of the output projection: byte offsets of row m, columns k.. of plane 0.
__device__ __forceinline__ uint32_t xf_bytes(int m, int k, int KS) { return ((uint32_t)(m >> 5) * (uint32_t)KS + (k >> 4)) * 1024u + (m & 31) * 16u + ((k & 15) >> 3) * 512u + (k & 7) * 2u; }
__device__ __forceinline__ void attn_store(const AttnArgs& A, __amdgpu_buffer_rsrc_t xf, int m, int k, f32x4 v) {
  const int KS = A.H * A.kv.head_dim / 16;
  const uint32_t at = xf_bytes(m, k, KS), plane = (uint32_t)A.MT * (uint32_t)KS * 1024u;
  float r[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (q < A.nplanes) {
      u32x2 u; u.x = split_pair(r[0], r[1]); u.y = split_pair(r[2], r[3]);
      __builtin_amdgcn_raw_buffer_store_b64(u, xf, at, q * plane, 0);
    }
}

// The rows q0, q0 + RT, ... (IT of them) of one (sequence, head), columns d0..d0+3: all splits together.  at: byte offset of (row q0, split 0)'s outputs.
template <int DH, int IT>
__device__ __forceinline__ void attn_merge(const AttnArgs& A, __amdgpu_buffer_rsrc_t xf, int r0, int R, int hd, int q0, int d0, uint32_t at) {
  constexpr int RT = 256 / (DH / 4);
  const int n_splits = A.n_splits;
  const __amdgpu_buffer_rsrc_t po = coh_rsrc(A.part_o), pm = coh_rsrc(A.part_ml);
  const uint32_t row_o = (uint32_t)(RT * A.H * n_splits) * (DH * 4), row_ml = (uint32_t)(RT * A.H * n_splits) * 8u;
  const uint32_t ml_at = ((uint32_t)(r0 + q0) * A.H + hd) * n_splits * 8u;
  uint32_t oo[IT], om[IT];
  float mx[IT], den[IT];
  f32x4 x[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const bool row = q0 + RT * i < R;
    oo[i] = row ? at : OUT_OF_RANGE; om[i] = row ? ml_at : OUT_OF_RANGE;
    mx[i] = -INFINITY; den[i] = 0.f;
    x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#define CHUNK(NS, FIRST) attn_merge_chunk<DH, IT, NS, FIRST>(po, pm, oo, om, row_o, row_ml, mx, den, x)
  switch (min(n_splits, 8)) {                                  // uniform: exactly the loads that are needed
    case 2: CHUNK(2, true); break;
    case 3: CHUNK(3, true); break;
    case 4: CHUNK(4, true); break;
    case 5: CHUNK(5, true); break;
    case 6: CHUNK(6, true); break;
    case 7: CHUNK(7, true); break;
    default: CHUNK(8, true); break;
  }
  if (n_splits > 8) {                                           // (at most 16)
#pragma unroll
    for (int i = 0; i < IT; ++i) { oo[i] += 8 * (DH * 4); om[i] += 8 * 8; }
    switch (n_splits - 8) {
      case 1: CHUNK(1, false); break;
      case 2: CHUNK(2, false); break;
      case 3: CHUNK(3, false); break;
      case 4: CHUNK(4, false); break;
      case 5: CHUNK(5, false); break;
      case 6: CHUNK(6, false); break;
      case 7: CHUNK(7, false); break;
      default: CHUNK(8, false); break;
    }
  }
#undef CHUNK
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int q2 = q0 + RT * i;
    if (q2 >= R) continue;
    const float inv = den[i] > 0.f ? 1.0f / den[i] : 0.f;
    attn_store(A, xf, r0 + q2, hd * DH + d0, x[i] * inv);
  }
}

// Work-group = (KV split, query head, (sequence of the pass, 32-row block of that sequence's rows)).
template <typename CT, int DH>
__global__ __launch_bounds__(256) void k2_attn(AttnArgs A) {
  constexpr int KSN = DH / 16;              // k-steps of the QK product
  constexpr int DB = DH / 32;               // 32-wide blocks of the head dimension
  constexpr int OS = DH + 4;                // row stride of o_s: 16-byte accesses along d and across rows without bank conflicts
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_a[];
  float* o_s = (float*)smem_a;              // [4 waves][32 rows][OS]
  float* ml_s = o_s + 4 * 32 * OS;          // [4 waves][2][32]
  __shared__ int s_last;
  const int split = blockIdx.x, hd = blockIdx.y, z = blockIdx.z;
  const int H = A.H, n_splits = A.n_splits, n_new = A.n_new;
  const KVCache& kv = A.kv;
  const float* Q = A.Q;
  const int seq_l = z / A.rblocks, rblk = z % A.rblocks;
  // optional time stamps: 0 entered, 1 keys/values consumed, 2 waves merged + partials written, 3 arrived, 4 splits merged
  unsigned long long* tr = TRACE_PTR((A.trace && threadIdx.x == 0 && seq_l == 0) ? A.trace + ((size_t)hd * n_splits + split) * 8 : nullptr);
  TRACE_STAMP(tr, 0);
  const int r0 = seq_l * A.rows_per_seq + 32 * rblk;
  const int R = min(32, A.rows_per_seq - 32 * rblk);
  const int kvh = hd / (H / kv.n_kv_heads);
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int q = lane & 31, hh = lane >> 5;
  // the queries are requested before anything else: their address needs no load (wave w takes k-steps w, w + 4, ...)
  constexpr int QI = (KSN + 3) / 4;
  float qx[QI][8];
#pragma unroll
  for (int i = 0; i < QI; ++i)
    if (w + 4 * i < KSN) load8(Q + ((size_t)(r0 + min(q, R - 1)) * H + hd) * DH + 16 * (w + 4 * i) + 8 * hh, qx[i]);
  // (the rows' facts were written by the pass's first kernel)
  const bool causal = A.causal;
  const RowFact fq = A.facts[r0 + min(q, R - 1)];                 // this lane's query row
  int seq, base;
  if (A.slot0 >= 0) { seq = A.slot0 + seq_l; base = seq_l == 0 ? A.ctx[0] : seq_l == 1 ? A.ctx[1] : seq_l == 2 ? A.ctx[2] : A.ctx[3]; }
  else { seq = __builtin_amdgcn_readfirstlane(fq.seq); base = __builtin_amdgcn_readfirstlane(fq.base); }
  const int rel = fq.rel;
  const unsigned long long mask = (unsigned long long)fq.mask_hi << 32 | fq.mask_lo;
  // causal passes (prompt chunks, pending rows): the rows of this 32-row block see no new token beyond its own last row,
  // so the blocks of keys after it are not visited at all (they would contribute exp(-inf) = 0: same bits, less work)
  const int T = base + (causal ? min(n_new, 32 * rblk + R) : n_new);
  // the split boundaries depend on `base` only, so a row sees the same partition whatever else is in the pass
  const int span = base + max(64, (n_new + 63) / 64 * 64);   // passes with at most 64 new rows share one partition
  const int tps = ((span + n_splits - 1) / n_splits + 63) / 64 * 64;
  const int t_begin = split * tps, t_end = min(T, t_begin + tps);
  // Wave w takes every 4th 32-token block.  A block starts on a multiple of 32 and therefore lies inside one 64-token
  // (or larger) page.  The keys of the NEXT block are requested as soon as the scores of the current one are done
  // (the registers are free then), after the current block's values, so that they travel while the softmax and the
  // P V product run: a wave that walks several blocks pays about one memory round trip per block.
  // A block's address is the same for the whole wave and stays in scalar registers; a lane adds a 32-bit offset.  (With an address
  // per lane the 64 value loads of a block took their offsets from vector registers; that, a branch per score for the mask and
  // the queries requested behind the facts: 15.2 us a launch at 7B, 550 keys, 26 rows, 13.9 without.)
  // Where the host knows the cached lengths, the first block's address needs one look-up and its keys are requested before the queries are
  // converted.  (That, the merge of the waves with all its reads out at once, and the merge of the splits above: 13.6 -> 11.4 us.  With the first
  // values requested there too, the queries wait behind them: 12.3.)
  float kx[KSN][8];
  size_t blk = 0;
  auto block_of = [&](int tok) -> size_t {
    const int phys = ((const __attribute__((address_space(4))) int*)kv.page_table)[seq * kv.pages_per_seq + (tok >> kv.page_shift)];
    return (((size_t)phys * kv.n_kv_heads + kvh) << kv.page_shift | (size_t)(tok & ((1 << kv.page_shift) - 1))) * DH;
  };
  const uint32_t k_lane = (uint32_t)((lane & 31) * DH + 8 * hh), v_lane = (uint32_t)(4 * hh * DH + (lane & 31));
  auto load_keys = [&](size_t at) {
    const CT* kp = (const CT*)kv.k + at;
#pragma unroll
    for (int ks = 0; ks < KSN; ++ks) load8(kp + 16 * ks + k_lane, kx[ks]);
  };
  // slot t of lane-half hh in k-step j of the P V product is the token that accumulator register 8j+t of the same lane-half holds
  float vx[2][DB][8];
  auto load_values = [&](size_t at) {
    const CT* vp = (const CT*)kv.v + at;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int tl = 16 * j + 8 * (t >> 2) + (t & 3);       // + 4 * hh
          vx[j][b][t] = cache_load(vp + tl * DH + 32 * b + v_lane);
        }
  };
  {
    const int tok0 = t_begin + 32 * w;
    blk = block_of(tok0 < t_end ? tok0 : 0);                   // (a wave without a block requests one too: behind a branch its wait for the queries would be a wait for all)
    load_keys(blk);
  }
  // The scaled queries as bf16 hi + lo B-operand fragments live in LDS, built once by the four waves together (wave w
  // converts k-steps w, w+4, ...); they share the memory of o_s, which is not written before every wave has left the
  // key loop.  (One load and one conversion of the queries per work-group instead of one per wave.)
  bf16x8* q_s = (bf16x8*)smem_a;                               // [2 planes][KSN][64 lanes]
#pragma unroll
  for (int i = 0; i < QI; ++i) {
    const int ks = w + 4 * i;
    if (ks >= KSN) continue;
#pragma unroll
    for (int t = 0; t < 8; ++t) qx[i][t] = q < R ? qx[i][t] * A.scale : 0.f;
    bf16x8 h8, l8;
    split8(qx[i], h8, l8);
    q_s[(0 * KSN + ks) * 64 + lane] = h8;
    q_s[(1 * KSN + ks) * 64 + lane] = l8;
  }
  __syncthreads();
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[b][r] = 0.f;
  for (int tok0 = t_begin + 32 * w; tok0 < t_end; tok0 += 128) {
    const bool more = tok0 + 128 < t_end;
    const size_t blk_next = more ? block_of(tok0 + 128) : 0;   // look-up in flight during the scores
    f32x16 sacc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KSN; ++ks) {
      bf16x8 kh, kl;
      split8(kx[ks], kh, kl);
      const bf16x8 qh = q_s[(0 * KSN + ks) * 64 + lane], ql = q_s[(1 * KSN + ks) * 64 + lane];
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qh, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, ql, sacc, 0, 0, 0);
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kl, qh, sacc, 0, 0, 0);
    }
    load_values(blk);                                          // (out before the softmax arithmetic)
    if (more) load_keys(blk_next);
    blk = blk_next;
    // mask, running max and sum for this lane's query.  Bit i of vis: token tok0 + i is visible to the row.
    uint32_t vis = 0xFFFFFFFFu;
    if (tok0 + 32 > base || tok0 + 32 > t_end) {               // (uniform: most blocks hold cached tokens only)
      const int sh = tok0 - base;
      auto ones = [](int n) -> uint32_t { return n >= 32 ? 0xFFFFFFFFu : n <= 0 ? 0u : (1u << n) - 1u; };
      if (causal) vis = ones(rel + 1 - sh);
      else vis = ones(-sh) | (sh >= 64 || sh <= -32 ? 0u : sh >= 0 ? (uint32_t)(mask >> sh) : (uint32_t)(mask << -sh));
      vis &= ones(t_end - tok0);
    }
    vis = q < R ? vis >> (4 * hh) : 0u;
    float bmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sacc[r] = (vis >> (8 * (r >> 2) + (r & 3))) & 1u ? sacc[r] : -INFINITY;
      bmax = fmaxf(bmax, sacc[r]);
    }
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
    const float m_new = fmaxf(m_run, bmax);
    const float alpha = (m_run == -INFINITY) ? 0.f : __expf(m_run - m_new);
    float psum = 0.f, pv[2][8];                                // two arrays: a pointer into one of 16 ends up on the stack
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e = (m_new == -INFINITY) ? 0.f : __expf(sacc[r] - m_new);
      pv[r >> 3][r & 7] = e;
      psum += e;
    }
    psum += __shfl_xor(psum, 32, 64);
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[b][r] *= alpha;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 ph, pl;
      split8(pv[j], ph, pl);
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        bf16x8 vh, vl;
        split8(vx[j][b], vh, vl);
        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, ph, oacc[b], 0, 0, 0);
        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, pl, oacc[b], 0, 0, 0);
        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl, ph, oacc[b], 0, 0, 0);
      }
    }
  }
  TRACE_STAMP(tr, 1);
  __syncthreads();                          // every wave is done with the query fragments that o_s overlays
  // merge the 4 waves through LDS; accumulator register r of block b holds d = 32b + 8(r/4) + 4hh + r%4 of row q
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 v; v.x = oacc[b][4 * i]; v.y = oacc[b][4 * i + 1]; v.z = oacc[b][4 * i + 2]; v.w = oacc[b][4 * i + 3];
      *(f32x4*)(o_s + ((size_t)w * 32 + q) * OS + 32 * b + 8 * i + 4 * hh) = v;
    }
  if (hh == 0) { ml_s[(w * 2 + 0) * 32 + q] = m_run; ml_s[(w * 2 + 1) * 32 + q] = l_run; }
  __syncthreads();
  // thread = (four consecutive columns d0, rows tid / LD + RT * i): the lanes of a row write its partial output, and read the
  // other splits' below, in contiguous runs.  (With a row per lane each 16-byte access of a wave touched 64 cache lines.)
  constexpr int LD = DH / 4, RT = 256 / LD, NI = 32 / RT;       // lanes per row, rows at a time, items per thread
  const int d0 = (tid % LD) * 4, q0 = tid / LD;
  const uint32_t at = ((uint32_t)(r0 + q0) * H + hd) * n_splits * (DH * 4) + d0 * 4;   // outputs of (row q0, split 0)
  const __amdgpu_buffer_rsrc_t xf = __builtin_amdgcn_make_buffer_rsrc((void*)A.xf_out, 0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int q2 = q0 + RT * i;
    float mw[4], lw[4];
    f32x4 ow[4];
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
      mw[ww] = ml_s[(ww * 2) * 32 + q2]; lw[ww] = ml_s[(ww * 2 + 1) * 32 + q2];
      ow[ww] = *(const f32x4*)(o_s + ((size_t)ww * 32 + q2) * OS + d0);
    }
    float mm = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) mm = fmaxf(mm, mw[ww]);
    float L = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
      const float wgt = (mw[ww] == -INFINITY) ? 0.f : __expf(mw[ww] - mm);
      L += wgt * lw[ww];
      o += wgt * ow[ww];
    }
    if (q2 >= R) continue;
    if (n_splits == 1) {
      const float inv = L > 0.f ? 1.0f / L : 0.f;
      o *= inv;
      attn_store(A, xf, r0 + q2, hd * DH + d0, o);
    } else {
      coh_store16(A.part_o, at + (uint32_t)(RT * i * H * n_splits + split) * (DH * 4), o);
      if (d0 == 0) {
        const u32x2 u = {__builtin_bit_cast(uint32_t, mm), __builtin_bit_cast(uint32_t, L)};
        __builtin_amdgcn_raw_buffer_store_b64(u, coh_rsrc(A.part_ml), (uint32_t)(((r0 + q2) * H + hd) * n_splits + split) * 8u, 0, 16);
      }
    }
  }
  TRACE_STAMP(tr, 2);
  if (n_splits == 1) return;
  publish_wait();
  __syncthreads();
  if (tid == 0) {
    int* cnt = A.counters + (z * H + hd) * COUNTER_STRIDE;
    int old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (old == n_splits - 1);
    if (s_last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  TRACE_STAMP(tr, 3);
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  // merge the splits of (sequence, head).  Every load of up to 8 splits of a thread's rows -- (max, sum) pairs and partial outputs -- is in
  // flight at once, so the merge costs one memory round trip; more splits continue with a running rescale, in split order.
  if (R <= RT) attn_merge<DH, 1>(A, xf, r0, R, hd, q0, d0, at);
  else if (R <= 2 * RT) attn_merge<DH, 2>(A, xf, r0, R, hd, q0, d0, at);
  else attn_merge<DH, NI>(A, xf, r0, R, hd, q0, d0, at);
  TRACE_STAMP(tr, 4);
}

// ============================================================================ causal attention of a prompt pass
// The arithmetic of k2_attn (scores and outputs transposed, hi * hi + hi * lo + lo * hi on bf16 pieces of the fp32 values), for one
// sequence of many rows: a work-group owns 128 rows of a head, a wave 32 of them, and the keys and values of 32 tokens at a time
// are fetched, split into bf16 pieces and laid out as MFMA operands ONCE for the four waves, in LDS.  (k2_attn walks the tokens with
// all four waves on the same 32 rows: every work-group fetches and splits all keys and values for 32 rows, which is what bounds it
// there -- 41 GB/s a CU from the L2 and 64 four-byte loads a lane and block.)  Two tile buffers: the next tile is requested before
// the products of this one and written behind them, one barrier a tile.  Work-groups of the last rows, which see the most tokens,
// come first in the grid.
#define ATTN_PROMPT_THREADS 512
template <typename CT, int DH>
__global__ __launch_bounds__(ATTN_PROMPT_THREADS, 2) void k2_attn_prompt(AttnArgs A) {
  constexpr int KSN = DH / 16, DB = DH / 32, VP = 2 * DB;        // k-steps of the scores; (16 tokens, 32 dims) pieces of the values
  constexpr int TILE = (KSN + VP) * 2 * 64;                      // 16-byte units of a tile: keys [plane][k-step][lane], values [plane][piece][lane]
  constexpr int KI = (KSN + 3) / 4, VI = (VP + 3) / 4;           // a wave's share of a tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_a[];
  const int H = A.H, rows = A.rows_per_seq;
  const KVCache& kv = A.kv;
  // consecutive work-groups go round the 8 XCDs: an XCD gets neighbouring heads, which share keys and values in grouped-query models
  const int hd = H % 8 == 0 ? (int)(blockIdx.x % 8) * (H / 8) + (int)blockIdx.x / 8 : (int)blockIdx.x;
  const int blk = (int)gridDim.y - 1 - (int)blockIdx.y;
  const int kvh = hd / (H / kv.n_kv_heads);
  const int lane = threadIdx.x & 63, w = wave_id() & 3, kg = wave_id() >> 2, q = lane & 31, hh = lane >> 5;   // 32 rows w of the tiles kg, kg + 2, ...
  bf16x8* tiles = (bf16x8*)smem_a + kg * 2 * TILE;               // [2][TILE] of the half
  const int r0 = 128 * blk + 32 * w, row = min(r0 + q, rows - 1);
  const bool live = r0 + q < rows;
  bf16x8 qf[2][KSN];                                             // the wave's scaled queries, hi and lo
#pragma unroll
  for (int ks = 0; ks < KSN; ++ks) {
    float x[8];
    load8(A.Q + ((size_t)row * H + hd) * DH + 16 * ks + 8 * hh, x);
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] *= A.scale;
    split8(x, qf[0][ks], qf[1][ks]);
  }
  const RowFact fq = A.facts[row];
  const int seq = __builtin_amdgcn_readfirstlane(fq.seq), base = __builtin_amdgcn_readfirstlane(fq.base), rel = fq.rel;
  const int see = base + min(rows, 128 * blk + 128), see_w = base + min(rows, r0 + 32);   // tokens the work-group's / the wave's rows see
  const int nt = (see + 31) / 32;
  // page-table entries of 64 pages in the lanes of a register: no load stands in front of a tile's
  int pages = 0, page0 = -64;
  auto block_of = [&](int tok) -> size_t {
    const int pg = tok >> kv.page_shift;
    if (pg >= page0 + 64) { page0 = pg; pages = kv.page_table[seq * kv.pages_per_seq + min(pg + lane, kv.pages_per_seq - 1)]; }
    const int phys = __builtin_amdgcn_readlane(pages, pg - page0);
    return (((size_t)phys * kv.n_kv_heads + kvh) << kv.page_shift | (size_t)(tok & ((1 << kv.page_shift) - 1))) * DH;
  };
  float kx[KI][8], vx[VI][8];
  const uint32_t k_lane = (uint32_t)((lane & 31) * DH + 8 * hh), v_lane = (uint32_t)(4 * hh * DH + (lane & 31));
  auto fetch = [&](int tok) {
    const size_t at = block_of(tok);
    const CT *kp = (const CT*)kv.k + at, *vp = (const CT*)kv.v + at;
#pragma unroll
    for (int i = 0; i < KI; ++i)
      if (w + 4 * i < KSN) load8(kp + 16 * (w + 4 * i) + k_lane, kx[i]);
#pragma unroll
    for (int i = 0; i < VI; ++i) {
      const int pc = w + 4 * i, j = pc / DB, b = pc % DB;        // order of the tokens in a piece: see k2_attn
      if (pc < VP)
#pragma unroll
        for (int t = 0; t < 8; ++t) vx[i][t] = cache_load(vp + (16 * j + 8 * (t >> 2) + (t & 3)) * DH + 32 * b + v_lane);
    }
  };
  auto put = [&](bf16x8* tile) {
#pragma unroll
    for (int i = 0; i < KI; ++i)
      if (w + 4 * i < KSN) {
        bf16x8 h8, l8;
        split8(kx[i], h8, l8);
        tile[(w + 4 * i) * 64 + lane] = h8;
        tile[(KSN + w + 4 * i) * 64 + lane] = l8;
      }
#pragma unroll
    for (int i = 0; i < VI; ++i)
      if (w + 4 * i < VP) {
        bf16x8 h8, l8;
        split8(vx[i], h8, l8);
        tile[(2 * KSN + w + 4 * i) * 64 + lane] = h8;
        tile[(2 * KSN + VP + w + 4 * i) * 64 + lane] = l8;
      }
  };
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[b][r] = 0.f;
  if (kg < nt) { fetch(32 * kg); put(tiles); }
  __syncthreads();
  for (int i = 0; 2 * i < nt; ++i) {
    const int tok0 = 32 * (2 * i + kg);
    const bool more = tok0 + 64 < 32 * nt;
    const bf16x8* tile = tiles + (i & 1) * TILE;
    if (more) fetch(tok0 + 64);
    if (tok0 < see_w) {                                          // (uniform over the wave; the tiles behind hold only tokens its rows do not see)
      f32x16 sacc;
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KSN; ++ks) {
        const bf16x8 kh = tile[ks * 64 + lane], kl = tile[(KSN + ks) * 64 + lane];
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qf[0][ks], sacc, 0, 0, 0);
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qf[1][ks], sacc, 0, 0, 0);
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kl, qf[0][ks], sacc, 0, 0, 0);
      }
      if (tok0 + 32 > base + r0) {                               // the tile holds tokens that some row does not see
        const int n = live ? base + rel + 1 - tok0 : 0;          // token tok0 + i is visible iff i < n
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = 8 * (r >> 2) + 4 * hh + (r & 3) < n ? sacc[r] : -INFINITY;
      }
      float bmax = sacc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) bmax = fmaxf(bmax, sacc[r]);
      bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
      const float m_new = fmaxf(m_run, bmax);
      if (__any(m_new > m_run)) {                                // (otherwise the factor is 1 in every lane)
        const float alpha = m_run == -INFINITY ? 0.f : __expf(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[b][r] *= alpha;
        m_run = m_new;
      }
      const float m_sub = m_new == -INFINITY ? 0.f : m_new;      // (no visible token yet: every score is -inf, every weight 0)
      float psum = 0.f, pv[2][8];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = __expf(sacc[r] - m_sub);
        pv[r >> 3][r & 7] = e;
        psum += e;
      }
      psum += __shfl_xor(psum, 32, 64);
      l_run += psum;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bf16x8 ph, pl;
        split8(pv[j], ph, pl);
#pragma unroll
        for (int b = 0; b < DB; ++b) {
          const bf16x8 vh = tile[(2 * KSN + j * DB + b) * 64 + lane], vl = tile[(2 * KSN + VP + j * DB + b) * 64 + lane];
          oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, ph, oacc[b], 0, 0, 0);
          oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh, pl, oacc[b], 0, 0, 0);
          oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl, ph, oacc[b], 0, 0, 0);
        }
      }
    }
    if (more) put(tiles + ((i + 1) & 1) * TILE);
    __syncthreads();
  }
  // the second half's state goes through LDS to the first half's waves of the same rows
  float* st = (float*)smem_a + (size_t)w * (16 * DB + 2) * 64 + lane;
  if (kg == 1) {
    st[0] = m_run; st[64] = l_run;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) st[(2 + 16 * b + r) * 64] = oacc[b][r];
  }
  __syncthreads();
  if (kg == 1 || !live) return;
  {
    const float m1 = st[0], m_new = fmaxf(m_run, m1);            // (-inf: a half that holds no visible token, or a row whose scores are all -inf)
    const float w0 = m_run == -INFINITY ? 0.f : __expf(m_run - m_new), w1 = m1 == -INFINITY ? 0.f : __expf(m1 - m_new);
    l_run = l_run * w0 + st[64] * w1;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[b][r] = oacc[b][r] * w0 + st[(2 + 16 * b + r) * 64] * w1;
  }
  const float inv = l_run > 0.f ? 1.0f / l_run : 0.f;
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 o; o.x = oacc[b][4 * i]; o.y = oacc[b][4 * i + 1]; o.z = oacc[b][4 * i + 2]; o.w = oacc[b][4 * i + 3];
      xf_store4(A.xf_out, r0 + q, hd * DH + 32 * b + 8 * i + 4 * hh, A.MT, H * DH / 16, A.nplanes, o * inv);
    }
}
