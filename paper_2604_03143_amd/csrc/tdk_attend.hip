// Attention of new query tokens over the shared span of every mirror, computed from master + diff
// with no restored copy (Sec. 4.4, last paragraphs: the diff applied as attention tiles are loaded;
// Fig. 9: skip-or-correct per block).
//
// RoPE rotations are orthogonal, so q . (R(delta) k) = (R(-delta) q) . k: instead of rotating the
// master's keys once per agent, each agent's few query rows are rotated back by its offset and all
// agents of a session then attend to the SAME un-rotated master keys.  The query rows of a session
// (agents x query tokens x query heads of one KV head) become the N side of one dense product with
// the master's K and V tiles, which is MFMA work, and the master is read once per session instead of
// once per agent (the master pass).  Pages that an agent's diff lists are masked out of that product for
// that agent's rows and come from the payload instead, with the same tile arithmetic (the listed-pages
// pass, the "correct" half); a last kernel merges the partial results with their log-sum-exp weights.
// For the decode case (identity layouts, at most 32 rows per agent and KV head) the two passes share one launch,
// which also rotates the query rows itself; rounds whose agents bring more rows, and most rounds with per-agent
// block orders, give every wavefront one agent's rows (tdk_attend_rows_kernel); per-agent block orders with few rows
// of many agents run tdk_attend_qrot_kernel, tdk_attend_master_kernel and tdk_attend_diff16_kernel one after another.
#include "tdk_internal.h"

#include <algorithm>
#include <type_traits>

namespace tdk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2a __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2a __attribute__((ext_vector_type(2)));

namespace {

constexpr int kTile = 32;            // tokens per MFMA tile
constexpr int kRowsPerWave = 32;     // query rows per wavefront (the N side of the 32x32 MFMA)
constexpr int kRowsPerBlock = kRowsPerWave * kWaves;
constexpr int kKsStride = kHeadDim + 8;   // bf16 elements per staged K row (+16 bytes: spreads LDS banks)
constexpr int kBigTile = 2 * kTile;       // tokens per step of the master pass
constexpr int kVsStride = kHeadDim + 32;  // bf16 elements per staged V row (+64 bytes: four consecutive rows' 64-byte
                                          // pieces then fall into different LDS banks for the transposing reads)

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  f32x2a v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2a));
}

// position of a query row inside its session's row list, and where its data lives
struct RowRef {
  int agent;      // agent id, -1 for a padding row
  int64_t out;    // index of the row in q / out / lse: ((agent * n_q + qi) * Hq + hq)
};

__device__ __forceinline__ RowRef row_ref(const RoundDev& rd, const SessionDev& sd, const AttendDev& at, int h, int row) {
  RowRef r;
  const int per_agent = at.n_q * at.group;
  const int a_local = row / per_agent;
  if (a_local >= sd.n_agents) { r.agent = -1; r.out = 0; return r; }
  const int rem = row - a_local * per_agent;
  const int qi = rem / at.group, g = rem - qi * at.group;
  r.agent = rd.order[sd.order_begin + a_local];
  r.out = ((int64_t)r.agent * at.n_q + qi) * at.n_q_heads + h * at.group + g;
  return r;
}

// Running softmax of one query row (the lane pair n, n + 32 shares a row) and its output accumulators:
// oacc[b][i] is element 32 b + 8 (i / 4) + 4 hh + i % 4 of the row's un-normalised output.
struct RowState {
  float m_run, l_run;
  f32x16 oacc[4];
};

// The maximum that goes with a partial sum.  A NaN score keeps a row's reference point at -infinity for as long as no step is
// free of NaN, and the merge takes -infinity for an empty part: such a part says +infinity instead, and the row becomes NaN.
__device__ __forceinline__ float part_max(float m_run, float l_tot) { return m_run == -INFINITY && l_tot != l_tot ? INFINITY : m_run; }

// log-sum-exp of a row: -infinity for an empty one, NaN for a row with a NaN score
__device__ __forceinline__ float row_lse(float m, float l) { return l > 0.f ? m + __logf(l) : l != l ? l : -INFINITY; }

__device__ __forceinline__ void row_state_init(RowState& st) {
  st.m_run = -INFINITY;
  st.l_run = 0.f;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.oacc[b][i] = 0.f;
}

// Orders the LDS traffic of one wavefront (its lanes exchange data through a staging area no other
// wavefront touches): no hardware barrier, only a point the compiler may not move memory accesses across.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same for a 64-token step held in LDS (two independent score tiles): their MFMA chains interleave,
// the LDS reads of one hide behind the products of the other, and the softmax bookkeeping (exchange with
// the partner lane, reference point, rescale test) is paid once per 64 tokens.  Score i of a lane is token
// 32 (i / 16) + 8 ((i % 16) / 4) + 4 hh + i % 4 of the step.
// scores of a 64-token step for the wavefront's 32 rows: two independent MFMA chains
template <bool AHEAD>
__device__ __forceinline__ void scores64(const uint16_t* Ks, const bf16x8 (&qf)[8], int n, int hh, f32x16& s0, f32x16& s1) {
#pragma unroll
  for (int i = 0; i < 16; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
  if (!AHEAD) {                                             // the form that needs few registers
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const u32x4 a0 = *reinterpret_cast<const u32x4*>(Ks + n * kKsStride + 16 * kk + 8 * hh);
      const u32x4 a1 = *reinterpret_cast<const u32x4*>(Ks + (kTile + n) * kKsStride + 16 * kk + 8 * hh);
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a0), qf[kk], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a1), qf[kk], s1, 0, 0, 0);
    }
    return;
  }
  // all sixteen A operands are requested before the first product: the LDS round trips overlap instead of
  // each pair of products waiting for its own
  u32x4 a[16];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    a[2 * kk] = *reinterpret_cast<const u32x4*>(Ks + n * kKsStride + 16 * kk + 8 * hh);
    a[2 * kk + 1] = *reinterpret_cast<const u32x4*>(Ks + (kTile + n) * kKsStride + 16 * kk + 8 * hh);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);       // the 16 LDS reads first
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[2 * kk]), qf[kk], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[2 * kk + 1]), qf[kk], s1, 0, 0, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);       // then the 16 products
}

// O^T += V^T P^T for a 64-token step whose V rows sit row-major in LDS (Vs[token][d]).  The A operand of
// product (kk, b) is V^T[d = 32 b + n][tokens 16 kk + 8 hf + 4 hh + j], hf = 0, 1, j = 0..3: each half comes from
// one ds_read_b64_tr_b16.  Within a block of 16 lanes that instruction treats the 8-byte pieces the lanes
// address as the rows of a 16 x 4 matrix of 16-bit values and hands lane i the values (i / 4 + 4 j, i % 4),
// j = 0..3; with lane i addressing (token i / 4 of the four, d-quad i % 4 of its block's sixteen d) lane i gets
// element d = 16 (block % 2) + i of tokens 0..3 -- its own row of V^T.  p[i] is the weight of token
// 32 (i / 16) + 8 ((i % 16) / 4) + 4 hh + i % 4.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int NK>                             // NK products of 16 tokens each: 4 for a 64-token step, 2 for a 32-token tile
__device__ __forceinline__ void pv_tr(const uint16_t* Vs, const float (&p)[8 * NK], int lane, RowState& st) {
  const int i16 = lane & 15, blk = lane >> 4;
  const uint16_t* base = Vs + (4 * (blk >> 1) + (i16 >> 2)) * kVsStride + 16 * (blk & 1) + 4 * (i16 & 3);
  u32x4 va[4 * NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + (16 * kk) * kVsStride + 32 * b));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + (16 * kk + 8) * kVsStride + 32 * b));
      const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
      va[4 * kk + b] = u32x4{l2.x, l2.y, h2.x, h2.y};
    }
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    u32x4 pw;
#pragma unroll
    for (int e = 0; e < 4; ++e) pw[e] = pack2(p[8 * kk + 2 * e], p[8 * kk + 2 * e + 1]);
    const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
    for (int b = 0; b < 4; ++b)
      st.oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[4 * kk + b]), pb, st.oacc[b], 0, 0, 0);
  }
}

// One 32-token tile for the 32 query rows of a wavefront, K rows in registers: k[kk] holds, for lane (n, hh),
// elements 16 kk + 8 hh .. + 7 of the K row of token n.  S^T (tokens x rows) = K Q^T: lane (n, hh) then holds,
// for query row n, the scores of tokens 8 (i / 4) + 4 hh + i % 4; bit i of `live` says whether that token counts.
__device__ __forceinline__ void scores32(const u32x4 (&k)[8], const bf16x8 (&qf)[8], f32x16& sacc) {
#pragma unroll
  for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
    sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[kk]), qf[kk], sacc, 0, 0, 0);
}

__device__ __forceinline__ void softmax_pv32(const uint16_t* Vs, const f32x16& sacc, float scale, uint32_t live, int lane,
                                             RowState& st) {
  float p[16];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    p[i] = ((live >> i) & 1u) ? sacc[i] * scale : -INFINITY;
    mx = fmaxf(mx, p[i]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  constexpr float kLazy = 8.f;
  const float m_new = mx > st.m_run + kLazy || st.m_run == -INFINITY ? fmaxf(st.m_run, mx) : st.m_run;
  const float m_ref = m_new == -INFINITY ? 0.f : m_new;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) { p[i] = __expf(p[i] - m_ref); sum += p[i]; }
  if (__any(m_new != st.m_run)) {
    const float alpha = __expf(st.m_run - m_ref);      // 1 for the rows whose reference stays
    st.l_run *= alpha;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.oacc[b][i] *= alpha;
  }
  st.l_run += sum;
  st.m_run = m_new;
  pv_tr<2>(Vs, p, lane, st);
}

__device__ __forceinline__ void softmax_pv64(const uint16_t* Vs, const f32x16& s0, const f32x16& s1, float scale,
                                             uint32_t live, int lane, RowState& st) {
  float p[32];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    p[i] = ((live >> i) & 1u) ? s0[i] * scale : -INFINITY;
    p[16 + i] = ((live >> (16 + i)) & 1u) ? s1[i] * scale : -INFINITY;
    mx = fmaxf(mx, fmaxf(p[i], p[16 + i]));
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  constexpr float kLazy = 8.f;
  const float m_new = mx > st.m_run + kLazy || st.m_run == -INFINITY ? fmaxf(st.m_run, mx) : st.m_run;
  const float m_ref = m_new == -INFINITY ? 0.f : m_new;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i) { p[i] = __expf(p[i] - m_ref); sum += p[i]; }
  if (__any(m_new != st.m_run)) {
    const float alpha = __expf(st.m_run - m_ref);
    st.l_run *= alpha;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.oacc[b][i] *= alpha;
  }
  st.l_run += sum;
  st.m_run = m_new;
  pv_tr<4>(Vs, p, lane, st);
}

// The same with whole 16-token groups switched off instead of single tokens, for a positive scale: score i
// of a lane belongs to group i / 8 and bit g of m4 says whether group g takes part (four lane masks, one
// select per score); the scale and the reference point go into one fused multiply-add in base-2 units in
// front of v_exp_f32.  m_run stays in natural-log units of the scaled scores.
__device__ __forceinline__ void softmax_pv64_groups(const uint16_t* Vs, const f32x16& s0, const f32x16& s1, float scale,
                                                    uint32_t m4, int lane, RowState& st) {
  constexpr float kLog2e = 1.4426950408889634f;
  const bool on[4] = {(m4 & 1u) != 0, (m4 & 2u) != 0, (m4 & 4u) != 0, (m4 & 8u) != 0};
  float p[32];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    p[i] = on[i >> 3] ? s0[i] : -INFINITY;
    p[16 + i] = on[2 + (i >> 3)] ? s1[i] : -INFINITY;
    // (the NaN-propagating maximum: v_maximum3_f32, with no quieting of its operands first)
    mx = __builtin_elementwise_maximum(mx, __builtin_elementwise_maximum(p[i], p[16 + i]));
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32)) * scale;
  constexpr float kLazy = 8.f;
  const float m_new = mx > st.m_run + kLazy || st.m_run == -INFINITY ? fmaxf(st.m_run, mx) : st.m_run;
  const float m_ref = m_new == -INFINITY ? 0.f : m_new;
  const float c2 = scale * kLog2e, m2 = -m_ref * kLog2e;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i) { p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(p[i], c2, m2)); sum += p[i]; }
  if (__any(m_new != st.m_run)) {
    const float alpha = __expf(st.m_run - m_ref);
    st.l_run *= alpha;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.oacc[b][i] *= alpha;
  }
  st.l_run += sum;
  st.m_run = m_new;
  pv_tr<4>(Vs, p, lane, st);
}

// ---- the same tile for 16 query rows per wavefront (v_mfma_f32_16x16x32_bf16): for passes whose row
// blocks are nearly empty (the listed pages of one agent meet only its own few rows), a quarter of the
// scores per lane.  Lane (n, g) = (lane % 16, lane / 16) owns row n; of a 32-token tile it holds the scores
// of tokens 16 tt + 4 g + i (tt = 0, 1; i = 0..3) as p[4 tt + i], and elements 16 b + 4 g + i of the output.
typedef float f32x4a __attribute__((ext_vector_type(4)));

struct RowState16 {
  float m_run, l_run;
  f32x4a oacc[8];
};

__device__ __forceinline__ void row_state16_init(RowState16& st) {
  st.m_run = -INFINITY;
  st.l_run = 0.f;
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) st.oacc[b][i] = 0.f;
}

// k[2 kk + tt] holds, for lane (n, g), elements 32 kk + 8 g .. + 7 of the K row of token 16 tt + n
__device__ __forceinline__ void scores16(const u32x4 (&k)[8], const bf16x8 (&qf)[4], f32x4a& s0, f32x4a& s1) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[2 * kk]), qf[kk], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[2 * kk + 1]), qf[kk], s1, 0, 0, 0);
  }
}

// Vs holds the tile's V rows row-major (kVsStride); the A operands come from transposing reads as in pv_tr:
// lane i of a block of 16 addresses (token i / 4 of the block's four, d-quad i % 4) and receives d = 16 b + i.
__device__ __forceinline__ void softmax_pv16(const uint16_t* Vs, const f32x4a& s0, const f32x4a& s1, float scale, uint32_t live,
                                             int n, int g, RowState16& st) {
  float p[8];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = ((live >> i) & 1u) ? s0[i] * scale : -INFINITY;
    p[4 + i] = ((live >> (4 + i)) & 1u) ? s1[i] * scale : -INFINITY;
    mx = fmaxf(mx, fmaxf(p[i], p[4 + i]));
  }
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  constexpr float kLazy = 8.f;
  const float m_new = mx > st.m_run + kLazy || st.m_run == -INFINITY ? fmaxf(st.m_run, mx) : st.m_run;
  const float m_ref = m_new == -INFINITY ? 0.f : m_new;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) { p[i] = __expf(p[i] - m_ref); sum += p[i]; }
  if (__any(m_new != st.m_run)) {
    const float alpha = __expf(st.m_run - m_ref);
    st.l_run *= alpha;
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) st.oacc[b][i] *= alpha;
  }
  st.l_run += sum;
  st.m_run = m_new;
  u32x4 pw;
#pragma unroll
  for (int e = 0; e < 4; ++e) pw[e] = pack2(p[2 * e], p[2 * e + 1]);
  const bf16x8 pb = __builtin_bit_cast(bf16x8, pw);
  const uint16_t* base = Vs + (4 * g + (n >> 2)) * kVsStride + 4 * (n & 3);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + 16 * b));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(base + 16 * kVsStride + 16 * b));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    const u32x4 a = {l2.x, l2.y, h2.x, h2.y};
    st.oacc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), pb, st.oacc[b], 0, 0, 0);
  }
}

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two pairs of a query row turned back by (c0, s0) and (c1, s1): y_a = x_a cos + x_b sin, y_b = x_b cos - x_a sin in
// fp32, rounded to bf16.  wa, wb hold the a and the b elements (half style).
__device__ __forceinline__ void turn_back_half(uint32_t wa, uint32_t wb, float c0, float s0, float c1, float s1, uint32_t& ya, uint32_t& yb) {
  const float a0 = lo16(wa), a1 = hi16(wa), b0 = lo16(wb), b1 = hi16(wb);
  ya = pack2(__builtin_fmaf(a0, c0, __fmul_rn(b0, s0)), __builtin_fmaf(a1, c1, __fmul_rn(b1, s1)));
  yb = pack2(__builtin_fmaf(b0, c0, -__fmul_rn(a0, s0)), __builtin_fmaf(b1, c1, -__fmul_rn(a1, s1)));
}
// One pair held in one word (interleaved style).
__device__ __forceinline__ uint32_t turn_back_pair(uint32_t w, float c, float s) {
  const float a = lo16(w), b = hi16(w);
  return pack2(__builtin_fmaf(a, c, __fmul_rn(b, s)), __builtin_fmaf(b, c, -__fmul_rn(a, s)));
}

// The fragments of a row for the 32-row tiles (fragment kk of a lane: elements 16 kk + 8 hh .. + 7), turned back by tab.
__device__ __forceinline__ void turn_back32(const u32x4 (&raw)[8], const float* tab, bool interleaved, int hh, bf16x8 (&qf)[8]) {
  if (!interleaved) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {             // fragments kk (elements a) and kk + 4 (elements b = a + 64)
      u32x4 ya, yb;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int j = 16 * kk + 8 * hh + 2 * w;
        uint32_t a, b;
        turn_back_half(raw[kk][w], raw[kk + 4][w], tab[j], tab[kHalf + j], tab[j + 1], tab[kHalf + j + 1], a, b);
        ya[w] = a; yb[w] = b;
      }
      qf[kk] = __builtin_bit_cast(bf16x8, ya);
      qf[kk + 4] = __builtin_bit_cast(bf16x8, yb);
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {             // word w of a fragment holds the pair j = 8 kk + 4 hh + w
      u32x4 y;
#pragma unroll
      for (int w = 0; w < 4; ++w) { const int j = 8 * kk + 4 * hh + w; y[w] = turn_back_pair(raw[kk][w], tab[j], tab[kHalf + j]); }
      qf[kk] = __builtin_bit_cast(bf16x8, y);
    }
  }
}

// The same for the 16-row tiles (fragment kk: elements 32 kk + 8 g .. + 7), in place.
__device__ __forceinline__ void turn_back16(bf16x8 (&qf)[4], const float* tab, bool interleaved, int g) {
  u32x4 raw[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) raw[kk] = __builtin_bit_cast(u32x4, qf[kk]);
  if (!interleaved) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {             // fragments kk (elements a) and kk + 2 (elements b = a + 64)
      u32x4 ya, yb;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int j = 32 * kk + 8 * g + 2 * w;
        uint32_t a, b;
        turn_back_half(raw[kk][w], raw[kk + 2][w], tab[j], tab[kHalf + j], tab[j + 1], tab[kHalf + j + 1], a, b);
        ya[w] = a; yb[w] = b;
      }
      qf[kk] = __builtin_bit_cast(bf16x8, ya);
      qf[kk + 2] = __builtin_bit_cast(bf16x8, yb);
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {             // word w of a fragment holds the pair j = 16 kk + 4 g + w
      u32x4 y;
#pragma unroll
      for (int w = 0; w < 4; ++w) { const int j = 16 * kk + 4 * g + w; y[w] = turn_back_pair(raw[kk][w], tab[j], tab[kHalf + j]); }
      qf[kk] = __builtin_bit_cast(bf16x8, y);
    }
  }
}

// A query row as it is, in the order of the B operands for the 32-row tiles: fragment kk of a lane holds elements
// 16 kk + 8 hh .. + 7.  Only the loads: where others are asked for before the rows are
// used, own_rows() is called behind those.
__device__ __forceinline__ void raw_queries(const AttendDev& at, int64_t out, int lane, u32x4 (&raw)[8]) {
  const u32x4* qp = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.q) + out * kHeadDim);
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) raw[kk] = qp[2 * kk + (lane >> 5)];
}
// A negative scale's sign travels with the rows; a row that does not exist has read another and is zero.
__device__ __forceinline__ void own_rows(const AttendDev& at, bool on, u32x4 (&raw)[8]) {
  const uint32_t flip = at.q_flip ? 0x80008000u : 0u, keep = on ? 0xffffffffu : 0u;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
    raw[kk] = u32x4{(raw[kk].x ^ flip) & keep, (raw[kk].y ^ flip) & keep, (raw[kk].z ^ flip) & keep, (raw[kk].w ^ flip) & keep};
}

// Those rows turned back by the rotation whose table the wavefront's lanes hold (entries 2 lane and 2 lane + 1 of its
// 128); it goes through lds_tab (128 floats of this wavefront), so that the fragments are turned one pair at a time
// with few registers.
__device__ __forceinline__ void turn_queries(const u32x4 (&raw)[8], bool interleaved, float2 tab, float* lds_tab, int lane, bf16x8 (&qf)[8]) {
  const int hh = lane >> 5;
  wave_sync();                                           // an earlier table has been used
  reinterpret_cast<float2*>(lds_tab)[lane] = tab;
  wave_sync();
  if (!interleaved) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      float c[8], sn[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) { c[e] = lds_tab[16 * kk + 8 * hh + e]; sn[e] = lds_tab[kHalf + 16 * kk + 8 * hh + e]; }
      u32x4 ya, yb;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t a, b;
        turn_back_half(raw[kk][w], raw[kk + 4][w], c[2 * w], sn[2 * w], c[2 * w + 1], sn[2 * w + 1], a, b);
        ya[w] = a; yb[w] = b;
      }
      qf[kk] = __builtin_bit_cast(bf16x8, ya);
      qf[kk + 4] = __builtin_bit_cast(bf16x8, yb);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u32x4 y;
#pragma unroll
      for (int w = 0; w < 4; ++w) y[w] = turn_back_pair(raw[kk][w], lds_tab[8 * kk + 4 * hh + w], lds_tab[kHalf + 8 * kk + 4 * hh + w]);
      qf[kk] = __builtin_bit_cast(bf16x8, y);
      if (kk & 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Both: tab != NULL turns the rows back by that rotation, the same for all lanes of the wavefront.
__device__ __forceinline__ void load_queries(const AttendDev& at, bool interleaved, int64_t out, bool on, const float* tab, float* lds_tab,
                                             int lane, bf16x8 (&qf)[8]) {
  float2 t2 = make_float2(1.f, 0.f);
  if (tab) t2 = reinterpret_cast<const float2*>(tab)[lane];
  u32x4 raw[8];
  raw_queries(at, out, lane, raw);
  own_rows(at, on, raw);
  if (tab) {
    turn_queries(raw, interleaved, t2, lds_tab, lane, qf);
  } else {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, raw[kk]);
  }
}

// A wavefront's search in an ascending list: how many of the n entries from v on are smaller than x (64 probes a round).
__device__ __forceinline__ int count_below(const int32_t* v, int n, int x, int lane) {
  int at = 0;
  while (n > 64) {
    const int stride = (n + 63) >> 6, i = lane * stride;
    const int c = __popcll(__ballot(i < n && v[at + i] < x));
    if (c == 0) return at;
    const int skip = (c - 1) * stride + 1;
    at += skip;
    n = min(stride - 1, n - skip);
  }
  return at + __popcll(__ballot(lane < n && v[at + lane] < x));
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// q' = bf16(R(-delta_i) q): one wavefront per query row (all heads of one token of one agent)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void tdk_attend_qrot_kernel(const RoundDev rd, const AttendDev at) {
  const int64_t row = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);   // (agent, qi, hq)
  const int64_t n_rows = (int64_t)rd.n_agents * at.n_q * at.n_q_heads;
  if (row >= n_rows) return;
  const int lane = threadIdx.x & 63;
  const int agent = (int)(row / ((int64_t)at.n_q * at.n_q_heads));
  const uint16_t* src = reinterpret_cast<const uint16_t*>(at.q) + row * kHeadDim;
  const int ia = rd.interleaved ? 2 * lane : lane;
  const int ib = rd.interleaved ? 2 * lane + 1 : lane + kHalf;
  // the kernels after this one work with |scale|: a negative scale flips the sign of every query copy (exact)
  const uint32_t flip = at.q_flip ? 0x8000u : 0u;
  const float xa = __uint_as_float((uint32_t)(src[ia] ^ flip) << 16), xb = __uint_as_float((uint32_t)(src[ib] ^ flip) << 16);
  // one copy per segment of the agent's layout: every segment has its own offset
  const int seg0 = rd.seg_off[agent], nseg = rd.seg_off[agent + 1] - seg0;
  for (int k = 0; k < nseg; ++k) {
    const float* tab = rd.segtab + (size_t)(seg0 + k) * (2 * kHalf);
    uint16_t* dst = reinterpret_cast<uint16_t*>(at.qrot) + (row * at.max_seg + k) * kHeadDim;
    const float c = tab[lane], s = tab[kHalf + lane];
    // rotation by -delta: y_a = x_a cos + x_b sin, y_b = x_b cos - x_a sin
    dst[ia] = (uint16_t)(pack2(__builtin_fmaf(xa, c, __fmul_rn(xb, s)), 0.f) & 0xffffu);
    dst[ib] = (uint16_t)(pack2(__builtin_fmaf(xb, c, -__fmul_rn(xa, s)), 0.f) & 0xffffu);
  }
  // the queries the listed pages meet: as they are, or turned back by the distance the stored values
  // have moved since they were encoded (then one such copy per segment: diff_seg copies per row)
  for (int k = 0; k < (at.seg_moved ? nseg : 1); ++k) {
    uint16_t* dst2 = reinterpret_cast<uint16_t*>(at.qdiff) + (row * at.diff_seg + k) * kHeadDim;
    uint16_t za = (uint16_t)(src[ia] ^ flip), zb = (uint16_t)(src[ib] ^ flip);
    if (at.seg_moved) {
      const float* td = rd.segtab_diff + (size_t)(seg0 + k) * (2 * kHalf);   // identity tables copy exactly
      const float c2 = td[lane], s2 = td[kHalf + lane];
      if (c2 != 1.f || s2 != 0.f) {
        za = (uint16_t)(pack2(__builtin_fmaf(xa, c2, __fmul_rn(xb, s2)), 0.f) & 0xffffu);
        zb = (uint16_t)(pack2(__builtin_fmaf(xb, c2, -__fmul_rn(xa, s2)), 0.f) & 0xffffu);
      }
    }
    dst2[ia] = za;
    dst2[ib] = zb;
  }
}

// ---------------------------------------------------------------------------------------------
// master pass: S^T = K Q'^T and O^T += V^T P^T per 32-token tile, online softmax per query row
// grid: one linear id = KV head + heads * (block of 128 query rows + row blocks * (session * n_chunks + chunk))
// ---------------------------------------------------------------------------------------------
constexpr int kMasterKs = kBigTile * kKsStride, kMasterVs = kBigTile * kVsStride;      // bf16 elements of the two tiles
constexpr int kMaskWords = 2;                                                          // 64-bit words of a row's page mask: 128 pages per chunk
constexpr int kMasterLds = (kMasterKs + kMasterVs) * 2 + kRowsPerBlock * kMaskWords * 8;   // bytes, with the page masks

// One workgroup of the master pass: KV head h, chunk number `sc` = session * n_chunks + chunk, row block zb.
// lds: kMasterLds bytes, 16-byte aligned.
// Identity layouts: the query rows are rotated back here, from the caller's q.  SEG (per-agent block orders): they are
// read from the copies that the qrot kernel leaves, one per segment.
template <bool SEG>
__device__ __forceinline__ void attend_master_body(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const AttendDev& at,
                                                   unsigned char* lds, int h, int sc, int zb) {
  uint16_t* Ks = reinterpret_cast<uint16_t*>(lds);
  uint16_t* Vs = Ks + kMasterKs;
  uint64_t* s_mask = reinterpret_cast<uint64_t*>(Vs + kMasterVs);   // bit p: page p of this chunk is listed in the row's agent's diff

  const int session = sc / at.n_chunks, chunk = sc - session * at.n_chunks;
  const SessionDev sd = rd.sess[session];
  const int tok_begin = chunk * at.chunk_tokens;
  if (tok_begin >= sd.span || sd.n_agents == 0) return;
  const int rows = sd.n_agents * at.n_q * at.group;
  const int row_begin = zb * kRowsPerBlock;
  if (row_begin >= rows) return;
  const int T = rd.page_tokens;
  const int tok_end = min(sd.span, tok_begin + at.chunk_tokens);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;

  // which pages of this chunk each row's agent lists in its diff (those tokens belong to the other kernel)
  if (threadIdx.x < kRowsPerBlock) {
    uint64_t mask[kMaskWords] = {0, 0};
    const RowRef rr = row_ref(rd, sd, at, h, row_begin + threadIdx.x);
    if (rr.agent >= 0) {
      int64_t lo = d.offset[rr.agent], hi = lo + d.count[rr.agent];
      if (lo < 0) lo = 0;
      if (hi > d.capacity) hi = d.capacity;
      const int pg0 = tok_begin / T, pg1 = (tok_end - 1) / T;
      int64_t a = lo, b = hi;
      while (a < b) {                      // first listed page >= pg0
        const int64_t mid = (a + b) >> 1;
        if (d.idx[mid] < pg0) a = mid + 1; else b = mid;
      }
      for (; a < hi; ++a) {
        const int p = d.idx[a];
        if (p > pg1 || p < pg0) break;
        const int rel_p = p - pg0;
        if (rel_p < 64) mask[0] |= (uint64_t)1 << rel_p; else mask[1] |= (uint64_t)1 << (rel_p - 64);
      }
    }
    s_mask[kMaskWords * threadIdx.x] = mask[0];
    s_mask[kMaskWords * threadIdx.x + 1] = mask[1];
  }

  // this lane's query row: its B operands (8 steps of 16 along the head dimension) stay in registers.
  // With per-agent block layouts every segment has its own copy of the row (rotated back by that
  // segment's offset); seg_k follows the segment that holds the current token.
  const RowRef mine = row_ref(rd, sd, at, h, row_begin + wave * kRowsPerWave + n);
  const uint16_t* q_rows = reinterpret_cast<const uint16_t*>(at.qrot) + mine.out * at.max_seg * kHeadDim;
  auto load_q = [&](int k, bool on, bf16x8 (&f)[8]) {
    const u32x4* qp = reinterpret_cast<const u32x4*>(q_rows + (size_t)k * kHeadDim);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u32x4 v = {0, 0, 0, 0};
      if (on) v = qp[2 * kk + hh];
      f[kk] = __builtin_bit_cast(bf16x8, v);
    }
  };
  bf16x8 qf[8];
  int seg_base = 0, seg_n = 1, seg_k = 0;
  if (SEG && mine.agent >= 0) {
    seg_base = rd.seg_off[mine.agent];
    seg_n = rd.seg_off[mine.agent + 1] - seg_base;
    while (seg_k + 1 < seg_n && rd.seg_src[seg_base + seg_k + 1] <= tok_begin) ++seg_k;
  }
  if (!SEG) {
    // fragment kk of a lane = elements 16 kk + 8 hh .. + 7 of its row.  Rotation by -delta of the pair (a, b):
    // y_a = x_a cos + x_b sin, y_b = x_b cos - x_a sin, with pair j = (j, j + 64) or (2 j, 2 j + 1).
    u32x4 raw[8];
    const u32x4* qp = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.q) + mine.out * kHeadDim);
    const uint32_t flip = at.q_flip ? 0x80008000u : 0u;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u32x4 v = {0, 0, 0, 0};
      if (mine.agent >= 0) v = qp[2 * kk + hh];
      raw[kk] = u32x4{v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip};
    }
    turn_back32(raw, rd.tab + (size_t)(mine.agent >= 0 ? mine.agent : 0) * (2 * kHalf), rd.interleaved, hh, qf);
  }
  __syncthreads();
  const uint64_t* my_masks = s_mask + kMaskWords * (wave * kRowsPerWave + n);   // (read per step: two registers less)

  RowState rs;
  row_state_init(rs);

  const int64_t head_u4 = 16;                                  // 128 bf16 = 16 chunks of 16 bytes
  const int64_t row_u4 = (int64_t)rd.heads * head_u4;
  // staging: sixteen lanes per token row (coalesced 256-byte reads of one head's K and V), four rows per
  // wavefront instruction; both tiles are kept row-major in LDS (the V operands are read with transposing loads)
  const int st_tok = threadIdx.x >> 4, st_pc = threadIdx.x & 15;

  // 64 tokens per step: the next step's rows travel from HBM to registers while this one is multiplied.
  // kp / vp follow this thread's piece of the rows of the chunk (thread t: token t / 16 of each group of 16,
  // piece t % 16); a step whose 64 tokens all lie inside the span needs no bounds checks.
  u32x4 kv[8];
  const int64_t row16 = 16 * row_u4;                           // sixteen token rows, in 16-byte units
  const u32x4* kp = io.master_k + (sd.master_row0 + tok_begin + st_tok) * row_u4 + h * head_u4 + st_pc;
  const u32x4* vp = io.master_v + (sd.master_row0 + tok_begin + st_tok) * row_u4 + h * head_u4 + st_pc;
  auto fetch = [&](int t0) {                                   // advances kp / vp past the step
    if (t0 + kBigTile <= tok_end) {
#pragma unroll
      for (int e = 0; e < 4; ++e) { kv[e] = __builtin_nontemporal_load(kp + e * row16); kv[4 + e] = __builtin_nontemporal_load(vp + e * row16); }
    } else {
      const u32x4 z = {0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        kv[e] = z; kv[4 + e] = z;
        if (t0 + 16 * e + st_tok < tok_end) { kv[e] = __builtin_nontemporal_load(kp + e * row16); kv[4 + e] = __builtin_nontemporal_load(vp + e * row16); }
      }
    }
    kp += 4 * row16; vp += 4 * row16;
  };
  fetch(tok_begin);
  uint32_t touch = 0;
  // thread t looks after line t % 2 of the K (t % 4 < 2) or V row of token t / 4, two steps ahead
  const u32x4* tp = ((threadIdx.x & 2) ? io.master_v : io.master_k) +
                    (sd.master_row0 + tok_begin + 2 * kBigTile + (threadIdx.x >> 2)) * row_u4 + h * head_u4 + (threadIdx.x & 1) * 8;
  // one 64-token step; WHOLE: all 64 tokens lie inside the span (every step but a ragged last one)
  auto step = [&](int t0, auto whole_tag) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    __syncthreads();                                           // the previous step has been consumed
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      *reinterpret_cast<u32x4*>(Ks + (16 * e + st_tok) * kKsStride + 8 * st_pc) = kv[e];
      *reinterpret_cast<u32x4*>(Vs + (16 * e + st_tok) * kVsStride + 8 * st_pc) = kv[4 + e];
    }
    __syncthreads();
    if (WHOLE && t0 + kBigTile < tok_end) fetch(t0 + kBigTile);
    // The step after that is called into the caches now: one 4-byte read per 128-byte line of its K and V
    // rows (64 tokens x 2 lines x 2 planes = one line per thread), so that its rows, fetched a step from
    // now, come from L2 instead of HBM.  The value is not used.
    if (WHOLE) {
      if (t0 + 2 * kBigTile + (int)(threadIdx.x >> 2) < tok_end) touch = *reinterpret_cast<const uint32_t*>(tp);
      tp += 4 * row16;
    }
    // which of this lane's 32 scores take part: 16-token groups follow the page mask of the row's agent
    // (m4: bit g set = the g-th group of 16 tokens of this step takes part)
    uint32_t m4;
    {
      const uint32_t rel = (uint32_t)(t0 - tok_begin);
      if (T == 16) {
        const uint32_t pg = rel >> 4;                                        // four pages of 16 tokens
        m4 = ~(uint32_t)(my_masks[pg >> 6] >> (pg & 63u)) & 0xfu;
      } else {
        const uint32_t pg = rel >> 5;                                        // two pages of 32 tokens
        const uint32_t m2 = ~(uint32_t)(my_masks[pg >> 6] >> (pg & 63u)) & 0x3u;
        m4 = ((m2 & 1u) ? 0x3u : 0u) | ((m2 & 2u) ? 0xcu : 0u);
      }
      if (mine.agent < 0) m4 = 0;
    }
    f32x16 s0, s1;
    if (!SEG) {
      scores64<true>(Ks, qf, n, hh, s0, s1);
    } else {
      // The step may run over several segments of this row's agent: the scores are computed once per
      // segment met (each with that segment's copy of the query row) and every token keeps the one of the
      // segment it belongs to.  Rows differ in where their segments end; the loop runs while any row has one left.
#pragma unroll
      for (int i = 0; i < 16; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
      const int t_end = t0 + kBigTile;
      bool more = mine.agent >= 0;
      int k = seg_k;
      while (__any(more)) {
        load_q(k, more, qf);
        f32x16 p0, p1;
        scores64<false>(Ks, qf, n, hh, p0, p1);
        const int lo = more ? rd.seg_src[seg_base + k] : 0;
        const int hi = more ? (k + 1 < seg_n ? rd.seg_src[seg_base + k + 1] : sd.span) : 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int ta = t0 + 8 * (i >> 2) + 4 * hh + (i & 3), tb2 = ta + kTile;
          if (ta >= lo && ta < hi) s0[i] = p0[i];
          if (tb2 >= lo && tb2 < hi) s1[i] = p1[i];
        }
        more = more && hi < t_end && k + 1 < seg_n;
        if (more) ++k;
      }
      seg_k = k;                                  // the segment that holds the last token of this step
      if (mine.agent >= 0 && seg_k + 1 < seg_n && rd.seg_src[seg_base + seg_k + 1] <= t_end) ++seg_k;
    }
    if (WHOLE) {
      softmax_pv64_groups(Vs, s0, s1, at.scale, m4, lane, rs);
    } else {
      uint32_t live = ((m4 & 1u) ? 0x000000ffu : 0u) | ((m4 & 2u) ? 0x0000ff00u : 0u) |
                      ((m4 & 4u) ? 0x00ff0000u : 0u) | ((m4 & 8u) ? 0xff000000u : 0u);
#pragma unroll
      for (int i = 0; i < 32; ++i)                                           // ragged end of the span
        if (t0 + 32 * (i >> 4) + 8 * ((i & 15) >> 2) + 4 * hh + (i & 3) >= tok_end) live &= ~(1u << i);
      softmax_pv64(Vs, s0, s1, at.scale, live, lane, rs);
    }
  };
  const int whole_end = tok_begin + (tok_end - tok_begin) / kBigTile * kBigTile;
  for (int t0 = tok_begin; t0 < whole_end; t0 += kBigTile) step(t0, std::true_type{});
  if (whole_end < tok_end) step(whole_end, std::false_type{});
  asm volatile("" : : "v"(touch));                             // keeps the reads above alive

  const float l_tot = rs.l_run + __shfl_xor(rs.l_run, 32);
  if (mine.agent >= 0) {
    const int64_t slot = mine.out * at.n_parts + chunk;
    float4* po = reinterpret_cast<float4*>(at.part_o + slot * kHeadDim);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        po[(32 * b + 8 * q4 + 4 * hh) >> 2] = make_float4(rs.oacc[b][4 * q4], rs.oacc[b][4 * q4 + 1], rs.oacc[b][4 * q4 + 2], rs.oacc[b][4 * q4 + 3]);
    if (hh == 0) { at.part_m[slot] = part_max(rs.m_run, l_tot); at.part_l[slot] = l_tot; }
  }
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void tdk_attend_master_kernel(const RoundDev rd, const LayerDev io, const DiffDev d,
                                                                   const AttendDev at, const int row_blocks) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kMasterLds];
  // one linear id (grid dimensions y and z stop at 65535): KV head fastest, then the row block, then the chunk
  const int h = blockIdx.x % rd.heads, rest = blockIdx.x / rd.heads;
  attend_master_body<true>(rd, io, d, at, lds, h, rest / row_blocks, rest % row_blocks);
}

// ---------------------------------------------------------------------------------------------
// diff pass: the pages an agent's diff lists, from the payload (the "correct" half of skip-or-correct).
// One wavefront per (agent, KV head, piece): a piece is piece_tokens / 32 consecutive 32-token tiles of the agent's
// listed tokens and has its own partial result, so there is nothing to combine inside the kernel; workgroups
// whose piece lies past the end of the agent's list leave at once (the merge knows how many pieces an agent
// has).  The K rows go straight from the payload into the MFMA operand registers, the V rows through one
// row-major tile in LDS.  This form: 17 to 32 query rows per agent and KV head.
// ---------------------------------------------------------------------------------------------

// Vs: this wavefront's V tile, kTile * kVsStride bf16 elements; lane: 0..63.  MOVED: some agent's diff sits at other positions
template <bool MOVED>
__device__ __forceinline__ bool attend_diff32_piece(const RoundDev& rd, const DiffDev& d, const AttendDev& at, uint16_t* Vs,
                                                   int h, int agent, int piece, int lane) {
  const int T = rd.page_tokens;
  int64_t lo = d.offset[agent], hi = lo + d.count[agent];
  if (lo < 0) lo = 0;
  if (hi > d.capacity) hi = d.capacity;
  const int n_tok = hi > lo ? (int)((hi - lo) * T) : 0;
  const int n_tiles = (n_tok + kTile - 1) / kTile;
  const int piece_tiles = at.piece_tokens / kTile;
  const int tile_begin = piece * piece_tiles, tile_end = min(n_tiles, tile_begin + piece_tiles);
  if (tile_begin >= tile_end) return false;     // past the end of the list: so are the pieces after this one
  const int per_agent = at.n_q * at.group;
  const AgentDev ad = rd.agents[agent];
  const SessionDev sd = rd.sess[ad.session];
  const int n = lane & 31, hh = lane >> 5;
  const int64_t row_e = (int64_t)rd.heads * kHeadDim, page_e = (int64_t)T * row_e;
  const uint16_t* pay = reinterpret_cast<const uint16_t*>(d.payload);
  // (offsets inside the agent's part of the payload fit 32 bits: at most 2 P pages of 64 KB or less)
  const uint16_t* apay = pay + lo * 2 * page_e;
  const uint32_t row_u = (uint32_t)row_e, page_u = (uint32_t)page_e, tile_u = (uint32_t)(kTile / T) * 2u * page_u;
  auto tok_off = [&](int tk) { return (uint32_t)(tk / T) * 2u * page_u + (uint32_t)(tk % T) * row_u + (uint32_t)(h * kHeadDim); };
  const int st_row = lane >> 4, st_pc = lane & 15;

  // this lane's query row (at most 32 per agent and KV head: one block)
  const bool row_ok = n < per_agent;
  const int qi = row_ok ? n / at.group : 0, g = row_ok ? n - qi * at.group : 0;
  const int64_t out = ((int64_t)agent * at.n_q + qi) * at.n_q_heads + h * at.group + g;
  bf16x8 qf[8];
  {
    // the listed pages meet the caller's rows as they are, or turned back by the distance the stored values have moved
    const u32x4* qp = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.q) + out * kHeadDim);
    const uint32_t flip = at.q_flip ? 0x80008000u : 0u;
    u32x4 raw[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u32x4 v = {0, 0, 0, 0};
      if (row_ok) v = qp[2 * kk + hh];
      raw[kk] = u32x4{v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip};
      qf[kk] = __builtin_bit_cast(bf16x8, raw[kk]);
    }
    if (MOVED && ad.diff_rot) turn_back32(raw, rd.tab_diff + (size_t)agent * (2 * kHalf), rd.interleaved, hh, qf);
  }
  RowState rs;
  row_state_init(rs);
  // The next tile travels from the payload to registers while the current one is multiplied.  K: lane
  // (n, hh) loads what it multiplies, elements 16 kk + 8 hh .. + 7 of the row of token n.  V: sixteen lanes
  // per 256-byte row, four rows per instruction.  The payload address of a listed token depends on its place
  // in the list alone, so the rows are requested together with the page number; what the page number decides
  // (does the token lie inside the span, which segment holds it) is settled when the tile is used.
  u32x4 kreg[8], vreg[8];
  int p_next = -1;                             // master page of token lane % 32 of the fetched tile (-1: no such token)
  auto fetch = [&](int tile) {
    const int t = tile * kTile + n;
    const bool there = t < n_tok;
    p_next = there ? d.idx[lo + t / T] : -1;
    const u32x4 z = {0, 0, 0, 0};
    const uint32_t tile_off = (uint32_t)tile * tile_u;
    const uint32_t off = tile_off + tok_off(n) + 8u * hh;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      kreg[kk] = z;
      if (there) kreg[kk] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(apay + off + 16 * kk));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      vreg[j] = z;
      if (tile * kTile + 4 * j + st_row < n_tok)
        vreg[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(apay + tile_off + tok_off(4 * j + st_row) + page_u + 8u * st_pc));
    }
  };
  fetch(tile_begin);
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    wave_sync();                               // the previous tile has been consumed
    // bit t of valid: token t of the tile exists and lies inside the span (lanes 32..63 repeat lanes 0..31)
    bool ok = false;
    {
      const int rr = (tile * kTile + n) % T, p = p_next;
      ok = p >= 0 && p < sd.pages && p * T + rr < sd.span;
    }
    const uint32_t valid = (uint32_t)__ballot(ok);
    if (valid != 0xffffffffu) {                // rows of tokens that do not count are staged as zeros
      const u32x4 z = {0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (!((valid >> (4 * j + st_row)) & 1u)) vreg[j] = z;     // (their scores are switched off below)
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(Vs + (4 * j + st_row) * kVsStride + 8 * st_pc) = vreg[j];
    f32x16 sacc;
    scores32(kreg, qf, sacc);
    wave_sync();                               // the V tile is complete
    if (tile + 1 < tile_end) fetch(tile + 1);  // the K registers are free: the scores are taken
    // score i of a lane belongs to token 8 (i / 4) + 4 hh + i % 4: four nibbles of `valid`
    const uint32_t vs = valid >> (4 * hh);
    uint32_t live = (vs & 0xfu) | ((vs >> 4) & 0xf0u) | ((vs >> 8) & 0xf00u) | ((vs >> 12) & 0xf000u);
    if (!row_ok) live = 0;
    softmax_pv32(Vs, sacc, at.scale, live, lane, rs);
  }
  // this piece's partial result: lane (n, hh) holds elements 32 b + 8 q + 4 hh + (0..3) of row n
  const float l_tot = rs.l_run + __shfl_xor(rs.l_run, 32);
  if (row_ok) {
    const int64_t slot = out * at.n_parts + at.n_chunks + piece;
    float4* po = reinterpret_cast<float4*>(at.part_o + slot * kHeadDim);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        po[(32 * b + 8 * q4 + 4 * hh) >> 2] = make_float4(rs.oacc[b][4 * q4], rs.oacc[b][4 * q4 + 1], rs.oacc[b][4 * q4 + 2], rs.oacc[b][4 * q4 + 3]);
    if (hh == 0) { at.part_m[slot] = part_max(rs.m_run, l_tot); at.part_l[slot] = l_tot; }
  }
  return true;
}

// the pieces z, z + piece_grid, ... of one list, until one lies past its end
template <bool MOVED>
__device__ __forceinline__ void attend_diff32_body(const RoundDev& rd, const DiffDev& d, const AttendDev& at, uint16_t* Vs,
                                                   int h, int agent, int piece0, int lane) {
  for (int piece = piece0; piece < at.n_pieces; piece += at.piece_grid)
    if (!attend_diff32_piece<MOVED>(rd, d, at, Vs, h, agent, piece, lane)) break;
}

// The same pass with 16 query rows per wavefront: used when an agent brings at most 16 rows per KV head
// (decode: query tokens x heads per KV head), where the 32-row tiles would be five sixths padding.

// Vs: this wavefront's V tile, kTile * kVsStride bf16 elements (the K rows go straight from the payload into
// the MFMA operand registers); lane: 0..63
template <bool SEGMOVED, bool QDIRECT, bool MOVED>
__device__ __forceinline__ bool attend_diff16_piece(const RoundDev& rd, const DiffDev& d, const AttendDev& at, uint16_t* Vs,
                                                   int h, int agent, int piece, int lane) {
  const int T = rd.page_tokens;
  int64_t lo = d.offset[agent], hi = lo + d.count[agent];
  if (lo < 0) lo = 0;
  if (hi > d.capacity) hi = d.capacity;
  const int n_tok = hi > lo ? (int)((hi - lo) * T) : 0;
  const int n_tiles = (n_tok + kTile - 1) / kTile;
  const int piece_tiles = at.piece_tokens / kTile;
  const int tile_begin = piece * piece_tiles, tile_end = min(n_tiles, tile_begin + piece_tiles);
  if (tile_begin >= tile_end) return false;     // past the end of the list: so are the pieces after this one
  const int per_agent = at.n_q * at.group;     // at most 16: one row block
  const AgentDev ad = rd.agents[agent];
  const SessionDev sd = rd.sess[ad.session];
  const int n = lane & 15, g4 = lane >> 4;
  const int64_t row_e = (int64_t)rd.heads * kHeadDim, page_e = (int64_t)T * row_e;
  const uint16_t* pay = reinterpret_cast<const uint16_t*>(d.payload);

  // this lane's query row
  const bool row_ok = n < per_agent;
  const int qi = row_ok ? n / at.group : 0, g = row_ok ? n - qi * at.group : 0;
  const int64_t out = ((int64_t)agent * at.n_q + qi) * at.n_q_heads + h * at.group + g;
  bf16x8 qf[4];
  auto load_q = [&](int k) {
    // QDIRECT (identity layouts): the listed pages meet the caller's rows as they are (but for the sign), or turned back
    // by the distance the stored values have moved
    const u32x4* qp = QDIRECT ? reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.q) + out * kHeadDim)
                              : reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.qdiff) +
                                                               (out * at.diff_seg + k) * kHeadDim);
    const uint32_t flip = QDIRECT && at.q_flip ? 0x80008000u : 0u;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 v = {0, 0, 0, 0};
      if (row_ok) v = qp[4 * kk + g4];
      qf[kk] = __builtin_bit_cast(bf16x8, u32x4{v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip});
    }
    if (QDIRECT && MOVED && ad.diff_rot) turn_back16(qf, rd.tab_diff + (size_t)agent * (2 * kHalf), rd.interleaved, g4);
  };
  if (!SEGMOVED) load_q(0);
  const int seg_base = SEGMOVED ? rd.seg_off[agent] : 0;
  const int seg_n = SEGMOVED ? rd.seg_off[agent + 1] - seg_base : 1;
  RowState16 rs;
  row_state16_init(rs);
  // The next tile travels from the payload to registers while the current one is multiplied.
  // K: lane (n, g) loads what it multiplies -- elements 32 kk + 8 g .. + 7 of the rows of tokens n and 16 + n
  // (the A operands of the two 16-token score products).  V: sixteen lanes per 256-byte row, four rows per
  // instruction, staged row-major in LDS for the transposing reads.
  u32x4 kreg[8], vreg[8];
  int p_next = -1;                             // master page of token lane % 32 of the fetched tile (-1: no such token)
  const int st_row = lane >> 4, st_pc = lane & 15;
  // The payload address of a listed token depends on its place in the list alone, so the rows are requested
  // together with the page number; what the page number decides (does the token lie inside the span, which
  // segment holds it) is settled when the tile is used.
  // (offsets inside the agent's part of the payload fit 32 bits: at most 2 P pages of 64 KB or less)
  const uint16_t* apay = pay + lo * 2 * page_e;
  const uint32_t row_u = (uint32_t)row_e, page_u = (uint32_t)page_e, tile_u = (uint32_t)(kTile / T) * 2u * page_u;
  auto tok_off = [&](int tk) { return (uint32_t)(tk / T) * 2u * page_u + (uint32_t)(tk % T) * row_u + (uint32_t)(h * kHeadDim); };
  auto fetch = [&](int tile) {
    const int t = tile * kTile + (lane & 31);
    p_next = t < n_tok ? d.idx[lo + t / T] : -1;
    const u32x4 z = {0, 0, 0, 0};
    const uint32_t tile_off = (uint32_t)tile * tile_u;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const bool there = tile * kTile + 16 * tt + n < n_tok;
      const uint32_t off = tile_off + tok_off(16 * tt + n) + 8u * g4;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        kreg[2 * kk + tt] = z;
        if (there) kreg[2 * kk + tt] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(apay + off + 32 * kk));
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      vreg[j] = z;
      if (tile * kTile + 4 * j + st_row < n_tok)
        vreg[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(apay + tile_off + tok_off(4 * j + st_row) + page_u + 8u * st_pc));
    }
  };
  fetch(tile_begin);
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    wave_sync();                               // the previous tile has been consumed
    // bit t of valid: token t of the tile exists and lies inside the span (lanes 32..63 repeat lanes 0..31)
    int seg_cur = 0;
    bool ok = false;
    {
      const int rr = (tile * kTile + (lane & 31)) % T, p = p_next;
      if (p >= 0 && p < sd.pages && p * T + rr < sd.span) {
        ok = true;
        if (SEGMOVED)
          while (seg_cur + 1 < seg_n && rd.seg_src[seg_base + seg_cur + 1] <= p * T + rr) ++seg_cur;
      }
    }
    const uint32_t valid = (uint32_t)__ballot(ok);
    if (valid != 0xffffffffu) {                // rows of tokens that do not count are staged as zeros
      const u32x4 z = {0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (!((valid >> (4 * j + st_row)) & 1u)) vreg[j] = z;       // (their scores are switched off below)
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(Vs + (4 * j + st_row) * kVsStride + 8 * st_pc) = vreg[j];
    // scores 0..3 of a lane belong to tokens 4 g + i, scores 4..7 to tokens 16 + 4 g + i
    f32x4a s0, s1;
    if (!SEGMOVED) {
      scores16(kreg, qf, s0, s1);
    } else {
      // the tile's tokens come from up to four segments stored at different distances from today's
      // positions: scores once per segment present, with the queries turned back by that distance
      int sid[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) { sid[i] = __shfl(seg_cur, 4 * g4 + i); sid[4 + i] = __shfl(seg_cur, 16 + 4 * g4 + i); }
#pragma unroll
      for (int i = 0; i < 4; ++i) { s0[i] = 0.f; s1[i] = 0.f; }
      int done = -1;
      while (true) {
        int cand = (lane < kTile && ((valid >> lane) & 1u) && seg_cur > done) ? seg_cur : 0x7fffffff;
#pragma unroll
        for (int sft = 32; sft > 0; sft >>= 1) cand = min(cand, __shfl_xor(cand, sft));
        if (cand == 0x7fffffff) break;
        load_q(cand);
        f32x4a p0, p1;
        scores16(kreg, qf, p0, p1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (sid[i] == cand) s0[i] = p0[i];
          if (sid[4 + i] == cand) s1[i] = p1[i];
        }
        done = cand;
      }
    }
    wave_sync();                               // the V tile is complete
    if (tile + 1 < tile_end) fetch(tile + 1);  // the K registers are free: the scores are taken
    const uint32_t vs = valid >> (4 * g4);
    uint32_t live = (vs & 0xfu) | ((vs >> 12) & 0xf0u);
    if (!row_ok) live = 0;
    softmax_pv16(Vs, s0, s1, at.scale, live, n, g4, rs);
  }
  // this piece's partial result: lane (n, g) holds elements 16 b + 4 g + i of row n
  float l_tot = rs.l_run + __shfl_xor(rs.l_run, 16);
  l_tot += __shfl_xor(l_tot, 32);
  if (row_ok) {
    const int64_t slot = out * at.n_parts + at.n_chunks + piece;
    float4* po = reinterpret_cast<float4*>(at.part_o + slot * kHeadDim);
#pragma unroll
    for (int b = 0; b < 8; ++b) po[4 * b + g4] = make_float4(rs.oacc[b][0], rs.oacc[b][1], rs.oacc[b][2], rs.oacc[b][3]);
    if (g4 == 0) { at.part_m[slot] = part_max(rs.m_run, l_tot); at.part_l[slot] = l_tot; }
  }
  return true;
}

// the pieces z, z + piece_grid, ... of one list, until one lies past its end
template <bool SEGMOVED, bool QDIRECT = false, bool MOVED = false>
__device__ __forceinline__ void attend_diff16_body(const RoundDev& rd, const DiffDev& d, const AttendDev& at, uint16_t* Vs,
                                                   int h, int agent, int piece0, int lane) {
  for (int piece = piece0; piece < at.n_pieces; piece += at.piece_grid)
    if (!attend_diff16_piece<SEGMOVED, QDIRECT, MOVED>(rd, d, at, Vs, h, agent, piece, lane)) break;
}

template <bool SEGMOVED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void tdk_attend_diff16_kernel(const RoundDev rd, const DiffDev d, const AttendDev at) {
  __shared__ __attribute__((aligned(16))) uint16_t Vs[kTile * kVsStride];
  // one linear id: KV head fastest, then the agent, then the wavefront's number among those of its list
  const int h = blockIdx.x % rd.heads, rest = blockIdx.x / rd.heads;
  attend_diff16_body<SEGMOVED>(rd, d, at, Vs, h, rest % rd.n_agents, rest / rd.n_agents, threadIdx.x);
}

// ---------------------------------------------------------------------------------------------
// One agent per wavefront: attention of rounds whose agents bring enough query rows of their own (prefill), and calls with fewer rows
// that attend_plan gives it (short spans, per-agent block orders).  A wavefront owns 32 query rows of ONE agent and KV head and
// walks the span in 64-token steps; the four wavefronts of a workgroup share the master's K and V tiles in LDS,
// whatever agents they belong to.  Because the rows of a wavefront have one agent, everything that depends on
// the agent is uniform: the pages its diff lists (a bit mask in LDS; most steps have none and skip the masking),
// the segment of its layout (one reload of the query fragments per border; the steps run over the borders, and the
// scores of the tokens behind one are taken again).  The same wavefront then adds the
// listed pages from the payload to the same accumulators, so a span that is not split needs no partial results
// and no merge.
// The steps are software-pipelined: the score products of step i + 1 stand beside the exponentials of step i
// in one basic block (the matrix cores and the vector units then work at the same time within a wavefront),
// the K and V tiles are double-buffered with one barrier per step, and the rows of the tiles after that travel
// from memory straight to LDS meanwhile (through registers and LDS writes 204 to 217 us against 198 at the size below).
// What bounds it (25 agents x 64 query tokens x 40 heads over 5000 tokens, 2 wavefronts per SIMD, counters): matrix
// cores are busy 43 % of the time, vector units 47, LDS with operand reads 25, 1.8 us per step of both wavefronts of a SIMD; no
// single pipe is full, the rest is waiting between dependent stages (score products, maxima, exponentials, second
// products) and at the barrier.  64 rows per wavefront (half the LDS bytes per product, one wavefront per SIMD) measured
// the same.
// Measured against rows of all agents in one block plus separate listed-pages and merge launches: 64 query tokens
// per agent 462 -> 206 us (187 now), 16 tokens 140 -> 93 us, 8 tokens 94 -> 70 us.  Per-agent orders of blocks of 200 tokens, steps
// that ended at every border, a chain of reads to find a chunk's first segment and page, tiles through registers -> now:
// 25 agents x 5000 tokens, 20 rows 70 -> 54 us (48 now); 129 x 4307, 35 rows 502 -> 375; blocks of 64, 151 x 937, 80 rows 105 -> 81.
// ---------------------------------------------------------------------------------------------
constexpr int kRowsMaskWords = 32;                        // 32-bit words of a wavefront's page mask
constexpr int kRowsMaxPages = 32 * kRowsMaskWords;        // pages per chunk

struct RowsGrid {
  int32_t blocks;       // workgroups (four wavefronts) per (session, KV head, chunk), for the largest session
  int32_t per_agent;    // wavefronts per agent and KV head
  int32_t direct;       // the span is one chunk: write out / lse here instead of partial results
  int32_t session0;     // first session of this launch
};

// The tiles of these kernels: rows of 256 bytes without padding, as the loads that write LDS directly leave them (a wavefront
// instruction fills 1 KB: four rows), with the 16-byte pieces of a row exchanged so that the reads spread over the banks:
// piece c of K row r stands at place c ^ (r % 16) (the score operands of 16 rows fall on all 64 banks), piece c of
// V row r at c ^ 4 (r % 4) (the 64-byte parts of four rows that a transposing read meets do).
constexpr int kStepTile = kBigTile * kHeadDim * 2;        // bytes of one K or V tile of a step
__device__ __forceinline__ int k_place(int r, int c) { return r * (kHeadDim * 2) + 16 * (c ^ (r & 15)); }
__device__ __forceinline__ int v_place(int r, int c) { return r * (kHeadDim * 2) + 16 * (c ^ (4 * (r & 3))); }

// 16 bytes per lane from memory straight into LDS: lane l's piece goes to byte lds + 16 l.  base and lds are the same for
// all lanes.  The instruction writes no register; the compiler does not see that it is in flight: landed() waits for it,
// before the barrier that hands the tile over.  (The builtin makes every later LDS read of the kernel wait for the
// tile, also reads of the other buffer.)  The wait states: M0 before its use, and base, which a vector instruction may
// have written just before.  (M0 has no other use in these kernels, which a test of the assembly pins: the
// compiler reserves M0 and does not take it in the list of registers that a statement overwrites.)
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(off), "s"(base) : "memory");
}
__device__ __forceinline__ void landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint32_t lds_byte(const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p; }

// One thread's share of the loads of a step's tile: thread t brings piece t % 16 of rows t / 16, 16 + t / 16, ...
struct StepLoader {
  uint32_t row_bytes, k_off, v_off;      // distance of two tokens in memory; this thread's places in the first 16 rows
  int st_tok, st_pc;
  uint32_t lds_wave;                     // where this wavefront's four rows of every sixteen go
  __device__ __forceinline__ StepLoader(int heads) {
    st_tok = threadIdx.x >> 4;
    st_pc = threadIdx.x & 15;
    row_bytes = (uint32_t)heads * (kHeadDim * 2);
    k_off = (uint32_t)st_tok * row_bytes + 16u * (st_pc ^ (st_tok & 15));
    v_off = (uint32_t)st_tok * row_bytes + 16u * (st_pc ^ (4 * (st_tok & 3)));
    lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 1024u;
  }
  // rows 0 .. 63 from `tile` on into the LDS tile at byte `lds`; rows behind `last` repeat that one
  __device__ __forceinline__ void load(const char* tile, int last, uint32_t first, uint32_t lds) const {
    if (last >= kBigTile - 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) load_to_lds(tile + (size_t)(16 * e) * row_bytes, first, lds + 4096u * e + lds_wave);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        load_to_lds(tile, first - (uint32_t)st_tok * row_bytes + (uint32_t)min(16 * e + st_tok, last) * row_bytes, lds + 4096u * e + lds_wave);
    }
  }
};

struct RowsShared {
  unsigned char k[2][kStepTile];
  unsigned char v[2][kStepTile];
  float tab[kWaves][2 * kHalf];                           // rotation table of the query rows being loaded
  uint32_t mask[kWaves][kRowsMaskWords];                  // bit p: page p of the chunk is listed in the wavefront's agent's diff
};
static_assert(kWaves * 2 * kTile * kHeadDim * 2 <= sizeof(RowsShared::k) + sizeof(RowsShared::v),
              "the listed pages' tiles reuse the memory of the master's");

// maximum of a value over the lane pair (n, n + 32)
__device__ __forceinline__ float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int NT>
__device__ __forceinline__ void rows_max(const f32x16 (&s)[NT], float& mx) {
  mx = s[0][0];
#pragma unroll
  for (int i = 1; i < 16 * NT - 1; i += 2)
    mx = __builtin_elementwise_maximum(mx, __builtin_elementwise_maximum(s[i >> 4][i & 15], s[(i + 1) >> 4][(i + 1) & 15]));
  mx = __builtin_elementwise_maximum(mx, s[NT - 1][15]);
}

// mx: each lane's maximum of the masked scores to come (unscaled).  A row's reference point moves when the
// maximum has outgrown it by more than 8.
__device__ __forceinline__ void rows_settle(float mx, float scale, RowState& st) {
  constexpr float kLazy = 8.f;
  const float m = pair_max(mx) * scale;
  if (__any(m > st.m_run + kLazy || (st.m_run == -INFINITY && m != -INFINITY))) {
    const float m_new = m > st.m_run + kLazy || st.m_run == -INFINITY ? fmaxf(st.m_run, m) : st.m_run;
    const float alpha = __expf(st.m_run - (m_new == -INFINITY ? 0.f : m_new));     // 1 for the rows whose reference stays
    st.l_run *= alpha;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.oacc[q][i] *= alpha;
    st.m_run = m_new;
  }
}

// The operands of the two products, from tiles of rows of 256 bytes.  Score product: elements 16 kk + 8 hh .. + 7 of row n
// of the 32 rows from `Ks` on.  Second product: see pv_tr; tokens 16 kk .. + 15, elements 32 q .. + 31.
__device__ __forceinline__ bf16x8 k_operand(const unsigned char* Ks, int kk, int n, int hh) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Ks + (k_place(n, hh) ^ (32 * kk))));
}
__device__ __forceinline__ bf16x8 v_operand(const unsigned char* Vs, int kk, int q, int lane) {
  const int i16 = lane & 15, blk = lane >> 4;
  const unsigned char* p = Vs + (v_place(4 * (blk >> 1) + (i16 >> 2), 2 * (blk & 1)) ^ (64 * q)) + 8 * (i16 & 3);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + (16 * kk) * (kHeadDim * 2)));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + (16 * kk + 8) * (kHeadDim * 2)));
  const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
  return __builtin_bit_cast(bf16x8, u32x4{l2.x, l2.y, h2.x, h2.y});
}

// NT tiles of 32 tokens: weights from the settled scores, sums, and O^T += V^T P^T (see pv_tr for the operands).
template <int NT>
__device__ __forceinline__ void rows_weights_pv(const unsigned char* Vs, const f32x16 (&s)[NT], float scale, int lane, RowState& st) {
  constexpr float kLog2e = 1.4426950408889634f;
  const float c2 = scale * kLog2e;
  const float m2 = -(st.m_run == -INFINITY ? 0.f : st.m_run) * kLog2e;
#pragma unroll
  for (int kk = 0; kk < 2 * NT; ++kk) {
    float p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kk >> 1][8 * (kk & 1) + j], c2, m2));
      st.l_run += p[j];
    }
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack2(p[2 * e], p[2 * e + 1]);
    const bf16x8 pb = __builtin_bit_cast(bf16x8, w);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      st.oacc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(Vs, kk, q, lane), pb, st.oacc[q], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void rows_scores(const unsigned char* Ks, const bf16x8 (&qf)[8], int n, int hh, f32x16 (&s)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) s[t][i] = 0.f;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
#pragma unroll
    for (int t = 0; t < 2; ++t)
      s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(Ks + t * (kStepTile / 2), kk, n, hh), qf[kk], s[t], 0, 0, 0);
}

// One pipelined step: the score products of the next step's K tile (16 operands of 32 tokens x 16 elements), the
// weights of this step's scores, and the products of this step's V tile (16 operands of 32 elements x 16 tokens).
// The order is written down slot by slot, because a wavefront only keeps the matrix cores and the vector units
// busy together if their instructions alternate: a slot is the product(s) of one operand, the LDS read of the
// operand four slots ahead, and a few weights (scale and reference point in one fma, exp2, sum, packing), spread so
// that a slot's vector work takes about as long as its products; the maxima of the new scores stand in the last
// slots.  nx: the raw scores of the next step, mx: their maxima; s is used up.
__device__ __forceinline__ void rows_step(const unsigned char* Ks, const unsigned char* Vs, const bf16x8 (&qf)[8], f32x16 (&s)[2],
                                          f32x16 (&nx)[2], float& mx, float scale, int lane, RowState& st) {
  constexpr float kLog2e = 1.4426950408889634f;
  constexpr int kAhead = 4;                                 // (6 and 8 measured the same)
  const int n = lane & 31, hh = lane >> 5;
  const float c2 = scale * kLog2e;
  const float m2 = -(st.m_run == -INFINITY ? 0.f : st.m_run) * kLog2e;
  auto k_op = [&](int j) { return k_operand(Ks + (j & 1) * (kStepTile / 2), j >> 1, n, hh); };
  auto v_op = [&](int j) { return v_operand(Vs, j >> 2, j & 3, lane); };
  constexpr int kWeights = 32;
  // weight number w, in the order the second products need them: 16 tokens at a time
  uint32_t pw[4][4];
  // in three stages, each a slot after the one before: a chain of scaling, exponential, sum and packing inside one slot
  // is longer than its product and holds up the next one (12 agents x 2496 tokens x 320 rows 67.6 -> 64.8 us)
  auto tile = [](int w) { return w / 16; };
  auto elem = [](int w) { return 8 * ((w / 8) & 1) + w % 8; };
  auto weight = [&](int w) {
    if (w + 2 < kWeights) s[tile(w + 2)][elem(w + 2)] = __builtin_fmaf(s[tile(w + 2)][elem(w + 2)], c2, m2);
    if (w + 1 < kWeights) s[tile(w + 1)][elem(w + 1)] = __builtin_amdgcn_exp2f(s[tile(w + 1)][elem(w + 1)]);
    st.l_run += s[tile(w)][elem(w)];
    if (w & 1) pw[w / 8][(w % 8) >> 1] = pack2(s[tile(w - 1)][elem(w - 1)], s[tile(w)][elem(w)]);
  };
  // weights before the first product (while its operands arrive), per slot of the first and of the second products;
  // the eight weights of 16 tokens must stand before the four slots that use them
  constexpr int kPre = 4, kFirst = 1, kSecond = 1;
  static_assert(kPre + 16 * kFirst >= 8 && kPre + 16 * kFirst + 4 * kSecond >= 16 && kPre + 16 * kFirst + 8 * kSecond >= 24 &&
                kPre + 16 * kFirst + 12 * kSecond >= 32, "weights stand before their products");
  // The step goes before whatever the unit's other wavefront does between its own steps (tiles, masks, listed pages): with that, and
  // one weight per slot to the end instead of two in the first of the second products, 25 agents x 4992 tokens x 320 rows 196.8
  // -> 191.9 us, x 2496 with a fifth of the pages listed 139.5 -> 131.4.
  __builtin_amdgcn_s_setprio(1);
  bf16x8 ka[kAhead], va[kAhead];
#pragma unroll
  for (int j = 0; j < kAhead; ++j) ka[j] = k_op(j);
  s[tile(0)][elem(0)] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[tile(0)][elem(0)], c2, m2));
  s[tile(1)][elem(1)] = __builtin_fmaf(s[tile(1)][elem(1)], c2, m2);
#pragma unroll
  for (int w = 0; w < kPre; ++w) weight(w);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    f32x16 c;
    if (j < 2) {
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = 0.f;
    } else {
      c = nx[j & 1];
    }
    nx[j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[j % kAhead], qf[j >> 1], c, 0, 0, 0);
    if (j + kAhead < 16) ka[j % kAhead] = k_op(j + kAhead);
    else va[j % kAhead] = v_op(j + kAhead - 16);
#pragma unroll
    for (int w = 0; w < kFirst; ++w)
      if (kPre + kFirst * j + w < kWeights) weight(kPre + kFirst * j + w);
    __builtin_amdgcn_sched_barrier(0);
  }
  mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pw[j >> 2][0], pw[j >> 2][1], pw[j >> 2][2], pw[j >> 2][3]});
    st.oacc[j & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[j % kAhead], pb, st.oacc[j & 3], 0, 0, 0);
    if (j + kAhead < 16) va[j % kAhead] = v_op(j + kAhead);
#pragma unroll
    for (int w = 0; w < kSecond; ++w)
      if (kPre + 16 * kFirst + kSecond * j + w < kWeights) weight(kPre + 16 * kFirst + kSecond * j + w);
    if (j >= 8) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int i = 4 * (j - 8) + 2 * q;
        mx = __builtin_elementwise_maximum(mx, __builtin_elementwise_maximum(nx[i >> 4][i & 15], nx[i >> 4][(i & 15) + 1]));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
}

// The pages d.idx[l0 .. l1) of the agent's list, 32 tokens at a time, from the payload, through K and V tiles that
// only this wavefront uses (kListedLds bytes).  The payload address of a listed token depends on its place in the list
// alone, so the next tile travels to registers while this one is multiplied.  load_q(k) loads the query
// fragments for tokens of segment k (SEGMOVED; otherwise called once with 0).  Which segment a token belongs to is in the
// agent's page table (`pages`, tables counted from seg_base): one read, where a search through the segments' first tokens
// is a chain of reads per tile.
constexpr int kListedLds = 2 * kTile * kHeadDim * 2;

// 32 tokens of a list on their way to registers: four rows per access, sixteen lanes per 256-byte row.
struct ListedTile {
  u32x4 k[8], v[8];
  int page;                                      // master page of token lane % 32 (-1: no such token)
};
struct ListedRows {
  const u32x4* pay;                              // this lane's piece of the first row
  const int32_t* idx;
  uint32_t row_u, page_u;
  int n_tok, last, lg, T;                        // last: the list's last token (0 for an empty list)
  // elsewhere: memory to read where the list is empty
  __device__ __forceinline__ ListedRows(const RoundDev& rd, const DiffDev& d, int h, int64_t l0, int n_pages, int lane, const void* elsewhere) {
    T = rd.page_tokens;
    lg = T == 16 ? 4 : 5;
    n_tok = max(n_pages, 0) * T;
    last = max(n_tok - 1, 0);
    // (offsets inside the chunk's part of the payload fit 32 bits: at most 2 x 1024 pages of 64 KB or less)
    pay = n_pages > 0 ? d.payload + (l0 * 2 * T * rd.heads + h) * 16 + (lane & 15) : reinterpret_cast<const u32x4*>(elsewhere);
    idx = d.idx + l0;
    row_u = n_pages > 0 ? (uint32_t)rd.heads * 16u : 0u;
    page_u = (uint32_t)T * row_u;
  }
  __device__ __forceinline__ void fetch(int t0, int lane, ListedTile& x) const {      // (a token past the list's end reads the last one: no branch around the loads)
    x.page = t0 + (lane & 31) < n_tok ? idx[(t0 + (lane & 31)) >> lg] : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int t = min(t0 + 4 * j + (lane >> 4), last);
      const u32x4* p = pay + (uint32_t)(t >> lg) * 2u * page_u + (uint32_t)(t & (T - 1)) * row_u;
      x.k[j] = p[0];
      x.v[j] = p[page_u];
    }
  }
};

// x: the first tile, asked for earlier; qf: the rows that it meets (SEGMOVED: load_q)
template <bool SEGMOVED, class LoadQ>
__device__ __forceinline__ void rows_listed(const AttendDev& at, const SessionDev& sd, unsigned char* lds, const ListedRows& list, ListedTile& x,
                                            const PageTab* pages, int seg_base, int lane, bf16x8 (&qf)[8], LoadQ load_q, RowState& st) {
  if (list.n_tok <= 0) return;
  unsigned char* Ks = lds;
  unsigned char* Vs = lds + kTile * kHeadDim * 2;
  const int T = list.T, lg = list.lg, n_tok = list.n_tok, n = lane & 31, hh = lane >> 5, st_row = lane >> 4, st_pc = lane & 15;
  auto fetch = [&](int t0) __attribute__((always_inline)) { list.fetch(t0, lane, x); };
  int loaded = -1;                               // SEGMOVED: the segment whose turned rows qf holds
  for (int t0 = 0; t0 < n_tok; t0 += kTile) {
    wave_sync();                                 // the previous tile has been consumed
    int seg_cur = 0;
    bool ok = false;
    {
      const int m = (x.page << lg) + ((t0 + n) & (T - 1));
      if (x.page >= 0 && x.page < sd.pages && m < sd.span) {
        ok = true;
        if (SEGMOVED) {
          const PageTab pt = pages[x.page];
          seg_cur = (((uint32_t)pt.z >> (m & (T - 1))) & 1u ? pt.y : pt.x) - seg_base;
        }
      }
    }
    const uint32_t valid = (uint32_t)__ballot(ok);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      u32x4 v = x.v[j];
      if (!((valid >> (4 * j + st_row)) & 1u)) v = u32x4{0, 0, 0, 0};      // rows of tokens that do not count
      *reinterpret_cast<u32x4*>(Ks + k_place(4 * j + st_row, st_pc)) = x.k[j];
      *reinterpret_cast<u32x4*>(Vs + v_place(4 * j + st_row, st_pc)) = v;
    }
    wave_sync();                                 // the tile is complete
    if (!SEGMOVED && t0 + kTile < n_tok) fetch(t0 + kTile);
    f32x16 s[1];
    auto scores = [&](f32x16 (&sc)[1]) __attribute__((always_inline)) {
      f32x16 y;                                  // two chains of products
#pragma unroll
      for (int i = 0; i < 16; ++i) { sc[0][i] = 0.f; y[i] = 0.f; }
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const bf16x8 a = k_operand(Ks, kk, n, hh);
        if (kk & 1) y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], y, 0, 0, 0);
        else sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], sc[0], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[0][i] += y[i];
    };
    if (!SEGMOVED) {
      scores(s);
    } else {
      // tokens of several segments, stored at different distances from today's positions: scores once per
      // segment present, with the queries turned back by that distance, and every token keeps its own
#pragma unroll
      for (int i = 0; i < 16; ++i) s[0][i] = 0.f;
      uint32_t rest = valid;                     // tokens whose scores are still to come
      while (rest != 0u) {
        const int cand = __builtin_amdgcn_readlane(seg_cur, __builtin_ctz(rest));
        const uint32_t mine = (uint32_t)__ballot(ok && seg_cur == cand);     // (lanes 32..63 repeat lanes 0..31)
        rest &= ~mine;
        if (cand != loaded) load_q(cand);        // (lists ascend: the segment of the last tile often goes on in this one)
        loaded = cand;
        f32x16 one[1];
        scores(one);
        const uint32_t ms = mine >> (4 * hh);    // score i of a lane belongs to token 8 (i / 4) + 4 hh + i % 4
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if ((ms >> (8 * (i >> 2) + (i & 3))) & 1u) s[0][i] = one[0][i];
      }
      // (only now, although the rows arrive later: in flight during the loop above they cost registers that spill)
      if (t0 + kTile < n_tok) fetch(t0 + kTile);
    }
    if (valid != 0xffffffffu) {
      const uint32_t vs = valid >> (4 * hh);     // score i of a lane belongs to token 8 (i / 4) + 4 hh + i % 4
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (!((vs >> (8 * (i >> 2) + (i & 3))) & 1u)) s[0][i] = -INFINITY;
    }
    float mx;
    rows_max<1>(s, mx);
    rows_settle(mx, at.scale, st);
    rows_weights_pv<1>(Vs, s, at.scale, lane, st);
  }
  wave_sync();
}

template <bool SEG, bool APART>   // APART (SEG only): segments of one agent have moved by different distances since their diff was stored
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tdk_attend_rows_kernel(const RoundDev rd, const LayerDev io, const DiffDev d, const AttendDev at, const RowsGrid rg) {
  __shared__ __attribute__((aligned(16))) RowsShared sh;
  const int h = blockIdx.x % rd.heads, rest = blockIdx.x / rd.heads;
  const int wb = rest % rg.blocks, sc = rest / rg.blocks;
  const int n_ch = max(at.n_chunks, 1);
  const int s_local = sc / n_ch, chunk = sc - s_local * n_ch, session = rg.session0 + s_local;
  const SessionDev sd = scalar_read(rd.sess + session);
  if (wb * kWaves >= sd.n_agents * rg.per_agent) return;
  const int T = rd.page_tokens;
  const int tok_begin = chunk * at.chunk_tokens;
  if (tok_begin >= sd.span && !(rg.direct && sd.span == 0)) return;
  const int tok_end = min(sd.span, tok_begin + at.chunk_tokens);
  const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int a_local = (wb * kWaves + wave) / rg.per_agent;
  const int r0 = (wb * kWaves + wave - a_local * rg.per_agent) * kRowsPerWave;
  const bool active = a_local < sd.n_agents;            // (a wavefront without rows only helps to stage the tiles)
  const int agent = active ? scalar_read(rd.order + sd.order_begin + a_local) : 0;
  const int per_agent_rows = at.n_q * at.group;

  // this lane's query row
  const bool row_ok = active && r0 + n < per_agent_rows;
  const int rr = row_ok ? r0 + n : 0, qi = rr / at.group;
  const int64_t out = ((int64_t)agent * at.n_q + qi) * at.n_q_heads + h * at.group + (rr - qi * at.group);
  bf16x8 qf[8];
  auto load_q = [&](const float* tab) __attribute__((always_inline)) {      // tab: turn the rows back by this rotation (NULL: as they are)
    load_queries(at, rd.interleaved, out, row_ok, tab, sh.tab[wave], lane, qf);
  };
  const int moved = scalar_read(&rd.agents[agent].diff_rot);
  int seg_base = 0, seg_n = 1, seg_k = 0;
  if (SEG && active) {
    seg_base = scalar_read(rd.seg_off + agent);
    seg_n = scalar_read(rd.seg_off + agent + 1) - seg_base;
  }

  RowState st;
  row_state_init(st);

  const StepLoader ld(rd.heads);
  const char* mk = reinterpret_cast<const char*>(io.master_k) + (sd.master_row0 + tok_begin) * (int64_t)ld.row_bytes + h * 256;
  const char* mv = reinterpret_cast<const char*>(io.master_v) + (sd.master_row0 + tok_begin) * (int64_t)ld.row_bytes + h * 256;
  // the tile of the step that begins at token p (rows behind the chunk repeat its last token; their scores are masked)
  auto fetch_k = [&](int p, int buf) __attribute__((always_inline)) {
    const int at_tok = min(p, tok_end - 1);
    ld.load(mk + (int64_t)(at_tok - tok_begin) * ld.row_bytes, tok_end - 1 - at_tok, ld.k_off, lds_byte(sh.k[buf]));
  };
  auto fetch_v = [&](int p, int buf) __attribute__((always_inline)) {
    const int at_tok = min(p, tok_end - 1);
    ld.load(mv + (int64_t)(at_tok - tok_begin) * ld.row_bytes, tok_end - 1 - at_tok, ld.v_off, lds_byte(sh.v[buf]));
  };
  // Per-agent block orders: where a segment begins the rows are read again and turned by that segment's table.  The first tokens
  // of 64 segments stand in the lanes (`src`), from segment `win` on, so that finding the segment of a token is a vote;
  // the next segment's table is asked for when this one's has been used.
  int win = 0, src = 0, seg_next = 0x7fffffff;           // seg_next: where the next segment begins
  float2 seg_tab = make_float2(1.f, 0.f);                // the table that is asked for: segment seg_k
  auto window = [&](int k0) __attribute__((always_inline)) {
    win = k0;
    src = k0 + lane < seg_n ? rd.seg_src[seg_base + k0 + lane] : 0x7fffffff;
  };
  auto table = [&](int k) __attribute__((always_inline)) {
    seg_k = k;
    seg_tab = reinterpret_cast<const float2*>(rd.segtab + (size_t)(seg_base + min(k, seg_n - 1)) * (2 * kHalf))[lane];
  };
  // Asked for before anything else is looked up: the rows, their table, the first tiles.  (Short spans are all start-up and
  // end: with this and the rows written whole, 2 x 32 agents x 132 tokens, 128 rows 25.8 -> 23.5 us, 189 agents x 68 tokens, 256 rows
  // 121.7 -> 114.9; the tiles alone asked for first: no gain, they then delay the rows.  Tiles behind rows that have not arrived yet, and
  // the list in front of them, cost spans of a few steps with masters of several sessions: 10 sessions of 3 agents x 275 tokens, 160 rows 24.9
  // against 24.3 us, nothing listed 19.9 against 19.6; other calls 0.99 to 1.01.)
  u32x4 raw0[8];
  int first = 0x7fffffff;                                // the first 64 entries of the list
  if (tok_end > tok_begin) {
    if (active) {
      raw_queries(at, out, lane, raw0);
      own_rows(at, row_ok, raw0);
      if (SEG) window(0);
      else seg_tab = reinterpret_cast<const float2*>(rd.tab + (size_t)agent * (2 * kHalf))[lane];
    }
    fetch_k(tok_begin, 0);
    fetch_v(tok_begin, 0);
    fetch_k(min(tok_begin + kBigTile, tok_end), 1);
  }
  __builtin_amdgcn_sched_barrier(0);
  // the agent's list, by scalar reads: vector reads would wait for the tiles
  int64_t lo = scalar_read(d.offset + agent), hi = lo + scalar_read(d.count + agent);
  if (lo < 0) lo = 0;
  if (hi > d.capacity) hi = d.capacity;
  const int len = hi > lo ? (int)min<int64_t>(hi - lo, 1 << 30) : 0;
  const int32_t* list = d.idx + lo;
  if (active && tok_end > tok_begin && lane < len) first = list[lane];

  // the part of the agent's list that falls into this chunk, and its page mask
  int64_t l0 = 0, l1 = 0;
  const int pg0 = tok_begin / T;
  if (active && tok_end > tok_begin) {
    const int pg1 = (tok_end - 1) / T + 1;
    if (lane < kRowsMaskWords) sh.mask[wave][lane] = 0u;
    int i0, i1;
    if (len <= 64) {
      i0 = __popcll(__ballot(first < pg0));
      i1 = __popcll(__ballot(first < pg1));
    } else {
      i0 = count_below(list, len, pg0, lane);
      i1 = count_below(list, len, pg1, lane);
    }
    i1 = max(min(i1, i0 + kRowsMaxPages), i0);                                 // (a list this round did not produce)
    l0 = lo + i0;
    l1 = lo + i1;
    wave_sync();
    auto mark = [&](int page) __attribute__((always_inline)) {
      const int rel = page - pg0;
      if (rel >= 0 && rel < kRowsMaxPages) atomicOr(&sh.mask[wave][rel >> 5], 1u << (rel & 31));
    };
    if (len <= 64) {
      if (lane >= i0 && lane < i1) mark(first);
    } else {
      for (int i = i0 + lane; i < i1; i += 64) mark(list[i]);
    }
    wave_sync();
  }

  // ---- the master's tokens ----
  const int lg = T == 16 ? 4 : 5;
  // the two words of the page mask that hold a step's pages (read early, used by mask_scores)
  auto mask_words = [&](int p) __attribute__((always_inline)) {
    const int pg = (p - tok_begin) >> lg;
    return make_uint2(sh.mask[wave][min(pg >> 5, kRowsMaskWords - 1)], sh.mask[wave][min((pg >> 5) + 1, kRowsMaskWords - 1)]);
  };
  // Masks the scores of the step [p, end): listed pages and tokens behind its end.  Few steps need it; those get
  // their maxima again.
  auto mask_scores = [&](int p, int end, uint2 words, f32x16 (&s)[2], float& mx) __attribute__((always_inline)) {
    const int rel = p - tok_begin, pg = rel >> lg, n_pages = ((rel + kBigTile - 1) >> lg) - pg + 1;
    const uint64_t both = ((uint64_t)__builtin_amdgcn_readfirstlane(words.y) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane(words.x);
    const uint32_t listed = (uint32_t)(both >> (pg & 31)) & ((1u << n_pages) - 1u);      // bit q: page pg + q is listed (at most five pages)
    const int left = end - p;                            // tokens of this step
    if (listed == 0u && left >= kBigTile) return;
    uint64_t dead = left < kBigTile ? ~0ull << left : 0ull;                              // bit t: token t of the step does not count
    const uint64_t page_bits = T == 16 ? 0xffffull : 0xffffffffull;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int at_tok = (q << lg) - (rel & (T - 1));
      if (((listed >> q) & 1u) && at_tok < kBigTile) dead |= at_tok >= 0 ? page_bits << at_tok : page_bits >> -at_tok;
    }
    const uint32_t d0 = (uint32_t)dead >> (4 * hh), d1 = (uint32_t)(dead >> 32) >> (4 * hh);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if ((d0 >> (8 * (e >> 2) + (e & 3))) & 1u) s[0][e] = -INFINITY;
      if ((d1 >> (8 * (e >> 2) + (e & 3))) & 1u) s[1][e] = -INFINITY;
    }
    rows_max<2>(s, mx);
  };
  auto enter = [&](int p, const u32x4 (&raw)[8]) __attribute__((always_inline)) {      // the segment of token p, p not before the current one
    int c = __popcll(__ballot(src <= p));
    while (c == 64) { window(win + 63); c = __popcll(__ballot(src <= p)); }
    seg_next = __builtin_amdgcn_readlane(src, c);
    if (seg_k != win + c - 1) table(win + c - 1);
    turn_queries(raw, rd.interleaved, seg_tab, sh.tab[wave], lane, qf);
    table(seg_k + 1);
  };
  // The scores of the step [p, end) were taken with the rows of the segment of its first token: those of the tokens of
  // further segments are taken again, for the 32-token tiles that have some.  Leaves the rows of the segment of `end`.
  // (With steps that end at every border instead, blocks of 200 tokens took four steps per block.)
  auto follow = [&](const unsigned char* Ks, int p, int end, f32x16 (&s)[2], float& mx) __attribute__((always_inline)) {
    bool again = false;
    while (seg_next <= end && seg_next < tok_end) {
      const int b = seg_next - p;                        // the first token of the step that belongs to the next segment
      {
        u32x4 raw[8];
        raw_queries(at, out, lane, raw);
        own_rows(at, row_ok, raw);
        enter(seg_next, raw);
      }
      if (b >= kBigTile) break;
      again = true;
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (b >= kTile * (t + 1)) continue;
        f32x16 x;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(Ks + t * (kStepTile / 2), kk, ln & 31, ln >> 5), qf[kk], x, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) s[t][e] = kTile * t + 8 * (e >> 2) + 4 * (ln >> 5) + (e & 3) >= b ? x[e] : s[t][e];
      }
    }
    if (again) rows_max<2>(s, mx);
  };
  if (tok_end > tok_begin) {
    f32x16 s0[2], s1[2];
    // starts of this step and of the next one
    int p1 = tok_begin, p2 = min(p1 + kBigTile, tok_end);
    if (active) {
      if (SEG) {
        seg_k = -1;
        enter(p1, raw0);
      } else {
        turn_queries(raw0, rd.interleaved, seg_tab, sh.tab[wave], lane, qf);
      }
    }
    landed();
    __syncthreads();
    if (active) {
      float mx;
      rows_scores(sh.k[0], qf, n, hh, s0);
      rows_max<2>(s0, mx);
      if (SEG) follow(sh.k[0], p1, p2, s0, mx);
      mask_scores(p1, p2, mask_words(p1), s0, mx);
      rows_settle(mx, at.scale, st);
    }
    __syncthreads();                                     // the first step replaces its K tile
    // the weights and second products of the step whose scores are s (buffers `odd`), and the scores of the next one
    auto step = [&](int odd, f32x16 (&s)[2], f32x16 (&nx)[2]) __attribute__((always_inline)) {
      const int p3 = min(p2 + kBigTile, tok_end);
      fetch_k(p3, odd);                                  // the tiles after that travel to LDS meanwhile (nobody reads
      fetch_v(p2, odd ^ 1);                              // these two buffers in this step)
      uint2 words = make_uint2(0u, 0u);
      float mx;
      if (active) {
        words = mask_words(p2);
        int ln = lane;
        if (SEG) asm volatile("" : "+v"(ln));            // (the places in the tiles are worked out again: kept from step to step they spill)
        rows_step(sh.k[odd ^ 1], sh.v[odd], qf, s, nx, mx, at.scale, ln, st);        // (past the last step: scores that are not used)
      }
      if (active && p2 < tok_end) {
        if (SEG) follow(sh.k[odd ^ 1], p2, p3, nx, mx);
        mask_scores(p2, p3, words, nx, mx);
        rows_settle(mx, at.scale, st);
      }
      p1 = p2; p2 = p3;
      landed();
      __syncthreads();
    };
    if (SEG) {
      // (one copy of the step: two of them next to the reloads of the queries cost registers that spill; 83 -> 71 us)
      int odd = 0;
      while (p1 < tok_end) {
        step(odd, s0, s1);
        s0[0] = s1[0];
        s0[1] = s1[1];
        odd ^= 1;
      }
    } else {
      // (A last step without scores, with the first listed tile on its way to the registers that it leaves free, gains 3 to 6 % on spans
      // of a few steps, but the steps before it lose 2.5 %, which 25 agents x 5000 tokens, 320 rows do not get back.)
      while (p1 < tok_end) {
        step(0, s0, s1);
        if (p1 < tok_end) step(1, s1, s0);
      }
    }
  }

  // ---- the listed pages, from the payload ----
  if (active) {
    unsigned char* lds = sh.k[0] + wave * kListedLds;
    const ListedRows listed(rd, d, h, l0, (int)(l1 - l0), lane, mk);
    // Segments that have moved together meet the same rows, so one turn serves the whole list; only lists whose segments have
    // moved by different distances need a turn per segment.
    ListedTile tile;
    if (SEG && APART && moved == 1) {
      listed.fetch(0, lane, tile);
      rows_listed<true>(at, sd, lds, listed, tile, rd.pagetab + rd.agents[agent].flag_off, seg_base, lane, qf,
                            [&](int k) __attribute__((always_inline)) { load_q(rd.segtab_diff + (size_t)(seg_base + k) * (2 * kHalf)); }, st);
    } else if (listed.n_tok > 0) {
      const float* turn = moved == 0 ? nullptr : SEG ? rd.segtab_diff + (size_t)seg_base * (2 * kHalf) : rd.tab_diff + (size_t)agent * (2 * kHalf);
      // (the rows and their table travel with the first tile: nothing waits in between)
      float2 t2 = make_float2(1.f, 0.f);
      u32x4 raw[8];
      if (turn) t2 = reinterpret_cast<const float2*>(turn)[lane];
      raw_queries(at, out, lane, raw);
      listed.fetch(0, lane, tile);
      own_rows(at, row_ok, raw);
      if (turn) {
        turn_queries(raw, rd.interleaved, t2, sh.tab[wave], lane, qf);
      } else {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, raw[kk]);
      }
      rows_listed<false>(at, sd, lds, listed, tile, nullptr, 0, lane, qf, [](int) {}, st);
    }
  }

  // Lane (n, hh) holds elements 32 q + 8 j + 4 hh + (0..3) of row n.  They go out by way of LDS, so that a store instruction
  // writes whole rows (straight from the registers it writes 32 bytes of each of 32 rows; 2 x 79 agents x 90 tokens, 640 rows,
  // 0.4 GB of results: 244.8 -> 233.5 us).  Piece c of row r (16 bytes) stands at place c ^ r.  With 33 to 63 rows per agent, whose
  // second wavefront is mostly empty, the way through LDS is longer than what the stores gain (ten sessions of 5 agents x 73 tokens, 33
  // rows 15.4 against 15.0 us, 25 agents x 64 tokens, 40 rows 11.9 against 11.7; 64 rows 16.6 against 16.8, 32 rows 17.9 against 18.1;
  // own block orders the same or slower).
  if (!active) return;
  const float l_tot = st.l_run + __shfl_xor(st.l_run, 32);
  float f = 1.f;
  if (rg.direct) {
    f = l_tot > 0.f ? 1.f / l_tot : l_tot != l_tot ? l_tot : 0.f;
    if (hh == 0 && row_ok) at.lse[out] = row_lse(st.m_run, l_tot);
  } else if (hh == 0 && row_ok) {
    const int64_t slot = out * at.n_parts + chunk;
    at.part_m[slot] = part_max(st.m_run, l_tot);
    at.part_l[slot] = l_tot;
  }
  float* to = rg.direct ? at.out : at.part_o + (int64_t)chunk * kHeadDim;
  const int64_t pitch = (int64_t)kHeadDim * (rg.direct ? 1 : at.n_parts);
  if (!SEG && per_agent_rows > kRowsPerWave && per_agent_rows < 2 * kRowsPerWave) {
    float4* po = reinterpret_cast<float4*>(to + out * pitch) + hh;
    if (row_ok)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          po[8 * q + 2 * j] = make_float4(st.oacc[q][4 * j] * f, st.oacc[q][4 * j + 1] * f, st.oacc[q][4 * j + 2] * f, st.oacc[q][4 * j + 3] * f);
    return;
  }
  float4* rows = reinterpret_cast<float4*>(sh.k[0] + wave * kListedLds);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      rows[32 * n + ((8 * q + 2 * j + hh) ^ n)] = make_float4(st.oacc[q][4 * j] * f, st.oacc[q][4 * j + 1] * f,
                                                             st.oacc[q][4 * j + 2] * f, st.oacc[q][4 * j + 3] * f);
  wave_sync();
  const int there = min(kRowsPerWave, per_agent_rows - r0);
  for (int r8 = 0; r8 < there; r8 += 8)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r8 + 2 * i + hh;
      const int64_t row = __shfl(out, r);
      if (r < there) reinterpret_cast<float4*>(to + row * pitch)[n] = rows[32 * r + (n ^ r)];
    }
}

// ---------------------------------------------------------------------------------------------
// Packed rows (identity layouts, few rows per agent): the master pass for 128 query rows of a session's agents, whatever
// agents they belong to, with the pipelined steps of the kernel above.  Rows of one wavefront have different agents, so the
// listed pages are masked per lane; those pages are the listed-pages pass's work.
// Where it is used: attend_plan (at most 16 rows per agent and KV head, two row blocks over every tile, enough steps).  250
// agents, ten sessions, 5000 tokens: 1 query token (5 rows) 111 -> 109 us in a graph, 2 tokens (10 rows) 164 -> 153.
// ---------------------------------------------------------------------------------------------
struct PackedShared {
  unsigned char k[2][kStepTile];
  unsigned char v[2][kStepTile];
  uint64_t mask[kRowsPerBlock * kMaskWords];              // bit p: page p of this chunk is listed in the row's agent's diff
};

// KV head h, chunk number `sc` = session * n_chunks + chunk, row block zb
__device__ __forceinline__ void attend_packed_body(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const AttendDev& at,
                                                   PackedShared& sh, int h, int sc, int zb) {
  const int session = sc / at.n_chunks, chunk = sc - session * at.n_chunks;
  const SessionDev sd = rd.sess[session];
  const int tok_begin = chunk * at.chunk_tokens;
  if (tok_begin >= sd.span || sd.n_agents == 0) return;
  const int rows = sd.n_agents * at.n_q * at.group;
  const int row_begin = zb * kRowsPerBlock;
  if (row_begin >= rows) return;
  const int T = rd.page_tokens, lg = T == 16 ? 4 : 5;
  const int tok_end = min(sd.span, tok_begin + at.chunk_tokens);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;

  // rows past the end repeat the last one (their scores are masked), a step past the last one repeats it
  const StepLoader ld(rd.heads);
  const char* mk = reinterpret_cast<const char*>(io.master_k) + (sd.master_row0 + tok_begin) * (int64_t)ld.row_bytes + h * 256;
  const char* mv = reinterpret_cast<const char*>(io.master_v) + (sd.master_row0 + tok_begin) * (int64_t)ld.row_bytes + h * 256;
  const int steps = (tok_end - tok_begin + kBigTile - 1) / kBigTile, last = tok_end - tok_begin - 1;
  auto fetch_k = [&](int i, int buf) __attribute__((always_inline)) {
    const int t0 = min(i, steps - 1) * kBigTile;
    ld.load(mk + (int64_t)t0 * ld.row_bytes, last - t0, ld.k_off, lds_byte(sh.k[buf]));
  };
  auto fetch_v = [&](int i, int buf) __attribute__((always_inline)) {
    const int t0 = min(i, steps - 1) * kBigTile;
    ld.load(mv + (int64_t)t0 * ld.row_bytes, last - t0, ld.v_off, lds_byte(sh.v[buf]));
  };
  fetch_k(0, 0);                                          // (asked for before the page masks are looked up)
  fetch_v(0, 0);
  fetch_k(1, 1);

  // which pages of this chunk each row's agent lists in its diff
  if (threadIdx.x < kRowsPerBlock) {
    uint64_t mask[kMaskWords] = {0, 0};
    const RowRef rr = row_ref(rd, sd, at, h, row_begin + threadIdx.x);
    if (rr.agent >= 0) {
      int64_t lo = d.offset[rr.agent], hi = lo + d.count[rr.agent];
      if (lo < 0) lo = 0;
      if (hi > d.capacity) hi = d.capacity;
      const int pg0 = tok_begin / T, pg1 = (tok_end - 1) / T;
      int64_t a = lo, b = hi;
      while (a < b) {                      // first listed page >= pg0
        const int64_t mid = (a + b) >> 1;
        if (d.idx[mid] < pg0) a = mid + 1; else b = mid;
      }
      for (; a < hi; ++a) {
        const int p = d.idx[a];
        if (p > pg1 || p < pg0) break;
        const int rel_p = p - pg0;
        if (rel_p < 64) mask[0] |= (uint64_t)1 << rel_p; else mask[1] |= (uint64_t)1 << (rel_p - 64);
      }
    }
    sh.mask[kMaskWords * threadIdx.x] = mask[0];
    sh.mask[kMaskWords * threadIdx.x + 1] = mask[1];
  }

  // this lane's query row, rotated back by its agent's offset: its B operands stay in registers
  const RowRef mine = row_ref(rd, sd, at, h, row_begin + wave * kRowsPerWave + n);
  bf16x8 qf[8];
  {
    u32x4 raw[8];
    const u32x4* qp = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(at.q) + mine.out * kHeadDim);
    const uint32_t flip = at.q_flip ? 0x80008000u : 0u;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u32x4 v = {0, 0, 0, 0};
      if (mine.agent >= 0) v = qp[2 * kk + hh];
      raw[kk] = u32x4{v.x ^ flip, v.y ^ flip, v.z ^ flip, v.w ^ flip};
    }
    turn_back32(raw, rd.tab + (size_t)(mine.agent >= 0 ? mine.agent : 0) * (2 * kHalf), rd.interleaved, hh, qf);
  }
  landed();
  __syncthreads();

  // which 16-token groups of step i the lane's agent lists (bit g: group g), read ahead of their use
  const uint64_t* my_masks = sh.mask + kMaskWords * (wave * kRowsPerWave + n);
  auto listed = [&](int i) __attribute__((always_inline)) {
    const uint32_t pg = (uint32_t)min(i, steps - 1) * kBigTile >> lg;              // four pages of 16 tokens or two of 32
    const uint32_t m = (uint32_t)(my_masks[pg >> 6] >> (pg & 63u));
    if (T == 16) return m & 0xfu;
    return ((m & 1u) ? 0x3u : 0u) | ((m & 2u) ? 0xcu : 0u);
  };
  auto mask_scores = [&](int i, uint32_t m4, f32x16 (&s)[2], float& mx) __attribute__((always_inline)) {
    const int left = last + 1 - i * kBigTile;
    if (!__any(m4 != 0u) && left >= kBigTile) return;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const bool off = (m4 >> (2 * t + g)) & 1u;
#pragma unroll
        for (int e = 0; e < 8; ++e) s[t][8 * g + e] = off ? -INFINITY : s[t][8 * g + e];
      }
    if (left < kBigTile) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (32 * t + 8 * (e >> 2) + 4 * hh + (e & 3) >= left) s[t][e] = -INFINITY;
    }
    rows_max<2>(s, mx);
  };
  RowState st;
  row_state_init(st);
  f32x16 s0[2], s1[2];
  {
    float mx;
    rows_scores(sh.k[0], qf, n, hh, s0);
    rows_max<2>(s0, mx);
    mask_scores(0, listed(0), s0, mx);
    rows_settle(mx, at.scale, st);
  }
  __syncthreads();                                        // the first step replaces its K tile
  auto step = [&](int i, f32x16 (&s)[2], f32x16 (&nx)[2]) __attribute__((always_inline)) {
    fetch_k(i + 2, i & 1);                                // (nobody reads these two buffers in this step)
    fetch_v(i + 1, (i + 1) & 1);
    const uint32_t m4 = listed(i + 1);
    float mx;
    rows_step(sh.k[(i + 1) & 1], sh.v[i & 1], qf, s, nx, mx, at.scale, lane, st);
    if (i + 1 < steps) {
      mask_scores(i + 1, m4, nx, mx);
      rows_settle(mx, at.scale, st);
    }
    landed();
    __syncthreads();
  };
  for (int i = 0; i < steps; i += 2) {
    step(i, s0, s1);
    if (i + 1 < steps) step(i + 1, s1, s0);
  }

  const float l_tot = st.l_run + __shfl_xor(st.l_run, 32);
  if (mine.agent >= 0) {
    const int64_t slot = mine.out * at.n_parts + chunk;
    float4* po = reinterpret_cast<float4*>(at.part_o + slot * kHeadDim);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        po[(32 * b + 8 * q4 + 4 * hh) >> 2] = make_float4(st.oacc[b][4 * q4], st.oacc[b][4 * q4 + 1], st.oacc[b][4 * q4 + 2], st.oacc[b][4 * q4 + 3]);
    if (hh == 0) { at.part_m[slot] = part_max(st.m_run, l_tot); at.part_l[slot] = l_tot; }
  }
}

// Both passes in one launch, for rounds with identity layouts and few query rows per agent: one ramp and one drain instead of two, and the listed-pages pass (bound by HBM) streams while
// the master pass (bound by arithmetic and LDS latency) computes.  A workgroup of the listed-pages kind = four
// wavefronts = four KV heads of one agent's piece; the pieces past 0, most of which leave at once, come last.
// Where the kinds run (measured with clock stamps and the hardware ids of the compute units): the device deals
// consecutive workgroup ids to the 8 XCDs, inside an XCD to its 4 shader engines in turn, inside an engine to its
// compute units in turn, and the two slots of a compute unit receive ids 256 apart.  With the kinds alternating
// in groups of 8 ids every engine holds one kind only; alternating in blocks of 32 puts both kinds on every
// engine but still never on one compute unit; blocks of 256 pair one workgroup of each kind on every compute
// unit.  The launch takes the same time in all three (the master workgroups slow down by what the listed ones
// gain: both wait for memory, whose latency under this launch's own 60 MB in flight is 5 to 9 us), so the
// simplest form stays.
static_assert(kWaves * kTile * kVsStride * 2 <= (int)sizeof(PackedShared) && kMasterLds <= (int)sizeof(PackedShared), "one allocation for all");

// MOVED: some agent's diff was stored at other positions (a kernel of its own: turning rows costs registers that the 32-row
// tiles do not have; 100 agents x 1500 tokens, 20 rows, diffs not moved: 69.6 us in one kernel for both, 67.5 in its own).
template <bool ROWS32, bool PIPELINED, bool MOVED>    // PIPELINED: the master kind with pipelined steps; ROWS32: the listed-pages kind with 32-row tiles (17 to 32 rows per agent and KV head) or 16-row tiles
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void tdk_attend_fused_kernel(const RoundDev rd, const LayerDev io, const DiffDev d,
                                                                  const AttendDev at, const FusedGrid fg) {
  constexpr int kLds = PIPELINED ? (int)sizeof(PackedShared) : kMasterLds > kWaves * kTile * kVsStride * 2 ? kMasterLds : kWaves * kTile * kVsStride * 2;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
  const int bid = blockIdx.x;
  // ids alternate between the kinds in groups of eight while both last (consecutive ids go to different XCDs,
  // so both kinds reach every XCD, on different shader engines), then come the master workgroups that are left,
  // then the other kind's
  const int groups = min(fg.n_master, fg.n_diff0) >> 3;
  int m_id = -1, d_id = -1;
  if (bid < 16 * groups) {
    const int at8 = (bid >> 4) * 8 + (bid & 7);
    if (bid & 8) d_id = at8; else m_id = at8;
  } else {
    const int r = bid - 16 * groups, m_left = fg.n_master - 8 * groups;
    if (r < m_left) m_id = 8 * groups + r; else d_id = 8 * groups + (r - m_left);
  }
  if (m_id >= 0) {
    const int h = m_id % rd.heads, rest = m_id / rd.heads;
    // the row blocks of one (chunk, KV head) get ids 8 apart: same XCD, one after the other, so the second
    // finds the tiles in that XCD's L2
    if (PIPELINED) attend_packed_body(rd, io, d, at, *reinterpret_cast<PackedShared*>(lds), h, rest / fg.row_blocks, rest % fg.row_blocks);
    else attend_master_body<false>(rd, io, d, at, lds, h, rest / fg.row_blocks, rest % fg.row_blocks);
  } else {
    const int piece = d_id / fg.n_diff0, rem = d_id - piece * fg.n_diff0;
    const int agent = rem / fg.head_groups, h = (rem - agent * fg.head_groups) * kWaves + (threadIdx.x >> 6);
    if (h >= rd.heads) return;
    uint16_t* Vs = reinterpret_cast<uint16_t*>(lds) + (threadIdx.x >> 6) * (kTile * kVsStride);
    if (ROWS32) attend_diff32_body<MOVED>(rd, d, at, Vs, h, agent, piece, threadIdx.x & 63);
    else attend_diff16_body<false, true, MOVED>(rd, d, at, Vs, h, agent, piece, threadIdx.x & 63);
  }
}

// ---------------------------------------------------------------------------------------------
// merge: out = sum_c o_c e^(m_c - M) / sum_c l_c e^(m_c - M), lse = M + log(that sum); one wavefront per row
// A chain of small reads: what the row's agent lists decides which parts exist.  So the rows of the first chunks, up to eight and as
// many as every session has (reading eight of all sessions: one of 5000 and nine of 300 tokens, 25 agents each, 45.9 us instead of
// 41.9), and all maxima and sums (up to 64 parts) are asked for before that is known; what does not exist gets no weight.  A
// half-wavefront takes every other part, 16 bytes per lane.  2 x 8 agents x 1113 tokens, 4 rows 14.2 -> 13.1 us with
// its launch, 6 x 608 tokens, own orders 17.7 -> 16.6, the 10 000 rows of 250 agents x 5000 tokens 12 us as before.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void tdk_attend_merge_kernel(const RoundDev rd, const DiffDev d, const AttendDev at) {
  const int64_t row = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
  const int64_t n_rows = (int64_t)rd.n_agents * at.n_q * at.n_q_heads;
  if (row >= n_rows) return;
  constexpr int kFirst = 8;
  const int lane = threadIdx.x & 63, half = lane >> 5, n = lane & 31;
  const int64_t base = row * at.n_parts;
  const float4* part = reinterpret_cast<const float4*>(at.part_o + base * kHeadDim) + n;
  const int early = min(at.all_chunks, kFirst);
  f32x4a v[kFirst / 2];
  auto ask = [&](int j, int slot, bool there) {
    v[j] = f32x4a{0.f, 0.f, 0.f, 0.f};
    if (there) v[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4a*>(part + (int64_t)slot * (kHeadDim / 4)));
  };
  float m0 = -INFINITY, l0 = 0.f;
  if (lane < at.n_parts) { m0 = at.part_m[base + lane]; l0 = at.part_l[base + lane]; }
#pragma unroll
  for (int j = 0; j < kFirst / 2; ++j) ask(j, 2 * j + half, 2 * j + half < early);

  const int agent = (int)(row / ((int64_t)at.n_q * at.n_q_heads));
  const int span = rd.sess[rd.agents[agent].session].span;
  const int chunks = (span + at.chunk_tokens - 1) / at.chunk_tokens;
  // the chunks of this row's span, then the pieces of its agent's listed pages
  int pieces;
  {
    int64_t lo = d.offset[agent], hi = lo + d.count[agent];
    if (lo < 0) lo = 0;
    if (hi > d.capacity) hi = d.capacity;
    const int64_t n_tok = hi > lo ? (hi - lo) * rd.page_tokens : 0;
    pieces = (int)min<int64_t>((n_tok + at.piece_tokens - 1) / at.piece_tokens, at.n_pieces);   // (a count beyond the session's pages)
  }
  auto exists = [&](int slot) { return slot < chunks || (slot >= at.n_chunks && slot < at.n_chunks + pieces); };
  // a lane per part for the maxima and the weights
  float M = exists(lane) ? m0 : -INFINITY;
  for (int c = lane + 64; c < at.n_chunks + pieces; c += 64)
    if (exists(c)) M = fmaxf(M, at.part_m[base + c]);
#pragma unroll
  for (int sft = 32; sft > 0; sft >>= 1) M = fmaxf(M, __shfl_xor(M, sft));
  // lane n of a half keeps output elements 4 n .. 4 n + 3
  float L = 0.f, a[4] = {0.f, 0.f, 0.f, 0.f};
  auto weight = [&](int slot, float m, float l) {
    float w = 0.f;
    if (exists(slot) && m != -INFINITY) { w = __expf(m - M); L = __builtin_fmaf(l, w, L); }
    return w;
  };
  auto add = [&](int j, float w) {                       // (a part that does not exist or is empty has weight 0; its row was never written)
    if (w != 0.f)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = __builtin_fmaf(v[j][e], w, a[e]);
  };
  float w = weight(lane, m0, l0);
#pragma unroll
  for (int j = 0; j < kFirst / 2; ++j) {
    const float wj = __shfl(w, 2 * j + half);
    if (2 * j + half < early) add(j, wj);
  }
  // the other parts, eight at a time: chunks from `early` on, then pieces
  const int more = max(chunks - early, 0), rest = more + pieces;
  int w_of = 0;                                          // the weights in the lanes are those of slots 64 w_of ..
  for (int r0 = 0; r0 < rest; r0 += kFirst) {
    auto slot_of = [&](int r) { return r < more ? early + r : at.n_chunks + (r - more); };
#pragma unroll
    for (int j = 0; j < kFirst / 2; ++j) ask(j, slot_of(r0 + 2 * j + half), r0 + 2 * j + half < rest);
#pragma unroll
    for (int k = 0; k < kFirst; ++k) {
      const int r = r0 + k;
      if (r >= rest) break;
      const int slot = slot_of(r);
      if ((slot >> 6) != w_of) {                         // (slots ascend: each group of 64 is weighed once)
        w_of = slot >> 6;
        const int c = 64 * w_of + lane;
        w = exists(c) ? weight(c, at.part_m[base + c], at.part_l[base + c]) : 0.f;
      }
      const float wk = __shfl(w, slot & 63);
      if (half == (k & 1)) add(k >> 1, wk);
    }
  }
#pragma unroll
  for (int sft = 32; sft > 0; sft >>= 1) L += __shfl_xor(L, sft);
#pragma unroll
  for (int e = 0; e < 4; ++e) a[e] += __shfl_xor(a[e], 32);
  const float inv = L > 0.f ? 1.f / L : L != L ? L : 0.f;
  if (half == 0) reinterpret_cast<float4*>(at.out + row * kHeadDim)[n] = make_float4(a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv);
  if (lane == 0) at.lse[row] = row_lse(M, L);
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
hipError_t launch_attend_qrot(const RoundDev& rd, const AttendDev& at, hipStream_t st) {
  const int64_t rows = (int64_t)rd.n_agents * at.n_q * at.n_q_heads;
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(tdk_attend_qrot_kernel, dim3((unsigned)((rows + kWaves - 1) / kWaves)), dim3(kBlock), 0, st, rd, at);
  return hipGetLastError();
}

hipError_t launch_attend_master(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const AttendDev& at,
                                int max_rows, hipStream_t st) {
  if (rd.n_sessions == 0 || at.n_chunks == 0 || max_rows == 0) return hipSuccess;
  // the KV heads of one chunk get consecutive workgroup ids: they start together and read neighbouring
  // 256-byte pieces of the same master rows
  // and the row blocks of a chunk follow each other (the second finds the tiles in L2)
  const int row_blocks = (max_rows + kRowsPerBlock - 1) / kRowsPerBlock;
  const int64_t blocks = (int64_t)rd.heads * row_blocks * rd.n_sessions * at.n_chunks;
  if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)blocks);
  hipLaunchKernelGGL(tdk_attend_master_kernel, grid, dim3(kBlock), 0, st, rd, io, d, at, row_blocks);
  return hipGetLastError();
}

hipError_t launch_attend_diff(const RoundDev& rd, const DiffDev& d, const AttendDev& at, hipStream_t st) {
  if (rd.n_agents == 0) return hipSuccess;
  // piece_grid wavefronts per list (agent, KV head): wavefront z takes the pieces z, z + piece_grid, ...
  const int64_t blocks = (int64_t)rd.heads * rd.n_agents * at.piece_grid;
  if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)blocks);
  if (at.seg_moved) hipLaunchKernelGGL(tdk_attend_diff16_kernel<true>, grid, dim3(64), 0, st, rd, d, at);
  else hipLaunchKernelGGL(tdk_attend_diff16_kernel<false>, grid, dim3(64), 0, st, rd, d, at);
  return hipGetLastError();
}

hipError_t launch_attend_fused(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const AttendDev& at,
                               const FusedGrid& fg, bool pipelined, hipStream_t st) {
  const int64_t blocks = (int64_t)fg.n_master + (int64_t)fg.n_diff0 * at.piece_grid;
  if (blocks == 0) return hipSuccess;
  auto with = [](bool b, auto f) { if (b) f(std::true_type{}); else f(std::false_type{}); };
  with(at.diff_moved != 0, [&](auto moved) {
    constexpr bool M = decltype(moved)::value;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, rd, io, d, at, fg); };
    if (at.n_q * at.group > 16) launch(tdk_attend_fused_kernel<true, false, M>);
    else if (pipelined) launch(tdk_attend_fused_kernel<false, true, M>);
    else launch(tdk_attend_fused_kernel<false, false, M>);
  });
  return hipGetLastError();
}

hipError_t launch_attend_rows(const RoundDev& rd, const LayerDev& io, const DiffDev& d, const AttendDev& at, int max_agents,
                              int launch_sessions, hipStream_t st) {
  RowsGrid rg;
  rg.per_agent = (at.n_q * at.group + kRowsPerWave - 1) / kRowsPerWave;
  rg.blocks = (int)(((int64_t)max_agents * rg.per_agent + kWaves - 1) / kWaves);
  rg.direct = at.n_chunks <= 1;
  const int64_t per_session = (int64_t)rd.heads * rg.blocks * (at.n_chunks > 1 ? at.n_chunks : 1);
  for (int s0 = 0; s0 < rd.n_sessions && per_session > 0; s0 += launch_sessions) {     // (nearly always one launch)
    const int64_t blocks = per_session * std::min(launch_sessions, rd.n_sessions - s0);
    if (blocks >= ((int64_t)1 << 31)) return hipErrorInvalidConfiguration;
    rg.session0 = s0;
    const dim3 grid((unsigned)blocks);
    if (rd.seg && at.seg_apart) hipLaunchKernelGGL((tdk_attend_rows_kernel<true, true>), grid, dim3(kBlock), 0, st, rd, io, d, at, rg);
    else if (rd.seg) hipLaunchKernelGGL((tdk_attend_rows_kernel<true, false>), grid, dim3(kBlock), 0, st, rd, io, d, at, rg);
    else hipLaunchKernelGGL((tdk_attend_rows_kernel<false, false>), grid, dim3(kBlock), 0, st, rd, io, d, at, rg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_attend_merge(const RoundDev& rd, const DiffDev& d, const AttendDev& at, hipStream_t st) {
  const int64_t rows = (int64_t)rd.n_agents * at.n_q * at.n_q_heads;
  if (rows == 0) return hipSuccess;
  hipLaunchKernelGGL(tdk_attend_merge_kernel, dim3((unsigned)((rows + kWaves - 1) / kWaves)), dim3(kBlock), 0, st, rd, d, at);
  return hipGetLastError();
}

}  // namespace tdk
