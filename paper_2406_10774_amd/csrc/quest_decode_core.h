// Device-side pieces of the paged decode attention (Figure 5 stage 2 of arXiv
// 2406.10774): streaming one (page, head) block of keys and values through a
// wave with an online softmax.  See quest_decode.hip for the scheme.
#pragma once

#include <type_traits>

#include "quest_common.h"

namespace quest {

#if defined(__HIPCC__)

constexpr float kNegBig = -1.0e30f;  // "no token yet": finite, so exp2(m - m) never sees inf - inf
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Registers of one unit of streaming: up to 16 consecutive tokens of one (page,
// head): kLoads = 4 wave-wide 16-byte loads of keys and 4 of values (2 and 2 for
// pages of 8 tokens).  Pages of 32 or 64 tokens are walked as 2 or 4 such units.
template <int kLoads>  // 2 or 4
struct PageRegsT {
  uint4 k[kLoads], v[kLoads];
  int n_valid;
};

__device__ __forceinline__ float lo(uint32_t h2) {
  return (float)__builtin_bit_cast(half2_t, h2)[0];
}
__device__ __forceinline__ float hi(uint32_t h2) {
  return (float)__builtin_bit_cast(half2_t, h2)[1];
}

struct Softmax {
  float m, l, acc[8];
};

// Unit `unit` (tokens [unit * 4 kLoads, (unit + 1) * 4 kLoads)) of logical page
// `logical_page`, stored in physical page `phys`; pages hold 1 << page_shift tokens.
template <int kLoads>
__device__ __forceinline__ void load_unit(PageRegsT<kLoads>& r, const char* __restrict__ k_pool,
                                          const char* __restrict__ v_pool, int num_heads, int h,
                                          int seq_len, int logical_page, int phys, int unit,
                                          int page_shift, int lane) {
  const size_t row = (((size_t)phys * num_heads + h) << page_shift) + (size_t)unit * (4 * kLoads);
  const size_t off = row * kRowBytes + lane * 16;
#pragma unroll
  for (int i = 0; i < kLoads; ++i) r.k[i] = ld16_stream(k_pool + off + i * 1024);
#pragma unroll
  for (int i = 0; i < kLoads; ++i) r.v[i] = ld16_stream(v_pool + off + i * 1024);
  r.n_valid = min(4 * kLoads, seq_len - (logical_page << page_shift) - unit * (4 * kLoads));
}

// n_valid may be anything up to 4 kLoads, also <= 0 (a unit past the end of a
// partial page): such tokens contribute nothing.
template <int kLoads>
__device__ __forceinline__ void fold_page(Softmax& st, PageRegsT<kLoads>& r, const uint4 qv,
                                          float scale_log2, int grp) {
  float z[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) z[i] = row16_sum(dot8(qv, r.k[i], 0.f)) * scale_log2;
  if (r.n_valid < 4 * kLoads) {  // partial last page: stale slots contribute nothing
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      if (grp + 4 * i >= r.n_valid) {
        z[i] = -INFINITY;
        r.v[i] = make_uint4(0, 0, 0, 0);
      }
    }
  }
  float m_new = st.m;
#pragma unroll
  for (int i = 0; i < kLoads; ++i) m_new = fmaxf(m_new, z[i]);
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
  float p[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) p[i] = __builtin_amdgcn_exp2f(z[i] - m_new);
  float p_sum = p[0] + p[1];
  if (kLoads == 4) p_sum += p[kLoads - 2] + p[kLoads - 1];
  st.l = st.l * alpha + p_sum;
#pragma unroll
  for (int j = 0; j < 8; ++j) st.acc[j] *= alpha;
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    st.acc[0] += p[i] * lo(r.v[i].x);
    st.acc[1] += p[i] * hi(r.v[i].x);
    st.acc[2] += p[i] * lo(r.v[i].y);
    st.acc[3] += p[i] * hi(r.v[i].y);
    st.acc[4] += p[i] * lo(r.v[i].z);
    st.acc[5] += p[i] * hi(r.v[i].z);
    st.acc[6] += p[i] * lo(r.v[i].w);
    st.acc[7] += p[i] * hi(r.v[i].w);
  }
  st.m = m_new;
}

// Merge the online-softmax states of the wave's four DPP rows (lanes 16 apart, then lanes
// 32 apart); every lane ends up with the merged state of its channels.
__device__ __forceinline__ float as_f(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u(float f) { return __builtin_bit_cast(uint32_t, f); }
template <bool kAcross32>
__device__ __forceinline__ void merge_rows_step(Softmax& st) {
  auto pair = [](float v) { return kAcross32 ? pair_across32(as_u(v)) : pair_across16(as_u(v)); };
  const LanePair m = pair(st.m), l = pair(st.l);
  const float m_n = fmaxf(as_f(m.first), as_f(m.second));
  const float a = __builtin_amdgcn_exp2f(as_f(m.first) - m_n);
  const float b = __builtin_amdgcn_exp2f(as_f(m.second) - m_n);
  st.l = as_f(l.first) * a + as_f(l.second) * b;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const LanePair p = pair(st.acc[j]);
    st.acc[j] = as_f(p.first) * a + as_f(p.second) * b;
  }
  st.m = m_n;
}
__device__ __forceinline__ void merge_rows(Softmax& st) {
  merge_rows_step<false>(st);
  merge_rows_step<true>(st);
}

// Partial results of the same outputs, one in each of the first n <= 16 lanes of every DPP row:
// their maximum, the sum of their denominators relative to it, and the lane's weight.  The weights
// are worked out once per wave, side by side, not once per output one after the other.  A wave has
// all of a group's head, two channels a lane, so that a head's weights are worked out once, and a wave that
// has two heads waits twice for the chain over its lanes, not four times (lists of 512 tokens,
// 2 sequences of 64 query / 8 KV heads, 8 splits: 8.2 us, 10.5 with one channel a lane, 10.1 with every output's
// weights its own; 2048 tokens, 16 splits: 10.7, 12.9 and 14.6).  With one head's outputs on two
// waves the chain is longer than their own weights (32 heads 19.9 us a step, 19.8).
struct Merged {
  float m, l, weight;
};
__device__ __forceinline__ Merged merge_parts(float m, float l, int n, int lane) {
  const bool there = (lane & 15) < n;
  Merged r;
  r.m = row16_max(there ? m : kNegBig);
  r.weight = __builtin_amdgcn_exp2f(m - r.m);
  r.l = row16_sum(there ? l * r.weight : 0.f);
  return r;
}
__device__ __forceinline__ float from_lane(float v, int lane) {
  return as_f((uint32_t)__builtin_amdgcn_readlane((int)as_u(v), lane));
}

// ---- Grouped-query attention: one wave, up to kGroupHeads query heads that share the KV
// head, one unit of 16 tokens at a time (pages of 8 tokens: two pages), on the matrix
// cores.  Per unit 4 v_mfma_f32_16x16x32_f16 give the logits (16 tokens x 16 columns) and
// 8 v_mfma_f32_16x16x16_f16 add the weighted values.  At 4 heads the same work is about
// 450 vector instructions per unit, 1720 cycles on a SIMD for 8 KiB; here it is 12 matrix
// instructions and about 100 others, the same for 2 or 8 heads.
//
// Columns: column n belongs to query head n % 8 (heads past the group: a zero query), in
// two copies.  The weights are fp32, at most 2 and the largest at least 1; columns 0-7 carry
// 2^14 times their value rounded to fp16 and columns 8-15 the fp16 of 2^12 times what that
// leaves, so the products with the fp16 values keep 23 bits of every weight down to 2^-28 of
// the largest (below, fp16's subnormal step costs it up to 2^-51 of the largest), and the
// copies are added at the end.
//
// Error against 64 bits, 2-norm of the outputs, over 31 cases of 16 to 64 query heads
// (ratio to the error of the query heads one by one on the vector unit, geometric mean): 0.94, lse
// 1.00.  Two things matter for that.  Logits: the four products of 32 channels go to sums of
// their own and are added as a tree; one after the other into one sum they gave 1.28.
// Weights: exp2 takes the distance to the largest logit, which is exact near it, and the power
// of two is multiplied on; with the power in the exponent the error of lse was 1.7 times as large.
//
// Operand layouts (lane l: c = l % 16, g = l / 16).  Logits: row m of the first operand is
// token 4 (m % 4) + m / 4, so the result leaves lane (c, g) with column c, tokens 4i + g, i =
// 0..3, which is what the second product wants as its second operand.  Values: load r
// of a unit leaves lane (c, g) with token 4r + g, channels 8c..8c+7; half e of the four
// loads is row c (channel 8c + e) of the first operand of the e-th product.  Nothing moves
// between lanes.  Keys are loaded like values and turned into rows through LDS (4 KiB per
// wave, the 16-byte chunks of token t exclusive-ored with t: no bank conflicts); loaded as
// the operand wants them, 64 bytes of each token per load, they held a compute unit to 30
// KiB per us.
constexpr int kGroupHeads = 8;
constexpr float kWeightScale = 16384.f, kRestScale = 4096.f;  // 2^14, 2^12: a rest is at most 2^3
constexpr int kGroupStride = kHeadDim + 4;  // floats per head in LDS: lanes spread over the banks
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

// Tokens of a unit that hold data: tokens [0, first) of the first eight and, of the others,
// [8, 8 + second); anything from below zero to above eight.
struct GroupRegs {
  uint4 k[4], v[4];
  int first, second;
};

struct GroupState {
  char* stage;      // kRowBytes * 16 bytes of LDS of this wave
  uint4 q[4];       // query of column c's head: channels 32j + 8g .. +7
  f32x4_t acc[8];   // [e]: channels 8 (4g + i) + e of column c
  float ref, l;     // exponent reference of the column (log2), this lane's share of its sum
};

__device__ __forceinline__ void group_init(GroupState& st, char* stage, const char* __restrict__ q,
                                           int heads, int lane) {
  st.stage = stage;
  const int head = lane & (kGroupHeads - 1);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 v = ld16(q + (head < heads ? head : 0) * kRowBytes + j * 64 + (lane >> 4) * 16);
    st.q[j] = head < heads ? v : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) st.acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  st.ref = kNegBig;
  st.l = 0.f;
}

// base_a: byte offset of the unit's first token in the pools; base_b: offset that token 8
// has minus 8 rows (the same as base_a unless a unit is two pages).
__device__ __forceinline__ void group_load(GroupRegs& r, const char* __restrict__ k_pool,
                                           const char* __restrict__ v_pool, size_t base_a,
                                           size_t base_b, int lane) {
#pragma unroll
  for (int i = 0; i < 4; ++i) r.k[i] = ld16_stream(k_pool + (i < 2 ? base_a : base_b) + i * 1024 + lane * 16);
#pragma unroll
  for (int i = 0; i < 4; ++i) r.v[i] = ld16_stream(v_pool + (i < 2 ? base_a : base_b) + i * 1024 + lane * 16);
}

__device__ __forceinline__ void group_fold(GroupState& st, GroupRegs& r, float scale_log2, int lane) {
  const int g = lane >> 4, c = lane & 15;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = 4 * i + g;
    st16(st.stage + t * kRowBytes + ((c ^ t) << 4), r.k[i]);
  }
  lds_in_order();
  f32x4_t s[4];
  const int token = 4 * (c & 3) + (c >> 2);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 k = ld16(st.stage + token * kRowBytes + (((4 * j + g) ^ token) << 4));
    s[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, k),
                                                  __builtin_bit_cast(half8_t, st.q[j]),
                                                  f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  }
  lds_in_order();
  float z[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) z[i] = ((s[0][i] + s[1][i]) + (s[2][i] + s[3][i])) * scale_log2;
  if (r.first < 8 || r.second < 8) {  // stale slots contribute nothing, whatever they hold
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = 4 * (i & 1) + g;  // token within its eight
      if (t >= (i < 2 ? r.first : r.second)) {
        z[i] = -INFINITY;
        r.v[i] = make_uint4(0, 0, 0, 0);
      }
    }
  }
  float top = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
  LanePair p2 = pair_across16(as_u(top));
  p2 = pair_across32(as_u(fmaxf(as_f(p2.first), as_f(p2.second))));
  top = fmaxf(as_f(p2.first), as_f(p2.second));
  // weights stay at or below 2: the reference moves only when a logit passes that
  const bool move = top > st.ref + 1.f;
  if (__ballot(move)) {
    const float ref = move ? top : st.ref;
    const float alpha = __builtin_amdgcn_exp2f(st.ref - ref);
    st.ref = ref;
    st.l *= alpha;
#pragma unroll
    for (int e = 0; e < 8; ++e) st.acc[e] *= alpha;
  }
  half4_t w;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p = __builtin_amdgcn_exp2f(z[i] - st.ref);
    sum += p;
    const float scaled = p * kWeightScale;
    const _Float16 part = (_Float16)scaled;
    w[i] = (lane & 8) ? (_Float16)((scaled - (float)part) * kRestScale) : part;
  }
  st.l += sum;
  // halves 2d and 2d + 1 of the four loads
  auto pick = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t sel) {
    const uint2 u = make_uint2(__builtin_amdgcn_perm(b, a, sel), __builtin_amdgcn_perm(d, c, sel));
    return __builtin_bit_cast(half4_t, u);
  };
#define QUEST_PV(d, member)                                                                          \
  st.acc[2 * d] = __builtin_amdgcn_mfma_f32_16x16x16f16(                                             \
      pick(r.v[0].member, r.v[1].member, r.v[2].member, r.v[3].member, 0x05040100u), w,              \
      st.acc[2 * d], 0, 0, 0);                                                                       \
  st.acc[2 * d + 1] = __builtin_amdgcn_mfma_f32_16x16x16f16(                                         \
      pick(r.v[0].member, r.v[1].member, r.v[2].member, r.v[3].member, 0x07060302u), w,              \
      st.acc[2 * d + 1], 0, 0, 0);
  QUEST_PV(0, x)
  QUEST_PV(1, y)
  QUEST_PV(2, z)
  QUEST_PV(3, w)
#undef QUEST_PV
}

// Whether every sum of the wave is finite.  Two parts of a weight times an infinite value are
// not the weight times that value: one of them may be zero or negative.
__device__ __forceinline__ bool group_finite(const GroupState& st) {
  float s = st.l * 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i) s = __builtin_fmaf(st.acc[e][i], 0.f, s);
  return __ballot(s != 0.f) == 0;  // NaN if one of them is not
}

// The wave's result: acc[head * kGroupStride + channel], ref[head], l[head] (LDS).
__device__ __forceinline__ void group_finish(GroupState& st, float* acc, float* ref, float* l,
                                             int lane) {
  LanePair s = pair_across16(as_u(st.l));
  s = pair_across32(as_u(as_f(s.first) + as_f(s.second)));
  const int head = lane & 15, g = lane >> 4;
  const float unscale = (lane & 8) ? 1.f / (kWeightScale * kRestScale) : 1.f / kWeightScale;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = row_ror_add<8>(st.acc[e][i] * unscale);  // the two parts of the weights
    if (head < kGroupHeads) {
      float4* to = reinterpret_cast<float4*>(acc + head * kGroupStride + 8 * (4 * g + i));
      to[0] = make_float4(v[0], v[1], v[2], v[3]);
      to[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
  }
  if (lane < kGroupHeads) {
    ref[lane] = st.ref;
    l[lane] = as_f(s.first) + as_f(s.second);
  }
}

// The same value in a register that no load is outstanding for: the compiler waits for
// `v` here, once, instead of before every later use it cannot order against other loads.
__device__ __forceinline__ int settled(int v) {
  int r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
  return r;
}

// What every attention launch is given.
struct AttnArgs {
  const char* k_pool;
  const char* v_pool;
  const char* q;
  const int32_t* page_table;
  const int32_t* seq_lens;
  float* part_acc;      // un-normalised accumulators of the partial results, [..][D]
  float* part_ml;       // their running max (log2 domain) and denominator, [..][2]
  void* out;
  float* lse;
  uint64_t* counters;   // arrival counters, one per 256-byte slot (quest_team.h); zero between launches
  int batch, num_heads, max_pages, out_is_fp16;
  int device_fences;    // QUEST_FLAG_DEVICE_FENCES: fences around the exchange as well
  int kv_heads, group;  // KV heads; query heads per KV head (num_heads = kv_heads * group)
  int subs;             // work-groups per KV head: ceil(group / kGroupHeads)
  int page_shift;       // log2(tokens per page)
  int unit_shift;       // log2(streaming units per page): 0 up to 16 tokens, 1 for 32, 2 for 64
  float scale_log2;     // sm_scale * log2(e)
};

inline int attention_subs(const quest_cache& c) { return (group_size(c) + kGroupHeads - 1) / kGroupHeads; }

// All but the workspace.
inline void fill_attn_args(AttnArgs& a, const quest_cache& c, const void* q, float sm_scale, void* out,
                           int out_is_fp16, float* lse) {
  a.k_pool = (const char*)c.k_pool;
  a.v_pool = (const char*)c.v_pool;
  a.q = (const char*)q;
  a.page_table = c.page_table;
  a.seq_lens = c.seq_lens;
  a.out = out;
  a.lse = lse;
  a.batch = c.batch;
  a.num_heads = c.num_heads;
  a.max_pages = c.max_pages_per_seq;
  a.out_is_fp16 = out_is_fp16;
  a.device_fences = (c.flags & QUEST_FLAG_DEVICE_FENCES) != 0;
  a.kv_heads = kv_heads(c);
  a.group = group_size(c);
  a.subs = attention_subs(c);
  a.page_shift = page_shift_of(c.page_size);
  a.unit_shift = a.page_shift > 4 ? a.page_shift - 4 : 0;
  a.scale_log2 = sm_scale * kLog2e;
}

// A wave's attention state: one query head on the vector unit, or up to kGroupHeads query
// heads of a KV head on the matrix cores.
// kLoads: wave-wide 16-byte loads per unit of keys (and of values) of one query head: 4, or
// 2 for 8-token pages.  A group's unit is 16 tokens for every page size.
template <int kLoads, bool kGroup>
struct HeadState {
  static constexpr int kSlots = kGroup ? kGroupHeads : 1;             // query heads
  static constexpr int kStride = kGroup ? kGroupStride : kHeadDim;    // floats per head in LDS
  static constexpr bool kTwoPages = kGroup && kLoads == 2;            // pages per unit
  using Regs = typename std::conditional<kGroup, GroupRegs, PageRegsT<kLoads>>::type;
  typename std::conditional<kGroup, GroupState, Softmax>::type st;
  uint4 qv;

  // q: vectors of the first of `heads` query heads; lds: the wave's kSlots * kStride floats,
  // where finish may leave the result.  Loads only (and constants): what it sets is first
  // used by fold.
  __device__ __forceinline__ void init(float* lds, const char* q, int heads, int lane) {
    if constexpr (kGroup) {
      static_assert(kSlots * kStride * sizeof(float) >= 16 * kRowBytes, "keys of a unit");
      group_init(st, reinterpret_cast<char*>(lds), q, heads, lane);
    } else {
      qv = ld16(q + (lane & 15) * 16);
      st.m = kNegBig;
      st.l = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) st.acc[j] = 0.f;
    }
  }
  __device__ __forceinline__ void load(Regs& r, const AttnArgs& a, int hk, int seq_len, int lp, int ph,
                                       int unit, int lp2, int ph2, int lane) {
    if constexpr (!kGroup) {
      load_unit<kLoads>(r, a.k_pool, a.v_pool, a.kv_heads, hk, seq_len, lp, ph, unit, a.page_shift, lane);
    } else {
      const auto row = [&](int p) { return (((size_t)p * a.kv_heads + hk) << a.page_shift) * kRowBytes; };
      if constexpr (kTwoPages) {
        group_load(r, a.k_pool, a.v_pool, row(ph), row(ph2) - 8 * kRowBytes, lane);
        r.first = lp < 0 ? 0 : seq_len - lp * 8;
        r.second = lp2 < 0 ? 0 : seq_len - lp2 * 8;
      } else {
        const size_t base = row(ph) + (size_t)unit * (16 * kRowBytes);
        group_load(r, a.k_pool, a.v_pool, base, base, lane);
        r.first = seq_len - (lp << a.page_shift) - unit * 16;
        r.second = r.first - 8;
      }
    }
  }
  __device__ __forceinline__ void fold(Regs& r, float scale_log2, int lane) {
    if constexpr (kGroup)
      group_fold(st, r, scale_log2, lane);
    else
      fold_page(st, r, qv, scale_log2, lane >> 4);
  }
  // The wave's result per query head: acc[head * kStride + channel], m[head], l[head] (LDS).
  __device__ __forceinline__ void finish(float* acc, float* m, float* l, int lane) {
    if constexpr (kGroup) {
      group_finish(st, acc, m, l, lane);
    } else {
      merge_rows(st);
      if (lane < 16) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[lane * 8 + j] = st.acc[j];
        if (lane == 0) m[0] = st.m, l[0] = st.l;
      }
    }
  }
};

// Stream `units` units through the wave.  at(i, lp, ph, unit, lp2, ph2) says, lane by lane,
// what the wave's i-th unit is: logical and physical page (and those of the second page of
// a pair) and the unit within the page; a negative logical page: nothing there.  at is asked
// for 64 units at a time, one per lane.
template <int kLoads, bool kGroup, class At>
__device__ __forceinline__ void stream_units(HeadState<kLoads, kGroup>& st, const AttnArgs& a, int hk,
                                             int seq_len, int units, int lane, At at) {
  using Head = HeadState<kLoads, kGroup>;
  for (int chunk = 0; chunk < units; chunk += kWave) {
    int lp_v = -1, ph_v = 0, un_v = 0, lp2_v = -1, ph2_v = 0;
    at(chunk + lane, lp_v, ph_v, un_v, lp2_v, ph2_v);
    if (Head::kTwoPages) {
      if (lp_v < 0) ph_v = 0;  // half a unit may be missing: it is read from page 0, and not used
      if (lp2_v < 0) ph2_v = 0;
    }
    // The units to stream are moved to the first n lanes (lists from the selection are
    // ascending and padded at the end, so normally they are there already; a caller's
    // list may have negative or out-of-range entries anywhere: those are skipped).
    // Two units in flight per wave: the next one is requested before the current one is
    // folded.  Every load inside the loop is unconditional and the index registers are
    // detached from the loads that produced them (one wait here), so the compiler's
    // wait counts inside the loop are exact: a conditional load, or an index still
    // marked as in flight, makes it wait for everything outstanding at every step,
    // which leaves a single unit in flight.
    const bool mine = lp_v >= 0 || lp2_v >= 0;
    const unsigned long long live = __ballot(mine);
    const int n = __popcll(live);
    if (live & (live + 1)) {  // not a prefix of the lanes: compact (wave-uniform branch)
      const int to = mine ? (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u)) : kWave - 1;
      // a dead lane's target is lane 63, which no live lane can have unless all 64 are
      // live (then this branch is not taken); its value there is never used (63 >= n)
      lp_v = __builtin_amdgcn_ds_permute(to * 4, lp_v);
      ph_v = __builtin_amdgcn_ds_permute(to * 4, ph_v);
      un_v = __builtin_amdgcn_ds_permute(to * 4, un_v);
      if (Head::kTwoPages) {
        lp2_v = __builtin_amdgcn_ds_permute(to * 4, lp2_v);
        ph2_v = __builtin_amdgcn_ds_permute(to * 4, ph2_v);
      }
    }
    lp_v = settled(lp_v);
    ph_v = settled(ph_v);
    if (Head::kTwoPages) {
      lp2_v = settled(lp2_v);
      ph2_v = settled(ph2_v);
    }
    auto load = [&](typename Head::Regs& r, int i) {
      st.load(r, a, hk, seq_len, __builtin_amdgcn_readlane(lp_v, i), __builtin_amdgcn_readlane(ph_v, i),
              __builtin_amdgcn_readlane(un_v, i), Head::kTwoPages ? __builtin_amdgcn_readlane(lp2_v, i) : -1,
              Head::kTwoPages ? __builtin_amdgcn_readlane(ph2_v, i) : 0, lane);
    };
    typename Head::Regs ra, rb;
    if (n > 0) {
      load(ra, 0);
      int j = 0;
      for (; j + 2 < n; j += 2) {
        load(rb, j + 1);
        st.fold(ra, a.scale_log2, lane);
        load(ra, j + 2);
        st.fold(rb, a.scale_log2, lane);
      }
      if (j + 1 < n) {
        load(rb, j + 1);
        st.fold(ra, a.scale_log2, lane);
        st.fold(rb, a.scale_log2, lane);
      } else {
        st.fold(ra, a.scale_log2, lane);
      }
    }
  }
}

// The wave's `units` units (see stream_units) with its n_heads query heads q: what finish
// leaves in LDS.  Where a group's sums are not finite, head by head on the vector unit.
template <int kLoads, bool kGroup, class At>
__device__ __forceinline__ void attend(HeadState<kLoads, kGroup>& st, const AttnArgs& a, int hk, int seq_len,
                                       int units, const char* q, int n_heads, float* acc, float* m, float* l,
                                       int lane, At at) {
  stream_units<kLoads, kGroup>(st, a, hk, seq_len, units, lane, at);
  if constexpr (kGroup) {
    if (!group_finite(st.st)) {
      constexpr bool kTwo = HeadState<kLoads, kGroup>::kTwoPages;
#pragma unroll 1
      for (int g = 0; g < n_heads; ++g) {
        HeadState<kLoads, false> one;
        one.init(nullptr, q + g * kRowBytes, 1, lane);
        stream_units<kLoads, false>(one, a, hk, seq_len, kTwo ? 2 * units : units, lane,
                                    [&](int i, int& lp, int& ph, int& un, int& lp2, int& ph2) {
          if constexpr (kTwo) {
            int lp_b = -1, ph_b = 0;
            at(i >> 1, lp, ph, un, lp_b, ph_b);
            if (i & 1) lp = lp_b, ph = ph_b;
          } else {
            at(i, lp, ph, un, lp2, ph2);
          }
        });
        one.finish(acc + g * HeadState<kLoads, kGroup>::kStride, m + g, l + g, lane);
      }
      return;
    }
  }
  st.finish(acc, m, l, lane);
}

__device__ __forceinline__ void store_out(void* out, int out_is_fp16, size_t idx, float v) {
  if (out_is_fp16)
    reinterpret_cast<_Float16*>(out)[idx] = (_Float16)v;
  else
    reinterpret_cast<float*>(out)[idx] = v;
}
// Two neighbours.
__device__ __forceinline__ void store_out2(void* out, int out_is_fp16, size_t idx, float v0, float v1) {
  store_out(out, out_is_fp16, idx, v0);
  store_out(out, out_is_fp16, idx + 1, v1);
}

#endif  // __HIPCC__

}  // namespace quest
