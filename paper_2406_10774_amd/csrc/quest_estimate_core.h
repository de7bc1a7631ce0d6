// Device-side core of the criticality estimate (attention half of Algorithm 1,
// Section 3.4 of arXiv 2406.10774).
#pragma once

#include "quest_common.h"

namespace quest {

#if defined(__HIPCC__)

constexpr int kEstIters = 4;                     // wave-wide load pairs per wave (large tables)
constexpr int kEstPagesPerWave = 4 * kEstIters;  // 16

// kAppend: the wave that owns the newest token's page first performs the
// insertion half of Algorithm 1 for it (store k/v into the slot, fold k into
// the page's min/max, write the entry back) on the registers it scores from.
struct EstimateArgs {
  char* meta;
  const char* q;
  const int32_t* page_table;
  const int32_t* seq_lens;
  float* scores;
  int num_heads, max_pages;  // num_heads: KV heads (rows of meta, pools, scores)
  int group;                 // query heads per KV head: q has num_heads * group heads
  int64_t num_phys_pages;
  const char* k_new;  // kAppend only
  const char* v_new;
  char* k_pool;
  char* v_pool;
  int k_pool_write;
  int page_shift;  // log2(tokens per page)
};

// Per half: 0xffff where q is negative (min row wins), 0 elsewhere (max row wins).
__device__ __forceinline__ uint4 negative8(const uint4 q) {
  const auto of = [](uint32_t v) { return __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2_t, v) >> 15); };
  return make_uint4(of(q.x), of(q.y), of(q.z), of(q.w));
}

// One wave scores the 4 * kIters logical pages starting at `base` of (sequence b,
// head h): DPP row g takes pages base + kIters*g .. + kIters - 1, one per
// wave-wide load pair.
// kQ: query heads of a KV head: 1 to 4, or 0 for any number, scored on the matrix cores (`stage`: 512
// bytes of LDS of this wave per page, unused otherwise).
template <bool kAppend, int kIters, int kQ>
__device__ __forceinline__ void estimate_wave(const EstimateArgs& a, int b, int h, int base, char* stage) {
  char* __restrict__ meta = a.meta;
  const char* __restrict__ q = a.q;
  const int32_t* __restrict__ page_table = a.page_table;
  const int32_t* __restrict__ seq_lens = a.seq_lens;
  float* __restrict__ scores = a.scores;
  const int num_heads = a.num_heads, max_pages = a.max_pages;
  const char* __restrict__ k_new = a.k_new;
  const char* __restrict__ v_new = a.v_new;
  char* __restrict__ k_pool = a.k_pool;
  char* __restrict__ v_pool = a.v_pool;
  const int k_pool_write = a.k_pool_write;
  const int lane = lane_id();
  const int grp = lane >> 4;  // DPP row: pages base + kIters*grp + it
  const int c = lane & 15;    // channels 8c..8c+7
  const size_t bh = (size_t)b * num_heads + h;

  // What the first loads need comes from the kernel's arguments in one go, and the length
  // and the page-table entries are asked for together: left to itself the compiler asks for
  // the length first, leaves if the wave has nothing to do, and starts the next trips after.
  asm volatile("" ::"s"(meta), "s"(q), "s"(page_table), "s"(seq_lens), "s"(max_pages), "s"(a.page_shift),
               "s"(a.num_phys_pages), "s"(num_heads));
  // The wave's page-table entries in one load (whether a page holds tokens is decided
  // afterwards): lane c of row g fetches entry c % kIters of the row's, and the quad hands
  // them round.  (A load per page, each under its own condition, is a chain of kIters trips
  // to the cache.)  Together 7.6 us instead of 7.9 us in the case above, 13.8 us instead of
  // 14.5 us at 4105 pages of 32 heads, 2.8 us instead of 3.0 us at one head.
  const int32_t* pt = page_table + (size_t)b * max_pages;
  static_assert(kIters == 2 || kIters == 4, "entries of a quad");
  int entry = pt[min(base + kIters * grp + (c & (kIters - 1)), max_pages - 1)];
  const int seq_len = __builtin_amdgcn_readfirstlane(seq_lens[b]);
  // The query vectors in front of the metadata.  Up to four: lane c has channels 8c .. +7 of
  // each.  Any number: as rows of a matrix operand, lane c of row g has channels 32j + 8g .. +7 of head c (heads
  // past the group: the last one again).
  constexpr bool kMatrix = kQ == 0;
  const int group = kMatrix ? a.group : kQ;
  constexpr int kQueries = kMatrix ? 4 : kQ;
  uint4 qv[kQueries];
  auto load_queries = [&](int g0) {
#pragma unroll
    for (int i = 0; i < kQueries; ++i)
      qv[i] = kMatrix ? ld16(q + (bh * group + min(g0 + c, group - 1)) * (kHeadDim * 2) + i * 64 + grp * 16)
                      : ld16(q + (bh * group + i) * (kHeadDim * 2) + c * 16);
  };
  load_queries(0);
  asm volatile("" : "+v"(entry) : "s"(seq_len));
  const int page_shift = a.page_shift;
  const int num_pages = (seq_len + (1 << page_shift) - 1) >> page_shift;
  if (base >= num_pages) return;

  // The wave that holds the newest token's page (wave-uniform) asks for the token in front of
  // the metadata; at the end of the launch nothing waits but this wave.
  const int pos = seq_len - 1;
  const int last = pos >> page_shift;
  const bool appends = kAppend && last >= base && last < base + 4 * kIters;
  uint4 kn = make_uint4(0, 0, 0, 0), vn = kn;
  if (appends) {
    kn = ld16(k_new + bh * (kHeadDim * 2) + c * 16);
    if (k_pool_write) vn = ld16(v_new + bh * (kHeadDim * 2) + c * 16);
  }

  uint4 mn[kIters], mx[kIters];
  int phys[kIters];
  phys[0] = __builtin_amdgcn_update_dpp(0, entry, 0x00, 0xf, 0xf, true);  // quad_perm: lane 0 to all
  phys[1] = __builtin_amdgcn_update_dpp(0, entry, 0x55, 0xf, 0xf, true);
  if constexpr (kIters == 4) {
    phys[2] = __builtin_amdgcn_update_dpp(0, entry, 0xaa, 0xf, 0xf, true);
    phys[3] = __builtin_amdgcn_update_dpp(0, entry, 0xff, 0xf, 0xf, true);
  }
  // Pages past the end are read from the wave's first page instead, and not used: no load
  // stands under a condition.
  const int some = __builtin_amdgcn_readfirstlane(entry);
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    if (base + kIters * grp + it >= num_pages) phys[it] = some;
    const char* e = meta + meta_offset(a.num_phys_pages, phys[it], h) + c * 16;
    mn[it] = ld16_stream(e);
    mx[it] = ld16_stream(e + kHeadDim * 2);
  }
  // Where the scores go is worked out while the metadata is on its way, and the last sums in front of the
  // branch around the store: the compiler would put both behind it, at the wave's end (8100 entries or less:
  // 1.5 % of the launch).
  float* row = scores + bh * max_pages;
  asm volatile("" : "+s"(row));

  if (appends) {
    const int slot = pos - (last << page_shift);
    const uint4 key = order_key8(kn);
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      if (base + kIters * grp + it == last) {
        const size_t ph = (size_t)phys[it] * num_heads + h;
        if (k_pool_write) {
          const size_t off = ((ph << page_shift) + slot) * kRowBytes + c * 16;
          st16(k_pool + off, kn);
          st16(v_pool + off, vn);
        }
        if (slot == 0) {
          mn[it] = kn;
          mx[it] = kn;
        } else {
          mn[it] = order_key8(key_min8(order_key8(mn[it]), key));
          mx[it] = order_key8(key_max8(order_key8(mx[it]), key));
        }
        char* e = meta + meta_offset(a.num_phys_pages, phys[it], h) + c * 16;
        st16(e, mn[it]);
        st16(e + kHeadDim * 2, mx[it]);
      }
    }
  }

  if constexpr (kMatrix) {
    // Several query heads meet every entry: a contraction over twice the channels.  13 vector
    // instructions per head and load pair held a wave longer than its loads; here it is eight matrix
    // instructions and about 110 others for up to 16 heads and 16 pages.  us an append and estimate, before /
    // now: 4 sequences of up to 32k tokens, 8 KV heads, groups of four 7.1 / 6.4, of eight 9.7 / 6.4; 16
    // sequences of up to 64k, of eight 38.4 / 26.1 (one query head per KV head: 25.4, 6.6 TB/s); one of
    // 32k, of eight 5.2 / 3.8.  Against 64 bits, 2-norm over nine shapes: 4.09e-8 (4.11e-8 before).
    // Turned through LDS: entries as columns of a matrix operand, lane c of row g with channels
    // 32j + 8g .. +7 of page c (of eight pages: twice).  The 16-byte chunks of page p are exclusive-ored
    // with p, so neither side has bank conflicts.
    constexpr int kPages = 4 * kIters;
    uint4 lo[4], hi[4];
    auto split_queries = [&] {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint4 neg = negative8(qv[j]);
        lo[j] = make_uint4(qv[j].x & neg.x, qv[j].y & neg.y, qv[j].z & neg.z, qv[j].w & neg.w);
        hi[j] = make_uint4(qv[j].x & ~neg.x, qv[j].y & ~neg.y, qv[j].z & ~neg.z, qv[j].w & ~neg.w);
      }
    };
    split_queries();  // while the metadata is on its way
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int p = kIters * grp + it;
      st16(stage + p * kMetaBytes + ((c ^ p) << 4), mn[it]);
      st16(stage + p * kMetaBytes + kHeadDim * 2 + ((c ^ p) << 4), mx[it]);
    }
    lds_in_order();
    const int page = c & (kPages - 1);
    const char* entry_of = stage + page * kMetaBytes;
    float keep = -INFINITY;
    bool odd = false;
    // 16 heads against the pages: q where it is positive meets the max row, where it is negative the
    // min row; the other of the two products is zero.  Eight sums of 32 channels, added as a tree.
    auto score_heads = [&] {
      f32x4_t s[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int at = ((4 * j + grp) ^ page) << 4;
        const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
        s[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, lo[j]),
                                                      __builtin_bit_cast(half8_t, ld16(entry_of + at)), zero, 0, 0, 0);
        s[j] += __builtin_amdgcn_mfma_f32_16x16x32_f16(
            __builtin_bit_cast(half8_t, hi[j]), __builtin_bit_cast(half8_t, ld16(entry_of + kHeadDim * 2 + at)), zero, 0, 0, 0);
        // Operands of one j at a time, or of two: registers for seven waves per SIMD, or for four (five are what
        // LDS has room for).
        if (kIters == 2 || j == 1) __builtin_amdgcn_sched_barrier(0);
      }
      float z[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = (s[0][i] + s[1][i]) + (s[2][i] + s[3][i]);
      odd |= !((z[0] + z[1]) + (z[2] + z[3]) > -INFINITY);
      keep = fmaxf(keep, fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));  // heads 4g .. 4g + 3
    };
    score_heads();
    for (int g0 = 16; g0 < group; g0 += 16) {
      load_queries(g0);
      split_queries();
      score_heads();
    }
    // An infinite entry, or one that is no number, may have met a zero.  Such pages, which a cache
    // hardly ever holds, are scored head by head.
    if (__ballot(odd) == 0) {
      LanePair s = pair_across16(__builtin_bit_cast(uint32_t, keep));
      s = pair_across32(__builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, s.first), __builtin_bit_cast(float, s.second))));
      keep = fmaxf(__builtin_bit_cast(float, s.first), __builtin_bit_cast(float, s.second));
      if (lane < kPages && base + lane < num_pages) row[base + lane] = keep;
      return;
    }
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int p = kIters * grp + it;
      mn[it] = ld16(stage + p * kMetaBytes + ((c ^ p) << 4));
      mx[it] = ld16(stage + p * kMetaBytes + kHeadDim * 2 + ((c ^ p) << 4));
    }
  }

  // One query head against the pages this wave holds: lane c of a row keeps the
  // score of the row's c-th page.
  auto score_pages = [&](const uint4 qh) {
    const uint4 neg = negative8(qh);
    float mine = 0.f;
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      uint4 sel;
      sel.x = (mn[it].x & neg.x) | (mx[it].x & ~neg.x);
      sel.y = (mn[it].y & neg.y) | (mx[it].y & ~neg.y);
      sel.z = (mn[it].z & neg.z) | (mx[it].z & ~neg.z);
      sel.w = (mn[it].w & neg.w) | (mx[it].w & ~neg.w);
      const float s = row16_sum(dot8(qh, sel, 0.f));
      if (c == it) mine = s;
    }
    return mine;
  };
  // The page's score for the KV head: the largest of its query heads' scores
  // (one query head per KV head in the paper's models: no further round).
  float keep;
  if constexpr (kMatrix) {
    const char* heads = q + bh * group * (kHeadDim * 2) + c * 16;
    keep = score_pages(ld16(heads));
#pragma unroll 1
    for (int i = 1; i < group; ++i) keep = fmaxf(keep, score_pages(ld16(heads + i * (kHeadDim * 2))));
  } else {
    keep = score_pages(qv[0]);
#pragma unroll
    for (int i = 1; i < kQ; ++i) keep = fmaxf(keep, score_pages(qv[i]));
  }
  // lanes c < 4 of each row hold 4 consecutive pages: 16 consecutive floats per wave
  asm volatile("" : "+v"(keep));
  const int p = base + kIters * grp + c;
  if (c < kIters && p < num_pages) row[p] = keep;
}

#endif  // __HIPCC__

}  // namespace quest
