// Device-side core of the criticality estimate (attention half of Algorithm 1,
// Section 3.4 of arXiv 2406.10774).
#pragma once

#include <type_traits>

#include "quest_common.h"
#include "quest_team.h"

namespace quest {

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

EstimateArgs estimate_args(const quest_cache& c, const void* k_new, const void* v_new, int k_pool_write, const void* q,
                           float* scores);
// Whether groups are scored on the matrix cores (else on the vector unit; the sums differ in their order).
bool estimate_on_matrix_cores(const quest_cache& c);

#if defined(__HIPCC__)

// Per half: 0xffff where q is negative (min row wins), 0 elsewhere (max row wins).
__device__ __forceinline__ uint4 negative8(const uint4 q) {
  const auto of = [](uint32_t v) { return __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2_t, v) >> 15); };
  return make_uint4(of(q.x), of(q.y), of(q.z), of(q.w));
}

// Query vectors of one (sequence, KV head) as a wave holds them.  Up to four (kQ of them): lane c has channels
// 8c .. +7 of each.  Any number (kQ == 0): as rows of a matrix operand, lane c of row g has channels
// 32j + 8g .. +7 of head c (heads past the group: the last one again).
template <int kQ>
struct Queries {
  static constexpr bool kMatrix = kQ == 0;
  static constexpr int kRegs = kMatrix ? 4 : kQ;
  const char* first;  // the first head's
  int group;
  uint4 v[kRegs];
  // kUpTo: up to kQ heads (the last one again in the others' place)
  template <bool kUpTo = false>
  __device__ __forceinline__ void load(int g0, int lane) {
    const int grp = lane >> 4, c = lane & 15;
#pragma unroll
    for (int i = 0; i < kRegs; ++i)
      v[i] = kMatrix ? ld16(first + (uint32_t)(min(g0 + c, group - 1) * (kHeadDim * 2) + i * 64 + grp * 16))
                     : ld16(first + (kUpTo && kQ > 1 ? min(i, group - 1) : i) * (kHeadDim * 2) + c * 16);
  }
};

// Sums over the 16 lanes of a DPP row of two or four values at once, each added up as row16_sum does (the same bits):
// halves, then quarters of the row go on with a value of their own.  Lane c ends up with the sum of value
// row16_sums_index(c), and row16_sums_has(c) names one lane for each.  Four of them take 12 instructions, one by one
// and put into their lanes 20.
template <int kCount>
__device__ __forceinline__ int row16_sums_index(int c) {
  return kCount == 2 ? c >> 3 : (c >> 3) + ((c >> 1) & 2);
}
template <int kCount>
__device__ __forceinline__ bool row16_sums_has(int c) {
  return (c & (kCount == 2 ? 7 : 3)) == 0;
}
__device__ __forceinline__ float row_swap_add4(float keep, float give) {  // keep + the give of lane c ^ 4
  const int g = __builtin_bit_cast(int, give);
  int got = __builtin_amdgcn_update_dpp(0, g, 0x104, 0xf, 0x5, false);  // row_shl:4 to the first and third four
  got = __builtin_amdgcn_update_dpp(got, g, 0x114, 0xf, 0xa, false);    // row_shr:4 to the others
  return keep + __builtin_bit_cast(float, got);
}
template <int kCtrl>
__device__ __forceinline__ float quad_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_swap_add8(float a, float b, int c) {  // lanes below 8: a, above: b
  const float keep = c < 8 ? a : b, give = c < 8 ? b : a;
  const int g = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), 0x128, 0xf, 0xf, true);  // row_ror:8
  return keep + __builtin_bit_cast(float, g);
}
__device__ __forceinline__ float row16_sums(const float (&v)[2], int c) {
  const float s = row_swap_add8(v[0], v[1], c);
  return quad_add<0xb1>(quad_add<0x4e>(row_swap_add4(s, s)));
}
__device__ __forceinline__ float row16_sums(const float (&v)[4], int c) {
  const float a = row_swap_add8(v[0], v[1], c), b = row_swap_add8(v[2], v[3], c);
  const bool second = c & 4;
  return quad_add<0xb1>(quad_add<0x4e>(row_swap_add4(second ? b : a, second ? a : b)));
}

// The scores of the 4 * kIters pages that a wave holds the entries of (DPP row g: pages kIters * g
// + it), of which the first `pages` are of the sequence: emit(has, page, score), where has says that the
// lane has a page to emit.
// stage: for kQ == 0, 512 bytes of LDS of this wave per page.
template <int kIters, int kQ, class Emit>
__device__ __forceinline__ void score_wave(Queries<kQ>& q, uint4 (&mn)[kIters], uint4 (&mx)[kIters], int pages,
                                           char* stage, int lane, Emit emit) {
  constexpr bool kMatrix = kQ == 0;
  const int grp = lane >> 4, c = lane & 15;
  const int group = kMatrix ? q.group : kQ;
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
        const uint4 neg = negative8(q.v[j]);
        lo[j] = make_uint4(q.v[j].x & neg.x, q.v[j].y & neg.y, q.v[j].z & neg.z, q.v[j].w & neg.w);
        hi[j] = make_uint4(q.v[j].x & ~neg.x, q.v[j].y & ~neg.y, q.v[j].z & ~neg.z, q.v[j].w & ~neg.w);
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
      q.load(g0, lane);
      split_queries();
      score_heads();
    }
    // An infinite entry, or one that is no number, may have met a zero.  Such pages, which a cache
    // hardly ever holds, are scored head by head.
    if (__ballot(odd & (page < pages)) == 0) {
      LanePair s = pair_across16(__builtin_bit_cast(uint32_t, keep));
      s = pair_across32(__builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, s.first), __builtin_bit_cast(float, s.second))));
      keep = fmaxf(__builtin_bit_cast(float, s.first), __builtin_bit_cast(float, s.second));
      emit(lane < kPages, lane, keep);
      return;
    }
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int p = kIters * grp + it;
      mn[it] = ld16(stage + p * kMetaBytes + ((c ^ p) << 4));
      mx[it] = ld16(stage + p * kMetaBytes + kHeadDim * 2 + ((c ^ p) << 4));
    }
  }

  // One query head against the pages this wave holds: the four (or eight) lanes of page_of's page keep its score.
  auto score_pages = [&](const uint4 qh) {
    const uint4 neg = negative8(qh);
    float part[kIters];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      uint4 sel;
      sel.x = (mn[it].x & neg.x) | (mx[it].x & ~neg.x);
      sel.y = (mn[it].y & neg.y) | (mx[it].y & ~neg.y);
      sel.z = (mn[it].z & neg.z) | (mx[it].z & ~neg.z);
      sel.w = (mn[it].w & neg.w) | (mx[it].w & ~neg.w);
      part[it] = dot8(qh, sel, 0.f);
    }
    return row16_sums(part, c);
  };
  // The page's score for the KV head: the largest of its query heads' scores
  // (one query head per KV head in the paper's models: no further round).
  float keep;
  if constexpr (kMatrix) {
    const char* heads = q.first + c * 16;
    keep = score_pages(ld16(heads));
#pragma unroll 1
    for (int i = 1; i < group; ++i) keep = fmaxf(keep, score_pages(ld16(heads + i * (kHeadDim * 2))));
  } else {
    keep = score_pages(q.v[0]);
#pragma unroll
    for (int i = 1; i < kQ; ++i) keep = fmaxf(keep, score_pages(q.v[i]));
  }
  asm volatile("" : "+v"(keep));
  emit(row16_sums_has<kIters>(c), kIters * grp + row16_sums_index<kIters>(c), keep);
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
  // The query vectors in front of the metadata.
  const int group = kQ == 0 ? a.group : kQ;
  Queries<kQ> queries{q + bh * group * (kHeadDim * 2), group};
  queries.load(0, lane);
  asm volatile("" : "+v"(entry) : "s"(seq_len));
  const int page_shift = a.page_shift;
  const int num_pages = (seq_len + (1 << page_shift) - 1) >> page_shift;
  if (base >= num_pages) return;

  // The wave that holds the newest token's page (wave-uniform) asks for the token in front of
  // the metadata; at the end of the launch nothing waits but this wave.
  const int pos = seq_len - 1;
  const int last = pos >> page_shift;
  const bool appends = kAppend && (unsigned)(last - base) < 4u * kIters;
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

  score_wave<kIters, kQ>(queries, mn, mx, num_pages - base, stage, lane, [&](bool has, int page, float score) {
    if (has & (base + page < num_pages)) row[base + page] = score;  // (&: one branch, not two)
  });
}

struct RowOfPages {
  int seq_len, num_pages;
  int newest_phys;   // physical page of the newest token, in the wave that has it ...
  bool mine;         // ... and its entry with the key folded in, in the lanes that have it
  uint4 low, high;
};

// One work-group scores a whole row, (sequence b, head h): the scores (those of estimate_wave) and the physical
// pages go to LDS.  A row has at most kWaves * kPasses * 4 kIters pages;
// wave w takes blocks w, w + kWaves, .. of 4 kIters pages, with the entries of up to four blocks in flight, and
// folds them in the order they come.  What bounds it: the launch's start and two trips to memory, 1.5 us, then
// 64 bytes a clock from L2 or, where few compute units share a row, about 27 KiB per us from memory.  (A row
// is fetched into L2 once: in eight splits of 124 or 188 pages, 32 heads, a step fetches 1.02 times its bytes.)
// Nobody has inserted the newest token yet: every work-group of the row stores its key and value (the
// same bytes; each later reads what it stored itself) and folds the key into the entry it scores, and
// one of them writes that entry back (store_row).  Another work-group may find the entry as it was or with the key folded in,
// element by element: min and max with the same key again change nothing, and a page's first token
// does not look at the entry.
// kQ: 1, 0 (matrix cores, groups of up to 16), or 4 (up to four).
template <int kWaves, int kPasses, int kIters, int kQ>
__device__ __forceinline__ RowOfPages estimate_row(const EstimateArgs& a, int b, int h, int wave, char* stage,
                                                   float* sm_score, int* sm_phys) {
  constexpr int kBlock = 4 * kIters, kDepth = kPasses < 4 ? kPasses : 4;
  const int lane = lane_id();
  const int grp = lane >> 4, c = lane & 15;
  const size_t bh = (size_t)b * a.num_heads + h;
  const int32_t* pt = a.page_table + (size_t)b * a.max_pages;
  int entry[kPasses];
#pragma unroll
  for (int p = 0; p < kPasses; ++p)
    entry[p] = pt[min((p * kWaves + wave) * kBlock + kIters * grp + (c & (kIters - 1)), a.max_pages - 1)];
  const int seq_len = __builtin_amdgcn_readfirstlane(a.seq_lens[b]);
  Queries<kQ> queries{a.q + bh * a.group * (kHeadDim * 2), a.group};
  queries.template load<true>(0, lane);
  // (addresses that may be read, whether or not there is a new token)
  const bool stores = a.k_new && a.k_pool_write;
  const uint4 kn = ld16((a.k_new ? a.k_new + bh * (kHeadDim * 2) : queries.first) + c * 16);
  const uint4 vn = ld16((stores ? a.v_new + bh * (kHeadDim * 2) : queries.first) + c * 16);
  const int num_pages = min((seq_len + (1 << a.page_shift) - 1) >> a.page_shift, a.max_pages);
  const int pos = seq_len - 1, last = pos >> a.page_shift, slot = pos - (last << a.page_shift);
  const auto base_of = [&](int p) { return (p * kWaves + wave) * kBlock; };
  // The newest token's page, if this wave has it: in this pass.
  const int newest_block = last / kBlock;
  const int newest_pass = a.k_new && last >= 0 && last < num_pages && newest_block % kWaves == wave ? newest_block / kWaves : -1;
  // (left to itself the compiler asks for the query and the new token behind the metadata)
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < kPasses; ++p)
    if (c < kIters) sm_phys[base_of(p) + kIters * grp + c] = entry[p];

  // Entries of pages past the end lie past the end of the buffer: such loads touch no memory.
  const __amdgpu_buffer_rsrc_t table = __builtin_amdgcn_make_buffer_rsrc(
      a.meta + meta_offset(a.num_phys_pages, 0, h), 0, (uint32_t)a.num_phys_pages * kMetaBytes, 0x00020000);
  uint4 mn[kDepth][kIters], mx[kDepth][kIters];
  const auto load = [&](int p) {
    const int page = base_of(p) + kIters * grp + (c & (kIters - 1));
    const uint32_t offset = page < num_pages ? (uint32_t)entry[p] * kMetaBytes : 0xfffff000u;
    const auto spread = [&](auto ctrl) {  // quad_perm: one lane's to all
      return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)offset, decltype(ctrl)::value, 0xf, 0xf, true) + c * 16;
    };
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const uint32_t at = it == 0   ? spread(std::integral_constant<int, 0x00>{})
                          : it == 1 ? spread(std::integral_constant<int, 0x55>{})
                          : it == 2 ? spread(std::integral_constant<int, 0xaa>{})
                                    : spread(std::integral_constant<int, 0xff>{});
      mn[p % kDepth][it] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(table, at, 0, 0));
      mx[p % kDepth][it] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(table, at + kHeadDim * 2, 0, 0));
    }
  };
#pragma unroll
  for (int p = 0; p < kDepth; ++p) load(p);
  __builtin_amdgcn_sched_barrier(0);
  // The newest token is stored behind the loads of the metadata, and what only others read is left to store_row:
  // the selection waits for neither.
  RowOfPages r{seq_len, num_pages, 0, false, kn, kn};
  if (newest_pass >= 0) {
    r.newest_phys = __builtin_amdgcn_readfirstlane(sm_phys[last]);
    const size_t off = (((((size_t)r.newest_phys * a.num_heads + h) << a.page_shift) + slot) * kRowBytes) + c * 16;
    if (stores && grp < 2) st16((grp == 0 ? a.k_pool : a.v_pool) + off, grp == 0 ? kn : vn);
  }
  const uint4 key = order_key8(kn);
#pragma unroll
  for (int p = 0; p < kPasses; ++p) {
    uint4(&low)[kIters] = mn[p % kDepth];
    uint4(&high)[kIters] = mx[p % kDepth];
    if (p == newest_pass) {
#pragma unroll
      for (int it = 0; it < kIters; ++it) {
        if (base_of(p) + kIters * grp + it == last) {
          low[it] = slot == 0 ? kn : order_key8(key_min8(order_key8(low[it]), key));
          high[it] = slot == 0 ? kn : order_key8(key_max8(order_key8(high[it]), key));
          r.low = low[it], r.high = high[it];
          r.mine = true;
        }
      }
    }
    if (base_of(p) < num_pages) {
      score_wave<kIters, kQ>(queries, low, high, num_pages - base_of(p), stage, lane, [&](bool has, int page, float score) {
        if (has) sm_score[base_of(p) + page] = score;
      });
    }
    if (p + kDepth < kPasses) load(p + kDepth);
  }
  wait_stores();  // the attention of this work-group reads the newest key and value
  return r;
}

// What the writer stores of it, behind the barrier that follows: the scores and the newest page's entry.
template <int kThreads>
__device__ __forceinline__ void store_row(const EstimateArgs& a, int b, int h, const float* sm_score, const RowOfPages& r) {
  float* row = a.scores + ((size_t)b * a.num_heads + h) * a.max_pages;
  for (int i = threadIdx.x; i < r.num_pages; i += kThreads) row[i] = sm_score[i];
  if (r.mine) {
    char* e = a.meta + meta_offset(a.num_phys_pages, r.newest_phys, h) + (lane_id() & 15) * 16;
    st16(e, r.low);
    st16(e + kHeadDim * 2, r.high);
  }
}

#endif  // __HIPCC__

}  // namespace quest
