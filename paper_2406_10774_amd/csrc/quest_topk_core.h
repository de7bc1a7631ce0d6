// Device-side core of the Top-K page selection (Section 3.4 of arXiv
// 2406.10774), shared by the stand-alone kernel and the attention launch that
// selects its pages itself.  See quest_topk.hip for the algorithm.
#pragma once

#include <type_traits>

#include "quest_common.h"

namespace quest {

#if defined(__HIPCC__)

// An unsigned key in the order of the scores, -0 equal to +0 (the negation of its bits is +0's
// key), and never 0.
__device__ __forceinline__ uint32_t score_key(float s) {
  const uint32_t u = __builtin_bit_cast(uint32_t, s);
  return (int32_t)u < 0 ? 0u - u : u | 0x80000000u;
}
__device__ __forceinline__ float score_of(uint32_t key) {
  return __builtin_bit_cast(float, (int32_t)key < 0 ? key ^ 0x80000000u : 0u - key);
}

// Inclusive prefix sum over the 64 lanes: DPP row shifts inside each 16-lane row, then the
// last lane of a row to the next row, and of the second row to the two behind it.
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 to rows 2 and 3
  return v;
}

// The same way: lane 63 ends up with the largest value of the 64 lanes.
__device__ __forceinline__ uint32_t wave_max_in_last(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
  return v;
}

// The bin of a 256-bin histogram in which the need-th entry lies, counting from bin 0.  Lane
// l owns bins 4l .. 4l + 3.  Every lane returns the same (bin, entries before the bin,
// entries in the bin).  No branches: one costs as much as ten instructions here.
struct BinHit {
  int bin, before, count;
};
template <int kCopies = 1>  // the histogram is the sum of that many
__device__ __forceinline__ BinHit find_bin(const uint32_t* hist, int need, int lane) {
  int4 c = reinterpret_cast<const int4*>(hist)[lane];
#pragma unroll
  for (int i = 1; i < kCopies; ++i) {
    const int4 more = reinterpret_cast<const int4*>(hist)[i * kWave + lane];
    c.x += more.x, c.y += more.y, c.z += more.z, c.w += more.w;
  }
  const int tot = c.x + c.y + c.z + c.w;
  const int incl = wave_incl_scan(tot);
  const int b0 = incl - tot, b1 = b0 + c.x, b2 = b1 + c.y, b3 = b2 + c.z;
  const bool p1 = b1 < need, p2 = b2 < need, p3 = b3 < need;  // the entry is past the lane's bin 0, 1, 2
  const int bin = 4 * lane + p1 + p2 + p3;
  const int before = p3 ? b3 : p2 ? b2 : p1 ? b1 : b0;
  const int count = p3 ? c.w : p2 ? c.z : p1 ? c.y : c.x;
  const int src = __popcll(__ballot(incl < need));  // the first lane that reaches it
  BinHit r;
  r.bin = __builtin_amdgcn_readlane(bin, src);
  r.before = __builtin_amdgcn_readlane(before, src);
  r.count = __builtin_amdgcn_readlane(count, src);
  return r;
}

// Pages kept whatever their score (quest.h: QUEST_FLAG_KEEP_FIRST_PAGE,
// QUEST_FLAG_KEEP_NEWEST_PAGE); the page of the newest token is the last valid one.
struct ForcedPages {
  bool first, newest;
  int newest_page, count;
  __device__ __forceinline__ bool is(int page) const {
    return (first && page == 0) || (newest && page == newest_page);
  }
};
__device__ __forceinline__ ForcedPages forced_pages(int policy, int num_pages) {
  ForcedPages f;
  f.newest_page = num_pages - 1;
  f.first = (policy & QUEST_FLAG_KEEP_FIRST_PAGE) != 0;
  f.newest = (policy & QUEST_FLAG_KEEP_NEWEST_PAGE) != 0 && !(f.first && f.newest_page == 0);
  f.count = (int)f.first + (int)f.newest;
  return f;
}

// Keys left in the threshold bin that are ranked directly, one per lane.
constexpr int kFewKeys = 64;

// Digits and places beside the keys are three registers a key.  Where those would spill, the keys
// alone tell all: radix digits of the key from the first pass on, and a place is handed out when a
// key turns out to be of the last bin.  32 rows of 65535 scores, K = 64: 19.6 us, 42.3 with digits and
// places partly in scratch memory; 512 rows 50 and 229; 49152 scores 15.7 and 28.0, 512 rows 37 and 128.
// (All but five of 49152: 36.1 us, 32.2: their leading bits need a pass more than bins of equal width.)
// 33 keys per thread fit (12.6 us; 12.7 to 15.8 from the keys alone).
constexpr bool keys_only(int threads, int items) { return 3 * items > 128 * 1024 / threads - 24; }

template <int kThreads, int kItems>
struct TopkShared {
  static constexpr int kWaves = kThreads / kWave;
  static constexpr int kRuns = kItems * kWaves;  // runs of 64 consecutive pages, one per wave and item
  static constexpr int kRunsPerLane = kRuns <= 64 ? 1 : kRuns <= 128 ? 2 : kRuns <= 256 ? 4 : kRuns <= 512 ? 8 : 16;
  static_assert(kItems <= kWave, "a lane per item");
  static_assert(kRuns <= kWave * kRunsPerLane && kWaves % kRunsPerLane == 0, "a wave's runs at one place of the lanes'");
  // Leading bits put many keys into the same few bins, and lanes with the same bin wait for each
  // other: a histogram for each quarter of the lanes (32 rows of 65535 scores on both sides of zero,
  // K = 32767: 61 us, 96 with one histogram).
  static constexpr int kCopies = keys_only(kThreads, kItems) ? 4 : 1;
  static constexpr int kSpare = 256 * kCopies;
  static_assert(kSpare <= kThreads, "cleared by one store a thread");
  // Entries for lanes that have nothing to write stand behind the others: a store or an atomic
  // without a condition is cheaper than a branch around it.
  uint32_t hist[kSpare + kWave];
  uint32_t few_key[kFewKeys + kWave], few_page[kFewKeys + kWave];  // the threshold bin's, in any order
  uint2 range[kWaves];                       // lower bound of the threshold (inverted) and largest key, by wave
  uint32_t count[kWave * kRunsPerLane];      // of each run: keys in front of the threshold bin (see topk_block_put)
  uint32_t few_count;                        // keys of the bin that have their place (if there are keys only)
};

// What a row of scores is, given the sequence length: its number of valid entries and
// which of them are kept whatever their score (QUEST_FLAG_KEEP_* bits).
struct RowShape {
  int num_pages, policy;
};
// The row holds the scores of all pages of the sequence.
struct WholeRow {
  int page_shift, policy;
  __device__ __forceinline__ RowShape operator()(int seq_len) const {
    return {(seq_len + (1 << page_shift) - 1) >> page_shift, policy};
  }
};

// The row holds the scores of the candidates that the chunks of the row left.
struct CandidateRow {
  int page_shift, policy, k_pages, chunk_pages;
  __device__ __forceinline__ RowShape operator()(int seq_len) const {
    const int pages = (seq_len + (1 << page_shift) - 1) >> page_shift;
    const int full = pages / chunk_pages;
    return {full * k_pages + min(k_pages, pages - full * chunk_pages), policy};
  }
};

// Inside a lane group of kGroup (2, 4, 8 or 16) lanes, one step towards the group's maximum: the
// value of a lane kGroup / 2 away, whose half of the group has its own maximum already.
template <int kGroup>
__device__ __forceinline__ uint32_t group_max_step(uint32_t v) {
  constexpr int kCtrl = kGroup == 2 ? 0xb1 : kGroup == 4 ? 0x4e : kGroup == 8 ? 0x141 : 0x140;
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true));
}

typedef unsigned long long LaneMask;
// `start` plus the lanes of the mask in front of this one.
__device__ __forceinline__ int lanes_before(LaneMask mask, int start) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, start));
}
// 1 if a < b, else 0: a compare would leave it in a lane mask, which the next instruction waits for.
__device__ __forceinline__ uint32_t is_less(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_sub_u32 %0, %1, %2 clamp" : "=v"(d) : "v"(b), "v"(a));  // 0 if b < a
  return min(d, 1u);
}
// v of one lane (a constant) becomes the wave-uniform value.
__device__ __forceinline__ void set_lane(uint32_t& v, int lane, uint32_t value) {
  asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(value), "n"(lane));
}
__device__ __forceinline__ bool in_mask(LaneMask mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// The part of topk_block_put that ranks: of the keys of pages first .. end - 1, all among the first
// kUsed pages of each thread, the `need` best go to put at positions from `first` on.
template <int kThreads, int kItems, int kUsed, class Put>
__device__ __forceinline__ void topk_rank(TopkShared<kThreads, kItems>& sm, const float (&raw)[kItems],
                                          int first, int end, int need, Put put) {
  constexpr int kWaves = kThreads / kWave;
  using Shared = TopkShared<kThreads, kItems>;
  constexpr bool kKeysOnly = keys_only(kThreads, kUsed);
  constexpr int kCopies = kKeysOnly ? Shared::kCopies : 1;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- A lower bound of the need-th largest key: the smallest of the largest keys of any
  // `need` or more disjoint sets of pages.  The sets are the pages of a thread, or of 2, 4,
  // .. 16 adjacent ones, or 2, 4, .. 16 equal parts of a thread's, whichever leave just enough of
  // them; a thread's pages lie kThreads apart, so every set samples the whole context.  Few
  // keys pass the bound (650 to 1500 of 8193 for 256).
  constexpr int kClasses = kUsed >= 16 ? 16 : kUsed >= 8 ? 8 : kUsed >= 4 ? 4 : kUsed >= 2 ? 2 : 1;
  uint32_t key[kUsed], best[kClasses];  // (key 0: none)
#pragma unroll
  for (int j = 0; j < kUsed; ++j) {
    const bool is_key = tid < end - j * kThreads && (j > 0 || tid >= first);
    key[j] = is_key ? score_key(raw[j]) : 0u;
    best[j % kClasses] = j < kClasses ? key[j] : max(best[j % kClasses], key[j]);
  }
  uint32_t lo = 0xffffffffu, hi = best[0];
#pragma unroll
  for (int c = 1; c < kClasses; ++c) hi = max(hi, best[c]);
  // (with page 0 kept, thread 0's sets may be empty: they stay out of the bound and of the count)
  const int spread = min(end, kThreads);
  if (spread - first >= need) {
    int group = 1;
    uint32_t v = hi;
    const auto widen = [&](int to, uint32_t wider) {
      const bool enough = (int)((unsigned)spread / to) - first >= need;
      v = enough ? wider : v;
      group = enough ? to : group;
    };
    widen(2, group_max_step<2>(v));
    widen(4, group_max_step<4>(v));
    widen(8, group_max_step<8>(v));
    widen(16, group_max_step<16>(v));
    const int leader = tid & -group;
    lo = leader >= first && leader < end ? v : lo;
  } else if (min(end, kClasses * kThreads) - kClasses * first >= need) {
    bool done = false;
    const auto parts = [&](auto parts_of_thread) {
      constexpr int kParts = decltype(parts_of_thread)::value;
      if constexpr (kParts <= kClasses) {
        if (done || min(end, kParts * kThreads) - kParts * first < need) return;
        done = true;
#pragma unroll
        for (int c = 0; c < kParts; ++c) {
          uint32_t v = best[c];
#pragma unroll
          for (int i = c + kParts; i < kClasses; i += kParts) v = max(v, best[i]);
          if (tid >= first && tid + c * kThreads < end) lo = min(lo, v);
        }
      }
    };
    parts(std::integral_constant<int, 2>{});
    parts(std::integral_constant<int, 4>{});
    parts(std::integral_constant<int, 8>{});
    parts(std::integral_constant<int, 16>{});
  } else {  // as many pages as that: the smallest key
#pragma unroll
    for (int j = 0; j < kUsed; ++j)
      if (key[j] > 0u) lo = min(lo, key[j]);
  }
  const uint2 reach = make_uint2(wave_max_in_last(~lo), wave_max_in_last(hi));
  if (lane == kWave - 1) sm.range[wave] = reach;
  __syncthreads();
  uint32_t not_lo = 0u;
  hi = 0u;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) not_lo = max(not_lo, sm.range[w].x), hi = max(hi, sm.range[w].y);
  lo = ~__builtin_amdgcn_readfirstlane(not_lo);
  hi = __builtin_amdgcn_readfirstlane(hi);

  // ---- Count the keys from lo on in 256 bins of equal width between the scores hi and lo: the bin never
  // decreases as scores fall, whatever the rounding, and equal keys share one (if the width is no
  // number or no finite one, all share bin 0).  Scores rather than their bits: those of a range that
  // spans zero are nearly all exponents.  The list takes every key in front of the bin in which the
  // need-th lies, and then `need` of the keys in it: 5 to 50 with the bound above, few enough to
  // rank directly.
  const uint32_t range = hi - lo;
  uint32_t digit[kUsed];  // the bin; behind all bins for what does not count
  uint32_t slot[kUsed];   // a key's place among those of its bin, in any order
  BinHit hit = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < kUsed; ++j) key[j] = hi - key[j];  // 0: the best; what is no key ranks behind every key
  if constexpr (!kKeysOnly) {
    const float hi_score = score_of(hi), bins = 256.f * __builtin_amdgcn_rcpf(hi_score - score_of(lo));
    const float hi_bins = hi_score * bins;
#pragma unroll
    for (int j = 0; j < kUsed; ++j) {
      const float x = __builtin_fmaf(raw[j], -bins, hi_bins);
      uint32_t bin;
      asm("v_cvt_u32_f32 %0, %1" : "=v"(bin) : "v"(x));  // below 0 and NaN: 0; too large: the largest
      digit[j] = key[j] <= range ? min(bin, 255u) : Shared::kSpare + lane;
      slot[j] = atomicAdd(&sm.hist[digit[j]], 1u);
    }
    __syncthreads();
    hit = find_bin(sm.hist, need, lane);
    need -= hit.before;
  }
  // The bin's keys: those from `base` to `base + last` (with digits, of those in the bin).
  uint32_t base = 0u, last = range;
  if (kKeysOnly || (need != hit.count && hit.count > kFewKeys)) {
    // Radix select among the bin's keys, 8-bit digits from the leading bit of the range, until the
    // keys left are few or equal.  Then keys in front, in the last bin and behind are told apart.
    const uint32_t bin0 = hit.bin;
    int shift = range ? 32 - __builtin_clz(range) : 0;
    bool clear = !kKeysOnly;
#pragma unroll 1
    do {
      shift = max(shift - 8, 0);
      if (clear) {
        __syncthreads();
        if (tid < 256 * kCopies) sm.hist[tid] = 0;
        __syncthreads();
      }
      clear = true;
#pragma unroll
      for (int j = 0; j < kUsed; ++j) {
        const uint32_t rest = key[j] - base;
        const bool counts = (kKeysOnly || digit[j] == bin0) && rest <= last;
        const uint32_t bin = (rest >> shift) + (lane & (kCopies - 1)) * 256;
        const uint32_t at = atomicAdd(&sm.hist[counts ? bin : Shared::kSpare + lane], 1u);
        if constexpr (!kKeysOnly) slot[j] = at;
      }
      __syncthreads();
      hit = find_bin<kCopies>(sm.hist, need, lane);
      base += (uint32_t)hit.bin << shift;
      last = min(last - ((uint32_t)hit.bin << shift), (1u << shift) - 1u);
      need -= hit.before;
    } while (need != hit.count && hit.count > kFewKeys && shift > 0);
    if constexpr (!kKeysOnly) {
#pragma unroll
      for (int j = 0; j < kUsed; ++j) {
        const bool front = digit[j] < bin0 || (digit[j] == bin0 && key[j] < base);
        const bool inside = digit[j] == bin0 && !front && key[j] - base <= last;
        digit[j] = front ? 0u : inside ? 1u : 2u;
      }
      hit.bin = 1;
    }
  }
  const bool whole = need == hit.count;                    // the list takes all of the bin
  const int n_few = !whole && hit.count <= kFewKeys ? hit.count : 0;
  const bool ties = !whole && n_few == 0;                  // more equal keys than places: the lowest pages

  // ---- List positions in page order.  A wave's j-th pages are a run of 64 consecutive ones,
  // runs follow each other by (j, wave); the runs' counts go through LDS, and so do, in
  // any order, the few keys of the bin with their pages.
  const uint32_t bin_at = kKeysOnly ? base : hit.bin, bin_end = kKeysOnly ? base + last + 1u : hit.bin + 1;
  const uint32_t front_end = whole ? bin_end : bin_at;
  const auto in_front = [&](int j) { return (kKeysOnly ? key[j] : digit[j]) < front_end; };
  const auto in_bin = [&](int j) { return kKeysOnly ? key[j] - base <= last : digit[j] == bin_at; };
  uint32_t my_count = 0;
#pragma unroll
  for (int j = 0; j < kUsed; ++j)
    set_lane(my_count, j, __popcll(__ballot(in_front(j))));
  if (n_few > 0) {
#pragma unroll
    for (int j = 0; j < kUsed; ++j) {
      if constexpr (kKeysOnly) {
        if (in_bin(j)) {
          const uint32_t to = atomicAdd(&sm.few_count, 1u);
          sm.few_key[to] = key[j];
          sm.few_page[to] = tid + j * kThreads;
        }
      } else {
        const uint32_t to = in_bin(j) ? slot[j] : kFewKeys + lane;
        sm.few_key[to] = key[j];
        sm.few_page[to] = tid + j * kThreads;
      }
    }
  } else if (ties) {  // rows have fewer than 2^16 pages
#pragma unroll
    for (int j = 0; j < kUsed; ++j) {
      const uint32_t n = __popcll(__ballot(in_bin(j)));
      my_count += lane == j ? n << 16 : 0u;
    }
  }
  if (lane < kUsed) sm.count[lane * kWaves + wave] = my_count;
  __syncthreads();
  constexpr int kPerLane = Shared::kRunsPerLane;
  uint32_t part[kPerLane];
  int sum = 0;
#pragma unroll
  for (int i = 0; i < kPerLane; ++i) {
    part[i] = sm.count[lane * kPerLane + i];  // (lanes past the runs get what is there, and nobody looks at them)
    sum += (int)part[i];
  }
  // The few keys, one per lane: those with fewer than `need` better ones are taken, unless
  // equal keys stand at the threshold: then the lowest of their pages.  Every wave does it.
  uint32_t threshold = 0u;           // the last key that the list takes
  uint32_t few_page = 0xffffffffu;   // of a key that is taken
  uint32_t last_page = 0u;           // the last page that it takes of keys equal to that one
  bool split_ties = false;
  if (n_few > 0) {
    const uint32_t mine = sm.few_key[lane];
    few_page = sm.few_page[lane];
    uint32_t better = 0;
#pragma unroll 1
    for (int i = 0; i < n_few; i += 16) {
      const uint4* them = reinterpret_cast<const uint4*>(sm.few_key + i);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint4 t = them[k];
        better += is_less(t.x, mine) + is_less(t.y, mine);
        better += is_less(t.z, mine) + is_less(t.w, mine);
      }
    }
    const LaneMask filled = ~0ull >> (kWave - n_few);
    const LaneMask at_threshold = filled & __ballot(better == (uint32_t)need - 1u);
    LaneMask taken;
    if (__popcll(at_threshold) == 1) {
      threshold = __builtin_amdgcn_readlane((int)mine, __ffsll((long long)at_threshold) - 1);
      taken = filled & __ballot(mine <= threshold);
    } else {
      taken = filled & __ballot(better < (uint32_t)need);
      split_ties = true;
      const uint32_t most = wave_max_in_last(in_mask(taken) ? better : 0u);
      int places = __builtin_amdgcn_readlane((int)most, kWave - 1);
      LaneMask left = taken & __ballot(better == (uint32_t)places);
      threshold = __builtin_amdgcn_readlane((int)mine, __ffsll((long long)left) - 1);
      taken &= ~left;
      places = need - places;
#pragma unroll 1
      for (int bit = 15; bit >= 0; --bit) {
        const LaneMask zeros = left & ~__ballot((few_page >> bit) & 1u);
        const int c = __popcll(zeros);
        if (c >= places) {
          left = zeros;
        } else {
          taken |= zeros;
          left &= ~zeros;
          places -= c;
        }
      }
      taken |= left;
      last_page = wave_max_in_last(in_mask(taken) && mine == threshold ? few_page : 0u);
      last_page = __builtin_amdgcn_readlane((int)last_page, kWave - 1);
    }
    few_page = in_mask(taken) ? few_page : 0xffffffffu;
  }
  int before = wave_incl_scan(sum) - sum;
#pragma unroll
  for (int i = 0; i + 1 < kPerLane; ++i)
    if (i < (wave & (kPerLane - 1))) before += (int)part[i];
  const auto front_before = [&](int j) {
    return (uint32_t)__builtin_amdgcn_readlane(before, (j * kWaves + wave) / kPerLane);
  };
  const auto few_before = [&](int j) {
    return __popcll(__ballot(few_page < (uint32_t)(j * kThreads + wave * kWave)));
  };
  if (!split_ties && !ties) {
    const uint32_t upto = whole ? bin_end - 1u : threshold;
#pragma unroll
    for (int j = 0; j < kUsed; ++j) {
      const LaneMask sel = __ballot((whole && !kKeysOnly ? digit[j] : key[j]) <= upto);
      const int at = (int)front_before(j) + few_before(j) + first;
      put(in_mask(sel), lanes_before(sel, at), tid + j * kThreads, j, raw[j]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < kUsed; ++j) {
      LaneMask sel;
      const uint32_t b = front_before(j);  // with ties: and the equal keys before, in the upper half
      int at = (int)(b & 0xffffu) + few_before(j) + first;
      if (split_ties) {
        const uint32_t page = tid + j * kThreads;
        sel = __ballot(key[j] < threshold || (key[j] == threshold && page <= last_page));
      } else {
        const LaneMask equal = __ballot(in_bin(j));
        const int ties_before = (int)(b >> 16);
        sel = __ballot(in_front(j)) | (equal & __ballot(lanes_before(equal, ties_before) < need));
        at += min(ties_before, need);
      }
      put(in_mask(sel), lanes_before(sel, at), tid + j * kThreads, j, raw[j]);
    }
  }
}

// Selection for one row of scores by one work-group of kThreads threads (all of
// them must call): thread t has the scores of entries t + j * kThreads (whatever stands past the
// valid ones).  row_shape describes the row (it has room for max_pages
// entries); put(selected, position, page, j, score) receives the list from the threads that pass
// selected (the others' arguments mean nothing, but position is at least 0): positions 0 .. k_pages-1,
// pages ascending, -1 past the K_b selected ones; j >= 0 says that the page is the calling
// thread's j-th one (page == threadIdx.x + j * kThreads) and `score` its score as loaded,
// j < 0 that it is not (then `score` carries nothing).  A put that needs per-page data
// takes it from what the thread already holds whenever j >= 0: a load issued from inside
// put is waited for before the next page's put starts.
template <int kThreads, int kItems, class Put>
__device__ __forceinline__ void topk_select(TopkShared<kThreads, kItems>& sm, const float (&raw)[kItems],
                                            const RowShape row_shape, int max_pages, int k_pages, Put put,
                                            int32_t* __restrict__ k_eff_slot) {
  using Shared = TopkShared<kThreads, kItems>;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  if (tid < Shared::kSpare) sm.hist[tid] = 0;
  if (wave == 0) sm.few_key[lane] = 0xffffffffu;
  if constexpr (Shared::kCopies > 1)
    if (tid == 0) sm.few_count = 0;

  const int num_pages = min(row_shape.num_pages, max_pages);  // whatever the length says: no entry past the row
  const int K = min(k_pages, num_pages);
  if (tid == 0 && k_eff_slot != nullptr) *k_eff_slot = K;
  if (K == num_pages) {  // everything is selected: identity list, padded with -1
    for (int i = tid; i < k_pages; i += kThreads) put(true, i, i < K ? i : -1, -1, 0.f);
    return;
  }

  // Pages that are kept whatever their score rank above every score and, like
  // equal scores, by page index: they are no keys, take their places off the count,
  // and are the first and the last entry of the list.
  const ForcedPages forced = forced_pages(row_shape.policy, num_pages);
  if (forced.count >= K) {  // K is 1 or 2 here: the list is the forced pages, lowest first
    if (tid == 0) {
      put(true, 0, forced.first ? 0 : num_pages - 1, -1, 0.f);
      if (K == 2) put(true, 1, num_pages - 1, -1, 0.f);
    }
    return;
  }
  const int first = forced.first, end = num_pages - (int)forced.newest;  // the keys: pages first .. end - 1
  int need = K - forced.count;  // how many of them the list takes, at least one

  // A sequence that ends far in front of a long row's end leaves most of a thread's pages empty: the
  // work is then done for the first of them only (rows of 8704 pages of which 435 hold tokens, K = 32, a launch
  // that selects and attends: 7.9 us, 9.2 for all of them; quest_topk of rows of 6100 pages, a tenth of them in use,
  // 32 rows 4.1 and 5.0 us).
  constexpr int kPart = kItems >= 10 ? kItems * 3 / 8 : kItems;
  const auto rank = [&](auto items) {
    topk_rank<kThreads, kItems, decltype(items)::value>(sm, raw, first, end, need, put);
  };
  if (kPart < kItems && end <= kPart * kThreads)
    rank(std::integral_constant<int, kPart>{});
  else
    rank(std::integral_constant<int, kItems>{});
  if (forced.count > 0) {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int page = tid + j * kThreads;
      put(forced.first && page == 0, 0, page, j, raw[j]);
      put(forced.newest && page == num_pages - 1, K - 1, page, j, raw[j]);
    }
  }
}

// The same for a row of scores in memory.  shape(seq_len) describes the row.
// after_loads() is called once, right after the loads of the scores have been issued:
// the place for loads the caller wants in flight behind them.
template <int kThreads, int kItems, class Put, class Shape, class AfterLoads>
__device__ __forceinline__ void topk_block_put(TopkShared<kThreads, kItems>& sm,
                                               const float* __restrict__ row,
                                               const int32_t* __restrict__ seq_len_ptr,
                                               int max_pages, int k_pages, Put put,
                                               int32_t* __restrict__ k_eff_slot, Shape shape,
                                               AfterLoads after_loads) {
  const int tid = threadIdx.x;

  // issue every load first: this thread's scores (entries past the valid pages
  // are inside the row, so reading them is safe; they are masked later) and the
  // sequence length
  float raw[kItems];
  const uint32_t last_offset = ((uint32_t)max_pages - 1u) * (uint32_t)sizeof(float);
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    // clamped, not predicated: the loads stay independent and all in flight at once
    const uint32_t at = min((uint32_t)(tid + j * kThreads) * (uint32_t)sizeof(float), last_offset);
    raw[j] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + at);
  }
  const int seq_len = __builtin_amdgcn_readfirstlane(*seq_len_ptr);
  after_loads();
  topk_select<kThreads, kItems>(sm, raw, shape(seq_len), max_pages, k_pages, put, k_eff_slot);
}

// The list goes to memory.
template <int kThreads, int kItems>
__device__ __forceinline__ void topk_block(TopkShared<kThreads, kItems>& sm, const float* __restrict__ row,
                                           const int32_t* __restrict__ seq_len_ptr, int max_pages,
                                           int k_pages, int32_t* __restrict__ out,
                                           int32_t* __restrict__ k_eff_slot, int page_shift,
                                           int policy) {
  topk_block_put<kThreads, kItems>(
      sm, row, seq_len_ptr, max_pages, k_pages, [out](bool sel, int pos, int page, int, float) {
        if (sel) out[pos] = page;
      },
      k_eff_slot, WholeRow{page_shift, policy}, [] {});
}

#endif  // __HIPCC__

}  // namespace quest
