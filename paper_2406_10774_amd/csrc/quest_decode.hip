// Sparse paged decode attention (Figure 5 stage 2 / Section 3.4 of arXiv
// 2406.10774): ordinary softmax attention of one query per (sequence, head)
// over the tokens of the selected pages only.  Attention over every page is
// quest_dense.hip, with rows of few tokens and little work done here: their list is the row.
//
// Split-K flash-decoding.  One work-group per (sequence, head, split); each work-group of
// four waves owns a contiguous slice of the head's page list, its waves take
// the slice's pages round-robin.  A wave streams one unit (up to 16 tokens of one
// page: 4 KiB of keys and 4 KiB of values = 4 + 4 wave-wide 16-byte loads; pages
// of 32 or 64 tokens are 2 or 4 units, pages of 8 tokens units of 2 + 2 loads) per
// step, double-buffered in registers so the next unit's loads are in flight while
// the current one is reduced.  Lane l holds channels 8*(l%16)..+7 of tokens
// l/16 + 4r; q.k is a v_dot2_f32_f16 chain plus a reduction inside the 16-lane
// DPP row; each DPP row keeps its own online softmax state (running max,
// denominator, 8 accumulator channels per lane) in fp32, in the log2 domain.
// Rows, waves and finally splits are merged with the usual (max, sum,
// accumulator) rescaling; the split that finishes last merges the partial
// results of all splits of its head.
//
// With one query head per KV head this is a matrix-vector product (about one flop per
// byte read): no matrix cores, the kernel is bound by how fast HBM delivers the 8 KiB per
// selected (page, head).  With grouped-query attention up to eight query heads meet each
// key and value; a work-group serves them all from one load on the matrix cores
// (GroupState in quest_decode_core.h).  32 query / 8 KV heads, 4 sequences of up to 32k
// tokens: a step takes 23 us instead of 40 us (2048-token budget; every query head loaded
// its pages and selected its list alone).  Short lists of few heads are the exception: see
// heads_apart.
#include "quest_common.h"
#include "quest_decode_core.h"
#include "quest_estimate_core.h"
#include "quest_team.h"
#include "quest_topk_core.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace quest {

namespace {

constexpr long kComputeUnits = 256, kDies = 8;  // MI355X; only used to decide how finely to split
constexpr int kDecWaves = 4;
// With the selection done in the same launch (see decode_split_kernel): room in LDS for a page list
// of this many entries, scores per thread up to which their page-table entries are fetched with
// them, and the longest row.
constexpr int kSelListCap = 2048;
constexpr int kLookAhead = 8;
constexpr int kMostSelected = 512 * 17, kMostSelectedOfGroup = 512 * 10;

struct DecodeArgs : AttnArgs {
  const int32_t* topk_idx;  // the page list [B][kv heads][k_pages] (nullptr: selected inside the launch, or every page)
  const float* scores;      // selection inside the launch: scores [B][kv heads][max_pages] ...
  int32_t* topk_out;        // ... the list is also written here [B][kv heads][k_pages] ...
  int32_t* k_eff;           // ... and K_b here (nullable)
  const int32_t* cand_page; // their pages, if the scores are those of candidates
  int row_len;              // entries of a row of scores: max_pages, or candidates
  int chunk_pages;          // pages that k_pages candidates stand for
  int policy;               // QUEST_FLAG_KEEP_* bits
  int k_pages, splits;
  int list_len;             // entries of the page list the splits divide
  int per_split;            // ceil(list_len / splits)
  uint32_t seq_inverse;     // ceil(2^32 / items per sequence), if that is exact for every item; else 0
};

struct StepArgs : DecodeArgs {
  EstimateArgs est;
};

// All splits of one (sequence, head) get work-group ids that are equal modulo 8
// (grid.x is a multiple of 8), so under the usual round-robin placement they run on
// one die and their traffic stays in one L2.  Nothing depends on that: partial results
// are handed over with device-scope stores and loads (quest_team.h), correct wherever
// the splits run; the split that finishes last merges them, without a second launch.
// kLoads, kGroup: see HeadState; a work-group serves one query head, or up to kGroupHeads
// of a KV head, so that a page is loaded (and a list selected) once for all of them.
// a.subs: work-groups per KV head and split that this takes.
//
// kSelItems > 0: the page list does not exist yet.  Every work-group first selects the
// pages of its head itself from the scores (the same selection as quest_topk, kSelItems
// scores per thread), keeps the list in LDS and uses its own slice; split 0 also writes
// the list out.  The selection is repeated by every split of a head, which costs nothing
// that matters (the compute units would idle meanwhile) and saves a launch and the trip
// of the list through memory.
//
// kCand: the scores are those of candidates that a launch before has picked from the chunks
// of a longer row, each with its page.
//
// kEstPasses > 0: the scores do not exist either: the whole step is this launch.  Every work-group scores
// its row itself (estimate_row, with kEstPasses and kEstQ), then selects; step_in_one_launch says when.
//
// kSelWaves: waves that select; those past kWaves end when the list is there (a barrier counts the waves that
// are left).
template <int kLoads, bool kGroup, int kWaves, int kSelItems, bool kCand, int kEstPasses = 0, int kEstQ = 0,
          int kSelWaves = kWaves>
__global__ __launch_bounds__(kSelWaves* kWave) void decode_split_kernel(
    const typename std::conditional<(kEstPasses > 0), StepArgs, DecodeArgs>::type a) {
  using Head = HeadState<kLoads, kGroup>;
  static_assert(kSelWaves == kWaves || kEstPasses == 0, "the others have nothing but the list to do");
  constexpr int kThreads = kWaves * kWave, kSelThreads = kSelWaves * kWave;
  constexpr int kSlots = Head::kSlots, kStride = Head::kStride;
  __shared__ __align__(16) float sm_acc[kWaves][kSlots * kStride];
  __shared__ float sm_m[kWaves][kSlots], sm_l[kWaves][kSlots];
  __shared__ uint32_t sm_before;
  // the selection's LDS only where there is a selection; the list as (logical page,
  // physical page) pairs
  __shared__ __align__(16) typename std::conditional<(kSelItems > 0), TopkShared<kSelThreads, kSelItems>, char>::type sm_topk;
  __shared__ int2 sm_list[kSelItems > 0 ? kSelListCap + kWave : 1];
  // of a row that is scored here: scores and physical pages, and where groups turn the metadata (a group's
  // attention has room for that)
  constexpr int kIters = kEstQ == 0 ? 2 : 4;  // pages per wave and pass: four times that
  constexpr int kRow = kEstPasses > 0 ? kWaves * kEstPasses * 4 * kIters : 1;
  constexpr int kStage = 4 * kIters * kMetaBytes;
  __shared__ float sm_score[kRow];
  __shared__ int sm_phys[kRow];
  __shared__ __align__(16) char sm_stage[kEstPasses > 0 && kEstQ == 0 && !kGroup ? kWaves * kStage : 16];
  static_assert(kEstQ != 0 || !kGroup || kEstPasses == 0 || sizeof(sm_acc[0]) >= kStage, "metadata of a wave");

  // Every argument in one trip to memory, not one per use: 0.2 us less until the first score.
  asm volatile("" ::"s"(a.batch), "s"(a.kv_heads), "s"(a.subs), "s"(a.group), "s"(a.num_heads), "s"(a.max_pages), "s"(a.seq_inverse),
               "s"(a.page_table), "s"(a.seq_lens), "s"(a.q), "s"(a.scores), "s"(a.row_len), "s"(a.k_pages));
  asm volatile("" ::"s"(a.k_pool), "s"(a.v_pool), "s"(a.counters), "s"(a.per_split), "s"(a.list_len), "s"(a.splits),
               "s"(a.page_shift), "s"(a.unit_shift), "s"(a.scale_log2), "s"(a.policy), "s"(a.topk_out), "s"(a.k_eff));
  if constexpr (kEstPasses > 0)
    asm volatile("" ::"s"(a.est.meta), "s"(a.est.q), "s"(a.est.scores), "s"(a.est.k_new), "s"(a.est.v_new), "s"(a.est.k_pool),
                 "s"(a.est.v_pool), "s"(a.est.k_pool_write), "s"(a.est.num_phys_pages));
  // blockIdx.x = slot + 8 * split, blockIdx.y = group of 8 items: the linear work-group
  // id is slot + 8 * (split + splits * blockIdx.y).  The usual shapes are taken apart without
  // integer divisions: they sit in front of the first load of every work-group.
  const int slot = blockIdx.x & 7;
  const int split = blockIdx.x >> 3;
  const int item = blockIdx.y * 8 + slot;  // (sequence, KV head, query heads of its group)
  const int subs = a.subs;
  const int per_seq = a.kv_heads * subs;
  if (item >= a.batch * per_seq) return;
  const int b = a.batch == 1 ? 0 : a.seq_inverse ? (int)__umulhi(item, a.seq_inverse) : item / per_seq;
  const int in_seq = item - b * per_seq;
  const int hk = subs == 1 ? in_seq : in_seq / subs;  // the KV head: its pages, its page list
  const int sub = in_seq - hk * subs;
  const int h = hk * a.group + sub * kSlots;  // first query head served here
  const int n_heads = kGroup ? min(kSlots, a.group - sub * kSlots) : 1;
  const size_t bh = (size_t)b * a.num_heads + h;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = lane_id();
  uint32_t* arrivals = reinterpret_cast<uint32_t*>(a.counters + bh * kTeamWordStride);

  // This work-group's share of the page list: positions begin .. end - 1 (two pages per
  // unit: pairs of positions).  The list length is known on the host, so list entries and
  // page-table entries are fetched without waiting for seq_lens; entries past the valid
  // pages are dropped afterwards.
  const int begin = split * a.per_split;
  const int end = min(a.list_len, begin + a.per_split);
  const int entries = Head::kTwoPages ? (a.per_split + 1) >> 1 : a.per_split;
  const int32_t* pt = a.page_table + (size_t)b * a.max_pages;
  const char* q = a.q + bh * (kHeadDim * 2);
  int seq_len;
  Head st;
  if constexpr (kSelItems > 0) {
    const size_t row = (size_t)b * a.kv_heads + hk;
    const bool writer = split == 0 && sub == 0;  // one work-group per list writes it out
    // Behind the loads of the scores (loads complete in order, so nothing may be in front
    // of what the selection waits for): the page-table entries of this thread's pages,
    // which travel with their scores so that the list needs no look-up afterwards, and
    // what the attention needs besides the pages.
    // (of candidates: their logical pages)
    constexpr bool kLate = !kCand && kSelItems > kLookAhead;
    int mine[kSelItems];
    const int32_t* per_score = kCand ? a.cand_page + row * a.row_len : pt;
    auto more_loads = [&] {
#pragma unroll
      for (int j = 0; j < (kLate ? 0 : kSelItems); ++j)
        mine[j] = per_score[min((int)threadIdx.x + j * kSelThreads, a.row_len - 1)];
      seq_len = a.seq_lens[b];
      st.init(sm_acc[kSelWaves > kWaves ? min(wave, kWaves - 1) : wave], q, n_heads, lane);
    };
    // Lanes without a page write to entries of their own behind the list.
    auto put = [&](bool selected, int pos, int entry, int j, float) {
      int of = kCand ? -1 : 0;
      if (kLate) {
      } else if (j >= 0) {
#pragma unroll
        for (int jj = 0; jj < kSelItems; ++jj)
          if (jj == j) of = mine[jj];
      } else if (entry >= 0) {
        of = kEstPasses > 0 ? sm_phys[entry] : per_score[entry];
      }
      sm_list[selected ? pos : kSelListCap + lane] = make_int2(kCand ? of : entry, of);
    };
    int32_t* k_eff = (writer && hk == 0 && a.k_eff != nullptr) ? a.k_eff + b : nullptr;
    const float* scores = a.scores + row * a.row_len;
    if constexpr (kEstPasses > 0) {
      st.init(sm_acc[wave], q, n_heads, lane);
      char* stage = kGroup ? reinterpret_cast<char*>(sm_acc[wave]) : sm_stage + (sizeof(sm_stage) > 16 ? wave * kStage : 0);
      const RowOfPages r = estimate_row<kWaves, kEstPasses, kIters, kEstQ>(a.est, b, hk, wave, stage, sm_score, sm_phys);
      seq_len = r.seq_len;
      __syncthreads();
      if (writer) store_row<kThreads>(a.est, b, hk, sm_score, r);
      float raw[kSelItems];
#pragma unroll
      for (int j = 0; j < kSelItems; ++j) {
        const int at = min((int)threadIdx.x + j * kThreads, kRow - 1);
        raw[j] = sm_score[at];
        mine[j] = sm_phys[at];
      }
      topk_select<kThreads, kSelItems>(sm_topk, raw, WholeRow{a.page_shift, a.policy}(seq_len), a.row_len, a.k_pages, put,
                                       k_eff);
    } else if constexpr (kCand)
      topk_block_put<kSelThreads, kSelItems>(sm_topk, scores, a.seq_lens + b, a.row_len, a.k_pages, put, k_eff,
                                          CandidateRow{a.page_shift, a.policy, a.k_pages, a.chunk_pages}, more_loads);
    else
      topk_block_put<kSelThreads, kSelItems>(sm_topk, scores, a.seq_lens + b, a.row_len, a.k_pages, put, k_eff,
                                          WholeRow{a.page_shift, a.policy}, more_loads);
    __syncthreads();
    if (writer)
      for (int i = threadIdx.x; i < a.k_pages; i += kSelThreads) a.topk_out[row * a.k_pages + i] = sm_list[i].x;
    if (kSelWaves > kWaves && wave >= kWaves) return;
  } else {
    seq_len = a.seq_lens[b];
    st.init(sm_acc[wave], q, n_heads, lane);
  }

  // A page is streamed as 1 << unit_shift units of up to 16 tokens, which the waves take in
  // turn (so that a split of few large pages still occupies all of them).
  const int units = ((entries << a.unit_shift) + kWaves - 1) / kWaves;
  const int num_pages = (seq_len + (1 << a.page_shift) - 1) >> a.page_shift;
  attend<kLoads, kGroup>(st, a, hk, seq_len, units, q, n_heads, sm_acc[wave], sm_m[wave], sm_l[wave], lane,
                         [&](int i, int& lp, int& ph, int& un, int& lp2, int& ph2) {
    const int u = wave + kWaves * i;
    const int e = u >> a.unit_shift;
    un = u & ((1 << a.unit_shift) - 1);
    auto entry_at = [&](int pos, int& l, int& p) {
      if constexpr (kSelItems > 0) {
        if (pos < end) {
          const int2 entry = sm_list[pos];
          l = entry.x, p = entry.y;
          if ((kCand || kSelItems > kLookAhead) && l >= 0) p = pt[l];
        }
      } else {
        if (pos < end) l = a.topk_idx ? a.topk_idx[((size_t)b * a.kv_heads + hk) * a.k_pages + pos] : pos;
        if (l >= 0 && l < a.max_pages) p = pt[l];
      }
      if (l >= num_pages) l = -1;
    };
    if constexpr (Head::kTwoPages) {
      entry_at(begin + 2 * e, lp, ph);
      entry_at(begin + 2 * e + 1, lp2, ph2);
    } else {
      entry_at(begin + e, lp, ph);
    }
  });

  __syncthreads();
  const int t = threadIdx.x;
  // ---- this split's result per query head: written out if it is the only split, else
  // published as a partial; the split that arrives last merges
  if constexpr (kGroup) {  // a head per wave, two channels a lane: its weights once
    for (int g = wave; g < n_heads; g += kWaves) {
      const int part = lane & (kWaves - 1);
      const Merged all = merge_parts(sm_m[part][g], sm_l[part][g], kWaves, lane);
      float2 acc = make_float2(0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float2 x = *reinterpret_cast<const float2*>(&sm_acc[w][g * kStride + 2 * lane]);
        const float f = from_lane(all.weight, w);
        acc.x += x.x * f, acc.y += x.y * f;
      }
      if (a.splits == 1) {
        store_out2(a.out, a.out_is_fp16, (bh + g) * kHeadDim + 2 * lane, acc.x / all.l, acc.y / all.l);
        if (lane == 0 && a.lse) a.lse[bh + g] = (all.m + __builtin_amdgcn_logf(all.l)) * kLn2;
      } else {
        const size_t ps = (bh + g) * a.splits + split;
        dev_st2(a.part_acc + ps * kHeadDim + 2 * lane, acc);
        if (lane == 0) dev_st2(a.part_ml + ps * 2, make_float2(all.m, all.l));
      }
    }
  } else {
    for (int ch = t; ch < kHeadDim; ch += kThreads) {
      float m_tot = sm_m[0][0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) m_tot = fmaxf(m_tot, sm_m[w][0]);
      float l_tot = 0.f, acc = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(sm_m[w][0] - m_tot);
        l_tot += sm_l[w][0] * f;
        acc += sm_acc[w][ch] * f;
      }
      if (a.splits == 1) {
        store_out(a.out, a.out_is_fp16, bh * kHeadDim + ch, acc / l_tot);
        if (ch == 0 && a.lse) a.lse[bh] = (m_tot + __builtin_amdgcn_logf(l_tot)) * kLn2;
      } else {
        const size_t ps = bh * a.splits + split;
        dev_st(a.part_acc + ps * kHeadDim + ch, acc);
        if (ch == 0) {
          dev_st(a.part_ml + ps * 2 + 0, m_tot);
          dev_st(a.part_ml + ps * 2 + 1, l_tot);
        }
      }
    }
  }
  if (a.splits == 1) return;
  wait_stores();
  __syncthreads();
  if (t == 0) sm_before = team_arrive(arrivals, a.device_fences);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(sm_before) != (uint32_t)a.splits - 1) return;
  team_acquire(a.device_fences);
  if (t == 0) team_reset(arrivals);

  // one pass over the splits in chunks of 8 (a group's of 16), all loads of a chunk in flight at
  // once, with a running maximum (the same rescaling as between pages); always in split order, so
  // the result does not depend on which split arrived last
  if constexpr (kGroup) {
#pragma unroll 1
    for (int g = wave; g < n_heads; g += kWaves) {
      const float* ml = a.part_ml + (bh + g) * a.splits * 2;
      const float* pacc = a.part_acc + (bh + g) * a.splits * kHeadDim + 2 * lane;
      float mx = kNegBig, l_all = 0.f;
      float2 o = make_float2(0.f, 0.f);
      for (int s0 = 0; s0 < a.splits; s0 += 16) {
        const int n = min(16, a.splits - s0);
        const float2 pml = dev_ld2(ml + 2 * (s0 + min(lane & 15, n - 1)));
        float2 pa[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) pa[i] = dev_ld2(pacc + (size_t)(s0 + min(i, n - 1)) * kHeadDim);
        if (n > 8) {
#pragma unroll
          for (int i = 8; i < 16; ++i) pa[i] = dev_ld2(pacc + (size_t)(s0 + min(i, n - 1)) * kHeadDim);
        }
        const Merged part = merge_parts(pml.x, pml.y, n, lane);
        const float cm = fmaxf(mx, part.m);
        const float rescale = __builtin_amdgcn_exp2f(mx - cm), scale = __builtin_amdgcn_exp2f(part.m - cm);
        l_all = l_all * rescale + part.l * scale;
        o.x *= rescale, o.y *= rescale;
        const float weight = part.weight * scale;
        const auto add = [&](int i) {
          const float f = from_lane(weight, i);
          o.x += pa[i].x * f, o.y += pa[i].y * f;
        };
        // (what is not there is left out, not taken times zero: the values may be infinite)
        if (n >= 8) {
#pragma unroll
          for (int i = 0; i < 8; ++i) add(i);
#pragma unroll
          for (int i = 8; i < 16; ++i)
            if (i < n) add(i);
        } else {
#pragma unroll
          for (int i = 0; i < 7; ++i)
            if (i < n) add(i);
        }
        mx = cm;
      }
      store_out2(a.out, a.out_is_fp16, (bh + g) * kHeadDim + 2 * lane, o.x / l_all, o.y / l_all);
      if (lane == 0 && a.lse) a.lse[bh + g] = (mx + __builtin_amdgcn_logf(l_all)) * kLn2;
    }
  } else {
#pragma unroll 1
    for (int ch = t; ch < kHeadDim; ch += kThreads) {
      const float* ml = a.part_ml + bh * a.splits * 2;
      const float* pacc = a.part_acc + bh * a.splits * kHeadDim + ch;
      float mx = kNegBig, l_all = 0.f, o = 0.f;
      for (int s0 = 0; s0 < a.splits; s0 += 8) {
        float2 pml[8];
        float pa[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int sidx = min(s0 + i, a.splits - 1);
          pml[i] = dev_ld2(ml + 2 * sidx);
          pa[i] = dev_ld(pacc + (size_t)sidx * kHeadDim);
        }
        float cm = mx;
#pragma unroll
        for (int i = 0; i < 8; ++i) cm = fmaxf(cm, pml[i].x);
        const float rescale = __builtin_amdgcn_exp2f(mx - cm);
        l_all *= rescale;
        o *= rescale;
        const auto add = [&](int i) {
          const float f = __builtin_amdgcn_exp2f(pml[i].x - cm);
          l_all += pml[i].y * f;
          o += pa[i] * f;
        };
        if (s0 + 8 <= a.splits) {
#pragma unroll
          for (int i = 0; i < 8; ++i) add(i);
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (s0 + i < a.splits) add(i);  // not a factor of zero: the values may be infinite
        }
        mx = cm;
      }
      store_out(a.out, a.out_is_fp16, bh * kHeadDim + ch, o / l_all);
      if (ch == 0 && a.lse) a.lse[bh] = (mx + __builtin_amdgcn_logf(l_all)) * kLn2;
    }
  }
}

}  // namespace

// How finely the page lists are split.
namespace {
struct SplitPlan {
  int list_len, per_split, splits;
};
// With a page list: one work-group per compute unit, no more.  A second one on the same
// unit competes for its load path (about 25 KiB per us), repeats the selection and
// adds a partial result to merge: 6 sequences of 32 heads, 2048-token budget, selecting
// launch: 36.0 us with 1 split, 39.6 with 2, 42.5 with 4; 8 sequences 46.8 / 49.2 / 49.8;
// 40 heads of one sequence 13.4 us with 6 splits, 14.7 with 8; 16 sequences of 8 KV heads
// with 4 query heads each 29.2 us with 2 splits, 35.0 with 4.  Only when the items
// themselves leave a second round that is nearly empty are three splits of each better, as
// long as those make four rounds: 9 sequences of 32 heads 64.5 us with 1, 57.7 with 3 (10
// sequences: 65.7 and 60.3; 12: 69.4 and 72.5; 43 of 8 heads 78.4 and 79.9; at 512 tokens 1 is better
// everywhere).  More than 300 up to 2048 tokens only in rows of twice the list: in short rows the
// shorter sequences leave splits empty (10 sequences of 151 to 1317 tokens, 32 heads, a list of 1040:
// 26.5 us with 1, 31.0 with 3; but 7 of 1017 to 1887, 40 heads, 52.1 and 47.6).
// All splits of an item run on one die (see decode_split_kernel), so that is counted per die: its
// 32 units for the items that fall to it.  15 heads of one KV head, a list of 6024 tokens: 12.6 us
// with 16 splits, 15.3 with 17; attention over whole rows of 20000 tokens, 10 heads, 21.5 us with
// 16, 26.8 with 24; 5 sequences of 5000 to 9000, 10 heads, 32.5 with 4, 45.5 with 5.
// Short lists: a split merges in about 2.3 us, so 256 tokens stay whole (7.5 us against
// 7.9 us), 512 and 1024 tokens are worth 8 splits (8.4 us against 10.1 us), more tokens
// 16 (8 heads, 4096 tokens: 10.4 us, 12.1 with 8 splits, 11.0 with 32), very long lists a
// split per 256 tokens.
// per_unit: work-groups per compute unit.
long list_splits(long items, long tokens, int per_unit = 1) {
  if (items > kComputeUnits) return 3 * items <= 4 * kComputeUnits && tokens >= 1024 ? 3 : 1;
  if (tokens <= 256) return 1;
  const long useful = std::max(8l, std::min(tokens / 128, std::max(16l, tokens / 256)));
  return std::max(1l, std::min(per_unit * kComputeUnits / kDies / ((items + kDies - 1) / kDies), useful));
}
// One head's pages of 8 tokens leave a wave half the bytes in flight.  Few heads: splits of half the
// tokens, up to the 16 that long lists have (2 sequences, 8 heads, 1464 tokens: 7.2 us with 16 splits,
// 7.6 with 11; 32 heads, 256 tokens 5.6 with 8, 6.6 with 1; but 160 tokens 5.4 and 5.2, and of 616 tokens
// nine, merged in two rounds, cost more than eight).  More heads over a given list: two
// work-groups per unit (11 sequences of 8 heads, 736 tokens 8.8 us with 5 splits, 10.4 with 2; 3 of 32,
// 6680 tokens 51.9 and 56.7; 6 of 32, 2048 tokens 35.9 with 2, 34.9 with 1); selecting launches are as
// fast either way.
// 129 to 170 heads, lists of 3072 tokens or more: three splits, as fast as one where all sequences
// are longer than the list, faster where they are not (a step of 4 sequences of 2621 to 3960 tokens,
// 40 heads, all attended: 49.2 us, 52.7; groups, which have more to merge, lose: 20 of 32 query / 8 KV
// heads 56.7 and 52.9).
// items: work-groups per split.
long most_splits(const quest_cache& c, long items, int list_len, bool select) {
  long tokens = (long)list_len * c.page_size;
  int per_unit = 1;
  if (items > 300 && tokens < 2048 && c.max_pages_per_seq < 2 * (long)list_len) return 1;
  if (group_size(c) == 1) {
    const bool small = c.page_size == 8;
    if (items > 128 && items <= 170 && tokens >= 3072) per_unit = 2;
    if (small && !select && items > 64 && items <= 170 && tokens >= 512) per_unit = 2;
    if (small && items <= 64 && (tokens >= 1024 || (tokens > 192 && tokens <= 256)))
      tokens = std::max(tokens, std::min(2 * tokens, 4096l));
  }
  return std::min(list_splits(items, tokens, per_unit), std::min<long>(list_len, kMaxTeamSize));
}
SplitPlan split_list(int list_len, long splits) {
  SplitPlan p;
  p.list_len = list_len;
  p.per_split = (int)((p.list_len + splits - 1) / splits);
  p.splits = (p.list_len + p.per_split - 1) / p.per_split;  // no empty split
  return p;
}
long group_items(const quest_cache& c) { return (long)c.batch * kv_heads(c) * attention_subs(c); }
SplitPlan plan_splits(const quest_cache& c, int k_pages, bool select) {
  const int list_len = std::min(k_pages, c.max_pages_per_seq);
  return split_list(list_len, most_splits(c, group_items(c), list_len, select));
}
// Query heads of a group in work-groups of their own, on the vector unit: their pages then come
// from memory once and from the caches for the others, and a launch takes about 1 us less to
// get going and to finish (no keys through LDS, one head's outputs to merge), as long as that
// is little to load.  us a launch over a given list, apart / together, query heads / KV heads: 32/8 of
// 512 tokens 6.3 / 7.6, 1024 7.4 / 8.3, 2048 10.6 / 9.7; 16/8 of 2048 8.0 / 8.1, 4096 10.3 / 9.5; 4
// sequences of 32/8, 256 6.9 / 7.1, 512 10.6 / 8.4; 8/1 of 4096 9.5 / 14.0; 32/4 of 2048 11.3 / 13.0.
// Where the launch selects its list, the selection is repeated for more work-groups: 16/8 of 1024
// tokens 11.3 / 11.8 (a step), 32/8 of 512 11.2 / 11.8, 1024 12.5 / 12.4, 64/8 of 256 12.4 / 11.9, 32/4 of
// 1024 13.5 / 13.9, 8/1 of 4096 15.9 / 17.4; groups of two gain little from each other: 16/8 of 1952
// (every page) 11.1 / 11.6.
bool heads_apart(const quest_cache& c, int k_pages, bool select) {
  if (group_size(c) == 1) return false;
  const int64_t tokens = (int64_t)std::min(k_pages, c.max_pages_per_seq) * c.page_size;
  const int64_t heads = (int64_t)c.batch * c.num_heads, kv = (int64_t)c.batch * kv_heads(c);
  const bool few = group_items(c) <= 4;
  const int group = group_size(c);
  if (select) return (heads - kv) * tokens <= (few ? 32 : group == 2 ? 16 : group <= 4 ? 14 : 12) * 1024;
  return heads * tokens <= (few ? 72 : group >= 8 ? 52 : 44) * 1024;
}
// No more splits than plan_splits has: less work-groups are left for each item.
SplitPlan plan_apart(const quest_cache& c, int k_pages) {
  const int list_len = std::min(k_pages, c.max_pages_per_seq);
  return split_list(list_len, most_splits(c, (long)c.batch * c.num_heads, list_len, true));
}
// Every page of a row: the same rule, with two work-groups per compute unit for 64 to 170 heads,
// which even out ragged sequences (7 sequences of 500 to 2500 tokens, 20 heads, 26.1 us with 3
// splits, 29.2 with 1; 4 of 751 to 2221, 40 heads, 26.0 and 28.7; but 5 of 1000, 32 heads, 17.3 and
// 15.9), and for all above 48 of 8-token pages, which leave a wave half the bytes in flight (3 of
// 400 to 1200, 32 heads: 12.3 us with 5 splits, 14.4 with 2; 4 of 3000 to 6000 50.1 with 4, 53.0 with
// 2).  16 or 24 splits past 16, which are merged eight at a time (32 query / 8 KV heads of 32000
// tokens: 26.7 us with 24, 27.5 with 32; 8 heads of 8000 10.8 and 11.0).  Of few tokens one: 13
// sequences of 64 / 8 heads, 300 tokens, 9.4 and 11.3 with 2; 10 of 151 to 1317 tokens, 32 heads, 24.4,
// 25.6 with 3.
SplitPlan plan_rows(const quest_cache& c) {
  const long items = group_items(c);
  const long tokens = (long)c.max_pages_per_seq * c.page_size;
  long splits;
  if (group_size(c) > 1) {
    splits = items > 64 && tokens <= 512 ? 1 : list_splits(items, tokens);
  } else {
    const bool two = c.page_size == 8 ? items > 48
                                      : items >= (tokens <= 3072 ? 64 : 65) && items <= 170 && tokens >= 1024;
    splits = items > kComputeUnits && tokens < 2048 ? 1 : list_splits(items, tokens, two ? 2 : 1);
  }
  if (splits > 16) splits = splits < 24 ? 16 : 24;
  return split_list(c.max_pages_per_seq, std::min<long>(splits, c.max_pages_per_seq));
}
// One arrival counter per (sequence, head), each in a 256-byte slot of its own.
size_t counter_bytes(const quest_cache& c) {
  return (size_t)c.batch * c.num_heads * kTeamWordStride * sizeof(uint64_t);
}
}  // namespace

size_t decode_counter_bytes(const quest_cache& c) { return counter_bytes(c); }

namespace {
size_t split_bytes(const quest_cache& c, size_t splits) {
  if (splits == 1) return 0;
  return counter_bytes(c) + (size_t)c.batch * c.num_heads * splits * (kHeadDim + 2) * sizeof(float);
}
}  // namespace

size_t decode_workspace_bytes(const quest_cache& c, int k_pages) {
  return split_bytes(c, plan_splits(c, k_pages, true).splits);
}

// One split needs none, but every dense call of a cache shape asks for the counters.
size_t row_workspace_bytes(const quest_cache& c) {
  return std::max(split_bytes(c, plan_rows(c).splits), counter_bytes(c));
}

// most_splits of the longest list there is: no shorter one has more.
size_t attention_workspace_bytes(const quest_cache& c) {
  return std::max(dense_workspace_bytes(c), split_bytes(c, most_splits(c, group_items(c), c.max_pages_per_seq, false)));
}

namespace {
// scores != nullptr: select inside the launch (topk_out, k_eff receive the list and K_b), or
// among the candidates if there are some; the caller has checked that it can.
int launch_decode(const quest_cache& c, const void* q, const int32_t* topk_idx, const float* scores,
                  const Candidates* cand, int32_t* topk_out, int32_t* k_eff, int k_pages, float sm_scale,
                  void* out, int out_is_fp16, float* lse, void* workspace, size_t workspace_bytes,
                  hipStream_t s, const EstimateArgs* est = nullptr) {
  const bool select = scores != nullptr || cand != nullptr;
  const bool rows = !select && topk_idx == nullptr;  // every page of a row
  const bool apart = !rows && heads_apart(c, k_pages, select);
  SplitPlan p = rows ? plan_rows(c) : apart ? plan_apart(c, k_pages) : plan_splits(c, k_pages, select);
  StepArgs a;
  if (est) a.est = *est;
  fill_attn_args(a, c, q, sm_scale, out, out_is_fp16, lse);
  a.topk_idx = topk_idx;
  a.scores = cand ? cand->score : scores;
  a.cand_page = cand ? cand->page : nullptr;
  a.row_len = cand ? cand->row_len : c.max_pages_per_seq;
  a.chunk_pages = cand ? cand->chunk_pages : 0;
  a.topk_out = topk_out;
  a.k_eff = k_eff;
  a.policy = c.flags;
  a.k_pages = k_pages;
  if (workspace_bytes < split_bytes(c, p.splits) && !rows && !apart) p = plan_splits(c, k_pages, true);
  if (workspace_bytes < split_bytes(c, p.splits)) p = split_list(p.list_len, 1);
  a.splits = p.splits;
  a.list_len = p.list_len;
  a.per_split = p.per_split;
  const size_t n_part = (size_t)c.batch * c.num_heads * a.splits;
  a.counters = (uint64_t*)workspace;
  a.part_acc = workspace ? (float*)((char*)workspace + counter_bytes(c)) : nullptr;
  a.part_ml = a.part_acc ? a.part_acc + n_part * kHeadDim : nullptr;
  const bool group = a.group > 1 && !apart;
  if (apart) a.subs = a.group;
  const long items = (long)c.batch * a.kv_heads * a.subs, items8 = (items + 7) / 8;
  const long heads8 = ((long)c.batch * c.num_heads + 7) / 8;
  // item * ceil(2^32 / d) / 2^32 is item / d as long as item * d < 2^32
  const uint64_t per_seq = (uint64_t)a.kv_heads * a.subs;
  a.seq_inverse = per_seq > 1 && 8 * (uint64_t)items8 * per_seq < (1ull << 32) ? (uint32_t)(((1ull << 32) + per_seq - 1) / per_seq) : 0;
  if (heads8 > 65535 && !rows) {  // items8 <= heads8 (launch_dense_decode has a limit of its own)
    set_error("quest_sparse_decode: batch * heads = %ld exceeds the launch limit", heads8 * 8);
    return QUEST_ERR_SHAPE;
  }
  const dim3 grid((unsigned)(8 * a.splits), (unsigned)items8);
#define QUEST_LAUNCH(L, G, W, I, C) \
  hipLaunchKernelGGL((decode_split_kernel<L, G, W, I, C>), grid, dim3((W) * kWave), 0, s, a)
#define QUEST_LAUNCH_FOR_PAGE(G, W, I, C)           \
  do {                                              \
    if (c.page_size == 8) QUEST_LAUNCH(2, G, W, I, C); \
    else QUEST_LAUNCH(4, G, W, I, C);               \
  } while (0)
  if (est) {
#define QUEST_STEP(L, G, W, I, P, Q) \
  hipLaunchKernelGGL((decode_split_kernel<L, G, W, I, false, P, Q>), grid, dim3((W) * kWave), 0, s, a)
#define QUEST_STEP_CASE(G, W, I, P, Q)                                                     \
  if (group == G && (Q) == queries && a.max_pages <= (W) * (P) * ((Q) ? 16 : 8)) {         \
    if (c.page_size == 8) QUEST_STEP(2, G, W, I, P, Q); else QUEST_STEP(4, G, W, I, P, Q); \
    return check_launch("quest_decode_step");                                              \
  }
    const int queries = a.group == 1 ? 1 : estimate_on_matrix_cores(c) ? 0 : 4;
    // Waves, scores per thread, passes (estimate_row).  Four waves up to 256 pages; more pages of more rows are streamed faster by
    // eight (192 rows of 313 pages, 64 tokens each, 22.9 us a step, 23.6 with four), but those take a compute unit each
    // (384 rows of 434 pages 47.3 us with four, 52.6 with eight).
    QUEST_STEP_CASE(false, 4, 1, 2, 1)
    QUEST_STEP_CASE(false, 4, 1, 4, 1)
    if (items <= kComputeUnits) {
      QUEST_STEP_CASE(false, 8, 1, 4, 1)
      QUEST_STEP_CASE(false, 8, 2, 8, 1)
    } else {
      QUEST_STEP_CASE(false, 4, 2, 8, 1)
    }
    QUEST_STEP_CASE(true, 8, 1, 1, 4)
    QUEST_STEP_CASE(false, 8, 1, 1, 4)
    QUEST_STEP_CASE(true, 8, 1, 1, 0)
    QUEST_STEP_CASE(false, 8, 1, 1, 0)
    QUEST_STEP_CASE(true, 8, 1, 2, 0)
#undef QUEST_STEP_CASE
#undef QUEST_STEP
    set_error("quest_decode_step: internal: no one-launch step for rows of %d pages", a.max_pages);
    return QUEST_ERR_SHAPE;
  }
  if (select) {
#define QUEST_SELECT_CASE(G, C, W, I)                                                      \
  if (group == G && (cand != nullptr) == C && a.row_len <= (W) * kWave * (I)) {            \
    QUEST_LAUNCH_FOR_PAGE(G, W, I, C);                                                     \
    return check_launch("quest_select_decode");                                            \
  }
#define QUEST_LONG_CASE(G, I)                                                                             \
  if (group == G && cand == nullptr && eight_select && a.row_len <= 8 * kWave * (I)) {                                  \
    if (c.page_size == 8)                                                                                 \
      hipLaunchKernelGGL((decode_split_kernel<2, G, 4, I, false, 0, 0, 8>), grid, dim3(8 * kWave), 0, s, a); \
    else                                                                                                  \
      hipLaunchKernelGGL((decode_split_kernel<4, G, 4, I, false, 0, 0, 8>), grid, dim3(8 * kWave), 0, s, a); \
    return check_launch("quest_select_decode");                                                           \
  }
    // Waves and scores per thread.  Four waves select short rows as fast as eight and have less to
    // merge (32 heads, 438 pages: 12.3 us a step, 12.9 with eight); a group's matrix products are better off
    // on eight (4 sequences of up to 2050 pages, 32 query / 8 KV heads: 21.4 us, 22.6 with four), and so
    // is the selection in the middle (32 heads, 2053 pages: 19.8 and 20.1 us).  Rows of more than 4096 pages: four waves
    // attend, so that the sums are those of attention over a given list, which the same call makes
    // with QUEST_FLAG_SEPARATE_LAUNCHES, and up to a number of work-groups eight select (half the scores per thread each, two
    // waves to hide each other's waits on a SIMD: 8193 pages of 32 heads, 256 in the list, 19.8 us a launch with four, 18.8
    // with eight, 19.3 with sixteen; 64 in the list 12.2, 11.0 and 11.0; 32 query / 8 KV heads of 4600 pages 9.7, 9.1).  More
    // give a compute unit several work-groups, which hide each other's waits themselves as far as they fit on it.  A
    // group's: a list of 16 pages of 8 tokens, 256 of them 8.1 us with four, 7.5 with eight, but 264 10.7 and 14.7, 384
    // 11.7 and 15.9; 64 pages of 16 tokens, 264 35.1 and 45.3, 512 48.3 and 53.8.  One query head's: 16 pages
    // of 8 tokens, 512 11.8 and 11.2, but 640 15.1 and 17.6, 1024 18.5 and 21.5 (other row lengths 0 to 3 % less);
    // 64 pages of 16 tokens, 320 items of three splits 32.5 and 35.1; 16 ragged sequences of 32 heads and up to 4099 pages
    // (512), 128 pages in the list, 88.6 and 88.2.
#define QUEST_SELECT_CASES(C)     \
  QUEST_SELECT_CASE(false, C, 4, 2) \
  QUEST_SELECT_CASE(false, C, 4, 4) \
  QUEST_SELECT_CASE(false, C, 8, 3) \
  QUEST_SELECT_CASE(false, C, 8, 5) \
  QUEST_SELECT_CASE(false, C, 8, 8) \
  QUEST_SELECT_CASE(true, C, 8, 1)  \
  QUEST_SELECT_CASE(true, C, 8, 2)  \
  QUEST_SELECT_CASE(true, C, 8, 3)  \
  QUEST_SELECT_CASE(true, C, 8, 5)  \
  QUEST_SELECT_CASE(true, C, 8, 8)
    QUEST_SELECT_CASES(false)
    QUEST_SELECT_CASES(true)
    const bool eight_select = items * a.splits <= (group ? kComputeUnits : 2 * kComputeUnits);
    QUEST_LONG_CASE(false, 10)
    QUEST_LONG_CASE(false, 14)
    QUEST_LONG_CASE(false, 17)
    QUEST_LONG_CASE(true, 10)
    QUEST_SELECT_CASE(false, false, 4, 20)
    QUEST_SELECT_CASE(false, false, 4, 27)
    QUEST_SELECT_CASE(false, false, 4, 34)
    QUEST_SELECT_CASE(true, false, 4, 20)
#undef QUEST_LONG_CASE
#undef QUEST_SELECT_CASES
#undef QUEST_SELECT_CASE
    set_error("quest_select_decode: internal: no selecting kernel for rows of %d scores", a.row_len);
    return QUEST_ERR_SHAPE;
  }
  // Whole rows of a group, one work-group per compute unit: eight waves (32 query / 8 KV heads of
  // 8000 tokens 13.2 us, 15.1 with four; several per unit: 128 sequences of 64 tokens 18.6 and 12.9).
  if (rows && group && items <= kComputeUnits)
    QUEST_LAUNCH_FOR_PAGE(true, 8, 0, false);
  else if (group)
    QUEST_LAUNCH_FOR_PAGE(true, kDecWaves, 0, false);
  else
    QUEST_LAUNCH_FOR_PAGE(false, kDecWaves, 0, false);
#undef QUEST_LAUNCH_FOR_PAGE
#undef QUEST_LAUNCH
  return check_launch("quest_sparse_decode");
}
}  // namespace

int launch_sparse_decode(const quest_cache& c, const void* q, const int32_t* topk_idx, int k_pages,
                         float sm_scale, void* out, int out_is_fp16, float* lse, void* workspace,
                         size_t workspace_bytes, hipStream_t s) {
  return launch_decode(c, q, topk_idx, nullptr, nullptr, nullptr, nullptr, k_pages, sm_scale, out, out_is_fp16,
                       lse, workspace, workspace_bytes, s);
}

int launch_row_decode(const quest_cache& c, const void* q, float sm_scale, void* out, int out_is_fp16,
                      float* lse, void* workspace, size_t workspace_bytes, hipStream_t s) {
  return launch_decode(c, q, nullptr, nullptr, nullptr, nullptr, nullptr, 0, sm_scale, out, out_is_fp16, lse,
                       workspace, workspace_bytes, s);
}

namespace {
// Rows short enough for a launch that selects from the whole row.
bool selected_whole(const quest_cache& c) {
  return c.max_pages_per_seq <= (group_size(c) == 1 ? kMostSelected : kMostSelectedOfGroup);
}
}  // namespace

// Selection and attention in one launch: while a row of scores fits the in-register selection
// and the list fits in LDS.  Every split of a head repeats the selection, which costs less than the
// launches it saves.  The lines lie where the tilings end, us a call this way / with candidates picked by a launch of
// their own, rows of 8704 pages: 32 heads, lists of 64 pages 11.8 / 12.2, 256 18.1 / 19.4, 1024 47.5 / 50.9; 16
// sequences of them 50.0 / 59.7 and 169 / 180; with 2611 pages of the row in use 10.1 / 12.3 and 17.5 / 20.1, with
// 435 and 256 in the list 16.7 / 17.6; 8 heads, 64 pages 10.2 / 10.9.  Rows of 5120 pages of 32 query / 8 KV heads, lists
// of 64: 10.1 / 12.3, 3 sequences 10.9 / 13.4, 32 26.9 / 30.5, 40 40.2 / 50.5.  (Tilings for longer rows would gain as
// well: 2 to 18 % at 8720 to 10240 pages, groups 2 to 20 % at 5200 to 8210.)
bool select_decode_supported(const quest_cache& c, int k_pages) {
  return !(c.flags & QUEST_FLAG_SEPARATE_LAUNCHES) && k_pages <= kSelListCap && selected_whole(c);
}

namespace {
// Longer rows: a launch picks candidates from the chunks of the rows, and the attention launch
// selects among those, as long as they are as few as the scores of a short row: a step of
// 32 heads 49.6 us instead of 55.6 us at 12500 pages (Top-K of whole rows and attention over
// its list), 106.3 instead of 108.2 us at 32769 (Top-K in two stages).  Chunks of 4096 pages where
// 2048 leave too many candidates.
constexpr int kMostCandidatesOfRow = 4096;  // that a launch selects among
int chunk_to_select_from(const quest_cache& c, int k_pages, size_t room) {
  if ((c.flags & QUEST_FLAG_SEPARATE_LAUNCHES) || selected_whole(c) || k_pages > kSelListCap) return 0;
  for (const int chunk : {kSmallChunk, kLargeChunk})
    if (candidates_per_row(c, k_pages, chunk) <= kMostCandidatesOfRow && candidate_bytes(c, k_pages, chunk) > 0 &&
        candidate_bytes(c, k_pages, chunk) <= room)
      return chunk;
  return 0;
}
}  // namespace

// The most candidates that a row can have (candidate_bytes): at most half of its pages.
size_t selection_workspace_bytes(const quest_cache& c) {
  const bool select = !selected_whole(c) && !(c.flags & QUEST_FLAG_SEPARATE_LAUNCHES);
  const size_t most = c.max_pages_per_seq >= kChunkedFromPages ? kMaxCandidates : select ? kMostCandidatesOfRow : 0;
  return (size_t)c.batch * kv_heads(c) * std::min<size_t>(most, c.max_pages_per_seq / 2) * (sizeof(float) + sizeof(int32_t));
}

// The whole step as one launch (decode_split_kernel with kEstPasses): the estimate's launch, the gap between
// two launches and the trip of the scores through memory go, about 3.4 us of 11 to 12. Against that every
// work-group of a row scores all of it, which its compute unit's path to L2 (64 bytes a clock) and its vector unit
// have to carry, and a row that comes from memory reaches one unit at 25 to 30 KiB per us.  The lines lie where 5700
// calls of random shapes (1 to 64 sequences, ragged or in wide tables, pages of 8 to 64 tokens, lists of one page to all)
// stop being faster on either side; replayed, us a step, two launches / one:
//   up to 8 rows, 256 pages: one head, 61 pages 8.0 / 6.8, 124 8.5 / 7.4, 252 9.3 / 9.2, but 257 8.7 / 9.7, 314 9.2 / 9.6;
//   9 to 112 rows, 192 pages: 32 heads of 61 9.7 / 8.1, of 124 11.0 / 9.5; but 32 of 249, all attended, 12.0 / 13.0, of 257
//   17.0 / 19.0; 38 of 288 8.9 / 9.6; with more than half of the pages in the list 128: 64 rows of 161, all
//   attended, 13.6 / 14.4;
//   113 to 160 rows, 512 pages: 144 of 434 16.5 / 14.3, 128 of 507 18.2 / 17.5; but 120 of 740 16.6 / 18.3, 160
//   of 881 19.5 / 20.7; more rows up to 256, 1024 pages: 6 sequences of 32 heads, 434 pages 27.8 / 26.6, 996
//   36.5 / 34.3; but 5 to 8 of 1500 to 2000 pages, 2 to 10 % slower;
//   257 to 384 rows, which leave the second round of units half empty, 256 pages: 280 of 315 15.1 / 16.9, 336 of
//   305 18.0 / 19.8; up to 512 rows, 512 pages: 12 sequences of 32 heads, 434 49.5 / 47.3;
//   three splits of a row, or more rows, 256 pages: 640 rows of 500 up to 8 % slower; thousands of rows of a few pages
//   3 %, of 120 pages 4 % faster.
// Groups of query heads have each page scored for all of them, one work-group a unit: 64 pages (10 sequences of 64 / 8
// heads, 56 pages 13.4 / 12.5, one of 120 10.5 / 10.7), groups of up to four with half of the pages or less in the list 128
// (31 sequences of 32 / 8 heads, 109 pages 12.5 / 10.9, 10 of 64 / 16, 95 pages 17.1 / 15.7; all attended, 10 of 32 / 8, 71
// pages 14.6 / 15.3).  Query heads in work-groups of their own each score the row for the whole group: 64 pages (16 / 8 heads
// of 125 pages 9.3 / 9.6, 15 / 5 of 103 9.2 / 9.7), and it is those work-groups that have to fit (18
// sequences of 40 / 5 heads, one page, 720 of them: 8.0 / 11.1).  With 16 and more heads in a group 2 to 13 % slower.
bool step_in_one_launch(const quest_cache& c, int k_pages) {
  if (!select_decode_supported(c, k_pages) || c.num_phys_pages >= (1l << 22)) return false;  // (32-bit offsets)
  const long pages = c.max_pages_per_seq;
  const bool few_chosen = 2l * k_pages <= pages;
  if (const int group = group_size(c); group > 1) {
    const bool apart = heads_apart(c, k_pages, true);
    const long items = apart ? (long)c.batch * c.num_heads : group_items(c);
    return group <= 8 && items <= kComputeUnits && pages <= (group <= 4 && !apart && few_chosen ? 128 : 64);
  }
  const long items = group_items(c);
  if (items <= 112) return pages <= (items <= 8 ? 256 : few_chosen ? 192 : 128);
  if (items > 2 * kComputeUnits || plan_splits(c, k_pages, true).splits > 2)
    return pages <= 256 && (items <= 4 * kComputeUnits || pages >= 64);
  if (items > kComputeUnits) return pages <= (2 * items > 3 * kComputeUnits ? 512 : 256);
  return pages <= (items > 160 ? 1024 : 512);
}

// In two launches every wave has read the new token when the second one writes its results, and a
// work-group of the second reads no query vectors but those of the heads whose outputs it writes: a caller may have its
// results written over k_new and v_new, and fp16 outputs over q, head by head.  In one launch a
// work-group may end before another one of its launch has begun, so results must not lie on the new token; and where a
// group's query heads have a work-group each, every one of them scores with all the queries of the group.
bool step_reads_before_it_writes(const quest_cache& c, const void* k_new, const void* v_new, const void* q, int k_pages,
                                 const int32_t* topk_idx, const int32_t* k_eff, const void* out, int out_is_fp16,
                                 const float* lse, const Workspace& w) {
  const size_t heads = (size_t)c.batch * c.num_heads, kv = (size_t)c.batch * kv_heads(c);
  const size_t q_bytes = heads * kRowBytes, new_bytes = kv * kRowBytes, out_bytes = heads * kHeadDim * (out_is_fp16 ? 2 : 4);
  const auto meet = [](const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return a != nullptr && b != nullptr && x < y + nb && y < x + na;
  };
  const auto on = [&](const void* result, size_t bytes) {
    return meet(result, bytes, k_new, new_bytes) || meet(result, bytes, v_new, new_bytes);
  };
  const bool in_place = out == q && out_is_fp16 && !heads_apart(c, k_pages, true);
  if (meet(out, out_bytes, q, q_bytes) && !in_place) return false;
  return !on(out, out_bytes) && !on(lse, heads * sizeof(float)) && !on(topk_idx, kv * k_pages * sizeof(int32_t)) &&
         !on(k_eff, c.batch * sizeof(int32_t)) && !on(w.attention, w.attention_bytes);
}

int launch_step(const quest_cache& c, const void* k_new, const void* v_new, int k_pool_write, const void* q, int k_pages,
                float sm_scale, float* scores, int32_t* topk_idx, int32_t* k_eff, void* out, int out_is_fp16, float* lse,
                const Workspace& w, hipStream_t s) {
  const EstimateArgs est = estimate_args(c, k_new, v_new, k_pool_write, q, scores);
  return launch_decode(c, q, nullptr, scores, nullptr, topk_idx, k_eff, k_pages, sm_scale, out, out_is_fp16, lse,
                       w.attention, w.attention_bytes, s, &est);
}

int launch_select_decode(const quest_cache& c, const void* q, const float* scores, int k_pages,
                         float sm_scale, int32_t* topk_idx, int32_t* k_eff, void* out,
                         int out_is_fp16, float* lse, const Workspace& w, hipStream_t s) {
  if (select_decode_supported(c, k_pages))
    return launch_decode(c, q, nullptr, scores, nullptr, topk_idx, k_eff, k_pages, sm_scale, out,
                         out_is_fp16, lse, w.attention, w.attention_bytes, s);
  int r;
  if (const int chunk = chunk_to_select_from(c, k_pages, w.selection_bytes)) {
    Candidates cand;
    r = launch_topk_chunks(c, scores, k_pages, chunk, w.selection, &cand, s);
    if (r != QUEST_OK) return r;
    return launch_decode(c, q, nullptr, nullptr, &cand, topk_idx, k_eff, k_pages, sm_scale, out,
                         out_is_fp16, lse, w.attention, w.attention_bytes, s);
  }
  const size_t two_stages = topk_scratch_bytes(c, k_pages);
  r = two_stages > 0 && two_stages <= w.selection_bytes
          ? launch_topk_chunked(c, scores, k_pages, topk_idx, k_eff, w.selection, s)
          : launch_topk(c, scores, k_pages, topk_idx, k_eff, s);
  if (r != QUEST_OK) return r;
  return launch_sparse_decode(c, q, topk_idx, k_pages, sm_scale, out, out_is_fp16, lse, w.attention,
                              w.attention_bytes, s);
}

}  // namespace quest
