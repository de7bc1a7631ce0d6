// Decode attention over every page of every sequence: the dense baseline the paper compares
// against (Section 3.1 of arXiv 2406.10774), and what a model runs in the layers it does
// not sparsify.
//
// Rows of few tokens and little work: splits of each row (quest_decode.hip; equal_shares below).
// Else the pages of all sequences and heads are one line of work, cut into equal shares, one
// per work-group and at most one work-group per compute unit: sequences of any lengths keep
// every unit busy to the end.  (Splits of a fixed number of pages per head leave the shorter
// sequences' units idle: 8 sequences of 1000 to 20000 tokens, 32 heads, 245 us against 208; 5 of
// 300 to 24000 190 against 157.)  Items along the line are (sequence, block of heads); a share that covers an
// item in part leaves a partial result, and the last of the item's shares to finish merges
// them (quest_team.h).
//
// Bound by memory: 32 heads of 32k tokens, 537 MB, take 83 us (6.5 TB/s), against 94 us in
// 1024 work-groups of a head and 64 pages each.  One wave per SIMD and two units in flight
// per wave is all the memory system wants: plain reads of the same pages took 81 us this
// way, 84 us with twice and 85 to 96 us with four times the waves.  Where there are enough
// heads a work-group's four waves take four adjacent heads, each all pages of the share: a
// page of theirs is 16 KiB in a row (plain reads 81 us, against 86 to 92 us for four waves
// on pages of one head), and nothing has to be merged between the waves.
#include <algorithm>
#include <type_traits>

#include "quest_common.h"
#include "quest_decode_core.h"
#include "quest_team.h"
#include "quest_topk_core.h"

namespace quest {

namespace {

constexpr int waves_of(bool group) { return group ? 8 : 4; }
// Work-groups at most, of the 256 compute units: the memory system moves more with fewer
// streams as long as they can carry it (one sequence of 64k tokens, 32 heads: 162 us with 192
// work-groups, 168 with 224, 167 with 256; 8 of 1000 to 20000 tokens 208, 210, 214; one of 32k 85.6,
// 88.5, 88.5).  Groups have more to do per page: 32 sequences of 500 to 8000 tokens, 32 query / 8 KV
// heads, 108, 99 and 101; 8 of 1000 to 30000, 64 / 8 heads, 101, 94 and 95.
// Pages of 8 tokens leave a wave half the bytes in flight: 2 sequences of 30000 tokens, 32 heads,
// 162, 152 and 150; 6 of 1000 to 12000 113, 105 and 104.
int most_shares(const quest_cache& c) { return group_size(c) > 1 ? 224 : c.page_size == 8 ? 256 : 192; }

struct DenseArgs : AttnArgs {
  int shares;  // work-groups; partial results of share w are slots 2w and 2w + 1
};

// Query heads of one item and of one slot.
template <bool kGroup, int kBlock>
constexpr int slot_heads() { return kGroup ? kGroupHeads : kBlock; }

// kBlock: heads per item.  4 (not with kGroup): wave i has head i of the block and every
// page; 1: the waves share one head (or group of heads), unit by unit.
template <int kLoads, bool kGroup, int kBlock, int kWaves>
__global__ __launch_bounds__(kWaves* kWave) void dense_kernel(const DenseArgs a) {
  using Head = HeadState<kLoads, kGroup>;
  constexpr int kThreads = kWaves * kWave;
  constexpr int kSlots = Head::kSlots, kStride = Head::kStride;
  constexpr int kHeads = slot_heads<kGroup, kBlock>();
  __shared__ __align__(16) float sm_acc[kWaves * kSlots * kStride];
  __shared__ float sm_m[kWaves * kSlots], sm_l[kWaves * kSlots];
  __shared__ uint32_t sm_before;
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lane = lane_id();
  const int blocks = a.kv_heads * a.subs / kBlock;  // items per sequence
  // (a length past the end of the row, which a caller must not pass, reads no further than the row)
  auto pages_of = [&](int len) {
    return min((max(len, 0) + (1 << a.page_shift) - 1) >> a.page_shift, a.max_pages);
  };

  // ---- this work-group's share [off, end) of the line, and the sequence it begins in.  In front
  // of an item's pages the line is longer by what ending one item and beginning the next costs a
  // work-group, in pages: about 128 KiB of loads (partial results, the handing over, the first loads of
  // the next item).  Without it the work-groups with a border in their share finished last: 4
  // sequences of 5000 to 33000 tokens, 32 query / 8 KV heads, 55.6 us instead of 58.7 (57.6 with 64 KiB, 56.4
  // with 256); 32 of 500 to 8000 93.9 instead of 104.6; 5 of 300 to 24000, 32 heads, 152.0 instead of 158.3.
  // One sequence whose items are whole numbers of shares has no border inside a share.
  const int lead = a.batch == 1 && a.shares % blocks == 0 ? 0 : max(1, (128 * 1024 / (2 * kRowBytes * kBlock)) >> a.page_shift);
  auto length_of = [&](int pages) { return pages > 0 ? pages + lead : 0; };
  const int64_t w = blockIdx.x;
  int64_t total = 0;
  for (int b0 = 0; b0 < a.batch; b0 += kWave) {
    const int p = b0 + lane < a.batch ? length_of(pages_of(a.seq_lens[b0 + lane])) : 0;
    total += __builtin_amdgcn_readlane(wave_incl_scan(p), kWave - 1);
  }
  total *= blocks;
  // none is empty, but one may have no page: all of it in front of an item's
  const int64_t shares = total < a.shares ? total : a.shares;
  if (w >= shares) return;
  const int64_t begin = w * total / shares, end = (w + 1) * total / shares;
  int64_t off = begin;
  int64_t base = 0;  // where sequence b begins
  int b = 0;
  for (int b0 = 0; b0 < a.batch; b0 += kWave) {
    const int p = b0 + lane < a.batch ? length_of(pages_of(a.seq_lens[b0 + lane])) : 0;
    const int upto = wave_incl_scan(p);
    const int64_t after = base + (int64_t)__builtin_amdgcn_readlane(upto, kWave - 1) * blocks;
    if (off < after) {
      const int k = __popcll(__ballot(b0 + lane < a.batch && base + (int64_t)upto * blocks <= off));
      b = b0 + k;
      base += k > 0 ? (int64_t)__builtin_amdgcn_readlane(upto, k > 0 ? k - 1 : 0) * blocks : 0;
      break;
    }
    base = after;
  }
  auto share_of = [&](int64_t at) { return (int)(((at + 1) * shares - 1) / total); };

  while (off < end) {
    // ---- one item, or the part of it that lies in the share
    const int seq_len = __builtin_amdgcn_readfirstlane(a.seq_lens[b]);
    const int pages = pages_of(seq_len);
    if (pages == 0) {
      ++b;
      continue;
    }
    const int block = (int)((off - base) / length_of(pages));
    const int64_t item_at = base + (int64_t)block * length_of(pages) + lead;  // its first page
    off = off < item_at ? item_at : off;
    if (off >= end) break;
    const int p0 = (int)(off - item_at);
    const int n_pages = (int)(pages - p0 < end - off ? pages - p0 : end - off);
    const int virt = block * kBlock + (kBlock > 1 ? wave : 0);
    const int hk = a.subs == 1 ? virt : virt / a.subs;
    const int sub = virt - hk * a.subs;
    const int h = hk * a.group + sub * kSlots;  // first query head of this wave
    const int n_heads = kGroup ? min(kSlots, a.group - sub * kSlots) : 1;
    const size_t bh = (size_t)b * a.num_heads + h;
    const int32_t* pt = a.page_table + (size_t)b * a.max_pages + p0;

    Head st;
    st.init(sm_acc + wave * kSlots * kStride, a.q + bh * kRowBytes, n_heads, lane);
    constexpr int kStep = kBlock > 1 ? 1 : kWaves;
    const int first = kBlock > 1 ? 0 : wave;
    const int entries = Head::kTwoPages ? (n_pages + 1) >> 1 : n_pages;
    const int units = ((entries << a.unit_shift) - first + kStep - 1) / kStep;
    attend<kLoads, kGroup>(st, a, hk, seq_len, units, a.q + bh * kRowBytes, n_heads,
                           sm_acc + wave * kSlots * kStride, sm_m + wave * kSlots, sm_l + wave * kSlots, lane,
                           [&](int i, int& lp, int& ph, int& un, int& lp2, int& ph2) {
      const int u = first + kStep * i;
      const int e = u >> a.unit_shift;
      un = u & ((1 << a.unit_shift) - 1);
      auto entry_at = [&](int pos, int& l, int& p) {
        if (pos < n_pages) l = p0 + pos, p = pt[pos];
      };
      if constexpr (Head::kTwoPages) {
        entry_at(2 * e, lp, ph);
        entry_at(2 * e + 1, lp2, ph2);
      } else {
        entry_at(e, lp, ph);
      }
    });
    __syncthreads();

    // ---- the part's result: to the output if it is the whole item, else to a slot
    const size_t bh0 = (size_t)b * a.num_heads + (kBlock > 1 ? block * kBlock : h);
    const int n_out = (kGroup ? n_heads : kBlock) * kHeadDim;
    const bool whole = n_pages == pages;
    const size_t slot = 2 * (size_t)w + (item_at >= begin ? 1 : 0);  // items begun before: slot 0
    // (64 outputs of one head per wave)
    for (int x0 = wave * kWave; x0 < n_out; x0 += kThreads) {
      const int g = x0 / kHeadDim, ch = (x0 & (kHeadDim - 1)) + lane;
      float m_tot, l_tot, acc;
      if constexpr (kBlock > 1) {
        m_tot = sm_m[g], l_tot = sm_l[g], acc = sm_acc[g * kStride + ch];
      } else {
        const int part = (lane & (kWaves - 1)) * kSlots + g;
        const Merged all = merge_parts(sm_m[part], sm_l[part], kWaves, lane);
        m_tot = all.m, l_tot = all.l, acc = 0.f;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) acc += sm_acc[(i * kSlots + g) * kStride + ch] * from_lane(all.weight, i);
      }
      if (whole) {
        store_out(a.out, a.out_is_fp16, (bh0 + g) * kHeadDim + ch, acc / l_tot);
        if (ch == 0 && a.lse) a.lse[bh0 + g] = (m_tot + __builtin_amdgcn_logf(l_tot)) * kLn2;
      } else {
        const size_t ps = slot * kHeads + g;
        dev_st(a.part_acc + ps * kHeadDim + ch, acc);
        if (ch == 0) {
          dev_st(a.part_ml + ps * 2 + 0, m_tot);
          dev_st(a.part_ml + ps * 2 + 1, l_tot);
        }
      }
    }
    if (!whole) {
      const int from = share_of(item_at);
      const int parts = share_of(item_at + pages - 1) - from + 1;
      uint32_t* arrivals = reinterpret_cast<uint32_t*>(
          a.counters + ((size_t)b * blocks + block) * kTeamWordStride);
      wait_stores();
      __syncthreads();
      if (t == 0) sm_before = team_arrive(arrivals, a.device_fences);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sm_before) == (uint32_t)parts - 1) {
        team_acquire(a.device_fences);
        if (t == 0) team_reset(arrivals);
        // A head's parts are dealt to as many waves as there are for it, two channels a lane, 16 parts
        // at a time in flight per wave, and the waves' sums added through LDS.  Fixed order: the
        // result does not depend on who was last.
        const int heads = n_out / kHeadDim;  // at most kWaves
        const int ways_log2 = (kWaves == 8 ? 3 : 2) - (heads <= 1 ? 0 : heads <= 2 ? 1 : heads <= 4 ? 2 : 3);
        const int g = wave >> ways_log2, way = wave & ((1 << ways_log2) - 1);
        const float* head_ml = a.part_ml + ((size_t)2 * from * kHeads + g) * 2;  // part k: 2 k kHeads further,
        const float* head_acc = a.part_acc + ((size_t)2 * from * kHeads + g) * kHeadDim;  // the first in slot 1
        const auto place = [&](int k) { return (uint32_t)((2 * k + (k == 0 ? 1 : 0)) * kHeads); };
        const int mine = g < heads ? (parts - way + (1 << ways_log2) - 1) >> ways_log2 : 0;
        float mx = kNegBig, l_all = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll 1
        for (int i0 = 0; i0 < mine; i0 += 16) {
          const int n = min(16, mine - i0);
          const auto part_of = [&](int i) { return way + ((i0 + min(i, n - 1)) << ways_log2); };
          const float2 ml = dev_ld2(head_ml + place(part_of(lane & 15)) * 2);
          float2 pa[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) pa[i] = dev_ld2(head_acc + place(part_of(i)) * kHeadDim + 2 * lane);
          const Merged sum = merge_parts(ml.x, ml.y, n, lane);
          const float cm = fmaxf(mx, sum.m);
          const float rescale = __builtin_amdgcn_exp2f(mx - cm), scale = __builtin_amdgcn_exp2f(sum.m - cm);
          l_all = l_all * rescale + sum.l * scale;
          o0 *= rescale, o1 *= rescale;
          const float weight = sum.weight * scale;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            if (i < n) {  // not a factor of zero: the values may be infinite
              const float f = from_lane(weight, i);
              o0 += pa[i].x * f, o1 += pa[i].y * f;
            }
          }
          mx = cm;
        }
        *reinterpret_cast<float2*>(sm_acc + wave * kHeadDim + 2 * lane) = make_float2(o0, o1);
        if (lane == 0) sm_m[wave] = mx, sm_l[wave] = l_all;
        __syncthreads();
        for (int x0 = wave * kWave; x0 < n_out; x0 += kThreads) {
          const int hh = x0 / kHeadDim, ch = (x0 & (kHeadDim - 1)) + lane;
          const int first_way = hh << ways_log2, ways = 1 << ways_log2;
          const int part = first_way + (lane & (ways - 1));
          const Merged all = merge_parts(sm_m[part], sm_l[part], ways, lane);
          float acc = 0.f;
#pragma unroll
          for (int i = 0; i < kWaves; ++i)
            if (i < ways) acc += sm_acc[(first_way + i) * kHeadDim + ch] * from_lane(all.weight, i);
          store_out(a.out, a.out_is_fp16, (bh0 + hh) * kHeadDim + ch, acc / all.l);
          if (ch == 0 && a.lse) a.lse[bh0 + hh] = (all.m + __builtin_amdgcn_logf(all.l)) * kLn2;
        }
      }
    }
    __syncthreads();  // the LDS buffers are free again
    off += n_pages;
    if (off == base + (int64_t)blocks * length_of(pages)) base = off, ++b;
  }
}

// Four adjacent heads per work-group where that leaves an item at most about 32 parts to
// merge (256 shares over batch * heads / 4 items); fewer heads share a work-group's waves (one
// sequence of 30000 tokens, 8 heads: 30.1 us by fours, 24.5 one by one).
bool four_heads(const quest_cache& c) {
  return group_size(c) == 1 && kv_heads(c) % 4 == 0 && (long)c.batch * kv_heads(c) >= 32;
}

// Units of 16 tokens of all heads, of the longest sequences the page table has room for.
double dense_units(const quest_cache& c) {
  return (double)c.batch * kv_heads(c) * attention_subs(c) * c.max_pages_per_seq * c.page_size / 16;
}

// Long rows and much work are cut into equal shares; rows of few tokens, or little work, into
// splits (launch_row_decode): a share finds its place on the line only when it has the
// lengths, hands over twice if it ends one item and begins the next, and takes item after item
// where there are many short ones.  us a launch, splits / equal shares: 32 heads of 700 tokens
// 6.6 / 9.6, of 8000 tokens 24.1 / 26.7, of 16000 tokens (32k units) 43.7 / 45.8, of 32768 tokens (66k)
// 87.1 / 85.6; 64 sequences of 128 tokens 24.1 / 31.0, 128 of 100 to 1000 tokens, 32 query / 8 KV
// heads, 53.3 / 83.7, 16 of 1000 to 4000, 32 heads, 109.7 / 105.7, 8 of 1000 to 20000 251 / 209.
// A few heads of long rows need more parts than the splits of a row are good for: 4 heads of 8000
// tokens 10.1 / 9.3, 2 of 60000 29.8 / 16.4, 8 query / 2 KV heads of 30000 20.3 / 16.0 (but 2 sequences
// of 9000 11.9 / 17.1), 8 heads of 8000 10.8 / 11.4.  More than 128 items have one split each: 4 sequences
// of 1242 to 4314 tokens, 40 heads, 51.4 / 42.9, but 5 of 2000, 32 heads, 27.7 / 31.5.
bool equal_shares(const quest_cache& c) {
  const long tokens = (long)c.max_pages_per_seq * c.page_size;
  const long items = (long)c.batch * kv_heads(c) * attention_subs(c);
  return (tokens > 3072 && (dense_units(c) > 48 * 1024 || items > 128)) || (items < 8 && tokens > (group_size(c) > 1 ? 16384 : 6400));
}

// Work-groups: four units of 16 tokens per wave at least (a part costs about 2 us to hand
// over and merge).
int dense_shares(const quest_cache& c) {
  const double shares = std::min<double>(dense_units(c) / (4 * waves_of(group_size(c) > 1)), most_shares(c));
  return std::max(16, (int)((shares + 15) / 16) * 16);
}

int heads_per_slot(const quest_cache& c) { return group_size(c) > 1 ? kGroupHeads : four_heads(c) ? 4 : 1; }

size_t counter_bytes(const quest_cache& c) {
  return (size_t)c.batch * c.num_heads * kTeamWordStride * sizeof(uint64_t);
}

}  // namespace

size_t dense_workspace_bytes(const quest_cache& c) {
  if (!equal_shares(c)) return row_workspace_bytes(c);
  return counter_bytes(c) + (size_t)dense_shares(c) * 2 * heads_per_slot(c) * (kHeadDim + 2) * sizeof(float);
}

int launch_dense_decode(const quest_cache& c, const void* q, float sm_scale, void* out, int out_is_fp16,
                        float* lse, void* workspace, size_t workspace_bytes, hipStream_t s) {
  // The grid of heads one by one, by twos or by fours, whichever form runs.
  const int group = group_size(c), by = group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
  const long heads8 = ((long)c.batch * c.num_heads / by + 7) / 8;
  if (heads8 > 65535) {
    set_error("quest_sparse_decode: batch * heads = %ld exceeds the launch limit", heads8 * 8 * by);
    return QUEST_ERR_SHAPE;
  }
  if (!equal_shares(c) || workspace_bytes < dense_workspace_bytes(c))
    return launch_row_decode(c, q, sm_scale, out, out_is_fp16, lse, workspace, workspace_bytes, s);
  DenseArgs a;
  fill_attn_args(a, c, q, sm_scale, out, out_is_fp16, lse);
  const int block = four_heads(c) ? 4 : 1;
  a.shares = dense_shares(c);
  a.counters = (uint64_t*)workspace;
  a.part_acc = (float*)((char*)workspace + counter_bytes(c));
  a.part_ml = a.part_acc + (size_t)a.shares * 2 * heads_per_slot(c) * kHeadDim;
  const dim3 grid((unsigned)a.shares);
#define QUEST_DENSE_LAUNCH(L, G, B)                                                              \
  hipLaunchKernelGGL((dense_kernel<L, G, B, waves_of(G)>), grid, dim3(waves_of(G) * kWave), \
                     0, s, a)
  if (c.page_size == 8) {
    if (a.group > 1) QUEST_DENSE_LAUNCH(2, true, 1);
    else if (block == 4) QUEST_DENSE_LAUNCH(2, false, 4);
    else QUEST_DENSE_LAUNCH(2, false, 1);
  } else {
    if (a.group > 1) QUEST_DENSE_LAUNCH(4, true, 1);
    else if (block == 4) QUEST_DENSE_LAUNCH(4, false, 4);
    else QUEST_DENSE_LAUNCH(4, false, 1);
  }
#undef QUEST_DENSE_LAUNCH
  return check_launch("quest_sparse_decode");
}

}  // namespace quest
