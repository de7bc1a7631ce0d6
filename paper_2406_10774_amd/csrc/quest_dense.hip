// Decode attention over every page of every sequence: the dense baseline the paper compares
// against (Section 3.1 of arXiv 2406.10774), and what a model runs in the layers it does
// not sparsify.
//
// The pages of all sequences and heads are one line of work, cut into equal shares, one
// per work-group and at most one work-group per compute unit: sequences of any lengths keep
// every unit busy to the end.  (Splits of a fixed number of pages per head left the shorter
// sequences' units idle: 4 ragged sequences of 5k to 32k tokens, 32 query / 8 KV heads, 70
// us against 55 us.)  Items along the line are (sequence, block of heads); a share that covers an
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
// streams as long as they can carry it (2 layers of 32 heads, 32k tokens: 187 us with 128
// work-groups, 172.7 with 192, 174.5 with 224, 175.7 with 256, 189 with 512; 32 query / 8 KV
// heads, 4 ragged sequences: 133, 114.0, 113.3, 115.1, 127).
// Pages of 8 tokens leave a wave half the bytes in flight (one sequence of 42k tokens, 32 heads:
// 113.7 us with 192, 104.9 with 256, 115.9 with 384).
int most_shares(const quest_cache& c) { return group_size(c) > 1 ? 224 : c.page_size == 8 ? 256 : 192; }

struct DenseArgs : AttnArgs {
  int shares;  // work-groups; partial results of share w are slots 2w and 2w + 1
  int cuts;    // parts that every item is cut into, a work-group each; 0: equal shares of the line
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
  constexpr int kTeams = kThreads / 32;  // groups of threads that merge partial results
  constexpr int kSlots = Head::kSlots, kStride = Head::kStride;
  constexpr int kHeads = slot_heads<kGroup, kBlock>();
  constexpr int kAccFloats = kWaves * kSlots * kStride > kTeams * kHeadDim ? kWaves * kSlots * kStride : kTeams * kHeadDim;
  __shared__ __align__(16) float sm_acc[kAccFloats];
  __shared__ float sm_m[kWaves * kSlots > kTeams ? kWaves * kSlots : kTeams];
  __shared__ float sm_l[kWaves * kSlots > kTeams ? kWaves * kSlots : kTeams];
  __shared__ uint32_t sm_before;
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lane = lane_id();
  const int blocks = a.kv_heads * a.subs / kBlock;  // items per sequence
  // (a length past the end of the row, which a caller must not pass, reads no further than the row)
  auto pages_of = [&](int len) {
    return min((max(len, 0) + (1 << a.page_shift) - 1) >> a.page_shift, a.max_pages);
  };

  // ---- this work-group's share [off, end) of the line, and the sequence it begins in
  const int64_t w = blockIdx.x;
  int64_t total = 0, shares = 1, off, end;
  int64_t base = 0;  // where sequence b begins
  int b = 0;
  int parts_each = 0;
  if (a.cuts) {
    const int item = (int)w / a.cuts, part = (int)w - item * a.cuts;
    b = item / blocks;
    const int pages = pages_of(a.seq_lens[b]);
    parts_each = min(a.cuts, pages);  // none is empty
    if (part >= parts_each) return;
    off = end = (int64_t)(item - b * blocks) * pages;
    off += (int)((int64_t)part * pages / parts_each);
    end += (int)((int64_t)(part + 1) * pages / parts_each);
  } else {
    for (int b0 = 0; b0 < a.batch; b0 += kWave) {
      const int p = b0 + lane < a.batch ? pages_of(a.seq_lens[b0 + lane]) : 0;
      total += __builtin_amdgcn_readlane(wave_incl_scan(p, lane), kWave - 1);
    }
    total *= blocks;
    shares = total < a.shares ? total : a.shares;  // none is empty
    if (w >= shares) return;
    off = w * total / shares;
    end = (w + 1) * total / shares;
    for (int b0 = 0; b0 < a.batch; b0 += kWave) {
      const int p = b0 + lane < a.batch ? pages_of(a.seq_lens[b0 + lane]) : 0;
      const int upto = wave_incl_scan(p, lane);
      const int64_t after = base + (int64_t)__builtin_amdgcn_readlane(upto, kWave - 1) * blocks;
      if (off < after) {
        const int k = __popcll(__ballot(b0 + lane < a.batch && base + (int64_t)upto * blocks <= off));
        b = b0 + k;
        base += k > 0 ? (int64_t)__builtin_amdgcn_readlane(upto, k > 0 ? k - 1 : 0) * blocks : 0;
        break;
      }
      base = after;
    }
  }
  const int64_t begin = off;
  auto share_of = [&](int64_t at) { return (int)(((at + 1) * shares - 1) / total); };

  while (off < end) {
    // ---- one item, or the part of it that lies in the share
    const int seq_len = __builtin_amdgcn_readfirstlane(a.seq_lens[b]);
    const int pages = pages_of(seq_len);
    if (pages == 0) {
      ++b;
      continue;
    }
    const int block = (int)((off - base) / pages);
    const int64_t item_at = base + (int64_t)block * pages;
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
    for (int x = t; x < n_out; x += kThreads) {
      const int g = x / kHeadDim, ch = x & (kHeadDim - 1);
      float m_tot, l_tot, acc;
      if constexpr (kBlock > 1) {
        m_tot = sm_m[g], l_tot = sm_l[g], acc = sm_acc[g * kStride + ch];
      } else {
        m_tot = sm_m[g];
#pragma unroll
        for (int i = 1; i < kWaves; ++i) m_tot = fmaxf(m_tot, sm_m[i * kSlots + g]);
        l_tot = 0.f, acc = 0.f;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
          const float f = __builtin_amdgcn_exp2f(sm_m[i * kSlots + g] - m_tot);
          l_tot += sm_l[i * kSlots + g] * f;
          acc += sm_acc[(i * kSlots + g) * kStride + ch] * f;
        }
      }
      if (whole) {
        store_out(a.out, a.out_is_fp16, bh0 * kHeadDim + x, acc / l_tot);
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
      const int from = a.cuts ? (int)w / a.cuts * a.cuts : share_of(item_at);
      const int parts = a.cuts ? parts_each : share_of(item_at + pages - 1) - from + 1;
      uint32_t* arrivals = reinterpret_cast<uint32_t*>(
          a.counters + ((size_t)b * blocks + block) * kTeamWordStride);
      wait_stores();
      __syncthreads();
      if (t == 0) sm_before = team_arrive(arrivals, a.device_fences);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sm_before) == (uint32_t)parts - 1) {
        team_acquire(a.device_fences);
        if (t == 0) team_reset(arrivals);
        // Teams of 32 threads, four channels a thread: a head's parts are dealt to as
        // many teams as there are for it, eight at a time in flight per team, and the teams'
        // sums added through LDS.  Fixed order: the result does not depend on who was last.
        const int heads = n_out / kHeadDim;
        const int ways = kTeams / (heads <= 1 ? 1 : heads <= 2 ? 2 : heads <= 4 ? 4 : 8);  // teams per head
        const int team = t >> 5, quad = (t & 31) * 4;
        const int g = team / ways, way = team - g * ways;
        float mx = kNegBig, l_all = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
        if (g < heads) {
          for (int k0 = way; k0 < parts; k0 += 8 * ways) {
            float2 ml[8], pa[8], pb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int k = min(k0 + i * ways, parts - 1);
              const size_t ps = (2 * (size_t)(from + k) + (k == 0 ? 1 : 0)) * kHeads + g;
              ml[i] = dev_ld2(a.part_ml + ps * 2);
              pa[i] = dev_ld2(a.part_acc + ps * kHeadDim + quad);
              pb[i] = dev_ld2(a.part_acc + ps * kHeadDim + quad + 2);
            }
            float cm = mx;
#pragma unroll
            for (int i = 0; i < 8; ++i) cm = fmaxf(cm, ml[i].x);
            const float rescale = __builtin_amdgcn_exp2f(mx - cm);
            l_all *= rescale;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] *= rescale;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              if (k0 + i * ways >= parts) continue;  // not a factor of zero: the values may be infinite
              const float f = __builtin_amdgcn_exp2f(ml[i].x - cm);
              l_all += ml[i].y * f;
              o[0] += pa[i].x * f;
              o[1] += pa[i].y * f;
              o[2] += pb[i].x * f;
              o[3] += pb[i].y * f;
            }
            mx = cm;
          }
        }
        *reinterpret_cast<float4*>(sm_acc + team * kHeadDim + quad) = make_float4(o[0], o[1], o[2], o[3]);
        if ((t & 31) == 0) sm_m[team] = mx, sm_l[team] = l_all;
        __syncthreads();
        for (int x = t; x < n_out; x += kThreads) {
          const int hh = x / kHeadDim, ch = x & (kHeadDim - 1);
          float m_tot = kNegBig, l_tot = 0.f, acc = 0.f;
          for (int i = 0; i < ways; ++i) m_tot = fmaxf(m_tot, sm_m[hh * ways + i]);
          for (int i = 0; i < ways; ++i) {
            const float f = __builtin_amdgcn_exp2f(sm_m[hh * ways + i] - m_tot);
            l_tot += sm_l[hh * ways + i] * f;
            acc += sm_acc[(hh * ways + i) * kHeadDim + ch] * f;
          }
          store_out(a.out, a.out_is_fp16, bh0 * kHeadDim + x, acc / l_tot);
          if (ch == 0 && a.lse) a.lse[bh0 + hh] = (m_tot + __builtin_amdgcn_logf(l_tot)) * kLn2;
        }
      }
    }
    __syncthreads();  // the LDS buffers are free again
    off += n_pages;
    if (off == base + (int64_t)blocks * pages) base = off, ++b;
  }
}

// Four adjacent heads per work-group where that leaves an item at most about 32 parts to
// merge (256 shares over batch * heads / 4 items); fewer heads share a work-group's waves.
bool four_heads(const quest_cache& c) {
  return group_size(c) == 1 && kv_heads(c) % 4 == 0 && (long)c.batch * kv_heads(c) >= 32;
}

long dense_items(const quest_cache& c) {
  return (long)c.batch * kv_heads(c) * attention_subs(c) / (four_heads(c) ? 4 : 1);
}

// Little work: every item in as many parts, because a share that ends one item and begins the
// next hands over twice, one after the other (launches of 6 sequences of 900 tokens, 8 heads: 13.0
// us in equal shares, 10.9 in parts; 8 heads of 3000 tokens 8.9 and 7.7; 4 sequences of 900, 32
// query / 8 KV heads 16.2 and 11.5).  At
// most eight units per wave, so that ragged sequences cannot make one part long; two at least.
int dense_cuts(const quest_cache& c) {
  const long units = (long)c.max_pages_per_seq * c.page_size / 16 / (four_heads(c) ? 1 : waves_of(group_size(c) > 1));
  const long cuts = std::max(1l, std::min(256 / dense_items(c), units / 2));
  return dense_items(c) <= 256 && units <= 8 * cuts ? (int)cuts : 0;
}

// Work-groups: four units of 16 tokens per wave at least (a part costs about 2 us to hand
// over and merge), of the longest work the page table has room for.
int dense_shares(const quest_cache& c) {
  if (const int cuts = dense_cuts(c)) return (int)dense_items(c) * cuts;
  const bool group = group_size(c) > 1;
  const double heads = (double)c.batch * kv_heads(c) * attention_subs(c);
  const double units = heads * c.max_pages_per_seq * c.page_size / 16;
  const double shares = std::min<double>(units / (4 * waves_of(group)), most_shares(c));
  return std::max(16, (int)((shares + 15) / 16) * 16);
}

int heads_per_slot(const quest_cache& c) { return group_size(c) > 1 ? kGroupHeads : four_heads(c) ? 4 : 1; }

size_t counter_bytes(const quest_cache& c) {
  return (size_t)c.batch * c.num_heads * kTeamWordStride * sizeof(uint64_t);
}

}  // namespace

size_t dense_workspace_bytes(const quest_cache& c) {
  return counter_bytes(c) + (size_t)dense_shares(c) * 2 * heads_per_slot(c) * (kHeadDim + 2) * sizeof(float);
}

int launch_dense_decode(const quest_cache& c, const void* q, float sm_scale, void* out, int out_is_fp16,
                        float* lse, void* workspace, size_t workspace_bytes, hipStream_t s) {
  DenseArgs a;
  fill_attn_args(a, c, q, sm_scale, out, out_is_fp16, lse);
  const int block = four_heads(c) ? 4 : 1;
  const long items = dense_items(c);
  if (items > 8 * 65535l) {
    set_error("quest_sparse_decode: batch * heads = %ld exceeds the launch limit", items * block);
    return QUEST_ERR_SHAPE;
  }
  const bool whole = workspace_bytes < dense_workspace_bytes(c);  // no workspace: every work-group takes one item
  a.cuts = whole ? 1 : dense_cuts(c);
  a.shares = whole ? (int)items : dense_shares(c);
  a.counters = (uint64_t*)workspace;
  a.part_acc = whole ? nullptr : (float*)((char*)workspace + counter_bytes(c));
  a.part_ml = whole ? nullptr : a.part_acc + (size_t)a.shares * 2 * heads_per_slot(c) * kHeadDim;
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
