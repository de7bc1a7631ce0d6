// Query-aware page criticality (attention half of Algorithm 1, Section 3.4 of
// arXiv 2406.10774):  score[p] = sum_i max(q_i * m_{p,i}, q_i * M_{p,i}).
//
// Since m <= M per channel, max(q m, q M) is q * (q >= 0 ? M : m) exactly: the
// sign of q picks the row, done once per wave as a bit mask, and the products
// go through v_dot2_f32_f16 (fp16 products are exact in fp32, fp32 sum), or, where several
// query heads share a KV head, through matrix products with q split by its sign.
//
// One wavefront owns (head, block of 8 or 16 consecutive logical pages).  A 16-lane
// DPP row reads one metadata entry: 16 B per lane of the min row, then 16 B per
// lane of the max row (two 256 B segments, 512 B contiguous), so one wave-wide
// load instruction covers four pages; the 128-channel sum is a reduction inside
// the DPP row.  All loads of a wave are issued before the first use.
#include "quest_common.h"
#include "quest_estimate_core.h"

namespace quest {

namespace {

constexpr int kEstWaves = 4;
constexpr unsigned kLdsPerUnit = 160 * 1024;  // of a gfx950 compute unit

// Grid: x = blocks of pages, y = sequence, z = head.  The metadata table is head-major
// over the physical pages, so with the sequences' pages laid out one after the other
// consecutive work-groups walk memory in order (6.05 TB/s against 5.5 TB/s with the
// heads in y, at 16 sequences of 32k tokens).
//
// Large tables (kIters = 4): a wave asks for its page-table entries only once it has the
// length, so that the waves of a ragged batch that lie past the end of a sequence leave
// early (16 sequences of 8k to 64k tokens: 91.6 us against 93.3 us; one of 512k 80.2 against
// 81.9).  In a small table a trip to memory more would show (4 sequences, 8 heads: 7.0 us
// against 6.8 us).
template <bool kAppend, int kIters, int kQ>
__global__ __launch_bounds__(kEstWaves* kWave, kQ == 0 ? (kIters == 2 ? 7 : 4) : 1) void estimate_kernel(const EstimateArgs a) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int base = (blockIdx.x * kEstWaves + wave) * (4 * kIters);
  if (kIters == kEstIters && (long)base << a.page_shift >= a.seq_lens[blockIdx.y]) return;
  __shared__ __align__(16) char stage[kQ == 0 ? kEstWaves * 4 * kIters * kMetaBytes : 16];
  estimate_wave<kAppend, kIters, kQ>(a, blockIdx.y, blockIdx.z, base, stage + (kQ == 0 ? wave * 4 * kIters * kMetaBytes : 0));
}

}  // namespace

// The matrix cores score groups.  Two query heads meet the metadata of 16 sequences of up to 32k tokens
// in 14.7 us on the vector unit (one in 14.4), of 4 sequences in 6.1: no longer than four on the matrix
// cores (14.2 and 6.4).  Nor do three or four over small tables, where the turn through LDS shows: 2.85
// against 2.98 us at 8100 entries, but 4.08 against 3.75 at 16400.  Five and more are faster there in every
// table: five 3.00 and 2.83 at 256 entries, 4.03 and 3.73 at 9600; eight 3.17 and 2.93, 4.64 and 3.86.
bool estimate_on_matrix_cores(const quest_cache& c) {
  return group_size(c) > ((long)c.batch * kv_heads(c) * c.max_pages_per_seq <= (3l << 12) ? 4 : 2);
}

namespace {

// Pages per wave: 16 (eight wave-wide loads in flight) once the table is large; a smaller
// table is scanned faster by twice as many waves of half the size: 8.3 us against 8.75 us
// at 2049 pages of 32 heads, 13.6 against 14.2 at 4100, 23.0 against 23.4 at 8193; but 98.0
// against 93.7 us for 16 sequences of 8k to 64k tokens (1.2 M pages), and the calls of a layer
// 56.0 against 54.0 us for 2 sequences and 8 KV heads (0.49 M pages).
// On the matrix cores 16 pages fill an operand and eight leave half of it: 3.0 against 3.3 us at 4100
// entries, 4.7 against 4.8 at 33k, 6.6 against 6.4 at 66k, 15.7 against 14.2 at 263k.
// Not 12 for one query head in tables of 41k to 114k entries, where the waves of eight are about one round: full
// tables gain 2 to 8 % (66k 7.8 and 7.5), but where the sequences are shorter than the table's rows the waves with
// pages fall on the same units in every few rows once the work-groups of a row go into 256 a few times (2049 pages are
// 43 of 12 pages a wave, 65 of eight): at 0.3 of 2049 pages, 32 heads, 4.6 and 5.4; 576 rows of 183 pages, 0.27 of
// them in use, 6.0 and 9.0.  700 random tables: 1 % faster on average, a fifth of them up to 1.5 times slower.
int est_iters(const quest_cache& c) {
  const long entries = (long)c.batch * kv_heads(c) * c.max_pages_per_seq;
  return entries <= (group_size(c) > 2 ? 5l << 13 : 3l << 17) ? 2 : kEstIters;
}

template <bool kAppend, int kIters>
void launch_iters(const quest_cache& c, const EstimateArgs& a, hipStream_t s) {
  const int per_group = kEstWaves * 4 * kIters;
  const dim3 grid((c.max_pages_per_seq + per_group - 1) / per_group, c.batch, kv_heads(c));
  const dim3 block(kEstWaves * kWave);
  // LDS that nobody uses: it keeps the work-groups of a compute unit at five.  A large table
  // streams better that way than with more (512k tokens in order 80.2 us, 83.3 with six; two
  // sequences of 400k 123.5 and 128.9; 16 ragged ones 91.6 and 94.7); small ones do not care.
  // (On the matrix cores they use as much: 8 KiB per wave.)
  const unsigned lds = kIters == kEstIters && a.group <= 2 ? kLdsPerUnit / 5 : 0;
#define QUEST_ESTIMATE(Q) hipLaunchKernelGGL((estimate_kernel<kAppend, kIters, Q>), grid, block, lds, s, a)
  if (a.group == 1) QUEST_ESTIMATE(1);
  else if (a.group == 2) QUEST_ESTIMATE(2);
  else if (kIters == 2 && !estimate_on_matrix_cores(c)) {
    if constexpr (kIters == 2) {
      if (a.group == 3) QUEST_ESTIMATE(3);
      else QUEST_ESTIMATE(4);
    }
  } else {
    QUEST_ESTIMATE(0);
  }
#undef QUEST_ESTIMATE
}

template <bool kAppend>
void launch(const quest_cache& c, const EstimateArgs& a, hipStream_t s) {
  if (est_iters(c) == 2)
    launch_iters<kAppend, 2>(c, a, s);
  else
    launch_iters<kAppend, kEstIters>(c, a, s);
}

}  // namespace

EstimateArgs estimate_args(const quest_cache& c, const void* k_new, const void* v_new, int k_pool_write, const void* q,
                           float* scores) {
  EstimateArgs a;
  a.meta = (char*)c.meta;
  a.q = (const char*)q;
  a.page_table = c.page_table;
  a.seq_lens = c.seq_lens;
  a.scores = scores;
  a.num_heads = kv_heads(c);
  a.group = group_size(c);
  a.max_pages = c.max_pages_per_seq;
  a.num_phys_pages = c.num_phys_pages;
  a.page_shift = page_shift_of(c.page_size);
  a.k_new = (const char*)k_new;
  a.v_new = (const char*)v_new;
  a.k_pool = (char*)c.k_pool;
  a.v_pool = (char*)c.v_pool;
  a.k_pool_write = k_pool_write;
  return a;
}

int launch_estimate(const quest_cache& c, const void* q, float* scores, hipStream_t s) {
  launch<false>(c, estimate_args(c, nullptr, nullptr, 0, q, scores), s);
  return check_launch("quest_estimate");
}

int launch_append_estimate(const quest_cache& c, const void* k_new, const void* v_new,
                           int k_pool_write, const void* q, float* scores, hipStream_t s) {
  launch<true>(c, estimate_args(c, k_new, v_new, k_pool_write, q, scores), s);
  return check_launch("quest_append_estimate");
}

}  // namespace quest
