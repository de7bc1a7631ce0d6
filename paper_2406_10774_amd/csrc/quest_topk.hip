// Top-K page selection (Section 3.4 of arXiv 2406.10774: the K pages with the
// largest criticality score are the ones attended).  One work-group per
// (sequence, head).
//
// Scores are mapped to unsigned 32-bit keys whose integer order equals the order of the float
// values (-0 folded onto +0).  A lower bound of the K-th largest, from the largest keys of K or
// more sets of pages, leaves a fraction of the row; 256 bins of equal width between it and
// the largest score tell in which bin the K-th lies (LDS histogram); the few keys of that bin are
// ranked one by one, or, where they are many, narrowed down by a radix select first.
// Every page in front is emitted, and of the bin those that are left to take, each at the position given
// by a work-group-wide prefix count, so the output is ascending and the lowest page index wins
// among equal scores.  (quest_topk_core.h)
//
// The kernel is bound by instructions and latency (a few thousand keys per head): keys
// live in registers, the score loads are issued before seq_lens is known, every wave
// searches the histogram and ranks the bin's keys itself so that there are three barriers in
// all (more only where the radix select runs), atomics and stores to LDS go to spare entries instead of being branched around, and
// what is counted once per wave is kept in scalar registers.  32 rows of 2053 scores, K = 128: 3.8 us
// a launch, 5.4 with 8-bit digits of the keys from the first on; 8193, K = 256: 6.3 and 11.0 us.
#include "quest_common.h"
#include "quest_topk_core.h"

namespace quest {

namespace {

template <int kThreads, int kItems>
__global__ __launch_bounds__(kThreads) void topk_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ k_eff, int num_heads, int max_pages,
    int k_pages, int page_shift, int policy) {
  __shared__ __align__(16) TopkShared<kThreads, kItems> sm;
  const int h = blockIdx.x;
  const int b = blockIdx.y;
  const size_t bh = (size_t)b * num_heads + h;
  topk_block<kThreads, kItems>(sm, scores + bh * max_pages, seq_lens + b, max_pages, k_pages,
                                      topk_idx + bh * k_pages,
                                      (h == 0 && k_eff != nullptr) ? k_eff + b : nullptr, page_shift,
                                      policy);
}

// Fallback for rows too long for register-resident keys: keys are re-read from
// global memory (L2) in every pass; same algorithm without the shortcuts.
constexpr int kBigThreads = 1024;
__global__ __launch_bounds__(kBigThreads) void topk_big_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ k_eff, int num_heads, int max_pages,
    int k_pages, int page_shift, int policy) {
  constexpr int kWaves = kBigThreads / kWave;
  __shared__ __align__(16) uint32_t hist[256];
  __shared__ int wave_gt[kWaves], wave_eq[kWaves];
  const int h = blockIdx.x;
  const int b = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = tid >> 6;
  const int num_pages = (seq_lens[b] + (1 << page_shift) - 1) >> page_shift;
  const int K = min(k_pages, num_pages);
  const float* row = scores + ((size_t)b * num_heads + h) * max_pages;
  int32_t* out = topk_idx + ((size_t)b * num_heads + h) * k_pages;
  if (h == 0 && tid == 0 && k_eff != nullptr) k_eff[b] = K;
  if (K == num_pages) {
    for (int i = tid; i < k_pages; i += kBigThreads) out[i] = i < K ? i : -1;
    return;
  }
  const ForcedPages forced = forced_pages(policy, num_pages);
  if (forced.count >= K) {
    if (tid == 0) {
      out[0] = forced.first ? 0 : num_pages - 1;
      if (K == 2) out[1] = num_pages - 1;
    }
    return;
  }
  auto key_of = [&](int i) { return forced.is(i) ? 0xffffffffu : score_key(row[i]); };
  uint32_t prefix = 0;
  int need = K;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const uint32_t high_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int i = tid; i < num_pages; i += kBigThreads) {
      const uint32_t key = key_of(i);
      if ((key & high_mask) == prefix) atomicAdd(&hist[255u - ((key >> shift) & 255u)], 1u);
    }
    __syncthreads();
    const BinHit hit = find_bin(hist, need, lane);
    prefix |= (uint32_t)(255 - hit.bin) << shift;
    need -= hit.before;
    __syncthreads();
  }
  const uint32_t T = prefix;
  const int items = (num_pages + kBigThreads - 1) / kBigThreads;
  const int begin = min(tid * items, num_pages);
  const int end = min(begin + items, num_pages);
  int n_gt = 0, n_eq = 0;
  for (int i = begin; i < end; ++i) {
    const uint32_t key = key_of(i);
    n_gt += key > T;
    n_eq += key == T;
  }
  const int gt_incl = wave_incl_scan(n_gt);
  const int eq_incl = wave_incl_scan(n_eq);
  if (lane == kWave - 1) {
    wave_gt[wave] = gt_incl;
    wave_eq[wave] = eq_incl;
  }
  __syncthreads();
  int gt_before = gt_incl - n_gt, eq_before = eq_incl - n_eq;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) {
      gt_before += wave_gt[w];
      eq_before += wave_eq[w];
    }
  }
  for (int i = begin; i < end; ++i) {
    const uint32_t key = key_of(i);
    if (key > T) {
      out[gt_before + min(eq_before, need)] = i;
      ++gt_before;
    } else if (key == T) {
      if (eq_before < need) out[gt_before + eq_before] = i;
      ++eq_before;
    }
  }
}

// ---- Selection in two stages for very long rows.  One work-group per row is bound by
// what one compute unit can issue (about 0.75 us per key and thread at 1024 threads);
// here the row is cut into chunks of 2048 or 4096 pages, a work-group per chunk selects
// the chunk's own best K pages (the K best of the row are among them, ties included:
// fewer than K pages of the chunk rank above any of them), and a second launch selects
// among the candidates.  Candidates are stored densely in page order (every chunk
// before the last non-empty one is full and yields exactly k_pages of them), so
// positions in the candidate row order like pages do: equal scores still go to the
// lower page, page 0 is candidate 0 and the newest page is the last candidate whenever
// the policy flags keep them in their chunks.
// Threads: 4 keys each of a chunk of 2048 pages (512 threads; a step of 8 heads, 500k tokens, 31.2 us, 31.5
// with 8 keys each), 8 each of 4096 (512 threads: 32 heads, 512k tokens, 103.5 us a step, 104.5 with 1024
// threads, of which two work-groups fill a compute unit).
constexpr int kChunkThreads = 512;

struct ChunkOfRow {
  int page_shift, policy, chunk, chunk_pages;
  __device__ __forceinline__ RowShape operator()(int seq_len) const {
    const int pages = (seq_len + (1 << page_shift) - 1) >> page_shift;
    const int local = min(max(pages - chunk * chunk_pages, 0), chunk_pages);
    int pol = 0;
    if (chunk == 0) pol |= policy & QUEST_FLAG_KEEP_FIRST_PAGE;
    if (local > 0 && (chunk + 1) * chunk_pages >= pages) pol |= policy & QUEST_FLAG_KEEP_NEWEST_PAGE;
    return {local, pol};
  }
};

template <int kThreads, int kChunkItems>
__global__ __launch_bounds__(kThreads) void topk_chunk_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ seq_lens,
    float* __restrict__ cand_score, int32_t* __restrict__ cand_page, int num_heads, int max_pages,
    int k_pages, int num_chunks, int page_shift, int policy) {
  constexpr int kPages = kThreads * kChunkItems;
  __shared__ __align__(16) TopkShared<kThreads, kChunkItems> sm;
  // chunk-major launch order: the last chunk of a row, often a short one, must not take
  // the place of a full one on a compute unit that is still free
  const int h = blockIdx.x;
  const int chunk = blockIdx.y;
  const int b = blockIdx.z;
  const size_t bh = (size_t)b * num_heads + h;
  const float* row = scores + bh * max_pages + (size_t)chunk * kPages;
  const size_t at = (bh * num_chunks + chunk) * k_pages;
  float* out_score = cand_score + at;
  int32_t* out_page = cand_page + at;
  topk_block_put<kThreads, kChunkItems>(
      sm, row, seq_lens + b, min(kPages, max_pages - chunk * kPages), k_pages,
      [=](bool sel, int pos, int page, int j, float score) {
        if (sel && page >= 0) {
          out_page[pos] = page + chunk * kPages;
          out_score[pos] = j >= 0 ? score : row[page];
        }
      },
      nullptr, ChunkOfRow{page_shift, policy, chunk, kPages}, [] {});
}

template <int kThreads, int kItems>
__global__ __launch_bounds__(kThreads) void topk_candidates_kernel(
    const float* __restrict__ cand_score, const int32_t* __restrict__ cand_page,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx,
    int32_t* __restrict__ k_eff, int num_heads, int row_len, int k_pages, int page_shift,
    int policy) {
  __shared__ __align__(16) TopkShared<kThreads, kItems> sm;
  const int h = blockIdx.x;
  const int b = blockIdx.y;
  const size_t bh = (size_t)b * num_heads + h;
  const int32_t* pages = cand_page + bh * row_len;
  int32_t* out = topk_idx + bh * k_pages;
  // the pages of this thread's candidates travel behind their scores (entries past the
  // stored candidates are inside the row: never selected, safe to read)
  int32_t my_page[kItems];
  topk_block_put<kThreads, kItems>(
      sm, cand_score + bh * row_len, seq_lens + b, row_len, k_pages,
      [&](bool sel, int pos, int cand, int j, float) {
        int32_t page = -1;
        if (j >= 0) {
#pragma unroll
          for (int jj = 0; jj < kItems; ++jj)
            if (jj == j) page = my_page[jj];
        } else if (cand >= 0) {
          page = pages[cand];
        }
        if (sel) out[pos] = page;
      },
      (h == 0 && k_eff != nullptr) ? k_eff + b : nullptr, CandidateRow{page_shift, policy, k_pages, kLargeChunk},
      [&] {
#pragma unroll
        for (int jj = 0; jj < kItems; ++jj)
          my_page[jj] = pages[min((int)threadIdx.x + jj * kThreads, row_len - 1)];
      });
}

template <int kThreads, int kItems>
int launch_one(const quest_cache& c, const float* scores, int k_pages, int32_t* topk_idx,
               int32_t* k_eff, hipStream_t s) {
  hipLaunchKernelGGL((topk_kernel<kThreads, kItems>), dim3(kv_heads(c), c.batch), dim3(kThreads), 0,
                     s, scores, c.seq_lens, topk_idx, k_eff, kv_heads(c), c.max_pages_per_seq,
                     k_pages, page_shift_of(c.page_size), c.flags);
  return check_launch("quest_topk");
}

}  // namespace

int launch_topk(const quest_cache& c, const float* scores, int k_pages, int32_t* topk_idx,
                int32_t* k_eff, hipStream_t s) {
  const int mp = c.max_pages_per_seq;
#define QUEST_TOPK_CASE(T, I) \
  if (mp <= (T) * (I)) return launch_one<T, I>(c, scores, k_pages, topk_idx, k_eff, s)
  // up to 8192 pages: 512 threads, smallest ITEMS that covers the row
  QUEST_TOPK_CASE(512, 1);
  QUEST_TOPK_CASE(512, 2);
  QUEST_TOPK_CASE(512, 3);
  QUEST_TOPK_CASE(512, 4);
  QUEST_TOPK_CASE(512, 5);
  QUEST_TOPK_CASE(512, 6);
  QUEST_TOPK_CASE(512, 8);
  QUEST_TOPK_CASE(512, 10);
  QUEST_TOPK_CASE(512, 12);
  QUEST_TOPK_CASE(512, 16);
  QUEST_TOPK_CASE(512, 20);
  // up to 65536 pages (the packed prefix counts hold 16 bits each)
  QUEST_TOPK_CASE(1024, 12);
  QUEST_TOPK_CASE(1024, 17);
  QUEST_TOPK_CASE(1024, 24);
  QUEST_TOPK_CASE(1024, 33);
  QUEST_TOPK_CASE(1024, 48);
  if (mp < 65536) return launch_one<1024, 64>(c, scores, k_pages, topk_idx, k_eff, s);
#undef QUEST_TOPK_CASE
  hipLaunchKernelGGL(topk_big_kernel, dim3(kv_heads(c), c.batch), dim3(kBigThreads), 0, s, scores,
                     c.seq_lens, topk_idx, k_eff, kv_heads(c), c.max_pages_per_seq, k_pages,
                     page_shift_of(c.page_size), c.flags);
  return check_launch("quest_topk");
}

size_t candidate_bytes(const quest_cache& c, int k_pages, int chunk_pages) {
  const long cand = candidates_per_row(c, k_pages, chunk_pages);
  if (k_pages < 1 || k_pages > chunk_pages || cand > kMaxCandidates || 2 * cand > c.max_pages_per_seq) return 0;
  return (size_t)c.batch * kv_heads(c) * cand * (sizeof(float) + sizeof(int32_t));
}

size_t topk_scratch_bytes(const quest_cache& c, int k_pages) {
  return c.max_pages_per_seq < kChunkedFromPages ? 0 : candidate_bytes(c, k_pages, kLargeChunk);
}

int launch_topk_chunks(const quest_cache& c, const float* scores, int k_pages, int chunk_pages,
                       void* scratch, Candidates* out, hipStream_t s) {
  const int chunks = (c.max_pages_per_seq + chunk_pages - 1) / chunk_pages;
  float* cand_score = (float*)scratch;
  out->row_len = chunks * k_pages;
  out->chunk_pages = chunk_pages;
  out->score = cand_score;
  int32_t* cand_page = (int32_t*)(cand_score + (size_t)c.batch * kv_heads(c) * out->row_len);
  out->page = cand_page;
  const dim3 grid(kv_heads(c), chunks, c.batch);
#define QUEST_CHUNKS(T)                                                                           \
  hipLaunchKernelGGL((topk_chunk_kernel<kChunkThreads, (T) / kChunkThreads>), grid,               \
                     dim3(kChunkThreads), 0, s, scores, c.seq_lens, cand_score, cand_page,        \
                     kv_heads(c), c.max_pages_per_seq, k_pages, chunks, page_shift_of(c.page_size), c.flags)
  if (chunk_pages == kSmallChunk)
    QUEST_CHUNKS(kSmallChunk);
  else
    QUEST_CHUNKS(kLargeChunk);
#undef QUEST_CHUNKS
  return check_launch("quest_select_decode");
}

int launch_topk_chunked(const quest_cache& c, const float* scores, int k_pages, int32_t* topk_idx,
                        int32_t* k_eff, void* scratch, hipStream_t s) {
  Candidates cand;
  const int r = launch_topk_chunks(c, scores, k_pages, kLargeChunk, scratch, &cand, s);
  if (r != QUEST_OK) return r;
  const int row_len = cand.row_len;
  const float* cand_score = cand.score;
  const int32_t* cand_page = cand.page;
#define QUEST_CAND_CASE(I)                                                                       \
  if (row_len <= 512 * (I)) {                                                                    \
    hipLaunchKernelGGL((topk_candidates_kernel<512, I>), dim3(kv_heads(c), c.batch), dim3(512), 0, \
                       s, cand_score, cand_page, c.seq_lens, topk_idx, k_eff, kv_heads(c), row_len, \
                       k_pages, page_shift_of(c.page_size), c.flags);                            \
    return check_launch("quest_select_decode");                                                  \
  }
  QUEST_CAND_CASE(2)
  QUEST_CAND_CASE(5)
  QUEST_CAND_CASE(8)
  QUEST_CAND_CASE(16)
#undef QUEST_CAND_CASE
  set_error("quest_select_decode: internal: %d candidates per row", row_len);
  return QUEST_ERR_SHAPE;
}

}  // namespace quest
