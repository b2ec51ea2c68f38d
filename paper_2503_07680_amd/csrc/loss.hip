// Packed cross-entropy with the paper's loss normalisers (Section 4.3, normaliser equation), forward
// and backward in one pass over the logits, gfx950.
//
//   token loss      CE_r = logsumexp(z_r) - z_r[label_r]                     (rows with label < 0: none)
//   loss            sum_r w_r CE_r,  w_r by normaliser: token-mean 1 / sum_i T_i, sample-mean
//                   1 / (T_i B_l) for the row's sample i, stable 1 / (B_l T_ave)
//   d loss / d z_r  w_r (softmax(z_r) - onehot(label_r))
//
// HBM-bound: every logit is read once and every gradient written once.  One workgroup of 256, 512 or
// 1024 threads owns a row at a time and holds the whole row in registers as packed bf16 (up to 163840
// entries: 20 loads of 16 bytes per thread, each load instruction of the workgroup covering 16 bytes per
// thread of consecutive addresses), so the row maximum, the sum of exponentials and the gradient are all
// computed from that one read; the registers of a chunk are refilled with the next row while the
// gradient of this one is still being written.  Longer rows are streamed twice (running maximum and
// rescaled sum in the first pass; the second read mostly hits L2/MALL).
// The weighted token losses go to a workspace array and are summed by one workgroup in a fixed order,
// so the loss is bit-stable from run to run.
#include "common.hpp"
#include "loss_rules.hpp"

namespace hbp {

constexpr int kCeThreads = 1024;  // of the kernels with one workgroup, and the most of a row's workgroup
constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}
// block-wide reduction over 1024 threads through 16 LDS slots; every thread gets the result
template <bool IS_MAX>
__device__ __forceinline__ float block_reduce(float x, float* slots, int tid) {
  x = IS_MAX ? wave_max(x) : wave_sum(x);
  __syncthreads();  // the slots may still be read from the previous reduction
  if ((tid & 63) == 0) slots[tid >> 6] = x;
  __syncthreads();
  float r = slots[0];
#pragma unroll
  for (int i = 1; i < kCeThreads / 64; ++i) r = IS_MAX ? fmaxf(r, slots[i]) : r + slots[i];
  return r;
}

// loss tokens per sample
__global__ __launch_bounds__(256) void ce_count_kernel(const CeParams p) {
  __shared__ int part[4];
  const int i = blockIdx.x;
  const int a = max(p.cu[i], 0), b = min(p.cu[i + 1], p.T);  // a malformed list cannot take a read out of bounds
  int n = 0;
  for (int r = a + (int)threadIdx.x; r < b; r += 256) n += p.labels[r] >= 0 && p.labels[r] < p.V;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) n += __shfl_xor(n, m, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) p.counts[i] = part[0] + part[1] + part[2] + part[3];
  // a row that belongs to no sample has weight 0 (the weight kernel fills in the others)
  for (int r = i * 256 + (int)threadIdx.x; r < p.T; r += gridDim.x * 256) p.weighted[r] = 0.f;
}

// per-sample weight of a token's cross-entropy, written to every row of the sample (weighted[r] holds
// the row's weight until the main kernel replaces it with weight x loss); one workgroup per sample
__global__ __launch_bounds__(256) void ce_weight_kernel(const CeParams p) {
  __shared__ float part[4];
  const int tid = threadIdx.x, i = blockIdx.x;
  float total = 0.f;
  if (p.normalizer == HBP_LOSS_TOKEN_MEAN) {  // same order in every workgroup: the same bits
    for (int j = tid; j < p.n_samples; j += 256) total += (float)p.counts[j];
    total = wave_sum(total);
    if ((tid & 63) == 0) part[tid >> 6] = total;
    __syncthreads();
    total = (part[0] + part[1]) + (part[2] + part[3]);
  }
  const float c = (float)p.counts[i];
  float w;
  if (p.normalizer == HBP_LOSS_TOKEN_MEAN) w = total > 0.f ? 1.0f / total : 0.f;
  else if (p.normalizer == HBP_LOSS_SAMPLE_MEAN) w = c > 0.f ? 1.0f / (c * (float)p.n_samples) : 0.f;
  else w = 1.0f / ((float)p.n_samples * p.t_ave);
  if (tid == 0) p.weights[i] = w;
  const int a = max(p.cu[i], 0), b = min(p.cu[i + 1], p.T);
  for (int r = a + tid; r < b; r += 256) p.weighted[r] = w;
}

// Rows to workgroups: workgroup k of the main kernel takes the consecutive rows
// [row_start[k], row_start[k + 1]), cut so that every range carries the same memory traffic (a row
// with a loss is read and written, one without is only written, or skipped when no gradient is asked
// for).  row_start[k] = the first row whose preceding rows cost at least k / n_ranges of the total.
__device__ __forceinline__ int row_cost(int label, int V, bool with_grad) {
  return (label >= 0 && label < V ? 8 : 0) + (with_grad ? 8 : 0) + 1;
}
__global__ __launch_bounds__(kCeThreads) void ce_partition_kernel(const CeParams p, int n_ranges) {
  __shared__ int64_t part[kCeThreads];
  const int tid = threadIdx.x;
  const bool with_grad = p.dlogits != nullptr;
  const int slice = (p.T + kCeThreads - 1) / kCeThreads;
  const int a = min(tid * slice, p.T), b = min(a + slice, p.T);
  int64_t mine = 0;
  for (int r = a; r < b; ++r) mine += row_cost(p.labels[r], p.V, with_grad);
  part[tid] = mine;
  __syncthreads();
  for (int d = 1; d < kCeThreads; d <<= 1) {  // inclusive scan
    const int64_t add = tid >= d ? part[tid - d] : 0;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  const int64_t total = part[kCeThreads - 1];
  int64_t before = part[tid] - mine;  // cost of the rows before row a
  if (tid == 0) p.row_start[0] = 0;
  for (int r = a; r < b; ++r) {
    const int64_t after = before + row_cost(p.labels[r], p.V, with_grad);
    // ranges k with before < k total / n_ranges <= after begin at row r + 1
    for (int64_t k = before * n_ranges / total + 1; k <= after * n_ranges / total; ++k) p.row_start[k] = r + 1;
    before = after;
  }
}

// ---- what a workgroup of the main kernel works out for itself -----------------------------------
// Every workgroup needs its rows and the weights of their samples, and both follow from which
// rows have a loss.  Up to kCePlanRows rows each workgroup reads all labels itself (from L2; 4 bytes a row
// against the row's 2 V), keeps them as one bit a row with a running count per 64 rows, and finds its rows
// and any sample's number of loss tokens in that.  The three kernels that did this before the main one
// (count, weight, partition) each cost a launch: 22 us of 757 at T = 8192, V = 128256, and 12 us of 40 at
// T = 1000, V = 32000.  They stay for longer packs, whose bits and counts would not fit beside the others'.

struct CeRows {
  uint64_t* live;  // bit i of word w: row 64 w + i has a loss; one word of zeros behind the last
  int32_t* before; // loss rows in front of word w; one entry behind the last
  int32_t* cu;     // bounds of the samples, null: too many, read them from global memory
};
// loss rows in front of row x; x is clamped to the pack (a malformed list of samples stays in bounds)
__device__ __forceinline__ int ce_live_before(const CeRows& c, int x, int T) {
  x = min(max(x, 0), T);
  return c.before[x >> 6] + __popcll(c.live[x >> 6] & ((1ull << (x & 63)) - 1));
}
__device__ __forceinline__ int ce_sample_count(const CeRows& c, int a, int b, int T) {
  return max(ce_live_before(c, b, T) - ce_live_before(c, a, T), 0);
}
// Row number q (from 0) of those with a loss, or of those without.
__device__ __forceinline__ int ce_nth_row(const CeRows& c, int n_words, int q, bool with_loss) {
  auto in_front = [&](int w) { return with_loss ? c.before[w] : 64 * w - c.before[w]; };
  int lo = 0, hi = n_words;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (in_front(mid) <= q) lo = mid;
    else hi = mid;
  }
  const uint64_t bits = with_loss ? c.live[lo] : ~c.live[lo];
  const int k = q - in_front(lo);
  int i = 0;
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1)
    if (__popcll(bits & ((1ull << (i + step)) - 1)) <= k) i += step;
  return 64 * lo + i;
}
// Fills c and returns the loss tokens in all samples (token mean; else 0); RANGE: and range[0..1] = this workgroup's rows (the cut of
// ce_partition_kernel: the first row whose preceding rows cost at least k / n_ranges of the total).
template <int NT, bool RANGE>
__device__ __forceinline__ int ce_plan_rows(const CeParams& p, const CeRows& c, int tid, int* range, int* slots) {
  constexpr int NW = NT / 64, kBatch = 4;
  const int wave = tid >> 6, lane = tid & 63, nw = ce_plan_words(p.T);
  const int bound = c.cu ? p.cu[min(tid, p.n_samples)] : 0;  // in front of the labels: one wait for both
  for (int w0 = wave; w0 < nw; w0 += NW * kBatch) {
    int lab[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int r = (w0 + NW * j) * 64 + lane;
      lab[j] = r < p.T ? p.labels[r] : -1;
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const uint64_t bits = __builtin_amdgcn_ballot_w64(lab[j] >= 0 && lab[j] < p.V);
      if (lane == 0 && w0 + NW * j < nw) c.live[w0 + NW * j] = bits;
    }
  }
  if (c.cu) {
    if (tid <= p.n_samples) c.cu[tid] = bound;
    for (int i = tid + NT; i <= p.n_samples; i += NT) c.cu[i] = p.cu[i];
  }
  __syncthreads();
  // running counts: `per` consecutive words a thread
  const int per = (nw + NT - 1) / NT;
  const int w_begin = min(tid * per, nw), w_end = min(w_begin + per, nw);
  int mine = 0;
  for (int w = w_begin; w < w_end; ++w) mine += __popcll(c.live[w]);
  int incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) slots[wave] = incl;
  __syncthreads();
  int base = incl - mine, all = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i < wave) base += slots[i];
    all += slots[i];
  }
  const uint64_t row_c = (p.dlogits ? 8 : 0) + 1;  // row_cost(): 8 more for a row with a loss
  const uint64_t total = row_c * p.T + 8ull * all, n = gridDim.x;
  for (int w = w_begin; w < w_end; ++w) {
    c.before[w] = base;
    const uint64_t bits = c.live[w];
    if (!RANGE) {
      base += __popcll(bits);
      continue;
    }
    const uint64_t in_front = row_c * (64ull * w) + 8ull * base;
    base += __popcll(bits);
    const uint64_t behind = row_c * min(64 * (w + 1), p.T) + 8ull * base;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint64_t target = (blockIdx.x + j) * total;
      if (in_front * n < target && target <= behind * n) {
        int i = 0;  // first row of the word with the rows up to and including it costing >= target / n
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
          const int k = i + step;  // rows 0 .. k - 1 of the word
          if ((in_front + row_c * k + 8ull * __popcll(bits & ((1ull << k) - 1))) * n < target) i = k;
        }
        range[j] = 64 * w + i + 1;
      }
    }
  }
  if (tid == 0) {
    c.live[nw] = 0;
    c.before[nw] = all;
    if (RANGE && blockIdx.x == 0) range[0] = 0;
  }
  __syncthreads();
  if (p.normalizer != HBP_LOSS_TOKEN_MEAN) return 0;
  int in_samples = 0;
  if (p.n_samples <= 64 && c.cu) {  // every wavefront for itself: two barriers less (1000 rows of 32000: 26.7 -> 26.4 us with the bounds' load)
    if (lane < p.n_samples) in_samples = ce_sample_count(c, c.cu[lane], c.cu[lane + 1], p.T);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) in_samples += __shfl_xor(in_samples, m, 64);
    return __builtin_amdgcn_readfirstlane(in_samples);
  }
  for (int i = tid; i < p.n_samples; i += NT)
    in_samples += ce_sample_count(c, c.cu ? c.cu[i] : p.cu[i], c.cu ? c.cu[i + 1] : p.cu[i + 1], p.T);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) in_samples += __shfl_xor(in_samples, m, 64);
  if (lane == 0) slots[wave] = in_samples;  // the counts in it were read before the barrier
  __syncthreads();
  in_samples = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) in_samples += slots[i];
  return __builtin_amdgcn_readfirstlane(in_samples);
}
// the weight of row r's cross-entropy; 0 for a row that belongs to no sample.  tokens: what ce_plan_rows returned.
__device__ __forceinline__ float ce_row_weight(const CeParams& p, const CeRows& c, int r, int tokens) {
  auto cu = [&](int i) { return c.cu ? c.cu[i] : p.cu[i]; };
  int lo = 0, hi = p.n_samples;  // the last sample that begins at or in front of the row
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu(mid) <= r) lo = mid;
    else hi = mid;
  }
  const int a = cu(lo), b = cu(lo + 1);
  if (r < a || r >= b) return 0.f;
  if (p.normalizer == HBP_LOSS_TOKEN_MEAN) return tokens > 0 ? 1.0f / (float)tokens : 0.f;
  if (p.normalizer == HBP_LOSS_STABLE) return 1.0f / ((float)p.n_samples * p.t_ave);
  const float n = (float)ce_sample_count(c, a, b, p.T);
  return n > 0.f ? 1.0f / (n * (float)p.n_samples) : 0.f;
}

// NCH: 16-byte loads per thread that cover a row when HOLD (row kept in registers); with !HOLD the
// row is streamed in kCeChunk pieces, twice.
//
// Softmax statistics: every thread keeps a running maximum m_t and sum s_t = sum exp(z - m_t) over its
// own logits, chunk by chunk (the sum is rescaled when the maximum moves); the (m, s) pairs are merged
// per wave and then through LDS, s = sum_t s_t exp(m_t - m).  One workgroup barrier per row: the LDS
// slots alternate between two sets from row to row.
//
// HOLD form, one loop over the chunks per row with all of the row's memory traffic AND arithmetic in
// it: step c computes and stores chunk c of THIS row's gradient, refills the chunk's registers with
// chunk c of the workgroup's NEXT row, and adds chunk c - kLag of the next row (loaded kLag steps
// earlier) to that row's statistics.  A compute unit cannot queue a whole row of memory operations, so
// arithmetic outside this loop would run with the memory pipe idle.
#ifndef HBP_CE_LAG
#define HBP_CE_LAG 2
#endif
constexpr int kLag = HBP_CE_LAG;
constexpr int kRowBatch = kCeRowBatch;

// NT threads, by the length of a row (see launch_packed_ce).
template <int NT, int NCH, bool HOLD, bool WITH_GRAD>
__global__ __launch_bounds__(NT) void ce_main_kernel(const CeParams p) {
  constexpr int kCeChunk = NT * 8;  // logits covered by one load instruction of the workgroup
  constexpr int NW = NT / 64;
  __shared__ float slot_m[2][NW], slot_s[2][NW];
  const int tid = threadIdx.x;
  const u32x4 kNegInf = {0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};  // bf16 -inf pairs
  u32x4 held[HOLD ? NCH : 1];
  auto has_loss = [&](int label) { return label >= 0 && label < p.V; };  // an out-of-range label: no loss
  // HOLD: NCH = ceil(V / kCeChunk) exactly, so every chunk but the last has an entry for every thread
  // and the last one for the threads with tail_valid: which chunk needs a predicate is known at
  // compile time, and the chunk loops are straight-line code.
  const int last_chunk = HOLD ? NCH - 1 : (p.V + kCeChunk - 1) / kCeChunk - 1;
  const bool tail_valid = last_chunk * kCeChunk + tid * 8 < p.V;
  const int my_chunks = last_chunk + (tail_valid ? 1 : 0);
  const uint32_t byte_in_chunk = tid * 16;
  const uint32_t byte_in_tail = tail_valid ? byte_in_chunk : 0;  // a thread without an entry reads the chunk's first
  // The value again, opaque to the optimiser: keeps it from computing every chunk's predicate and
  // address ahead of the loops and holding them in registers the row needs.
  auto fresh = [](auto x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
    return x;
  };
  auto chunk_ptr = [&](const uint16_t* row, int c) {  // uniform base + one per-thread offset
    return (u32x4*)((char*)(row + c * kCeChunk) + fresh(byte_in_chunk));
  };
  // Unconditional for every thread (a predicated load would have to be waited for at once to merge it
  // with the "no entry" value): the partial chunk is masked where it is used, see entries().
  auto load_chunk = [&](const uint16_t* row, int c) {
    const uint32_t off = c == last_chunk ? byte_in_tail : byte_in_chunk;
    return __builtin_nontemporal_load((const u32x4*)((const char*)(row + c * kCeChunk) + fresh(off)));
  };
  auto entries = [&](const u32x4& v, int c) {  // the chunk as held, "no entry" = -inf
    u32x4 x = v;
    if (c == last_chunk) x = tail_valid ? v : kNegInf;
    return x;
  };

  // -inf stands for "no entry": its exponent offset is taken as 0 so that no inf - inf appears
  auto finite_or_zero = [](float m) { return m == -INFINITY ? 0.f : m; };
  // The instruction itself: fmaxf of unpacked bits costs another maximum an operand to quieten a NaN, 11 of a chunk's 58
  // instructions.  (A NaN among the entries makes the sum, and so the row's loss, a NaN whatever the maximum is.)
  auto max3 = [](float a, float b, float c) {
    float m = a;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
#endif
    return m;
  };
  // running (maximum, sum of exponentials) of this thread's entries, base 2 with log2(e) folded in
  float mx = -INFINITY, sm = 0.f;
  auto add_to_stats = [&](const u32x4& v) {
    float m_new = mx;
#pragma unroll
    for (int k = 0; k < 4; ++k) m_new = max3(m_new, bf16_lo(v[k]), bf16_hi(v[k]));
    const float m2 = finite_or_zero(m_new) * kLog2eF;
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a += __builtin_amdgcn_exp2f(__builtin_fmaf(bf16_lo(v[k]), kLog2eF, -m2));
      a += __builtin_amdgcn_exp2f(__builtin_fmaf(bf16_hi(v[k]), kLog2eF, -m2));
    }
    sm = sm * __builtin_amdgcn_exp2f(__builtin_fmaf(finite_or_zero(mx), kLog2eF, -m2)) + a;
    mx = m_new;
  };
  // The workgroup's rows.  With the gradient long rows are dealt in turn: of the rows with a loss every gridDim.x-th, and of
  // those without as well, beginning with the workgroups that have one row with a loss less.  The zeros of the latter are written
  // a share at a time in front of every other row's reduction, when nothing else is under way.  (Consecutive
  // rows a workgroup, cut by cost, lie all over the tensors, and a row without a loss between two with one leaves nothing to
  // read behind its zeros.  Plain copies of 8192 rows of 128256: 5.13 TB/s that way, 5.28 in turn; zeros alone 5.70.)
  // All zeros in front of the first row with a loss -> a share at a time, 30 % of the rows without, us: 8192 rows of 128256: 708
  // -> 693; 4096: 363 -> 352; 2048: 187 -> 180; 1000 of 32000: 26.8 -> 26.6; 300 of 65536: 21.1 -> 18.6.
  // Time of rows cut by cost / of dealt ones, T = 1000, 2500 and 8192, 0, 30 and 70 % of the rows without a loss:
  //   V = 1024, 2048        1.00 to 1.16       24576             1.06 to 1.18
  //       4096 to 8192       .81 to 1.10       32000              .99 to 1.24
  //       10240              .97 to 1.09       61440, 65536      1.00 to 1.23
  //       10248              .99 to 1.18       81920, 81928      1.02 to 1.28
  //       12288, 16384      1.04 to 1.26       90112 to 128256   1.03 to 1.16
  //       16392, 20480       .99 to 1.20       151936            1.04 to 1.29
  // (2.1 GB a tensor: with where in memory they lie.  8192 rows of 128256, 30 %, on four cards, us: 738 -> 707, 707 -> 693, 612
  // -> 646, 738 -> 696.)
  // Without the gradient consecutive rows, cut by cost, are as fast, and found sooner (300 of 128256: 14.9 against 16.0);
  // packs too long for ce_plan_rows have them as well, by ce_partition_kernel, and so have streamed rows (not measured).
  constexpr bool kDealt = ce_dealt(NT, NCH, HOLD, WITH_GRAD);
  //
  // Per-row scalars (label, weight, logit at the label; its number, where rows may be dealt) of the workgroup's next kRowBatch rows, staged
  // in LDS by one thread per row.  Read from global memory inside the row loop they would have to be
  // waited for with every outstanding store and load of the chunk pipeline (the counter is in order).
  __shared__ int row_index[kDealt ? kRowBatch : 1], row_label[kRowBatch];
  __shared__ float row_weight[kRowBatch], row_zlabel[kRowBatch];
  extern __shared__ uint64_t plan_lds[];
  __shared__ int plan_range[2], plan_slots[NW];
  CeRows rows;
  rows.live = plan_lds;
  rows.before = (int32_t*)(plan_lds + ce_plan_words(p.T) + 1);
  rows.cu = p.n_samples <= kCePlanCu ? rows.before + ce_plan_words(p.T) + 1 : nullptr;
  const int tokens = p.row_start ? 0 : ce_plan_rows<NT, !kDealt>(p, rows, tid, plan_range, plan_slots);
  // n rows, consecutive from `first`; or dealt: n with a loss and n_dead without.  The same in every thread and in
  // scalar registers.  Chosen by ?: it came from a load through
  // one pointer to either memory, whose result counts as different in every thread: a loop over rows by exec masks
  // and up to 10 more vector registers, of which the longest rows have none (20 chunks: a spill in the loop, whose
  // reload waits for the gradient stores; T = 8192, V = 160000: 933 -> 929 us).
  const bool dealt = kDealt && !p.row_start && (int)gridDim.x < p.T;
  int n, first, n_dead = 0, first_dead = 0;  // dealt: numbers of the first row of either kind among the rows of that kind
  if (p.row_start) {
    first = p.row_start[blockIdx.x];
    n = p.row_start[blockIdx.x + 1] - first;
  } else if (dealt) {
    const int G = gridDim.x, all_live = __builtin_amdgcn_readfirstlane(rows.before[ce_plan_words(p.T)]), all_dead = p.T - all_live;
    auto times = [G](int x) {  // x / G for x up to kCePlanRows: a division is 35 instructions
      const int q = (int)((float)x * __builtin_amdgcn_rcpf((float)G)), rest = x - q * G;
      return __builtin_amdgcn_readfirstlane(q + (rest >= G) - (rest < 0));
    };
    const int live = times(all_live), more_live = all_live - live * G, dead = times(all_dead), more_dead = all_dead - dead * G;
    first = blockIdx.x;
    first_dead = first - more_live + (first < more_live ? G : 0);
    n_dead = dead + (first_dead < more_dead);
    n = live + (first < more_live);
  } else if constexpr (kDealt) {  // a workgroup a row
    first = blockIdx.x;
    n = 1;
  } else {
    first = __builtin_amdgcn_readfirstlane(plan_range[0]);
    n = __builtin_amdgcn_readfirstlane(plan_range[1]) - first;
  }
  auto stage_rows = [&](int i0) {  // entries i0 + i, i < kRowBatch
    __syncthreads();                // the entries of the batch before have all been read
    if (tid < kRowBatch) {
      const int i = i0 + tid;
      int row = first + i, lab = -1;
      float wt = 0.f, zl = 0.f;
      if (i < n) {
        if (dealt) row = ce_nth_row(rows, ce_plan_words(p.T), first + i * (int)gridDim.x, true);
        lab = p.labels[row];
        if (has_loss(lab)) {
          wt = p.row_start ? p.weighted[row]  // the row's weight, put there by ce_weight_kernel
                           : ce_row_weight(p, rows, row, tokens);
          zl = __uint_as_float((uint32_t)p.logits[(int64_t)row * p.stride_t + lab] << 16);
        } else {
          lab = -1;
          if (HOLD && !WITH_GRAD) p.token_loss[row] = p.weighted[row] = 0.f;
        }
      }
      if (kDealt) row_index[tid] = row;
      row_label[tid] = lab;
      row_weight[tid] = wt;
      row_zlabel[tid] = zl;
    }
    __syncthreads();
  };
  // Dealt rows without a loss: their numbers, kRowBatch at a time, and their zeros, so many chunks at a time.
  __shared__ int dead_index[kDealt ? kRowBatch : 1];
  auto stage_dead = [&](int i0) {
    if (tid < kRowBatch && i0 + tid < n_dead) {
      const int row = ce_nth_row(rows, ce_plan_words(p.T), first_dead + (i0 + tid) * (int)gridDim.x, false);
      dead_index[tid] = row;
      p.token_loss[row] = p.weighted[row] = 0.f;
    }
    __syncthreads();
  };
  int zero_row = 0, zero_chunk = 0, zero_rows = 0;  // the next one to write, and how many rows there are
  auto write_zeros = [&](int chunks) {
    for (; chunks > 0 && zero_row < zero_rows; --chunks) {
      uint16_t* row = p.dlogits + (int64_t)__builtin_amdgcn_readfirstlane(dead_index[zero_row]) * p.V;
      if (zero_chunk < NCH - 1 || tail_valid) __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, chunk_ptr(row, zero_chunk));
      if (++zero_chunk == NCH) {
        zero_chunk = 0;
        ++zero_row;
      }
    }
  };
  int zeros_a_row = 0;  // chunks of zeros beside every row with a loss
  if constexpr (kDealt) {
    if (dealt) {
      for (int i0 = (n_dead - 1) / kRowBatch * kRowBatch; i0 >= 0 && n_dead > 0; i0 -= kRowBatch) {
        stage_dead(i0);
        zero_row = zero_chunk = 0;
        zero_rows = min(n_dead - i0, kRowBatch);
        if (i0 > 0 || n <= 0) {
          write_zeros(kRowBatch * NCH);
          __syncthreads();
        }
      }
      zeros_a_row = n > 0 ? (zero_rows * NCH + n - 1) / n : 0;
    }
  }
  if (n <= 0) return;
  // log2-sum-exp2 of a row from every thread's statistics; one barrier.  parity: which set of the slots
  auto row_lse2 = [&](int parity) {
    const float m_wave = wave_max(mx);
    sm *= __builtin_amdgcn_exp2f((finite_or_zero(mx) - finite_or_zero(m_wave)) * kLog2eF);
    sm = wave_sum(sm);
    if ((tid & 63) == 0) {
      slot_m[parity][tid >> 6] = m_wave;
      slot_s[parity][tid >> 6] = sm;
    }
    __syncthreads();
    float m_row = slot_m[parity][0];
#pragma unroll
    for (int i = 1; i < NW; ++i) m_row = fmaxf(m_row, slot_m[parity][i]);
    const float m_row0 = finite_or_zero(m_row);
    float s_row = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i)
      s_row += slot_s[parity][i] * __builtin_amdgcn_exp2f((finite_or_zero(slot_m[parity][i]) - m_row0) * kLog2eF);
    return m_row0 * kLog2eF + __builtin_amdgcn_logf(s_row);
  };
  if constexpr (HOLD && !WITH_GRAD) {
    // HBM-bound, reads alone.  A chunk is done with once it is in the statistics, so its registers take the same chunk of
    // the next row that has a loss at once: a whole row is always under way, over the reduction and over rows without a
    // loss too.  (The loop below waits for each load kLag chunks later, which is enough between the gradient's stores:
    // with it T = 4096, V = 151936, 30 % of the rows without a loss: 169 us, 5.1 TB/s; this way 146, 5.9.  V = 128256:
    // 146 -> 124; 65536: 79 -> 68; 50304: 66 -> 54; 32000: 40.6 -> 38.0; 4096: 17.9 -> 14.0; T = 1000, V = 65536: 30 -> 23.)
    // through a descriptor of the row: no address arithmetic for the vector unit, and the last chunk needs no clamp (the
    // offset opaque, or the compiler moves a load from the iteration before to its use)
    auto load_in_row = [&](int row, int c) {
      const auto src = __builtin_amdgcn_make_buffer_rsrc((void*)(p.logits + (int64_t)row * p.stride_t), 0, 2 * p.V, 0x00020000);
      return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, fresh(byte_in_chunk), c * 2 * kCeChunk, 2 /* nt */));
    };
    for (int i0 = 0, parity = 0; i0 < n; i0 += kRowBatch) {
      stage_rows(i0);
      const int base = first + i0, count = min(n - i0, kRowBatch);
      auto next_live = [&](int i) {  // the first row from i on with a loss; count: none
        while (i < count && row_label[i] < 0) ++i;
        return __builtin_amdgcn_readfirstlane(i);
      };
      int i = next_live(0);
      if (i == count) continue;
#pragma unroll
      for (int c = 0; c < NCH; ++c) held[c] = load_in_row(base + i, c);
      while (i < count) {
        const int i_next = next_live(i + 1);
        if (i_next < count) {
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            add_to_stats(entries(held[c], c));
            held[c] = load_in_row(base + i_next, c);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          // opaque: what both sides compute from a chunk is otherwise moved in front of the branch, for all chunks, with
          // registers that are not there
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            add_to_stats(entries(fresh(held[c]), c));
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        const float ce = row_lse2(parity) * kLn2F - row_zlabel[i];
        if (tid == 0) {
          p.token_loss[base + i] = ce;
          p.weighted[base + i] = row_weight[i] * ce;
        }
        parity ^= 1;
        mx = -INFINITY;
        sm = 0.f;
        i = i_next;
      }
    }
    return;
  }
  stage_rows(0);
  int r = kDealt ? __builtin_amdgcn_readfirstlane(row_index[0]) : first;
  int label = row_label[0];  // -1: no loss
  float w = row_weight[0], z_label = row_zlabel[0];
  if (HOLD && label >= 0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) held[c] = load_chunk(p.logits + (int64_t)r * p.stride_t, c);
    if constexpr (kDealt) write_zeros(zeros_a_row);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      add_to_stats(entries(held[c], c));
      __builtin_amdgcn_sched_barrier(0);  // one chunk at a time: bounds the temporaries
    }
  }
  for (int parity = 0, i_next = 1; i_next <= n; ++i_next) {
    if (i_next % kRowBatch == 0 && i_next < n) stage_rows(i_next);
    const int r_next = kDealt ? __builtin_amdgcn_readfirstlane(row_index[i_next % kRowBatch]) : r + 1;
    const int label_next = i_next < n ? row_label[i_next % kRowBatch] : -1;
    const float w_next = row_weight[i_next % kRowBatch], z_label_next = row_zlabel[i_next % kRowBatch];
    const bool fetch_next = HOLD && label_next >= 0;
    const bool live = label >= 0;  // a row without a loss: zero loss, zero gradient, no arithmetic
    const uint16_t* row = p.logits + (int64_t)r * p.stride_t;
    const uint16_t* row_next = p.logits + (int64_t)r_next * p.stride_t;
    uint16_t* grow = WITH_GRAD ? p.dlogits + (int64_t)r * p.V : nullptr;
    float lse2w = 0.f;
    if (live) {
      if (!HOLD) {
        for (int c = 0; c < my_chunks; ++c) add_to_stats(*chunk_ptr(row, c));
      }
      if constexpr (kDealt) {
        if (i_next > 1) write_zeros(zeros_a_row);
      }
      const float lse2 = row_lse2(parity);
      const float ce = lse2 * kLn2F - z_label;
      lse2w = lse2 - __builtin_amdgcn_logf(w);  // w exp2(x - lse2) = exp2(x - lse2w)
      if (tid == 0) {
        p.token_loss[r] = ce;
        p.weighted[r] = w * ce;
      }
      parity ^= 1;  // per row WITH a barrier: a set is written again only after the barrier of the row between
    } else if (tid == 0) {
      p.token_loss[r] = 0.f;
      p.weighted[r] = 0.f;
    }
    mx = -INFINITY;  // from here on: the statistics of the next row
    sm = 0.f;
    // gradient w (softmax - onehot): the one entry at the label is patched in by the thread that holds it
    const int label_chunk = label / kCeChunk, label_tid = (label % kCeChunk) >> 3;
    auto chunk_grad = [&](const u32x4& v, int c) {  // zeros for a row without a loss
      u32x4 g = {0, 0, 0, 0};
      if (live) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          g[k] = pack_bf16(__builtin_amdgcn_exp2f(__builtin_fmaf(bf16_lo(v[k]), kLog2eF, -lse2w)),
                           __builtin_amdgcn_exp2f(__builtin_fmaf(bf16_hi(v[k]), kLog2eF, -lse2w)));
        if (c == label_chunk && tid == label_tid) {
          const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(z_label, kLog2eF, -lse2w)) - w;
          const uint32_t bits = pack_bf16(a, 0.f) & 0xffffu;
          const int k_label = (label >> 1) & 3;
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k == k_label) g[k] = (label & 1) ? (g[k] & 0xffffu) | (bits << 16) : (g[k] & 0xffff0000u) | bits;
        }
      }
      return g;
    };
    if (HOLD) {
      // the only place (after the first row) where the held registers are written
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        // No store or load of this loop sits in a branch on a uniform condition (the arithmetic does):
        // with one there the compiler waits for ALL outstanding memory operations at every use of a
        // loaded chunk instead of for that chunk's load.
        const u32x4 g = chunk_grad(held[c], c);
        if (c < NCH - 1) __builtin_nontemporal_store(g, chunk_ptr(grow, c));
        else if (tail_valid) __builtin_nontemporal_store(g, chunk_ptr(grow, c));
        if (fetch_next) {
          held[c] = load_chunk(row_next, c);
          if (c >= kLag) add_to_stats(entries(held[c - kLag], c - kLag));
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the refill behind the store: hoisted loads would need a second set of registers
      }
      if (fetch_next) {
#pragma unroll
        for (int c = NCH > kLag ? NCH - kLag : 0; c < NCH; ++c) {
          add_to_stats(entries(held[c], c));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else if (WITH_GRAD) {
      for (int c = 0; c < my_chunks; ++c) __builtin_nontemporal_store(chunk_grad(*chunk_ptr(row, c), c), chunk_ptr(grow, c));
    }
    r = r_next;
    label = label_next;
    w = w_next;
    z_label = z_label_next;
  }
}

// loss = sum of the weighted token losses, fixed order
__global__ __launch_bounds__(kCeThreads) void ce_reduce_kernel(const CeParams p) {
  __shared__ float slots[kCeThreads / 64];
  const int tid = threadIdx.x;
  float acc = 0.f;
  for (int r = tid; r < p.T; r += kCeThreads) acc += p.weighted[r];
  acc = block_reduce<false>(acc, slots, tid);
  if (tid == 0) *p.loss_out = acc;
}

// Workgroups resident at once per compute unit.  The main kernel's grid is that times the compute
// units: a persistent loop over rows; a second batch of workgroups would start with an empty pipeline.
template <int NT, int NCH, bool HOLD, bool WITH_GRAD>
static int main_per_cu(int plan_lds) {
  static int by_registers = 0;  // without the planning's LDS; same on every device of this part
  if (by_registers == 0) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, ce_main_kernel<NT, NCH, HOLD, WITH_GRAD>, NT, 0) != hipSuccess || n < 1) n = 1;
    by_registers = n;
  }
  return ce_per_cu(by_registers, NT, NCH, HOLD, WITH_GRAD, plan_lds);
}
template <int NT, int NCH, bool HOLD, bool WITH_GRAD>
static void launch_main_g(CeParams p, int n_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const bool planned = p.T > kCePlanRows;
  const int lds = planned ? 0 : ce_plan_lds(p.T, p.n_samples);
  int64_t grid = (int64_t)main_per_cu<NT, NCH, HOLD, WITH_GRAD>(lds) * n_cu;
  if (grid > kCeMaxWorkgroups) grid = kCeMaxWorkgroups;
  if (grid > p.T) grid = p.T;
  if (planned) {
    hipLaunchKernelGGL(ce_count_kernel, dim3(p.n_samples), dim3(256), 0, s, p);
    hipLaunchKernelGGL(ce_weight_kernel, dim3(p.n_samples), dim3(256), 0, s, p);
    hipLaunchKernelGGL(ce_partition_kernel, dim3(1), dim3(kCeThreads), 0, s, p, (int)grid);
  } else {
    p.row_start = nullptr;
  }
  if (ev0) (void)hipEventRecord(ev0, s);
  hipLaunchKernelGGL((ce_main_kernel<NT, NCH, HOLD, WITH_GRAD>), dim3((unsigned)grid), dim3(NT), lds, s, p);
  if (ev1) (void)hipEventRecord(ev1, s);
}
template <int NT, int NCH, bool HOLD>
static void launch_main(const CeParams& p, int n_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (p.dlogits) launch_main_g<NT, NCH, HOLD, true>(p, n_cu, s, ev0, ev1);
  else launch_main_g<NT, NCH, HOLD, false>(p, n_cu, s, ev0, ev1);
}
// rows of LO to HI chunks of NT * 8 entries
template <int NT, int LO, int HI>
static bool launch_held(const CeParams& p, int n_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  switch ((p.V + NT * 8 - 1) / (NT * 8)) {
#define HBP_CE_HELD(N) case N: if constexpr (N >= LO && N <= HI) { launch_main<NT, N, true>(p, n_cu, s, ev0, ev1); return true; } return false;
    HBP_CE_HELD(1) HBP_CE_HELD(2) HBP_CE_HELD(3) HBP_CE_HELD(4) HBP_CE_HELD(5)
    HBP_CE_HELD(6) HBP_CE_HELD(7) HBP_CE_HELD(8) HBP_CE_HELD(9) HBP_CE_HELD(10)
    HBP_CE_HELD(11) HBP_CE_HELD(12) HBP_CE_HELD(13) HBP_CE_HELD(14) HBP_CE_HELD(15)
    HBP_CE_HELD(16) HBP_CE_HELD(17) HBP_CE_HELD(18) HBP_CE_HELD(19) HBP_CE_HELD(20)
#undef HBP_CE_HELD
    default: return false;
  }
}

// Threads a row.  A row costs its workgroup one reduction and one barrier whatever its length, with nothing
// else to run on the compute unit if the workgroup fills it; several smaller workgroups overlap theirs.  A
// longer row has to be spread over more threads to be held.  us at T = 8192 with the gradient, 30 % of the rows without a
// loss / without the gradient:
//   V        1024 threads   512          256
//   4096      62 /  41       43 /  27     36 /  22
//   16384    113 /  50       90 /  42     93 /  43
//   20480    132            114          117
//   32000    178 /  70      172 /  68    182 /  72
//   65536    349 / 130      356 / 130
//   81920    437 / 156      446 / 157
// With few rows, T = 64 / 1000 with the gradient:
//   4096      9.1 / 15.9     8.3 / 12.0     8.3 / 9.9
//   16384     9.6 / 24.0     9.0 / 17.7     8.9 / 16.3
//   20480    10.3 / 26.8     9.2 / 19.5     9.7 / 19.6
//   32000    10.7 / 29.5    10.0 / 24.8    10.9 / 28.7
// Few (up to two rows a compute unit, so that workgroups of 512 threads have a row each): 1024 threads have half the chain
// a row, as long as no more rows than compute units have a loss; with more of them some units have two rows after one
// another.  T = 280 / 512 with the gradient, 30 % of the rows without a loss, 1024 threads and 512: V = 65536: 18.2 / 27.6
// and 20.2 / 28.5; 81920: 21.2 / 33.7 and 25.8 / 34.6.  All with a loss: 25.7 / 29.5 and 18.8 / 24.1; 29.8 / 35.0 and 21.8 /
// 30.3.  The host does not know how many have one.  Up to 256 rows, V = 65536 to 81920, 512 threads are 0 to 3 % faster;
// V = 45056 to 61440: 1024 threads 3 to 7 % slower, T = 280: 5 % faster with 30 % without a loss, 27 % slower with none.
// Without the gradient both have one workgroup a compute unit and 512 threads are 0 to 3 % faster; the line is the same, so
// the losses are the same bits.
constexpr int kCeRow256 = 16384, kCeRow512 = 81920, kCeRow512Few = 61440;  // Few: a row a workgroup at most

int launch_packed_ce(const CeParams& p, int n_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (p.T > 0) {
    const int row512 = p.T <= 2 * n_cu ? kCeRow512Few : kCeRow512;
    if (p.V <= kCeRow256) (void)launch_held<256, 1, kCeRow256 / 2048>(p, n_cu, s, ev0, ev1);
    else if (p.V <= row512) (void)launch_held<512, kCeRow256 / 4096 + 1, kCeRow512 / 4096>(p, n_cu, s, ev0, ev1);
    else if (!launch_held<1024, kCeRow512Few / 8192 + 1, 20>(p, n_cu, s, ev0, ev1)) launch_main<1024, 1, false>(p, n_cu, s, ev0, ev1);
  }
  hipLaunchKernelGGL(ce_reduce_kernel, dim3(1), dim3(kCeThreads), 0, s, p);
  return (int)hipGetLastError();
}

}  // namespace hbp
