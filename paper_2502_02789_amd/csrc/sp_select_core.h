// Pieces of the chunk selection shared by sp_select.hip and the fused short-prompt kernel
// (sp_fused.hip): the kernel-side argument view, the order-preserving keys, and the single-sequence
// top-k + compaction done by one workgroup (Sec. 3.2.3 of arXiv 2502.02789: Top-K chunks, keep
// rate = ratio of chunks; equal scores go to the lower chunk index).
#pragma once

// the k formula below must stay a separate multiply and subtract (for every includer)
#pragma clang fp contract(off)

#include "sp_common.h"

namespace sp {

struct SelDev {
  int B;
  int T;
  int chunk, radius;
  double keep_rate;
  int64_t capacity;
  const int32_t* cu;
  const float* scores;
  int32_t* kept_idx;
  int32_t* cu_keep;
  float* chunk_scores_out;
  int table;            // the chunks are numbered without gaps by cu_chunks (the caller wants their scores)
  int32_t* cu_chunks;   // [B+1]
  int32_t* arrived;     // no table: sequences selected so far
  int32_t* seq_keep;    // [B]
  double* cs;           // [max_chunks]
  int32_t* chunk_off;   // [max_chunks]: rank of the chunk among its sequence's kept ones, or -1
  int n_chunks;         // one sequence: its chunks
};

// chunks of m tokens (a chunk may be as long as an int holds: the sum fits 32 bits without a sign, and no
// more; a test for m > 0 and a division of m - 1 instead made the selection of a batch 0.25 us longer)
__device__ __forceinline__ int chunk_count(int m, int chunk) { return (int)(((uint32_t)m + (uint32_t)chunk - 1u) / (uint32_t)chunk); }

// NaN, decided on the bit pattern (device code is compiled on the assumption that there are none)
__device__ __forceinline__ bool is_nan_bits(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  return (u & 0x7ff0000000000000ull) == 0x7ff0000000000000ull && (u & 0x000fffffffffffffull) != 0;
}

// monotone map double -> uint64 (larger value <-> larger key)
__device__ __forceinline__ uint64_t order_key(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Inclusive prefix sum over the 64 lanes of a wave; *total gets the wave's sum.  Inside each row
// of 16 lanes by DPP row shifts (lanes shifted in from outside the row contribute zero), the
// three row totals that lie below a lane through scalar registers: no LDS round trips.
__device__ __forceinline__ int wave_inclusive_scan(int v, int* total) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31);
  const int r2 = __builtin_amdgcn_readlane(v, 47), r3 = __builtin_amdgcn_readlane(v, 63);
  const int lane = threadIdx.x & 63;
  *total = r0 + r1 + r2 + r3;
  return v + (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
}

// The bucket holding the need-th largest of the keys still in play: the highest bucket whose
// count, added to the counts above it, reaches `need`.  Done by a whole wave (four buckets per
// lane, suffix sums by shuffles); every lane gets the bucket, how many keys of that bucket are
// still needed, and whether that is all of them.
__device__ __forceinline__ void find_bucket(const int* hist, int need, int* bucket_out, int* need_left, bool* all_of_it) {
  const int lane = threadIdx.x & 63;
  int h[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) h[u] = hist[4 * lane + u];
  const int own = h[0] + h[1] + h[2] + h[3];
  int all;
  const int upto = wave_inclusive_scan(own, &all);
  const int suffix = all - upto + own;  // counts of this lane's buckets and of all higher lanes'
  int above = suffix - own;
  int bucket = -1, left = 0, size = 0;
  if (above < need && need <= suffix) {  // exactly one lane: the keys still in play number at least `need`
    bucket = 4 * lane;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      if (above + h[u] >= need) { bucket = 4 * lane + u; size = h[u]; break; }
      above += h[u];
    }
    left = need - above;
  }
  const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)__ballot(bucket >= 0)) - 1);
  *bucket_out = __builtin_amdgcn_readlane(bucket, src);
  *need_left = __builtin_amdgcn_readlane(left, src);
  *all_of_it = __builtin_amdgcn_readlane(size, src) == *need_left;
}

// Chunks of a sequence in registers: wave w of the workgroup's sixteen owns chunks [w * 64 I, (w + 1) * 64 I), lane x of it
// chunk (w * I + i) * 64 + x as key[i].  (Re-reading the scores in every pass, a thread at a time in index order, made
// the selection of 9000 single tokens 71 us, nearly all of it memory latency.)
template <int I>
__device__ __forceinline__ int reg_chunk(int i) {
  return ((int)(threadIdx.x >> 6) * I + i) * 64 + (int)(threadIdx.x & 63);
}

// The k best of n chunks (scores cs[0..n), equal scores to the lower index) by one workgroup of 1024 threads:
// emit(j, rank) for every kept chunk j, the rank-th of them in index order, emit(j, -1) for the others; returns
// the number of kept chunks (*last_kept: chunk n - 1 among them), or -1 if a score is NaN (nothing is emitted then).
//
// The k-th largest key by counting in classes of equal width between the smallest and the largest key (their
// upper halves): the class that holds it is counted again in narrower classes until all of it is kept, all its keys are
// equal, or it has no more than 64 chunks, which are ranked among themselves -- after one or two passes as a rule.
// (Digits of eight fixed bits took three passes, the first of them with nearly all keys in one or two counters, whose
// additions LDS performs one after the other.  Whole selection, window 1, single tokens: eight sequences of 8000 29.2 -> 22.2 us,
// of 16000 36.1 -> 23.9, one of 2000 10.6 -> 7.6; 1024 and 2048 smoothed chunks of one sequence, a twentieth kept 9.2 -> 8.5 and
// 10.1 -> 9.4, three tenths 10.7 -> 9.9 and 12.8 -> 11.5, half 11.8 -> 10.9 and 15.7 -> 13.7.  Ranking up to 128 chunks
// took longer than the second pass.)
// `hist` has room for kSelectHist counters, `sh` for 48.
constexpr int kSelectHist = 1024 + 64;
// the least (MAX: the largest) of a wave's values
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  auto pick = [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return MAX ? max(a, b) : min(a, b); };
  v = pick(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));   // lane ^ 1, lane ^ 2 in the quad,
  v = pick(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));
  v = pick(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));  // the mirrored half row and row
  v = pick(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true));
  const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
  const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
  return pick(pick(a, b), pick(c, d));
}
template <int I, typename Emit>
__device__ __forceinline__ int select_chunks(const double* cs, int n, int k, int* hist, int* sh, bool* last_kept, Emit emit) {
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  // classes (a lane sums PER of them: a gap behind every PER)
  constexpr int LG_BINS = I <= 2 ? 9 : 10, BINS = 1 << LG_BINS, PER = BINS / 64;
  __shared__ uint64_t few_key[64], kth_sh;
  __shared__ int few_chunk[64], few, kth_chunk_sh;
  uint64_t key[I];
  int bad = 0;
  uint32_t least = ~0u, most = 0u;
  const uint64_t last_key = order_key(cs[n - 1]);
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = reg_chunk<I>(i);
    double v = 0.0;
    if (j < n) v = cs[j];
    bad |= is_nan_bits(v) ? 1 : 0;
    key[i] = order_key(v);
    const uint32_t top = (uint32_t)(key[i] >> 32);
    least = min(least, j < n ? top : ~0u);
    most = max(most, j < n ? top : 0u);
  }
  least = wave_extreme<false>(least);
  most = wave_extreme<true>(most);
  const int bad_wave = __ballot(bad != 0) != 0 ? 1 : 0;
  if (lane == 0) { sh[wave] = (int)least; sh[16 + wave] = (int)most; sh[32 + wave] = bad_wave; }
  if (t == 0) few = 0;
  for (int x = t; x < BINS + 64; x += 1024) hist[x] = 0;  // (for the first pass)
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    least = min(least, (uint32_t)sh[w]);
    most = max(most, (uint32_t)sh[16 + w]);
    bad |= sh[32 + w];
  }
  if (bad) return -1;  // (the same for all threads)

  // keys in play: lo .. lo + span; the k-th largest of all is the need-th largest of them
  uint64_t lo = (uint64_t)least << 32, span = ((uint64_t)(most - least) << 32) | 0xffffffffull;
  int shift = 64 - LG_BINS - __clzll((long long)span), need = k;
  // kept: key > kth, or == kth and the chunk no later than kth_chunk
  uint64_t kth;
  int kth_chunk = 0x7fffffff;
#pragma unroll 1
  for (;;) {
#pragma unroll
    for (int i = 0; i < I; ++i)
      if (reg_chunk<I>(i) < n && key[i] - lo <= span) {
        const int bin = (int)((key[i] - lo) >> shift);
        atomicAdd(&hist[bin + bin / PER], 1);
      }
    __syncthreads();
    // every wave finds the class by itself, lane x looking at the classes [BINS - PER (x + 1), BINS - PER x)
    const int group = 63 - lane;
    int h[PER], own = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) own += h[u] = hist[(PER + 1) * group + u];
    int all;
    const int upto = wave_inclusive_scan(own, &all);
    int above = upto - own, bin = -1, size = 0;
    if (above < need && need <= upto) {  // exactly one lane
#pragma unroll
      for (int u = PER - 1; u >= 0; --u) {
        if (bin < 0 && above + h[u] >= need) { bin = PER * group + u; size = h[u]; }
        if (bin < 0) above += h[u];
      }
    }
    const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)__ballot(bin >= 0)) - 1);
    need -= __builtin_amdgcn_readlane(above, src);
    size = __builtin_amdgcn_readlane(size, src);
    lo += (uint64_t)__builtin_amdgcn_readlane(bin, src) << shift;
    span = (1ull << shift) - 1;
    kth = lo;
    if (size == need) break;
    if (shift == 0) {
      // equal keys, of which the first `need` are kept: the last of those
      int equal = 0;
#pragma unroll
      for (int i = 0; i < I; ++i) equal += __popcll(__ballot(reg_chunk<I>(i) < n && key[i] == kth));
      if (lane == 0) sh[wave] = equal;
      __syncthreads();
      int before = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w)
        if (w < wave) before += sh[w];
#pragma unroll
      for (int i = 0; i < I; ++i) {
        const bool eq = reg_chunk<I>(i) < n && key[i] == kth;
        const unsigned long long mask = __ballot(eq);
        if (eq && before + __popcll(mask & ((1ull << lane) - 1ull)) == need - 1) kth_chunk_sh = reg_chunk<I>(i);
        before += __popcll(mask);
      }
      __syncthreads();
      kth_chunk = kth_chunk_sh;
      break;
    }
    if (size <= 64) {
#pragma unroll
      for (int i = 0; i < I; ++i)
        if (reg_chunk<I>(i) < n && key[i] - lo <= span) {
          const int at = atomicAdd(&few, 1);
          few_key[at] = key[i];
          few_chunk[at] = reg_chunk<I>(i);
        }
      __syncthreads();
      // A wave ranks four of them: lane x holds the x-th, a ballot finds those ahead.  (Every wave all of them for itself, a
      // key's index read behind the comparison of the keys, was a chain of two LDS round trips a chunk: 768 smoothed
      // chunks with 50 left to rank 13.3 us, 9.1 this way; by digits 10.0.)
      const uint64_t mine = few_key[lane];
      const int chunk = few_chunk[lane];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int x = wave * 4 + u;
        const uint64_t other = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), x) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)mine, x);
        const int other_chunk = __builtin_amdgcn_readlane(chunk, x);
        const bool ahead = (int)(lane < size) & ((int)(mine > other) | ((int)(mine == other) & (int)(chunk < other_chunk)));
        if (x < size && __popcll(__ballot(ahead)) == need - 1 && lane == 0) { kth_sh = other; kth_chunk_sh = other_chunk; }
      }
      __syncthreads();
      kth = kth_sh;
      kth_chunk = kth_chunk_sh;
      break;
    }
    shift = max(0, shift - LG_BINS);
    __syncthreads();
    for (int x = t; x < BINS + 64; x += 1024) hist[x] = 0;
    __syncthreads();
  }

  // in index order: rows of 64 chunks by ballots, the waves' totals through LDS
  int kept = 0;
  unsigned long long mask[I];
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = reg_chunk<I>(i);
    mask[i] = __ballot(j < n && (key[i] > kth || (key[i] == kth && j <= kth_chunk)));
    kept += __popcll(mask[i]);
  }
  if (lane == 0) sh[32 + wave] = kept;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int x = sh[32 + w];
    if (w < wave) before += x;
    total += x;
  }
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = reg_chunk<I>(i);
    const bool keep = (mask[i] >> lane) & 1ull;
    if (j < n) emit(j, keep ? before + __popcll(mask[i] & below) : -1);
    before += __popcll(mask[i]);
  }
  *last_kept = last_key > kth || (last_key == kth && n - 1 <= kth_chunk);
  return total;
}

// Single sequence with at most kSingleMaxChunks chunks: top-k, compaction and the kept-index
// list in one workgroup and one launch; kept tokens are written straight away.  The forms of the ranking: by one wave, a
// chunk a lane; by counting, four threads a chunk; by classes as in select_kernel.  The host knows the number of chunks, so
// a kernel has the code of one form only (all three in one: 0.2 us more for fetching instructions in between).
constexpr int kSingleMaxChunks = 2048;
constexpr int kWaveMaxChunks = 64, kCountMaxChunks = 256;
enum SingleForm { kRankByWave, kRankByCount, kRankByClasses };
inline SingleForm single_form(int64_t n_chunks) {
  return n_chunks <= kWaveMaxChunks ? kRankByWave : n_chunks <= kCountMaxChunks ? kRankByCount : kRankByClasses;
}
// `cs`: the chunk scores (global or LDS memory); `keys`: LDS room for kSingleMaxChunks 64-bit keys.
// Call with all 1024 threads of the workgroup.
template <SingleForm FORM>
__device__ __forceinline__ void select_emit_single(const SelDev& p, const double* cs, uint64_t* keys) {
  const int t = threadIdx.x;
  const int M = p.T;
  const int n = p.n_chunks;
  if (t == 0) p.cu_keep[0] = 0;
  if (n == 0) {
    if (t == 0) p.cu_keep[1] = 0;
    return;
  }
  const double scaled = p.keep_rate * (double)n;
  const double kd = ceil(scaled - 1e-9);
  const int k = (int)fmin((double)n, fmax(1.0, kd));
  // All kept chunks but possibly the very last are full: kept chunk number q starts at token q * chunk of the list.
  __shared__ unsigned short kept_list[kSingleMaxChunks];
  bool last_kept;
  int kept_chunks;
  if constexpr (FORM == kRankByWave) {
    // One wave ranks a chunk a lane and writes the list: one barrier, where the counting form has four.  (Chunks of 32, pooling
    // included, counting form and this one: 100 tokens 4.6 and 3.5 us, 1000 5.4 and 4.6, 64 chunks 6.4 and 6.2; the single-launch
    // kernel with a gather behind it: 100 tokens 14.4 and 13.5, 500 16.4 and 15.4; with the two barriers of a thread a chunk
    // in whole workgroups 14.1 and 16.1.)
    __shared__ int verdict;  // -1: invalid scores; else whether chunk n - 1 is kept
    if (t < 64) {
      const double v = t < n ? cs[t] : 0.0;
      const uint64_t mine = order_key(v);
      keys[t] = mine;
      const bool bad = __ballot(is_nan_bits(v)) != 0;
      int ahead = 0;
#pragma unroll 8
      for (int j = 0; j < n; ++j) {
        const uint64_t other = keys[j];
        ahead += (other > mine || (other == mine && j < t)) ? 1 : 0;
      }
      const uint64_t kept = __ballot(t < n && ahead < k);
      if ((kept >> t) & 1ull) kept_list[__popcll(kept & ((1ull << t) - 1ull))] = (unsigned short)t;
      if (t == 0) verdict = bad ? -1 : (int)((kept >> (n - 1)) & 1ull);
    }
    __syncthreads();
    if (verdict < 0) {  // reported in band, nothing kept
      if (t == 0) p.cu_keep[1] = -1;
      return;
    }
    kept_chunks = k;
    last_kept = verdict != 0;
  } else if constexpr (FORM == kRankByCount) {
    // Few chunks: a chunk is ranked by counting the chunks that come before it in the order (larger score, or equal score
    // and lower index), four threads a chunk, each a quarter of the others; the k first are kept.  (256 chunks of 32
    // tokens, pooling included: 15.6 us with a thread per chunk and every token looked at, 8.7 now.)
    __shared__ uint64_t kept_mask[kCountMaxChunks / 64];
    __shared__ unsigned char ahead[4][kCountMaxChunks];
    __shared__ int bad_wave[kCountMaxChunks / 64];
    if (t < kCountMaxChunks) {
      const double v = t < n ? cs[t] : 0.0;
      const bool bad = __ballot(is_nan_bits(v)) != 0;
      if ((t & 63) == 0) bad_wave[t >> 6] = bad ? 1 : 0;
      keys[t] = order_key(v);
    }
    __syncthreads();
    int bad = 0;
    for (int x = 0; x < kCountMaxChunks / 64; ++x) bad |= bad_wave[x];
    if (bad) {  // invalid scores: reported in band, nothing kept
      if (t == 0) p.cu_keep[1] = -1;
      return;
    }
    {
      const int c = t % kCountMaxChunks, quarter = t / kCountMaxChunks, per = (n + 3) / 4;
      const uint64_t mine = c < n ? keys[c] : 0;
      int count = 0;
#pragma unroll 8
      for (int j = quarter * per; j < min(n, (quarter + 1) * per); ++j) {
        const uint64_t other = keys[j];
        count += (other > mine || (other == mine && j < c)) ? 1 : 0;
      }
      ahead[quarter][c] = (unsigned char)count;
    }
    __syncthreads();
    const bool keep = t < n && ahead[0][t] + ahead[1][t] + ahead[2][t] + ahead[3][t] < k;
    const uint64_t ballot = __ballot(keep);
    if (t < kCountMaxChunks && (t & 63) == 0) kept_mask[t >> 6] = ballot;
    __syncthreads();
    kept_chunks = 0;
    for (int x = 0; x < kCountMaxChunks / 64; ++x) {
      if (keep && x == t >> 6) kept_list[kept_chunks + __popcll(ballot & ((1ull << (t & 63)) - 1ull))] = (unsigned short)t;
      kept_chunks += __popcll(kept_mask[x]);
    }
    last_kept = (kept_mask[(n - 1) >> 6] >> ((n - 1) & 63)) & 1ull;
  } else {
    __shared__ int hist[kSelectHist];
    __shared__ int sh[48];
    auto emit = [&](int j, int rank) __attribute__((always_inline)) {
      if (rank >= 0) kept_list[rank] = (unsigned short)j;
    };
    kept_chunks = n <= 1024 ? select_chunks<1>(cs, n, k, hist, sh, &last_kept, emit) : select_chunks<2>(cs, n, k, hist, sh, &last_kept, emit);
    if (kept_chunks < 0) {
      if (t == 0) p.cu_keep[1] = -1;
      return;
    }
  }
  const int64_t total_tokens = (int64_t)kept_chunks * p.chunk - (last_kept ? (int64_t)n * p.chunk - M : 0);
  if constexpr (FORM != kRankByWave) __syncthreads();
  // the kept tokens are written by all threads, a token each
  const uint32_t n_write = (uint32_t)min(total_tokens, p.capacity), chunk = (uint32_t)p.chunk;
  for (uint32_t pos = t; pos < n_write; pos += 1024) {
    const uint32_t q = pos / chunk;
    p.kept_idx[pos] = (int)(kept_list[q] * chunk + (pos - q * chunk));
  }
  if (t == 0) p.cu_keep[1] = (int32_t)total_tokens;
}

// Pooling and chunk means of one sequence whose scores are in LDS, by one workgroup of 1024 threads: `pooled` has room for
// kPoolRoom doubles, the chunks of up to kPoolSegment tokens at a time (a sequence with longer chunks must not be longer).
// Window sums, chunk sums and divisions are those of pool_chunk_kernel, in its order.
constexpr int kPoolSegment = 2048;
constexpr int kPoolRoom = kPoolSegment + kPoolSegment / 8;  // (chunks of eight and more tokens a double apart: no bank conflicts)
__device__ __forceinline__ void pool_chunks_in_lds(const SelDev& p, const float* score, double* pooled, double* cs) {
  const int n = p.n_chunks, per_segment = max(1, kPoolSegment / p.chunk), pad = p.chunk >= 8 ? 1 : 0;
  const uint32_t inverse = 0xffffffffu / (uint32_t)p.chunk + 1u;  // x / chunk = x * inverse >> 32 for x below 2^32 / chunk
  for (int j0 = 0; j0 < n; j0 += per_segment) {
    const int first = j0 * p.chunk, chunks = min(per_segment, n - j0), end = j0 + chunks == n ? p.T : first + chunks * p.chunk;
    for (int i = first + (int)threadIdx.x; i < end; i += 1024) {
      const int a = max(0, i - p.radius), e = min(p.T - 1, i + p.radius);
      double sum = 0.0;
#pragma unroll 8
      for (int x = a; x <= e; ++x) sum += (double)score[x];  // (sixteen masked reads, as from memory, are slower here)
      pooled[i - first + (pad ? (int)__umulhi((uint32_t)(i - first), inverse) : 0)] = sum / (double)(e - a + 1);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < chunks; j += 1024) {
      const int len = min(p.chunk, p.T - first - j * p.chunk);
      const double* v = pooled + j * (p.chunk + pad);
      double tot = 0.0;
#pragma unroll 8
      for (int x = 0; x < len; ++x) tot += v[x];
      const double mean = tot / (double)len;
      cs[j0 + j] = mean;
      if (p.chunk_scores_out) p.chunk_scores_out[j0 + j] = (float)mean;
    }
    __syncthreads();
  }
}

}  // namespace sp
