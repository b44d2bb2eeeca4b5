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
};

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

// Radix select over 64-bit keys in registers, eight bits a pass from the top: a chunk is kept if its key is above
// `prefix`, or equal to it and among the first `need` of those in index order.  Stops as soon as all keys of the bucket
// in hand are needed (usually after two or three passes; then need = n).  `skip_top`: all keys share their top
// byte, which is prefix's.  Call with all 1024 threads; `hist` has room for 3 x 256 counters.  One barrier per
// pass: the counters of pass i live in hist[i % 3], the next pass's are cleared meanwhile (their
// last readers finished two barriers ago), and every wave finds the bucket for itself.
template <int I>
__device__ __forceinline__ void radix_select_kth(const uint64_t (&key)[I], int n, int k, bool skip_top, uint64_t top, int* hist,
                                                 uint64_t* prefix_out, int* need_out) {
  const int t = threadIdx.x;
  const int first_pass = skip_top ? 1 : 0;
  if (t < 256) hist[first_pass * 256 + t] = 0;
  __syncthreads();
  uint64_t prefix = skip_top ? top : 0;
  int need = k;
#pragma unroll 1
  for (int pass = first_pass; pass < 8; ++pass) {
    int* cur = hist + (pass % 3) * 256;
    int* nxt = hist + ((pass + 1) % 3) * 256;
    if (t < 256) nxt[t] = 0;
    const int shift = (7 - pass) * 8;
    const uint64_t himask = (pass == 0) ? 0ull : (~0ull << (shift + 8));
#pragma unroll
    for (int i = 0; i < I; ++i) {
      const bool in_play = reg_chunk<I>(i) < n && (key[i] & himask) == prefix;
      const int digit = (int)((key[i] >> shift) & 255u);
      // Scores of one prompt share their sign and most exponent bits, so in the upper passes a
      // whole wave lands in one counter, and 64 additions to one LDS word are done one after
      // the other: where the wave's digits all agree, one lane adds the count.
      const unsigned long long mask = __ballot(in_play);
      if (mask == 0) continue;
      const int leader = __builtin_amdgcn_readfirstlane(__ffsll(mask) - 1);
      const int first = __builtin_amdgcn_readlane(digit, leader);
      if (__ballot(in_play && digit != first) == 0) {
        if ((t & 63) == leader) atomicAdd(&cur[first], __popcll(mask));
      } else if (in_play) {
        atomicAdd(&cur[digit], 1);
      }
    }
    __syncthreads();
    int bucket;
    bool all;
    find_bucket(cur, need, &bucket, &need, &all);
    prefix |= (uint64_t)bucket << shift;
    if (all) {  // every key with this prefix is kept, and none has smaller lower bits than zero
      need = n;
      break;
    }
  }
  *prefix_out = prefix;
  *need_out = need;
}

// The k best of n chunks (scores cs[0..n), equal scores to the lower index) by one workgroup of 1024 threads:
// emit(j, rank) for every kept chunk j, the rank-th of them in index order, emit(j, -1) for the others; returns
// the number of kept chunks (*last_kept: chunk n - 1 among them), or -1 if a score is NaN (nothing is emitted then).
template <int I, typename Emit>
__device__ __forceinline__ int select_chunks(const double* cs, int n, int k, int* hist, int* sh, bool* last_kept, Emit emit) {
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  __shared__ uint64_t key0;
  __shared__ int last_sh;
  uint64_t key[I];
  int bad = 0;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = reg_chunk<I>(i);
    double v = 0.0;
    if (j < n) v = cs[j];
    bad |= is_nan_bits(v) ? 1 : 0;
    key[i] = order_key(v);
  }
  if (t == 0) { key0 = key[0]; last_sh = 0; }
  if (__syncthreads_or(bad)) return -1;
  const uint64_t top = key0 & (255ull << 56);
  int differs = 0;
#pragma unroll
  for (int i = 0; i < I; ++i) differs |= (reg_chunk<I>(i) < n && (key[i] & (255ull << 56)) != top) ? 1 : 0;
  const bool skip_top = !__syncthreads_or(differs);
  uint64_t prefix;
  int need;
  radix_select_kth<I>(key, n, k, skip_top, top, hist, &prefix, &need);

  // in index order: rows of 64 chunks by ballots, the waves' totals through LDS
  int above = 0, equal = 0;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const bool in = reg_chunk<I>(i) < n;
    above += __popcll(__ballot(in && key[i] > prefix));
    equal += __popcll(__ballot(in && key[i] == prefix));
  }
  if (lane == 0) { sh[wave] = above; sh[16 + wave] = equal; }
  __syncthreads();
  int kept_before = 0, eq_before = 0, total = 0, eq_total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int a = sh[w], e = sh[16 + w];
    if (w < wave) { kept_before += a; eq_before += e; }
    total += a;
    eq_total += e;
  }
  kept_before += min(eq_before, need);
  total += min(eq_total, need);
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = reg_chunk<I>(i);
    const bool eq = j < n && key[i] == prefix;
    const unsigned long long eq_mask = __ballot(eq);
    const bool keep = j < n && (key[i] > prefix || (eq && eq_before + __popcll(eq_mask & below) < need));
    const unsigned long long mask = __ballot(keep);
    if (j < n) emit(j, keep ? kept_before + __popcll(mask & below) : -1);
    if (keep && j == n - 1) last_sh = 1;
    eq_before += __popcll(eq_mask);
    kept_before += __popcll(mask);
  }
  __syncthreads();
  *last_kept = last_sh != 0;
  return total;
}

// Single sequence with at most kSingleMaxChunks chunks: top-k, compaction and the kept-index
// list in one workgroup and one launch.  Above kCountMaxChunks chunks the chunks are selected as in
// select_kernel; kept tokens are written straight away.
constexpr int kSingleMaxChunks = 2048;
constexpr int kCountMaxChunks = 256;  // up to here the chunks are ranked by counting instead
// `cs`: the chunk scores (global or LDS memory); `keys`: LDS room for kSingleMaxChunks 64-bit keys.
// Call with all 1024 threads of the workgroup.
__device__ __forceinline__ void select_emit_single(const SelDev& p, const double* cs, uint64_t* keys) {
  __shared__ int hist[3 * 256];
  __shared__ int sh[32];
  const int t = threadIdx.x;
  const int M = p.T;
  const int n = (M + p.chunk - 1) / p.chunk;
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
  if (n <= kCountMaxChunks) {
    // Few chunks: a chunk is ranked by counting the chunks that come before it in the order (larger score, or equal score
    // and lower index), four threads a chunk, each a quarter of the others; the k first are kept.  (256 chunks of 32
    // tokens, pooling included: 15.6 us with a thread per chunk and every token looked at, 8.8 now.)
    __shared__ uint64_t kept_mask[kCountMaxChunks / 64];
    __shared__ unsigned char ahead[4][kCountMaxChunks];
    int bad = 0;
    if (t < n) {
      const double v = cs[t];
      bad = is_nan_bits(v) ? 1 : 0;
      keys[t] = order_key(v);
    }
    if (__syncthreads_or(bad)) {  // invalid scores: reported in band, nothing kept
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
  __syncthreads();
  // the kept tokens are written by all threads, a token each
  const int64_t n_write = min(total_tokens, p.capacity);
  for (int64_t pos = t; pos < n_write; pos += 1024) {
    const int q = (int)(pos / p.chunk);
    p.kept_idx[pos] = (int)kept_list[q] * p.chunk + (int)(pos - (int64_t)q * p.chunk);
  }
  if (t == 0) p.cu_keep[1] = (int32_t)total_tokens;
}

// Pooling and chunk means of one sequence whose scores are in LDS, by one workgroup of 1024 threads: `pooled` has room for
// kPoolRoom doubles, the chunks of up to kPoolSegment tokens at a time (a sequence with longer chunks must not be longer).  Window sums, chunk sums and divisions are those of pool_chunk_kernel, in its order.
constexpr int kPoolSegment = 2048;
constexpr int kPoolRoom = kPoolSegment + kPoolSegment / 8;  // (chunks of eight and more tokens a double apart: no bank conflicts)
__device__ __forceinline__ void pool_chunks_in_lds(const SelDev& p, const float* score, double* pooled, double* cs) {
  const int n = (p.T + p.chunk - 1) / p.chunk, per_segment = max(1, kPoolSegment / p.chunk), pad = p.chunk >= 8 ? 1 : 0;
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
