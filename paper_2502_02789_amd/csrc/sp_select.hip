// sp_pool_select: 1-D average pooling, chunk means, top-k chunks with a lower-index
// tie-break, and ordered compaction of the kept tokens (Sec. 3.2.3 and Algorithm 1,
// chunk_select_from_smoothed_attention, of arXiv 2502.02789; keep rate = ratio of
// chunks, Sec. 4.1).
//
// All arithmetic is fp64 on the fp32 input scores, summed in index order with adds and
// divides only, so the chunk scores (and therefore the kept set) do not depend on how the
// work is split over lanes.  Top-k is a selection of the k-th of order-preserving 64-bit keys held in registers, followed
// by an ordered count; equal scores are resolved to the lower chunk index.
#include <mutex>

// the k formula below must stay a separate multiply and subtract
#pragma clang fp contract(off)

#include "sp_select_core.h"

namespace sp {

// Where the chunks of sequence b sit in cs and chunk_off: without a table at cu[b] / chunk + b (every sequence has room
// for its chunks that way, T / chunk + B places in all); with one (the caller wants the chunk scores, which are
// numbered without gaps) where it says.
__device__ __forceinline__ int chunk_base(const SelDev& p, int b) {
  return p.table ? p.cu_chunks[b] : (int)((uint32_t)p.cu[b] / (uint32_t)p.chunk) + b;
}
// the largest b whose first chunk is <= j (`base`: where the sequences' chunks start, in LDS, or null)
__device__ __forceinline__ int sequence_of_chunk(const SelDev& p, int j, const int32_t* base) {
  int lo = 0, hi = p.B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((base ? base[mid] : chunk_base(p, mid)) <= j) lo = mid; else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(1024) void chunk_table_kernel(const SelDev p) {
  block_prefix_table(p.B, [&](int b) { return chunk_count(p.cu[b + 1] - p.cu[b], p.chunk); }, p.cu_chunks);
}

__device__ __forceinline__ double shfl_f64(double v, int src) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl(lo, src, kWave);
  hi = __shfl(hi, src, kWave);
  return __hiloint2double(hi, lo);
}

// tokens from chunk place j's start to the end of its sequence (<= 0: a place without a chunk)
template <bool SINGLE>
__device__ __forceinline__ int chunk_tokens(const SelDev& p, int j, int n_chunks, const int32_t* base) {
  if (j >= n_chunks) return 0;
  if (SINGLE) return p.T - j * p.chunk;
  const int b = sequence_of_chunk(p, j, base);
  return p.cu[b + 1] - p.cu[b] - (j - chunk_base(p, b)) * p.chunk;
}

// A workgroup serves 256 / chunk chunks (chunk <= 256): a thread pools one token (window sums in index order, the
// window's loads all in flight at once), then one lane per chunk adds the chunk's pooled values in token order.
// Bound by its dependent steps (loads, window, chunk sum), not by any throughput: 5.1 us before for 256 and 1024 chunks
// of 32 tokens with the chunk sums by shuffles, one value after the other.
constexpr int kPoolThreads = 256;
template <bool SINGLE>  // SINGLE: one sequence of T tokens
__global__ __launch_bounds__(kPoolThreads) void pool_chunk_kernel(const SelDev p) {
  __shared__ double pooled[2 * kPoolThreads];
  const int cpb = kPoolThreads / p.chunk;              // chunks per workgroup
  const int n_chunks = SINGLE ? p.n_chunks : p.table ? p.cu_chunks[p.B] : p.T / p.chunk + p.B;
  const int t = threadIdx.x;
  if (!SINGLE && !p.table && blockIdx.x == 0 && t == 0) *p.arrived = 0;  // (for the selection kernel behind this one)
  // (of a batch, the places of its sequences' chunks are searched in LDS, as the offsets in emit_kernel: whole selection of 16
  // sequences 13.2 -> 12.5 us, of 64 15.7 -> 14.4)
  __shared__ int32_t base_lds[kPoolThreads];
  const int32_t* base = nullptr;
  if (!SINGLE && p.B <= kPoolThreads) {
    if (t < p.B) base_lds[t] = chunk_base(p, t);
    __syncthreads();
    base = base_lds;
  }
  const int q = t / p.chunk, t_in = t - q * p.chunk;
  for (int j0 = blockIdx.x * cpb; j0 < n_chunks; j0 += gridDim.x * cpb) {
    const int j = j0 + q;
    int lo = 0, hi = 0, s0 = 0, s1 = 0;
    if (q < cpb && j < n_chunks) {
      if (SINGLE) {
        hi = p.T;
        s0 = j * p.chunk;
      } else {
        const int b = sequence_of_chunk(p, j, base);
        lo = p.cu[b];
        hi = p.cu[b + 1];
        s0 = lo + (j - chunk_base(p, b)) * p.chunk;
      }
      s1 = min(s0 + p.chunk, hi);                       // (<= s0: a place without a chunk)
    }
    const int i = s0 + t_in;
    if (i < s1) {
      const int a = max(lo, i - p.radius), e = min(hi - 1, i + p.radius);
      double sum = 0.0;
      for (int x0 = a; x0 <= e; x0 += 8) {              // eight loads at a time; adding zeros changes no sum
        float v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = p.scores[min(x0 + x, e)];
#pragma unroll
        for (int x = 0; x < 8; ++x) sum += x0 + x <= e ? (double)v[x] : 0.0;
      }
      pooled[q * (p.chunk + 1) + t_in] = sum / (double)(e - a + 1);
    }
    __syncthreads();
    if (t < cpb) {                                      // lane t: chunk j0 + t
      const int len = min(p.chunk, chunk_tokens<SINGLE>(p, j0 + t, n_chunks, base));
      if (len > 0) {
        double tot = 0.0;
#pragma unroll 8
        for (int x = 0; x < len; ++x) tot += pooled[t * (p.chunk + 1) + x];
        const double mean = tot / (double)len;
        p.cs[j0 + t] = mean;
        if (p.chunk_scores_out) p.chunk_scores_out[j0 + t] = (float)mean;
      }
    }
    __syncthreads();
  }
}

// The same for longer chunks: a wave per chunk, 64 tokens at a time, every lane adding the values in token order.
template <bool SINGLE>
__global__ __launch_bounds__(256) void pool_long_chunk_kernel(const SelDev p) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n_chunks = SINGLE ? p.n_chunks : p.table ? p.cu_chunks[p.B] : p.T / p.chunk + p.B;
  if (!SINGLE && !p.table && blockIdx.x == 0 && threadIdx.x == 0) *p.arrived = 0;
  for (int j = blockIdx.x * 4 + wave; j < n_chunks; j += gridDim.x * 4) {
    int lo = 0, hi = p.T, nth = j;
    if (!SINGLE) {
      const int b = sequence_of_chunk(p, j, nullptr);
      lo = p.cu[b];
      hi = p.cu[b + 1];
      nth = j - chunk_base(p, b);
    }
    if (nth >= chunk_count(hi - lo, p.chunk)) continue;  // (a place without a chunk)
    const int s0 = lo + nth * p.chunk, s1 = hi - s0 < p.chunk ? hi : s0 + p.chunk;
    double tot = 0.0;
    for (int seg = s0; seg < s1; seg += kWave) {
      const int i = seg + lane;
      double v = 0.0;
      if (i < s1) {
        const int a = max(lo, i - p.radius), e = min(hi - 1, i + p.radius);
        double sum = 0.0;
        for (int x = a; x <= e; ++x) sum += (double)p.scores[x];
        v = sum / (double)(e - a + 1);
      }
      const int have = min(kWave, s1 - seg);
      for (int x = 0; x < kWave; ++x) {  // uniform trip count
        const double y = shfl_f64(v, x);
        if (x < have) tot += y;
      }
    }
    if (lane == 0) {
      const double mean = tot / (double)(s1 - s0);
      p.cs[j] = mean;
      if (p.chunk_scores_out) p.chunk_scores_out[j] = (float)mean;
    }
  }
}

// cu_keep from the sequences' counts, by one workgroup of 1024 threads; up to 64 sequences by its first wave, without the
// barriers of the prefix over all threads (whole selection of 16 and of 64 sequences 15.6 -> 13.6 and 18.1 -> 16.1 us)
__device__ __forceinline__ void scan_seq_keep(const SelDev& p) {
  auto count = [&](int b) { return __hip_atomic_load(p.seq_keep + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  if (p.B <= kWave) {
    const int b = threadIdx.x;
    if (b >= kWave) return;
    const int n = b < p.B ? count(b) : 0;
    const bool bad = __ballot(n < 0) != 0;
    int all;
    const int upto = wave_inclusive_scan(n, &all);
    if (b == 0) p.cu_keep[0] = 0;
    if (b < p.B) p.cu_keep[b + 1] = bad ? -1 : upto;  // (some sequence had invalid scores: no keep set is handed on)
    return;
  }
  int bad = 0;
  for (int b = threadIdx.x; b < p.B; b += 1024) bad |= count(b) < 0 ? 1 : 0;
  bad = __syncthreads_or(bad);
  block_prefix_table(p.B, [&](int b) { return max(count(b), 0); }, p.cu_keep);
  if (bad)  // some sequence had invalid scores: no keep set is handed on
    for (int b = 1 + threadIdx.x; b <= p.B; b += 1024) p.cu_keep[b] = -1;
}

// More chunks than registers hold (a sequence of more than 16384): the same selection with the scores read again in
// every pass, thread t owning chunks [j0, j1) in the ordered count.
__device__ __forceinline__ int select_chunks_from_memory(const double* cs, int n, int k, int* hist, int* sh, bool* last_kept,
                                                         int32_t* rank_out) {
  const int t = threadIdx.x;
  __shared__ int last_sh;
  int bad = 0;
  for (int j = t; j < n; j += 1024) bad |= is_nan_bits(cs[j]) ? 1 : 0;
  if (t == 0) last_sh = 0;
  if (__syncthreads_or(bad)) return -1;
  uint64_t prefix = 0;
  int need = k;
#pragma unroll 1
  for (int pass = 0; pass < 8; ++pass) {
    if (t < 256) hist[t] = 0;
    __syncthreads();
    const int shift = (7 - pass) * 8;
    const uint64_t himask = (pass == 0) ? 0ull : (~0ull << (shift + 8));
    for (int j = t; j < n; j += 1024) {
      const uint64_t key = order_key(cs[j]);
      if ((key & himask) == prefix) atomicAdd(&hist[(int)((key >> shift) & 255u)], 1);
    }
    __syncthreads();
    int bucket;
    bool all;
    find_bucket(hist, need, &bucket, &need, &all);
    prefix |= (uint64_t)bucket << shift;
    __syncthreads();
    if (all) { need = n; break; }
  }
  const int per = (n + 1023) / 1024, j0 = min(n, t * per), j1 = min(n, j0 + per);
  int above = 0, equal = 0;
  for (int j = j0; j < j1; ++j) {
    const uint64_t key = order_key(cs[j]);
    above += key > prefix ? 1 : 0;
    equal += key == prefix ? 1 : 0;
  }
  const int wave = t >> 6;
  int wave_above, wave_equal;
  int kept_before = wave_inclusive_scan(above, &wave_above) - above;
  int eq_before = wave_inclusive_scan(equal, &wave_equal) - equal;
  if ((t & 63) == 0) { sh[wave] = wave_above; sh[16 + wave] = wave_equal; }
  __syncthreads();
  int total = 0, eq_total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) { kept_before += sh[w]; eq_before += sh[16 + w]; }
    total += sh[w];
    eq_total += sh[16 + w];
  }
  kept_before += min(eq_before, need);
  total += min(eq_total, need);
  for (int j = j0; j < j1; ++j) {
    const uint64_t key = order_key(cs[j]);
    const bool keep = key > prefix || (key == prefix && eq_before++ < need);
    rank_out[j] = keep ? kept_before++ : -1;
    if (keep && j == n - 1) last_sh = 1;
  }
  __syncthreads();
  *last_kept = last_sh != 0;
  return total;
}

// One workgroup per sequence; chunk_off gets the rank of every kept chunk among its sequence's, -1 for the others.
// Without a chunk table the workgroup that finishes last (a word the pooling kernel has cleared counts them) adds the
// sequences' counts up, which the table variant leaves to a launch of its own.
// MOST: chunks a sequence may have, as far as the host can tell from all the tokens: a kernel has the code for no more (all
// forms in one cost 0.2 us for fetching what lies in between).
template <int MOST>
__global__ __launch_bounds__(1024) void select_kernel(const SelDev p) {
  __shared__ int hist[kSelectHist];
  __shared__ int sh[48];
  const int b = blockIdx.x, t = threadIdx.x;
  const int M = p.cu[b + 1] - p.cu[b];
  const int c0 = chunk_base(p, b), n = chunk_count(M, p.chunk);
  int keep_tokens = 0;
  if (n > 0) {
    const double scaled = p.keep_rate * (double)n;
    const double kd = ceil(scaled - 1e-9);
    const int k = (int)fmin((double)n, fmax(1.0, kd));
    const double* cs = p.cs + c0;
    int32_t* rank_out = p.chunk_off + c0;
    auto emit = [&](int j, int rank) __attribute__((always_inline)) { rank_out[j] = rank; };
    bool last_kept = false;
    int kept;
    if (MOST <= 1024 || n <= 1024) kept = select_chunks<1>(cs, n, k, hist, sh, &last_kept, emit);
    else if (MOST <= 4096 || n <= 4096) kept = select_chunks<4>(cs, n, k, hist, sh, &last_kept, emit);
    else if (n <= 16384) kept = select_chunks<16>(cs, n, k, hist, sh, &last_kept, emit);
    else kept = select_chunks_from_memory(cs, n, k, hist, sh, &last_kept, rank_out);
    // invalid scores (NaN: the scorer's mark for "a device-side wait expired") are reported in band:
    // a negative count here turns every cu_keep entry after the first into -1
    keep_tokens = kept < 0 ? -1 : (int)((int64_t)kept * p.chunk - (last_kept ? (int64_t)n * p.chunk - M : 0));
    if (kept < 0)
      for (int j = t; j < n; j += 1024) rank_out[j] = -1;
  }
  if (p.table) {
    if (t == 0) p.seq_keep[b] = keep_tokens;
    return;
  }
  __shared__ int arrived;
  if (t == 0) {
    __hip_atomic_store(p.seq_keep + b, keep_tokens, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    arrived = __hip_atomic_fetch_add(p.arrived, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (arrived == p.B - 1) scan_seq_keep(p);
}

template <SingleForm FORM>
__global__ __launch_bounds__(1024) void select_emit_single_kernel(const SelDev p) {
  __shared__ uint64_t keys[kSingleMaxChunks];
  select_emit_single<FORM>(p, p.cs, keys);
}

// One short sequence: pooling, selection and compaction by one workgroup, all in LDS.
constexpr int kOneLaunchTokens = 2048;
template <SingleForm FORM>
__global__ __launch_bounds__(1024) void pool_select_single_kernel(const SelDev p) {
  __shared__ float score[kOneLaunchTokens];
  __shared__ double wide[kPoolRoom];  // first the pooled scores, then (as 64-bit keys) the selection's keys
  __shared__ double cs[kSingleMaxChunks];
  static_assert(kPoolRoom >= kSingleMaxChunks && kPoolSegment >= kPoolThreads, "the selection's keys reuse the pooled scores' room");
  for (int i = threadIdx.x; i < p.T; i += 1024) score[i] = p.scores[i];
  __syncthreads();
  pool_chunks_in_lds(p, score, wide, cs);
  select_emit_single<FORM>(p, cs, reinterpret_cast<uint64_t*>(wide));
}

__global__ __launch_bounds__(1024) void cu_keep_kernel(const SelDev p) { scan_seq_keep(p); }

// one thread per prompt token: if its chunk is kept, write its flat index to its slot
__global__ __launch_bounds__(256) void emit_kernel(const SelDev p) {
  __shared__ int32_t cu_lds[kStagedOffsets];
  const int32_t last = p.cu_keep[p.B];
  const int32_t* const cu = staged_offsets(p.cu, p.B, cu_lds);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= p.T || last < 0) return;
  const int b = upper_segment(cu, p.B, i);
  const int in_seq = i - cu[b];
  const int j = in_seq / p.chunk;
  const int kept_before = p.cu_keep[b];
  const int rank = p.chunk_off[(p.table ? p.cu_chunks[b] : (int)((uint32_t)cu[b] / (uint32_t)p.chunk) + b) + j];
  if (rank < 0) return;
  const int64_t slot = (int64_t)kept_before + (int64_t)rank * p.chunk + (in_seq - j * p.chunk);
  if (slot < p.capacity) p.kept_idx[slot] = i;
}

static bool select_shape_ok(const sp_pool_select_args* a) {
  if (a->B < 1 || a->T < 0 || a->T >= (int64_t)INT32_MAX) return false;
  if (a->chunk < 1 || a->pool_window < 1 || (a->pool_window & 1) == 0) return false;
  if (!finite_f64(a->keep_rate) || a->keep_rate <= 0.0 || a->keep_rate > 1.0) return false;
  return true;
}
static size_t select_max_chunks(const sp_pool_select_args* a) { return (size_t)(a->T / a->chunk) + a->B; }

}  // namespace sp

extern "C" int64_t sp_keep_upper_bound(int32_t B, const int32_t* h_seqlens, int32_t chunk, double keep_rate) {
  if (B < 0 || (B > 0 && !h_seqlens) || chunk < 1 || !sp::finite_f64(keep_rate) || keep_rate <= 0.0 || keep_rate > 1.0)
    return -1;
  int64_t total = 0;
  for (int b = 0; b < B; ++b) {
    const int64_t M = h_seqlens[b];
    if (M < 0) return -1;
    if (M == 0) continue;
    const int64_t n = (M + chunk - 1) / chunk;
    const double scaled = keep_rate * (double)n;
    int64_t k = (int64_t)ceil(scaled - 1e-9);
    k = k < 1 ? 1 : (k > n ? n : k);
    const int64_t toks = k * chunk;
    total += toks < M ? toks : M;
  }
  return total;
}

extern "C" size_t sp_pool_select_workspace_bytes(const sp_pool_select_args* a) {
  if (!a || !sp::select_shape_ok(a)) return 0;
  const size_t mc = sp::select_max_chunks(a);
  return sp::align_up(4 * ((size_t)a->B + 1), 256) + sp::align_up(4 * (size_t)a->B, 256) +
         sp::align_up(8 * mc, 256) + sp::align_up(4 * mc, 256);
}

namespace sp {

// argument checks shared by the two entry points (everything but the scratch space)
static sp_status check_select_args(const sp_pool_select_args* a) {
  if (!a) return SP_ENULL;
  if (!select_shape_ok(a)) return SP_EINVAL;
  if (!a->d_cu_seqlens || !a->d_scores || !a->d_kept_idx || !a->d_cu_keep) return SP_ENULL;
  if (a->kept_capacity < 0) return SP_EINVAL;
  return SP_OK;
}

// enqueue the selection with `scratch` (device memory, 256-byte aligned, at least
// sp_pool_select_workspace_bytes(a) bytes) as the kernels' scratch space
static sp_status run_pool_select(const sp_pool_select_args* a, void* scratch, hipStream_t stream) {
  const size_t mc = select_max_chunks(a);
  SelDev p;
  p.B = a->B; p.T = (int)a->T; p.chunk = a->chunk; p.radius = (a->pool_window - 1) / 2;
  p.keep_rate = a->keep_rate; p.capacity = a->kept_capacity;
  p.cu = a->d_cu_seqlens; p.scores = a->d_scores; p.kept_idx = a->d_kept_idx; p.cu_keep = a->d_cu_keep;
  p.chunk_scores_out = a->d_chunk_scores;
  char* ws = static_cast<char*>(scratch);
  p.cu_chunks = reinterpret_cast<int32_t*>(ws); ws += align_up(4 * ((size_t)a->B + 1), 256);
  p.seq_keep = reinterpret_cast<int32_t*>(ws);  ws += align_up(4 * (size_t)a->B, 256);
  p.cs = reinterpret_cast<double*>(ws);         ws += align_up(8 * mc, 256);
  p.chunk_off = reinterpret_cast<int32_t*>(ws);

  // (without a table its place holds the count of the workgroups that have finished)
  p.table = a->d_chunk_scores != nullptr;
  p.arrived = p.cu_chunks;
  const bool long_chunks = a->chunk > kPoolThreads;
  const size_t per_block = long_chunks ? 4 : kPoolThreads / a->chunk;
  const unsigned pool_blocks = (unsigned)std::max<size_t>(1, std::min<size_t>((mc + per_block - 1) / per_block, 65535));
  const int64_t chunks = (a->T + a->chunk - 1) / a->chunk;
  p.n_chunks = a->B == 1 ? (int)chunks : 0;
  if (a->B == 1 && chunks <= kSingleMaxChunks) {
    const SingleForm form = single_form(chunks);
    // One sequence (its length is T, known here): no chunk table, no cross-sequence scan.  One launch while one workgroup
    // pools in the time of a second launch (chunks of 32, window 13, one and two launches in us: 500 tokens 4.7 and 6.1,
    // 1000 5.1 and 6.3, 2048 6.4 and 6.8, 3001 9.0 and 7.4).  Its work is tokens times window,
    // which up to 1600 tokens it does as fast as many workgroups would, beyond for small windows only (windows 129, 513 and
    // 4095: 1500 tokens 9.1 and 10.2, 18.9 and 20.5, 45.9 and 46.5; 1700 tokens 9.8 and 10.3, 20.1 and 20.7, 57.4 and 51.5; 2048
    // tokens, window 33, 65, 129, 4095: 7.1 and 7.5, 8.3 and 8.3, 10.8 and 10.0, 84.0 and 60.4).
    const int64_t over = a->T - 1600;
    if (a->T <= kOneLaunchTokens && !long_chunks && (over <= 0 || over * a->pool_window <= 16000)) {
      auto kernel = form == kRankByWave ? pool_select_single_kernel<kRankByWave>
                    : form == kRankByCount ? pool_select_single_kernel<kRankByCount> : pool_select_single_kernel<kRankByClasses>;
      hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, stream, p);
      return launch_status();
    }
    if (long_chunks) hipLaunchKernelGGL(pool_long_chunk_kernel<true>, dim3(pool_blocks), dim3(256), 0, stream, p);
    else hipLaunchKernelGGL(pool_chunk_kernel<true>, dim3(pool_blocks), dim3(kPoolThreads), 0, stream, p);
    auto kernel = form == kRankByWave ? select_emit_single_kernel<kRankByWave>
                  : form == kRankByCount ? select_emit_single_kernel<kRankByCount> : select_emit_single_kernel<kRankByClasses>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, stream, p);
    return launch_status();
  }
  if (p.table) hipLaunchKernelGGL(chunk_table_kernel, dim3(1), dim3(1024), 0, stream, p);
  if (long_chunks) hipLaunchKernelGGL(pool_long_chunk_kernel<false>, dim3(pool_blocks), dim3(256), 0, stream, p);
  else hipLaunchKernelGGL(pool_chunk_kernel<false>, dim3(pool_blocks), dim3(kPoolThreads), 0, stream, p);
  hipLaunchKernelGGL(chunks <= 1024 ? select_kernel<1024> : chunks <= 4096 ? select_kernel<4096> : select_kernel<INT32_MAX>, dim3(a->B),
                     dim3(1024), 0, stream, p);
  if (p.table) hipLaunchKernelGGL(cu_keep_kernel, dim3(1), dim3(1024), 0, stream, p);
  if (a->T > 0)
    hipLaunchKernelGGL(emit_kernel, dim3((unsigned)((a->T + 255) / 256)), dim3(256), 0, stream, p);
  return launch_status();
}

}  // namespace sp

extern "C" sp_status sp_pool_select(const sp_pool_select_args* a, void* hip_stream) {
  using namespace sp;
  const sp_status st = check_select_args(a);
  if (st != SP_OK) return st;
  if (!a->d_workspace || a->workspace_bytes < sp_pool_select_workspace_bytes(a)) return SP_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(a->d_workspace) & 255u) return SP_EALIGN;
  return run_pool_select(a, a->d_workspace, static_cast<hipStream_t>(hip_stream));
}

// ---------------------------------------------------------------------------------------
// the variant for callers that cannot allocate: scratch space inside the library's image
// ---------------------------------------------------------------------------------------
// One copy per GPU (each device that loads the library's code object gets its own), alive until
// the process ends.  In host code this name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[SP_STATIC_SCRATCH_BYTES];

namespace sp {

// device address of `scratch` on the current GPU, looked up once per device
static void* static_scratch_address() {
  static std::mutex mu;
  static void* address[kMaxDevices] = {};
  std::lock_guard<std::mutex> lock(mu);
  const int slot = current_device();
  if (!address[slot]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    address[slot] = ptr;
  }
  return address[slot];
}

}  // namespace sp

extern "C" sp_status sp_pool_select_static(const sp_pool_select_args* a, void* hip_stream) {
  using namespace sp;
  const sp_status st = check_select_args(a);
  if (st != SP_OK) return st;
  if (a->B > SP_STATIC_MAX_SEQS || select_max_chunks(a) > (size_t)SP_STATIC_MAX_CHUNKS) return SP_EUNSUPPORTED;
  static_assert(256 * ((4 * ((size_t)SP_STATIC_MAX_SEQS + 1) + 255) / 256) + 256 * ((4 * (size_t)SP_STATIC_MAX_SEQS + 255) / 256) +
                        12 * (size_t)SP_STATIC_MAX_CHUNKS + 512 <= SP_STATIC_SCRATCH_BYTES,
                "the static scratch must hold the largest workspace the limits allow");
  if (sp_pool_select_workspace_bytes(a) > SP_STATIC_SCRATCH_BYTES) return SP_EUNSUPPORTED;
  void* ptr = static_scratch_address();
  if (!ptr) return SP_ELAUNCH;
  // nothing in the scratch has to start at zero: every word the kernels read was written earlier
  // in the same call (chunk table, chunk scores, per-chunk offsets, per-sequence counts)
  return run_pool_select(a, ptr, static_cast<hipStream_t>(hip_stream));
}
