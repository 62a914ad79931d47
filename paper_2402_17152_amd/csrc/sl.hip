// Stochastic Length (Eq. 4 and the subsequence selection appendix): shrinks
// a jagged batch before attention.  A sequence whose history (the tokens
// before its candidates) has n_h > L tokens keeps it whole with
// probability N_c^alpha / n_h^2 (the draw u_keep[b] and the numerator
// N_c^alpha are inputs) and otherwise
// keeps exactly L history tokens: those with the L smallest selection keys
// (equal keys: the later token first), in their original order.  The
// candidates always follow.  The result is a gather list of original
// token indices and the new offsets.
//
// Keys (the random draws e_rand are Exp(1) variates supplied by the
// caller): greedy = t_max - t_i (elapsed time, an integer); random = e_i;
// feature-weighted = e_i / (F - f_i), F = sum of f = t_max - t_i over the
// history, which orders the items as the exponential-race keys e_i / w_i
// of weighted sampling without replacement with w_i = 1 - f_i / F.  Keys
// are non-negative, so their bit patterns order like their values, and
// one workgroup per sequence finds the L-th smallest by a radix select over
// the 64-bit patterns (LDS histograms of 8-bit digits, at most 8 passes:
// it ends once every key sharing the known digits is chosen, for random
// keys after 3 or 4), then writes the chosen indices in order.
//
// Bound by the latency of the longest sequence's passes.  Keys of up to
// 8192 history tokens stay in the registers of 1024 threads, and one wave
// scans the histogram; a pass is two barriers.  (Recomputing the keys of 256
// threads from memory in each of 8 passes, with one thread scanning the
// bins, took 126 us on 64 sequences of up to 4096 tokens.)
#include "kernels.h"

namespace hstu {

namespace {

constexpr int kSlThreads = 1024;
constexpr int kSlWaves = kSlThreads / 64;
constexpr int kSlHeld = 8;  // keys a thread holds
// Up to this many sequences a select workgroup adds up the new lengths of
// the sequences before its own by itself, four per thread, instead of two
// launches before it (the keep decisions, their prefix sum: about 7 us).
constexpr int32_t kSlFusedSeqs = 4 * kSlThreads;

// log2 of the sequences per workgroup.  A CU holds one workgroup, so beyond a
// few times 256 sequences their number costs more than what they overlap: a
// workgroup then takes several sequences, copies those that stay whole side
// by side and shortens the others one after the other.  Sequences of 0 to 39
// tokens that all stay whole, one to a workgroup against several: 2048 of
// them 19.5 against 7.5 us, 4096 39.5 / 14.7, 60000 333 / 111; of 200 tokens
// shortened to 64: 55 / 44, 114 / 86, 1343 / 1105.
inline int sl_group_lg(int32_t B) { return B <= 1024 ? 0 : B <= kSlFusedSeqs ? 2 : 4; }

__device__ __forceinline__ bool keep_whole(int64_t n, int64_t t, int32_t L, double keep_num,
                                           double u) {
  const int64_t nh = n - t;
  return nh <= L || u < keep_num / ((double)nh * (double)nh);
}

__global__ __launch_bounds__(256) void sl_lengths_kernel(int32_t B,
                                                         const int64_t* __restrict__ offs,
                                                         const int64_t* __restrict__ nt, int32_t L,
                                                         double keep_num,
                                                         const double* __restrict__ u_keep,
                                                         int64_t* __restrict__ new_len) {
  for (int b = blockIdx.x * 256 + threadIdx.x; b < B; b += gridDim.x * 256) {
    const int64_t n = offs[b + 1] - offs[b];
    const int64_t t = nt ? nt[b] : 0;
    new_len[b] = keep_whole(n, t, L, keep_num, u_keep[b]) ? n : (int64_t)L + t;
  }
}

__device__ __forceinline__ uint64_t dbits(double x) { return (uint64_t)__double_as_longlong(x); }

struct SlKey {
  const int64_t* ts;
  const double* e;
  int64_t tmax, F;
  int mode;
  __device__ __forceinline__ uint64_t operator()(int i) const {
    if (mode == kSlGreedy) return (uint64_t)(tmax - ts[i]);
    const double ei = e[i] > 0.0 ? e[i] : 0.0;
    if (mode == kSlRandom || F == 0) return dbits(ei);
    const int64_t den = F - (tmax - ts[i]);
    if (den == 0) return dbits(__builtin_inf());
    return dbits(ei / (double)den);
  }
};

__device__ __forceinline__ int lanes_below(uint64_t m, int lane) {
  return __popcll(m & ((1ull << lane) - 1ull));
}

// Exclusive prefix count of `flag` over the workgroup in thread order;
// *total receives the workgroup's count.  Uses sc[0 .. kSlWaves - 1].
__device__ __forceinline__ int block_excl_count(bool flag, int* sc, int* total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t m = __ballot(flag);
  if (lane == 0) sc[wave] = __popcll(m);
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSlWaves; w++) {
    before += w < wave ? sc[w] : 0;
    tot += sc[w];
  }
  __syncthreads();
  *total = tot;
  return before + lanes_below(m, lane);
}

// Wave-wide reductions of 64-bit values.
__device__ __forceinline__ int64_t wave_add(int64_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Counts the digit of every active lane: the lanes that share the first
// active lane's digit (all of them, while the keys agree) add once.
__device__ __forceinline__ void count_digit(int* hist, bool active, int d, int lane) {
  const uint64_t act = __ballot(active);
  if (!act) return;
  const int first = __builtin_ctzll(act);
  const int d0 = __builtin_amdgcn_readlane(d, first);
  const uint64_t same = __ballot(active && d == d0);
  if (lane == first) atomicAdd(&hist[d0], __popcll(same));
  if (active && d != d0) atomicAdd(&hist[d], 1);
}

struct SlShared {
  int hist[256];
  int sc[kSlWaves];
  int64_t red[2][kSlWaves];
  int cnt[kSlHeld][kSlWaves];
  uint64_t prefix;
  int k, eq;
};

// Sum of v over the workgroup (`slot` of sm.red must not be in use).
__device__ __forceinline__ int64_t block_add(SlShared& sm, int slot, int64_t v) {
  v = wave_add(v);
  if ((threadIdx.x & 63) == 0) sm.red[slot][threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t s = 0;
#pragma unroll
  for (int w = 0; w < kSlWaves; w++) s += sm.red[slot][w];
  return s;
}

// Exclusive prefix over the (chunk, wave) counts in sm.cnt, in place.
__device__ __forceinline__ void scan_counts(SlShared& sm) {
  __syncthreads();
  if (threadIdx.x < 64) {
    int* c = &sm.cnt[0][0] + 2 * threadIdx.x;
    static_assert(kSlHeld * kSlWaves == 128, "two counts per lane");
    const int a = c[0], s = a + c[1];
    int run = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int x = __shfl_up(run, off, 64);
      if ((int)threadIdx.x >= off) run += x;
    }
    c[0] = run - s;
    c[1] = run - s + a;
  }
  __syncthreads();
}

// HELD: the history has at most kSlHeld * kSlThreads tokens, whose keys
// stay in registers; else they are recomputed in each pass.
template <bool HELD>
__device__ void select_tokens(SlShared& sm, const SlKey& key, int nh, int L, int64_t o,
                              int64_t* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int chunks = (nh + kSlThreads - 1) / kSlThreads;
  uint64_t held[HELD ? kSlHeld : 1];
  if constexpr (HELD) {
#pragma unroll
    for (int c = 0; c < kSlHeld; c++) {
      const int i = c * kSlThreads + tid;
      held[c] = i < nh ? key(i) : ~0ull;
    }
  }
  if (tid < 256) sm.hist[tid] = 0;
  __syncthreads();

  // Radix select: after pass p the top 8 (p + 1) bits of the L-th smallest
  // key are known; k is its rank among the keys sharing those bits.
  uint64_t prefix = 0, mask = 0;
  int k = L, eq = 0;
  for (int shift = 56; shift >= 0; shift -= 8) {
    auto count = [&](int i, uint64_t kv) {
      count_digit(sm.hist, i < nh && (kv & mask) == prefix, (int)(kv >> shift) & 255, lane);
    };
    if constexpr (HELD) {
#pragma unroll
      for (int c = 0; c < kSlHeld; c++)
        if (c < chunks) count(c * kSlThreads + tid, held[c]);
    } else {
      for (int c = 0; c < chunks; c++) {
        const int i = c * kSlThreads + tid;
        count(i, i < nh ? key(i) : ~0ull);
      }
    }
    __syncthreads();
    if (wave == 0) {
      // Lane l owns bins 4 l .. 4 l + 3; the digit is the first with k keys
      // in it and the bins before it.
      int h[4], sum = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        h[e] = sm.hist[4 * lane + e];
        sm.hist[4 * lane + e] = 0;
        sum += h[e];
      }
      int run = sum;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int x = __shfl_up(run, off, 64);
        if (lane >= off) run += x;
      }
      int before = run - sum;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (before < k && before + h[e] >= k) {
          sm.prefix = prefix | ((uint64_t)(4 * lane + e) << shift);
          sm.k = k - before;
          sm.eq = h[e];
        }
        before += h[e];
      }
    }
    __syncthreads();
    prefix = sm.prefix;
    k = sm.k;
    eq = sm.eq;
    mask |= 255ull << shift;
    if (eq == k) break;  // every key with these digits is chosen
  }

  // Of the eq tokens whose masked key equals prefix, the k with the largest
  // indices are chosen (with every smaller key).
  const int skip_eq = eq - k;
  if constexpr (HELD) {
    int rank[kSlHeld];
    if (skip_eq > 0) {
#pragma unroll
      for (int c = 0; c < kSlHeld; c++) {
        const uint64_t m = __ballot(c * kSlThreads + tid < nh && (held[c] & mask) == prefix);
        if (lane == 0) sm.cnt[c][wave] = __popcll(m);
        rank[c] = lanes_below(m, lane);
      }
      scan_counts(sm);
#pragma unroll
      for (int c = 0; c < kSlHeld; c++) rank[c] += sm.cnt[c][wave];
      __syncthreads();
    }
    uint32_t sel = 0;
    int pos[kSlHeld];
#pragma unroll
    for (int c = 0; c < kSlHeld; c++) {
      const bool is_eq = (held[c] & mask) == prefix;
      const bool take = c * kSlThreads + tid < nh &&
                        (is_eq ? (skip_eq == 0 || rank[c] >= skip_eq) : held[c] < prefix);
      const uint64_t m = __ballot(take);
      if (lane == 0) sm.cnt[c][wave] = __popcll(m);
      pos[c] = lanes_below(m, lane);
      sel |= take ? 1u << c : 0u;
    }
    scan_counts(sm);
#pragma unroll
    for (int c = 0; c < kSlHeld; c++) {
      const int x = pos[c] + sm.cnt[c][wave];
      if ((sel >> c & 1) && x < L) out[x] = o + c * kSlThreads + tid;
    }
  } else {
    int seen_eq = 0, written = 0;
    for (int c = 0; c < chunks; c++) {
      const int i = c * kSlThreads + tid;
      const uint64_t kv = i < nh ? key(i) : ~0ull;
      const bool is_eq = i < nh && (kv & mask) == prefix;
      int tot_eq, tot_sel;
      const int eq_before = seen_eq + block_excl_count(is_eq, sm.sc, &tot_eq);
      const bool take = i < nh && (is_eq ? eq_before >= skip_eq : kv < prefix);
      const int x = written + block_excl_count(take, sm.sc, &tot_sel);
      if (take && x < L) out[x] = o + i;
      seen_eq += tot_eq;
      written += tot_sel;
    }
  }
  __syncthreads();
}

// The L chosen history tokens of a sequence (tokens o .. o + n - 1, t of them
// candidates) and, after them, its candidates.
__device__ __forceinline__ void shorten(SlShared& sm, const int64_t* __restrict__ ts,
                                        const double* __restrict__ e_rand, int32_t L, int32_t mode,
                                        int64_t o, int n, int t, int64_t* __restrict__ out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nh = n - t;
  for (int c = tid; c < t; c += kSlThreads) out[L + c] = o + nh + c;

  // t_max and (feature-weighted) F = sum of t_max - t_i over the history;
  // random selection reads no timestamps.
  const int64_t* th = ts + o;
  int64_t tmax = 0, F = 0;
  if (mode != kSlRandom) {
    int64_t mx = (int64_t)(~0ull >> 1) * -1 - 1;
    for (int i = tid; i < nh; i += kSlThreads) mx = th[i] > mx ? th[i] : mx;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int64_t x = __shfl_xor(mx, off, 64);
      mx = x > mx ? x : mx;
    }
    if (lane == 0) sm.red[1][wave] = mx;
    __syncthreads();
    tmax = sm.red[1][0];
#pragma unroll
    for (int w = 1; w < kSlWaves; w++) tmax = max(tmax, sm.red[1][w]);
    __syncthreads();
  }
  if (mode == kSlWeighted) {
    int64_t sum = 0;
    for (int i = tid; i < nh; i += kSlThreads) sum += tmax - th[i];
    F = block_add(sm, 1, sum);
  }
  const SlKey key{th, e_rand ? e_rand + o : nullptr, tmax, F, mode};
  if (nh <= kSlHeld * kSlThreads)
    select_tokens<true>(sm, key, nh, L, o, out);
  else
    select_tokens<false>(sm, key, nh, L, o, out);
}

// FUSED: a workgroup adds up the new lengths of the sequences before its own
// and writes its new offsets; else new_offs holds them.  GROUP: 2^lg sequences
// (at most one per wave) to a workgroup; else one (FUSED only).
template <bool FUSED, bool GROUP>
__global__ __launch_bounds__(kSlThreads) void sl_select_kernel(
    int32_t B, int lg, const int64_t* __restrict__ offs, const int64_t* __restrict__ ts,
    const int64_t* __restrict__ nt, int32_t L, double keep_num, int32_t mode,
    const double* __restrict__ u_keep, const double* __restrict__ e_rand,
    int64_t* __restrict__ new_offs, int64_t* __restrict__ gather) {
  static_assert(FUSED || GROUP, "single sequences are few enough to be fused");
  __shared__ SlShared sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto new_len_before = [&](int b0) {
    int64_t sum = 0;
    for (int x = tid; x < b0; x += kSlThreads) {
      const int64_t xn = offs[x + 1] - offs[x], xt = nt ? nt[x] : 0;
      sum += keep_whole(xn, xt, L, keep_num, u_keep[x]) ? xn : (int64_t)L + xt;
    }
    return block_add(sm, 0, sum);
  };
  if constexpr (!GROUP) {
    const int b = blockIdx.x;
    const int64_t o = offs[b];
    const int n = (int)(offs[b + 1] - o), t = nt ? (int)nt[b] : 0;
    const bool whole = keep_whole(n, t, L, keep_num, u_keep[b]);
    const int64_t start = new_len_before(b);
    if (tid == 0) {
      if (b == 0) new_offs[0] = 0;
      new_offs[b + 1] = start + (whole ? n : (int64_t)L + t);
    }
    int64_t* out = gather + start;
    if (whole) {
      for (int i = tid; i < n; i += kSlThreads) out[i] = o + i;
    } else {
      shorten(sm, ts, e_rand, L, mode, o, n, t, out);
    }
    return;
  }
  for (int64_t first = (int64_t)blockIdx.x << lg; first < B; first += (int64_t)gridDim.x << lg) {
    const int b0 = (int)first, seqs = min(1 << lg, B - b0);
    // Lane l of every wave: sequence b0 + l.
    int64_t o_l = 0, start_l = 0;
    int n_l = 0, t_l = 0;
    bool whole_l = false;
    if (lane < seqs) {
      o_l = offs[b0 + lane];
      n_l = (int)(offs[b0 + lane + 1] - o_l);
      t_l = nt ? (int)nt[b0 + lane] : 0;
      whole_l = keep_whole(n_l, t_l, L, keep_num, u_keep[b0 + lane]);
      if constexpr (!FUSED) start_l = new_offs[b0 + lane];
    }
    if constexpr (FUSED) {
      const int64_t len = lane >= seqs ? 0 : whole_l ? n_l : (int64_t)L + t_l;
      int64_t run = len;
      for (int off = 1; off < 1 << lg; off <<= 1) {
        const int64_t x = __shfl_up(run, off, 64);
        if (lane >= off) run += x;
      }
      start_l = new_len_before(b0) + run - len;
      if (wave == 0 && lane < seqs) {
        if (b0 + lane == 0) new_offs[0] = 0;
        new_offs[b0 + lane + 1] = start_l + len;
      }
    }
    // Whole sequences, each by its share of the threads (whole waves).
    {
      const int sh = 10 - lg;  // 1024 >> lg threads
      const int k = __builtin_amdgcn_readfirstlane(tid >> sh);
      if (__builtin_amdgcn_readlane(whole_l, k)) {
        const int64_t o = readlane64(o_l, k);
        const int n = __builtin_amdgcn_readlane(n_l, k);
        int64_t* out = gather + readlane64(start_l, k);
        for (int i = tid & ((1 << sh) - 1); i < n; i += 1 << sh) out[i] = o + i;
      }
    }
    for (uint64_t left = __ballot(lane < seqs && !whole_l); left; left &= left - 1) {
      const int k = __builtin_ctzll(left);
      shorten(sm, ts, e_rand, L, mode, readlane64(o_l, k), __builtin_amdgcn_readlane(n_l, k),
              __builtin_amdgcn_readlane(t_l, k), gather + readlane64(start_l, k));
    }
    __syncthreads();  // sm.red is written again
  }
}

// dst row r = src row index[r] for r < *count (count read on the device).
// A row's words (of type W) are taken by 2^lg lanes (up to the whole
// workgroup), longer rows by as many columns of workgroups (blockIdx.x) as
// they have full ones, the first lanes taking what is left over; a workgroup
// takes kGatherUnroll sweeps of 256 >> lg consecutive rows, so that a lane has
// that many rows' loads in flight.  HBM-bound.  (With 64 lanes walking a whole
// row, few wide rows kept few lanes busy: 64 rows of 64 KB took 23 us, now 5;
// one of 1 MB 154, now 5; 36000 rows of 4 KB 56, now 46.  Columns of 64 words:
// 64 rows of 1 MB 24.1 us against 21.2, 36000 rows of 4112 bytes 54 against
// 49; a column of its own for what is left over: 76.)
constexpr int kGatherUnroll = 4;

template <typename W>
__global__ __launch_bounds__(256) void gather_rows_kernel(const char* __restrict__ src,
                                                          int64_t src_stride, int64_t words, int lg,
                                                          const int64_t* __restrict__ index,
                                                          const int64_t* __restrict__ count,
                                                          int64_t max_rows, char* __restrict__ dst,
                                                          int64_t dst_stride) {
  constexpr int U = kGatherUnroll;
  const int64_t rows = min(*count, max_rows);
  const int sub = threadIdx.x & ((1 << lg) - 1);
  const int step = 256 >> lg;
  for (int64_t r = (int64_t)blockIdx.y * (U * step) + (threadIdx.x >> lg); r < rows;
       r += (int64_t)gridDim.y * (U * step)) {
    int64_t from[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t x = r + u * step;
      from[u] = x < rows ? index[x] : 0;
    }
    for (int64_t w = ((int64_t)blockIdx.x << lg) + sub; w < words; w += (int64_t)gridDim.x << lg) {
      W v[U];
#pragma unroll
      for (int u = 0; u < U; u++)
        if (r + u * step < rows)
          v[u] = *reinterpret_cast<const W*>(src + from[u] * src_stride + w * (int)sizeof(W));
#pragma unroll
      for (int u = 0; u < U; u++)
        if (r + u * step < rows)
          *reinterpret_cast<W*>(dst + (r + u * step) * dst_stride + w * (int)sizeof(W)) = v[u];
    }
  }
}

template <typename W>
hipError_t gather_case(const void* src, int64_t src_stride, int64_t row_bytes,
                       const int64_t* index, const int64_t* count, int64_t max_rows, void* dst,
                       int64_t dst_stride, hipStream_t s) {
  const int64_t words = row_bytes / (int64_t)sizeof(W);
  int lg = 0;
  while (lg < 8 && (1 << lg) < words) lg++;
  const int64_t per_block = kGatherUnroll * (256 >> lg);
  const int64_t cols = max(min(words >> lg, (int64_t)65535), (int64_t)1);
  const int64_t blocks = min((max_rows + per_block - 1) / per_block, 65535 / cols);
  hipLaunchKernelGGL((gather_rows_kernel<W>), dim3((unsigned)cols, (unsigned)blocks), dim3(256), 0,
                     s, (const char*)src, src_stride, words, lg, index, count, max_rows,
                     (char*)dst, dst_stride);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stochastic_length(int32_t B, const int64_t* offs, const int64_t* ts,
                                    const int64_t* nt, int32_t L, double keep_num, int32_t mode,
                                    const double* u_keep, const double* e_rand, int64_t* new_len,
                                    int64_t* new_offs, int64_t* gather, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  const int lg = sl_group_lg(B);
  const int groups = (B + (1 << lg) - 1) >> lg;
  const dim3 grid((unsigned)(groups < 65535 ? groups : 65535));
  auto select = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(kSlThreads), 0, s, B, lg, offs, ts, nt, L, keep_num, mode,
                       u_keep, e_rand, new_offs, gather);
    return hipGetLastError();
  };
  if (lg == 0) return select(sl_select_kernel<true, false>);
  if (B <= kSlFusedSeqs) return select(sl_select_kernel<true, true>);
  const int blocks = (B + 255) / 256 < 1024 ? (B + 255) / 256 : 1024;
  hipLaunchKernelGGL(sl_lengths_kernel, dim3(blocks), dim3(256), 0, s, B, offs, nt, L, keep_num,
                     u_keep, new_len);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_complete_cumsum(B, new_len, new_offs, 0, s);
  if (e != hipSuccess) return e;
  return select(sl_select_kernel<false, true>);
}

hipError_t launch_gather_rows(const void* src, int64_t src_stride, int64_t row_bytes,
                              const int64_t* index, const int64_t* count, int64_t max_rows,
                              void* dst, int64_t dst_stride, hipStream_t s) {
  if (max_rows <= 0 || row_bytes <= 0) return hipSuccess;
  // The widest word that rows, strides and pointers are all multiples of.
  const uintptr_t all = (uintptr_t)row_bytes | (uintptr_t)src_stride | (uintptr_t)dst_stride |
                        (uintptr_t)src | (uintptr_t)dst;
  if (all % 16 == 0)
    return gather_case<u32x4>(src, src_stride, row_bytes, index, count, max_rows, dst,
                              dst_stride, s);
  if (all % 8 == 0)
    return gather_case<uint64_t>(src, src_stride, row_bytes, index, count, max_rows, dst,
                                 dst_stride, s);
  return gather_case<uint32_t>(src, src_stride, row_bytes, index, count, max_rows, dst,
                               dst_stride, s);
}

}  // namespace hstu
