// Jagged tile scheduler and small utility kernels.
//
// The scheduler turns the jagged batch into a list of (sequence, block)
// work items for the attention kernels -- the grouped computation over
// unpadded sequences of the paper (Sec. 3.2; appendix on the fused kernels):
// no padding, causally empty tiles never become work.  Items are written
// longest-first (counting sort by tile count) so that the hardware
// dispatcher, which hands out workgroups in index order, starts the
// longest items first.
#include "kernels.h"

namespace hstu {

namespace {

constexpr int kSchedThreads = 1024;

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Forward item (q-block qb): number of key tiles of kFwdBN the forward
// kernel visits.  Key tiles made only of candidates that lie before the
// block's first row are fully masked and skipped.
__device__ __forceinline__ int fwd_weight(int L, int n_h, int qb) {
  int i0 = qb * kFwdBM;
  int rows_end = min(i0 + kFwdBM, L);
  int kend = ceil_div(rows_end, kFwdBN);
  int skipped = max(0, i0 / kFwdBN - ceil_div(n_h, kFwdBN));
  return kend - skipped;
}

// Cross-mode forward item: key chunk c of a candidate block visits keys
// [c kCrossChunk, min(n_h, (c + 1) kCrossChunk)) of the cached prefix.
__device__ __forceinline__ int cross_weight(int n_h, int c) {
  return ceil_div(min(kCrossChunk, n_h - c * kCrossChunk), kFwdBN);
}

// Backward item (k-block kb): number of query steps of kBwdBM rows.
__device__ __forceinline__ int bwd_weight(int L, int n_h, int kb) {
  int j0 = kb * kBwdBN;
  int i_end = j0 >= n_h ? min(j0 + kBwdBN, L) : L;
  return ceil_div(i_end - j0, kBwdBM);
}

// Inclusive prefix sum over the workgroup's threads: shuffles inside a wave,
// one LDS exchange of the waves' sums (two barriers; a doubling scan through
// LDS took twenty).  `waves` holds a value per wave and may be used again
// after the call; *total receives the sum.
template <typename V>
__device__ __forceinline__ V block_scan(V v, V* waves, V* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const V x = __shfl_up(v, off, 64);
    if (lane >= off) v += x;
  }
  if (lane == 63) waves[wave] = v;
  __syncthreads();
  V before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kSchedThreads / 64; w++) {
    const V x = waves[w];
    before += w < wave ? x : 0;
    all += x;
  }
  __syncthreads();
  *total = all;
  return v + before;
}

// One workgroup of kSchedThreads builds the whole list; s_bins holds
// maxw + 1 ints (dynamic LDS), s_scan one per wave.  Bound by latency: a
// group keeps its first sequence's lengths over both passes.
__device__ void schedule_block(const JaggedArgs& ja, int mode, WorkItem* items, int32_t* count,
                               int* s_bins, int* s_scan) {
  const int tid = threadIdx.x;
  const int blk = mode == 0 ? kFwdBM : kBwdBN;
  const int maxw = mode == 0 ? ceil_div(ja.max_seq_len, kFwdBN) : ceil_div(ja.max_seq_len, kBwdBM);
  // (cross mode: a chunk's weight is at most kCrossChunk / kFwdBN <= maxw)
  const int nbins = maxw + 1;
  // Sequences are handed to groups of G lanes (G a power of two up to a
  // wave, larger for fewer sequences); a group's lanes share its items.
  int G = 1;
  while (G < 64 && G * ja.num_seqs < kSchedThreads) G <<= 1;
  const int group = tid / G, sub = tid % G, ngroups = kSchedThreads / G;
  const bool cross = mode == 0 && ja.key_offsets;
  struct Lens {
    int L, n_h;
  };
  auto lens_of = [&](int b) -> Lens {
    const int L = (int)(ja.seq_offsets[b + 1] - ja.seq_offsets[b]);
    const int n_h = cross ? (int)(ja.key_offsets[b + 1] - ja.key_offsets[b])
                          : L - (ja.num_targets ? (int)ja.num_targets[b] : 0);
    return Lens{L, n_h};
  };
  const Lens first = group < ja.num_seqs ? lens_of(group) : Lens{0, 0};
  // Calls f(seq, block, weight) for every item.
  auto for_items = [&](auto&& f) {
    for (int b = group; b < ja.num_seqs; b += ngroups) {
      const Lens len = b == group ? first : lens_of(b);
      const int L = len.L, n_h = len.n_h;
      const int nblk = ceil_div(L, blk);
      // (chunks past key_chunks exist only if n_h >= N: they are not scheduled)
      const int nch = cross ? min(ceil_div(n_h, kCrossChunk), ja.key_chunks) : 1;
      for (int e = sub; e < nblk * nch; e += G) {
        const int x = e / nch, c = e - x * nch;
        int w = cross       ? cross_weight(n_h, c)
                : mode == 0 ? fwd_weight(L, n_h, x)
                            : bwd_weight(L, n_h, x);
        w = min(max(w, 0), maxw);
        f(b, cross ? x * ja.key_chunks + c : x, w);
      }
    }
  };

  for (int i = tid; i < nbins; i += kSchedThreads) s_bins[i] = 0;
  __syncthreads();
  // Pass 1: histogram of item weights (bin index = maxw - weight, so that
  // an ascending scan orders items by descending weight).
  for_items([&](int, int, int w) { atomicAdd(&s_bins[maxw - w], 1); });
  __syncthreads();

  // Exclusive scan of the bins: each thread owns a contiguous run.
  const int per = ceil_div(nbins, kSchedThreads);
  const int lo = tid * per, hi = min(lo + per, nbins);
  int local = 0;
  for (int i = lo; i < hi; i++) local += s_bins[i];
  int items_total;
  int run = block_scan(local, s_scan, &items_total) - local;
  for (int i = lo; i < hi; i++) {
    int c = s_bins[i];
    s_bins[i] = run;
    run += c;
  }
  if (tid == 0) *count = items_total;
  __syncthreads();

  // Pass 2: scatter the items to their sorted positions.
  for_items([&](int b, int x, int w) {
    const int pos = atomicAdd(&s_bins[maxw - w], 1);
    WorkItem it;
    it.seq = b;
    it.blk = x;
    items[pos] = it;
  });
}

__global__ void fill_f32_kernel(float* p, int64_t n, float value) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = value;
}

// out[0] = 0, out[i+1] = out[i] + x_i; x_i = in[i], or (in[i+1]-in[i])^2
// when square_of_diff (pair offsets of the bucket matrices).
__global__ __launch_bounds__(kSchedThreads) void cumsum_kernel(int32_t n, const int64_t* in,
                                                               int64_t* out, int square_of_diff) {
  __shared__ int64_t s[kSchedThreads / 64];
  const int tid = threadIdx.x;
  int64_t carry = 0;
  if (tid == 0) out[0] = 0;
  for (int32_t base = 0; base < n; base += kSchedThreads) {
    int32_t i = base + tid;
    int64_t x = 0;
    if (i < n) {
      if (square_of_diff) {
        int64_t d = in[i + 1] - in[i];
        x = d * d;
      } else {
        x = in[i];
      }
    }
    int64_t total;
    const int64_t sum = block_scan(x, s, &total);
    if (i < n) out[i + 1] = carry + sum;
    carry += total;
  }
}

// acc is head-major [h][T][d] (fp32), dq token-major [T][h][d] (bf16);
// one thread per 4 features.
__global__ void dq_convert_kernel(const float* __restrict__ acc, uint16_t* __restrict__ dq,
                                  int64_t T, int32_t H, int32_t d4, float scale) {
  const int64_t n4 = T * H * d4;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    const int64_t row = i / d4;  // t * H + h
    const int64_t c = i - row * d4;
    const int64_t t = row / H, h = row - t * H;
    f32x4 a = reinterpret_cast<const f32x4*>(acc)[(h * T + t) * d4 + c];
    uint32_t lo = pack_bf16x2(a[0] * scale, a[1] * scale);
    uint32_t hi = pack_bf16x2(a[2] * scale, a[3] * scale);
    reinterpret_cast<uint2*>(dq)[i] = make_uint2(lo, hi);
  }
}

int grid_for(int64_t n, int threads) {
  int64_t g = (n + threads - 1) / threads;
  if (g > 65536) g = 65536;
  return (int)(g < 1 ? 1 : g);
}

// Per-sequence timestamp extremes (one workgroup per sequence; eight
// independent loads in flight per thread).  The attention kernels use them
// to pick 32-bit rebased time arithmetic when a sequence spans < 2^31.
__device__ void time_range_block(const JaggedArgs& ja, int b, int64_t* out,
                                 int64_t (*red)[kSchedThreads / 64]) {
  const int tid = threadIdx.x;
  const int64_t o = ja.seq_offsets[b];
  const int L = (int)(ja.seq_offsets[b + 1] - o);
  const int64_t* ts = ja.timestamps + o;
  int64_t lo = 0x7fffffffffffffffll, hi = -0x7fffffffffffffffll - 1;
  for (int x0 = 0; x0 < L; x0 += 8 * kSchedThreads) {
    int64_t v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = ts[min(x0 + k * kSchedThreads + tid, L - 1)];
#pragma unroll
    for (int k = 0; k < 8; k++) {
      lo = v[k] < lo ? v[k] : lo;
      hi = v[k] > hi ? v[k] : hi;
    }
  }
  // Cross mode: the cached prefix's timestamps count too.
  int Lk = 0;
  if (ja.key_offsets) {
    const int64_t ok = ja.key_offsets[b];
    Lk = (int)(ja.key_offsets[b + 1] - ok);
    const int64_t* tk = ja.key_timestamps + ok;
    for (int x = tid; x < Lk; x += kSchedThreads) {
      const int64_t v = tk[x];
      lo = v < lo ? v : lo;
      hi = v > hi ? v : hi;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int64_t a = __shfl_xor(lo, off, 64), c = __shfl_xor(hi, off, 64);
    lo = a < lo ? a : lo;
    hi = c > hi ? c : hi;
  }
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = lo;
    red[1][tid >> 6] = hi;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kSchedThreads / 64; w++) {
      lo = red[0][w] < lo ? red[0][w] : lo;
      hi = red[1][w] > hi ? red[1][w] : hi;
    }
    out[2 * b] = L + Lk > 0 ? lo : 0;
    out[2 * b + 1] = L + Lk > 0 ? hi : 0;
  }
}

// Zero fills: fill block f of nf covers a grid-stride share of every job.
__device__ void fill_blocks(const PrepFills& fills, int f, int nf) {
  const int64_t stride = (int64_t)nf * kSchedThreads;
  for (int k = 0; k < fills.n; k++) {
    float* p = fills.ptr[k];
    const int64_t n = fills.count[k];
    int64_t done = 0;
    if (((uintptr_t)p & 15) == 0) {
      const int64_t n4 = n / 4;
      const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
      for (int64_t i = (int64_t)f * kSchedThreads + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<f32x4*>(p)[i] = z;
      done = 4 * n4;
    }
    for (int64_t i = done + (int64_t)f * kSchedThreads + threadIdx.x; i < n; i += stride)
      p[i] = 0.0f;
  }
}

// Slot tables of the two-role backward's partial dQ blocks: bases[b] =
// sum over b' < b of ceil(L/32) (row blocks), bases[B + 1 + b] = sum over
// b' < b of K S - 2 K (K - 1) with K = ceil(L/128), S = ceil(L/32) (the
// 32-row steps of all 128-key blocks of a sequence).
__device__ void bases_block(const JaggedArgs& ja, int64_t* bases,
                            int64_t (*s)[kSchedThreads / 64]) {
  const int tid = threadIdx.x, B = ja.num_seqs;
  int64_t* rbase = bases;
  int64_t* pbase = bases + B + 1;
  if (tid == 0) {
    rbase[0] = 0;
    pbase[0] = 0;
  }
  int64_t carry_r = 0, carry_p = 0;
  for (int base = 0; base < B; base += kSchedThreads) {
    const int b = base + tid;
    int64_t r = 0, q = 0;
    if (b < B) {
      const int64_t L = ja.seq_offsets[b + 1] - ja.seq_offsets[b];
      const int64_t S = (L + kBwdBM - 1) / kBwdBM, K = (L + kBwdBN - 1) / kBwdBN;
      r = S;
      q = K * S - 2 * K * (K - 1);
    }
    int64_t total_r, total_p;
    r = block_scan(r, s[0], &total_r);
    q = block_scan(q, s[1], &total_p);
    if (b < B) {
      rbase[b + 1] = carry_r + r;
      pbase[b + 1] = carry_p + q;
    }
    carry_r += total_r;
    carry_p += total_p;
  }
}

// Column sums: workgroup g of ceil(2 D / 32) owns 32 columns; its 32 row
// groups each sum every 32nd row, then the group sums are added in order.
__device__ void col_sums_block(const ColSums& cs, int g, float (*red)[33]) {
  const int col = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int i = 32 * g + col, n = 2 * cs.D;
  float s = 0.0f;
  if (i < n) {
#pragma unroll 8
    for (int r = grp; r < cs.rows; r += 32) s += cs.part[(int64_t)r * n + i];
  }
  red[grp][col] = s;
  __syncthreads();
  if (grp == 0 && i < n) {
    float t = 0.0f;
#pragma unroll
    for (int q = 0; q < 32; q++) t += red[q][col];
    float* o = cs.out[i / cs.D];
    if (o) o[i % cs.D] = t;
  }
}

// Everything an attention call needs before its main kernel, in one
// launch: workgroup 0 builds the work list, workgroups 1..B take one
// sequence's timestamp range each (both only with `items`), the next ones
// zero the fills, the next take the column sums, and (if `bases` is set)
// the last one writes the backward's slot tables.
__global__ __launch_bounds__(kSchedThreads) void prep_kernel(JaggedArgs ja, int mode,
                                                             WorkItem* items, int32_t* count,
                                                             int64_t* trange, PrepFills fills,
                                                             int nfill_blocks, ColSums sums,
                                                             int nsum_blocks, int64_t* bases) {
  extern __shared__ int s_bins[];  // [maxw + 1]
  __shared__ int s_scan[kSchedThreads / 64];
  __shared__ int64_t red[2][kSchedThreads / 64];
  __shared__ int64_t s_bases[2][kSchedThreads / 64];
  __shared__ float s_sums[32][33];
  int g = (int)blockIdx.x;
  if (items) {
    if (g == 0) {
      schedule_block(ja, mode, items, count, s_bins, s_scan);
      return;
    }
    if (g <= ja.num_seqs) {
      time_range_block(ja, g - 1, trange, red);
      return;
    }
    g -= 1 + ja.num_seqs;
  }
  if (g < nfill_blocks)
    fill_blocks(fills, g, nfill_blocks);
  else if (g < nfill_blocks + nsum_blocks)
    col_sums_block(sums, g - nfill_blocks, s_sums);
  else
    bases_block(ja, bases, s_bases);
}

}  // namespace

hipError_t launch_prep(const JaggedArgs& ja, int mode, WorkItem* items, int32_t* count,
                       int64_t* trange, const PrepFills& fills, const ColSums& sums,
                       int64_t* bases, hipStream_t s) {
  const int maxw = mode == 0 ? (ja.max_seq_len + kFwdBN - 1) / kFwdBN
                             : (ja.max_seq_len + kBwdBM - 1) / kBwdBM;
  const size_t lds = items ? sizeof(int) * (size_t)(maxw + 1) : 0;
  int64_t work4 = 0;
  for (int k = 0; k < fills.n; k++) work4 += (fills.count[k] + 3) / 4;
  // About four float4 stores per thread for large fills, at most 1024 blocks.
  int64_t nf = (work4 + 4 * kSchedThreads - 1) / (4 * kSchedThreads);
  nf = nf > 1024 ? 1024 : nf;
  if (work4 > 0 && nf < 1) nf = 1;
  const int nsum = sums.rows > 0 ? (2 * sums.D + 31) / 32 : 0;
  const int64_t grid = (items ? 1 + (int64_t)ja.num_seqs : 0) + nf + nsum + (bases ? 1 : 0);
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(prep_kernel, dim3((unsigned)grid), dim3(kSchedThreads), lds, s, ja, mode,
                     items, count, trange, fills, (int)nf, sums, nsum, bases);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float value, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n, value);
  return hipGetLastError();
}

hipError_t launch_complete_cumsum(int32_t n, const int64_t* in, int64_t* out, int square_of_diff,
                                  hipStream_t s) {
  hipLaunchKernelGGL(cumsum_kernel, dim3(1), dim3(kSchedThreads), 0, s, n, in, out,
                     square_of_diff);
  return hipGetLastError();
}

hipError_t launch_dq_convert_bf16(const float* acc, void* dq, int64_t T, int32_t H, int32_t d,
                                  float scale, hipStream_t s) {
  const int64_t n4 = T * H * (d / 4);  // d is a multiple of 32
  if (n4 <= 0) return hipSuccess;
  hipLaunchKernelGGL(dq_convert_kernel, dim3(grid_for(n4, 256)), dim3(256), 0, s, acc,
                     (uint16_t*)dq, T, H, d / 4, scale);
  return hipGetLastError();
}

}  // namespace hstu
