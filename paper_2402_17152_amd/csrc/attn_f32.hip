// fp32 jagged pointwise attention, forward and backward: the HSTU_F32
// variant of the library, for problems where fp32 throughout is wanted.
//
// Same definitions as the bf16 kernels (Eq. 2 with the pointwise 1/N
// normaliser, rab^{p,t} from the two tables, Algorithm 1 mask), with every
// contraction on the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (fp32
// products and sums, the rounding of a plain multiply-add chain).
//
// A workgroup of 4 waves owns 32 consecutive token rows of one head and
// walks 32-wide tiles of the other side, of each sequence that its rows
// belong to in turn (rows of other sequences are masked, so one set of
// accumulators serves them all and no work list is needed):
//   forward    rows = queries, tiles = keys:  O += P V;
//   backward   two kinds of workgroups in one launch,
//     (a) rows = queries, tiles = keys:  dQ += dS K, and the bias gradients
//         in fp64: one sum per diagonal of a tile (history rows) or per key
//         (candidate rows, all at one position), and a running sum per
//         thread and time bucket, so that a bucket's millions of terms do
//         not pile up fp32 rounding;
//     (b) rows = keys, tiles = queries:  dV += P^T dO, dK += dS^T Q.
// Wave (wr, wc) computes the 16 x 16 quadrant of a tile's scores, which pass
// through LDS to become the operand of the second contraction.
//
// Bound by the latency of one tile after another: a tile's loads (operand
// rows, timestamps, the 64 entries of rab_pos it can use) are issued while
// the tile before is computed.  One thread per (row, head) with the keys
// one by one took 47 + 58 + 60 us (forward, dQ, dK / dV) on four sequences
// of up to 128 tokens (2 heads of 32).  Rows of sequences of at most 16
// tokens, of which a workgroup can hold 32, go row by row instead, 8 threads
// to a row.
#include "kernels.h"

namespace hstu {

namespace {

constexpr int kRows = 32;      // token rows of a workgroup, and width of a tile
constexpr int kScoreLd = 36;   // row pitch of the score tiles
constexpr int kThreads = 256;
constexpr int kBuckets = 64;   // time buckets that a 64-bit difference can reach

__device__ __forceinline__ f32x4 mfma16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool not_finite(float x) {
  return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u;
}

// One operand tile of 32 rows of D floats: global -> registers -> LDS rows
// of D + 4 floats.  Rows outside [0, L) read as zeros.
template <int D>
struct TileRegs {
  static constexpr int kPer = D / 32, kLd = D + 4;
  f32x4 v[kPer];
  __device__ __forceinline__ void load(const float* base, int64_t stride, int row0, int L,
                                       int tid) {
#pragma unroll
    for (int e = 0; e < kPer; e++) {
      const int c = tid + kThreads * e, r = row0 + c / (D / 4);
      v[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      if (r >= 0 && r < L)
        v[e] = *reinterpret_cast<const f32x4*>(base + (int64_t)r * stride + 4 * (c % (D / 4)));
    }
  }
  // Stores the tile; sets *special if it holds an infinity or a NaN.
  __device__ __forceinline__ void store(float* t, int tid, int* special) const {
    bool b = false;
#pragma unroll
    for (int e = 0; e < kPer; e++) {
      const int c = tid + kThreads * e;
      *reinterpret_cast<f32x4*>(t + (c / (D / 4)) * kLd + 4 * (c % (D / 4))) = v[e];
#pragma unroll
      for (int m = 0; m < 4; m++) b |= not_finite(v[e][m]);
    }
    if (b) *special = 1;
  }
};

// c[m][n] += sum over d of a[m0 + m][d] b[n0 + n][d]: the lane's 4
// consecutive d of a 16-byte read feed four matrix instructions (any order
// of the contraction index serves, as long as both operands share it).
template <int D>
__device__ __forceinline__ f32x4 dot_tile(const float* a, const float* b, int lane, f32x4 c) {
  const int off = (lane & 15) * (D + 4) + 4 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < D / 16; s++) {
    const f32x4 av = *reinterpret_cast<const f32x4*>(a + off + 16 * s);
    const f32x4 bv = *reinterpret_cast<const f32x4*>(b + off + 16 * s);
#pragma unroll
    for (int e = 0; e < 4; e++) c = mfma16x16x4(av[e], bv[e], c);
  }
  return c;
}

// acc[f] += sum over x of w[m][x] t[x][f] for 16 rows m of the score tile w
// and the wave's D / 2 features of the 32 tile rows x (acc element r of
// block nb: row 4 (lane / 16) + r, feature 16 nb + lane % 16).  A pair that
// the mask drops has w = 0, which a non-finite t would turn into NaN: in a
// tile holding one (`special`) those elements enter the product as 0, and
// the pairs that `keep(r, x)`s add theirs afterwards.  So what a dropped
// pair holds never reaches a bit of the result.
template <int D, typename Keep>
__device__ __forceinline__ void outer_tile(const float* w, const float* t, int f0, int lane,
                                           bool special, Keep&& keep, f32x4 (&acc)[D / 32]) {
  const int n = lane & 15, g = lane >> 4;
  auto product = [&](auto&& value) {
#pragma unroll
    for (int s = 0; s < 2; s++) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(w + n * kScoreLd + 16 * s + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int nb = 0; nb < D / 32; nb++)
          acc[nb] = mfma16x16x4(
              a[e], value(t[(16 * s + 4 * g + e) * (D + 4) + f0 + 16 * nb + n]), acc[nb]);
    }
  };
  if (!special) {
    product([](float v) { return v; });
    return;
  }
  product([](float v) { return not_finite(v) ? 0.0f : v; });
  for (int x = 0; x < kRows; x++)
#pragma unroll
    for (int nb = 0; nb < D / 32; nb++) {
      const float v = t[x * (D + 4) + f0 + 16 * nb + n];
      if (!not_finite(v)) continue;
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (keep(4 * g + r, x)) acc[nb][r] += w[(4 * g + r) * kScoreLd + x] * v;
    }
}

// Rows of a workgroup in sequences of at most kShort tokens go row by row
// (short_* below), the others by tiles.  The line depends on the sequence
// alone, so a row's sums run in one order wherever it lies in a batch.  By
// tiles, 32 rows of one-token sequences took 32 passes: 596 against 37 us
// forward for 20000 such tokens (8 heads of 64), 99 against 50 at 8 tokens;
// at 16 tokens the tiles are ahead, 59 against 74.
constexpr int kShort = 16;

__device__ __forceinline__ int pack_short(int L, int n_h, int i) { return L | n_h << 8 | i << 16; }

// The sequences that a workgroup's 32 rows belong to.
struct Seqs {
  // Those that go by tiles, in order (two full ones do not fit the rows).
  static constexpr int kLong = (kRows - 2) / (kShort + 1) + 2;
  int64_t o[kLong];
  int L[kLong], n_h[kLong];
  int short_row[kRows];  // rows of the others (see pack_short), 0 elsewhere
};

// The (sequence, tile) pairs a workgroup visits: rows r0 .. r0 + 31 (global
// tokens), tiles of 32 of the other side.  All values are uniform.
struct Walk {
  int64_t o, r0;           // first token of the sequence; of the rows
  int L, n_h;              // its length and history tokens
  int ra, rb;              // rows of this sequence: indices ra .. rb
  int x0, xend;            // current tile's first index, end of the tiles
  int seq, seqs;           // which of the sequences that go by tiles; their number
  bool rows_are_keys, any_short;

  // Fills q from the offsets and enters the first sequence.  64 sequences at
  // a time, one per lane: first probes for the one of row r0, until what is
  // left of the search is one such chunk, then that chunk and, while the
  // rows go on, the ones after it.  Wave 0 writes (read after a barrier).
  __device__ __forceinline__ void start(const JaggedArgs& ja, int64_t first_row, bool keys,
                                        Seqs& q) {
    const int lane = threadIdx.x & 63, B = ja.num_seqs;
    rows_are_keys = keys;
    r0 = first_row;
    seq = seqs = 0;
    any_short = false;
    if (threadIdx.x < kRows) q.short_row[threadIdx.x] = 0;
    int lo = 0, hi = B;  // seq_offsets[lo] <= r0 < seq_offsets[hi]
    int64_t base = 0;    // seq_offsets[lo]
    while (hi - lo > 64) {
      const int step = (hi - lo + 63) >> 6;
      const int64_t at = ja.seq_offsets[min(lo + (lane + 1) * step, hi)];
      // (lane 63's probe is hi, which lies above)
      const uint64_t above = __ballot(at > r0) | 1ull << 63;
      const int f = __builtin_amdgcn_readfirstlane(__builtin_ctzll(above));
      base = f ? readlane64(at, f - 1) : base;
      hi = min(lo + (f + 1) * step, hi);
      lo += f * step;
    }
    for (;;) {
      const int s = lo + lane;
      const int64_t end = ja.seq_offsets[min(s + 1, B)];
      const int64_t before = __shfl_up(end, 1, 64), so = lane ? before : base;
      const int len = s < B && end > r0 && so < r0 + kRows ? (int)(end - so) : 0;
      int nh = len;
      if (len && ja.num_targets) nh -= (int)ja.num_targets[s];
      if (threadIdx.x < 64 && len > 0 && len <= kShort) {
        const int first = (int)(so - r0);
        for (int i = max(-first, 0); i < len && first + i < kRows; i++)
          q.short_row[first + i] = pack_short(len, nh, i);
      }
      any_short |= __ballot(len > 0 && len <= kShort) != 0;
      for (uint64_t m = __ballot(len > kShort); m && seqs < Seqs::kLong; m &= m - 1) {
        const int f = __builtin_ctzll(m);
        const int64_t fo = readlane64(so, f);
        const int fl = __builtin_amdgcn_readlane(len, f), fh = __builtin_amdgcn_readlane(nh, f);
        if (seqs == 0) enter(fo, fl, fh);
        if (threadIdx.x == 0) {
          q.o[seqs] = fo;
          q.L[seqs] = fl;
          q.n_h[seqs] = fh;
        }
        seqs++;
      }
      base = readlane64(end, 63);
      lo += 64;
      if (lo >= B || base >= r0 + kRows) break;
    }
  }
  __device__ __forceinline__ void enter(int64_t first, int len, int hist) {
    o = first;
    L = len;
    n_h = hist;
    ra = (int)max(r0 - o, (int64_t)0);
    rb = (int)min(r0 + kRows - 1 - o, (int64_t)L - 1);
    // Tiles start at multiples of 32 of the sequence, whatever the rows.
    if (rows_are_keys) {
      x0 = ra & ~(kRows - 1);
      xend = ra >= n_h ? rb + 1 : L;  // a candidate key is seen by itself only
    } else {
      x0 = 0;
      xend = rb + 1;
      skip();
    }
  }
  // Key tiles made only of candidates before every row: nothing is kept.
  __device__ __forceinline__ void skip() {
    if (!rows_are_keys && x0 >= n_h && x0 + kRows - 1 < ra) x0 = max(x0, ra & ~(kRows - 1));
  }
  __device__ __forceinline__ bool done() const { return seq >= seqs; }
  __device__ __forceinline__ void next(const Seqs& q) {
    x0 += kRows;
    skip();
    if (x0 >= xend && ++seq < seqs) {
      const uint64_t fo = (uint64_t)q.o[seq];
      const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)fo);
      const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(fo >> 32));
      enter((int64_t)((uint64_t)hi << 32 | lo), __builtin_amdgcn_readfirstlane(q.L[seq]),
            __builtin_amdgcn_readfirstlane(q.n_h[seq]));
    }
  }
  // Index of rab_pos that entry 0 of the tile's 64-entry window holds:
  // p(j) - p(i) spans at most 63 values from p(first key) - p(last row).
  __device__ __forceinline__ int window_base(int N) const {
    const int j = rows_are_keys ? ra : x0, i = rows_are_keys ? x0 + kRows - 1 : rb;
    return (N - 1) + bias_pos(j, n_h) - bias_pos(i, n_h);
  }
};

// What a tile brings besides its operand rows, one element per thread.
struct SideRegs {
  int64_t t;   // threads 0..31: timestamp of a tile row
  float win;   // threads 64..127: rab_pos window entry
  __device__ __forceinline__ void load(const JaggedArgs& ja, const Walk& w, int tid) {
    if (tid < kRows) {
      const int x = min(w.x0 + tid, w.L - 1);
      t = ja.timestamps[w.o + x];
    } else if (tid >= 64 && tid < 128) {
      const int idx = w.window_base(ja.max_seq_len) + tid - 64;
      win = ja.rab_pos[min(max(idx, 0), 2 * ja.max_seq_len - 2)];
    }
  }
  __device__ __forceinline__ void store(int64_t* st, float* sw, int tid) const {
    if (tid < kRows)
      st[tid] = t;
    else if (tid >= 64 && tid < 128)
      sw[tid - 64] = win;
  }
};

template <int DQK, int DV>
struct FwdLds {
  __align__(16) float q[kRows * (DQK + 4)];
  __align__(16) float k[kRows * (DQK + 4)];
  __align__(16) float v[2][kRows * (DV + 4)];
  __align__(16) float p[kRows * kScoreLd];
  int64_t t[kRows];
  float win[64];
  float tab[kBuckets];
  // Whether the tile of this parity holds an infinity or a NaN: set before a
  // tile's first barrier, read after its second, cleared between the next's.
  int special[2];
  Seqs seqs;
};

// ---- rows of short sequences: 8 threads each, a wave 8 rows ----
// Thread `sub` of a row holds features 4 (sub + 8 e) .. +3 of it.

struct ShortRow {
  int L, n_h, i;     // its sequence (L = 0: not a short one), its index there
  int64_t r;         // the token (r0 for a row that is none)
  __device__ __forceinline__ ShortRow(const int* short_row, int64_t r0) {
    const int x = threadIdx.x >> 3, v = short_row[x];
    L = v & 255;
    n_h = v >> 8 & 255;
    i = v >> 16;
    r = L ? r0 + x : r0;
  }
};

template <int D>
__device__ __forceinline__ void load_slice(const float* row, int sub, f32x4 (&v)[D / 32]) {
#pragma unroll
  for (int e = 0; e < D / 32; e++) v[e] = *reinterpret_cast<const f32x4*>(row + 4 * (sub + 8 * e));
}

template <int D>
__device__ __forceinline__ void store_slice(float* row, int sub, const f32x4 (&v)[D / 32],
                                            float scale) {
#pragma unroll
  for (int e = 0; e < D / 32; e++)
    *reinterpret_cast<f32x4*>(row + 4 * (sub + 8 * e)) = v[e] * scale;
}

// Dot product over the row's 8 threads, in each of them.
template <int D>
__device__ __forceinline__ float dot_slices(const f32x4 (&a)[D / 32], const f32x4 (&b)[D / 32]) {
  float s = 0.0f;
#pragma unroll
  for (int e = 0; e < D / 32; e++)
#pragma unroll
    for (int m = 0; m < 4; m++) s = __builtin_fmaf(a[e][m], b[e][m], s);
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) s += __shfl_xor(s, off, 64);
  return s;
}

template <int D>
__device__ __forceinline__ void add_slice(f32x4 (&acc)[D / 32], float w, const f32x4 (&v)[D / 32]) {
#pragma unroll
  for (int e = 0; e < D / 32; e++)
#pragma unroll
    for (int m = 0; m < 4; m++) acc[e][m] = __builtin_fmaf(w, v[e][m], acc[e][m]);
}

// Largest of the wave's 8 rows' counts.
__device__ __forceinline__ int rows_max(int v) {
#pragma unroll
  for (int off = 8; off < 64; off <<= 1) v = max(v, __shfl_xor(v, off, 64));
  return __builtin_amdgcn_readfirstlane(v);
}

// Key of row i at distance d in position: itself, then the history backwards.
__device__ __forceinline__ int key_at(const ShortRow& w, int d) {
  return d ? min(w.i, w.n_h) - d : w.i;
}
__device__ __forceinline__ int keys_of(const ShortRow& w) {
  return !w.L ? 0 : w.i < w.n_h ? w.i + 1 : w.n_h + 1;
}

// Pairs in flight: as many as leave the registers of the tile loop unchanged.
template <int DQK, int DV>
constexpr int kShortStep = DQK + DV <= 128 ? 4 : 2;

template <int DQK, int DV, typename Lds>
__device__ __forceinline__ void short_fwd(const Lds& sm, const JaggedArgs& ja, const Tensors& t,
                                          float* __restrict__ out, int64_t r0, int head) {
  const ShortRow w(sm.seqs.short_row, r0);
  const int steps = rows_max(keys_of(w));
  if (!steps) return;
  constexpr int U = kShortStep<DQK, DV>;
  const int sub = threadIdx.x & 7, H = ja.num_heads, N = ja.max_seq_len;
  const float* kg = (const float*)t.k + head * DQK;
  const float* vg = (const float*)t.v + head * DV;
  f32x4 q[DQK / 32], acc[DV / 32];
  load_slice<DQK>(sm.q + (threadIdx.x >> 3) * (DQK + 4), sub, q);
#pragma unroll
  for (int e = 0; e < DV / 32; e++) acc[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t ti = ja.timestamps[w.r];
  for (int d0 = 0; d0 < steps; d0 += U) {
    f32x4 k[U][DQK / 32], v[U][DV / 32];
    int64_t tj[U];
    float pos[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      ok[u] = d0 + u < keys_of(w);
      const int64_t r = ok[u] ? w.r + key_at(w, d0 + u) - w.i : w.r;
      load_slice<DQK>(kg + r * t.k_stride, sub, k[u]);
      load_slice<DV>(vg + r * t.v_stride, sub, v[u]);
      tj[u] = ja.timestamps[r];
      pos[u] = ja.rab_pos[max(N - 1 - d0 - u, 0)];
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const float s = dot_slices<DQK>(q, k[u]) +
                      (pos[u] + sm.tab[time_bucket64(ti - tj[u], ja.num_buckets)]);
      if (ok[u]) add_slice<DV>(acc, s * sigmoid_fast(s), v[u]);
    }
  }
  if (w.L) store_slice<DV>(out + (w.r * H + head) * DV, sub, acc, 1.0f / (float)N);
}

template <int DQK, int DV>
__global__ __launch_bounds__(kThreads) void fwd_f32_kernel(JaggedArgs ja, Tensors t,
                                                           float* __restrict__ out) {
  __shared__ FwdLds<DQK, DV> sm;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
  const int64_t r0 = (int64_t)blockIdx.x * kRows, T = ja.total_tokens;
  const int head = blockIdx.y, H = ja.num_heads, N = ja.max_seq_len;
  const float* kg = (const float*)t.k + head * DQK;
  const float* vg = (const float*)t.v + head * DV;
  Walk w;
  w.start(ja, r0, false, sm.seqs);
  TileRegs<DQK> kr;
  TileRegs<DV> vr;
  SideRegs sr;
  auto load = [&](const Walk& x) {
    kr.load(kg + x.o * t.k_stride, t.k_stride, x.x0, x.L, tid);
    vr.load(vg + x.o * t.v_stride, t.v_stride, x.x0, x.L, tid);
    sr.load(ja, x, tid);
  };
  if (!w.done()) load(w);
  {
    TileRegs<DQK> qr;
    int ignored;
    qr.load((const float*)t.q + head * DQK + r0 * t.q_stride, t.q_stride, 0,
            (int)min((int64_t)kRows, T - r0), tid);
    qr.store(sm.q, tid, &ignored);
  }
  if (tid < min(ja.num_buckets, kBuckets)) sm.tab[tid] = ja.rab_time[tid];
  if (tid < 2) sm.special[tid] = 0;
  __syncthreads();
  const int64_t my_r = r0 + 16 * wr + n;
  const int64_t ti = ja.timestamps[min(my_r, T - 1)];
  f32x4 acc[DV / 32];
#pragma unroll
  for (int nb = 0; nb < DV / 32; nb++) acc[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // Per tile: K, V (two buffers: the slower waves may still read the last
  // one), timestamps and window to LDS; scores; their weights to LDS; O.
  for (int par = 0; !w.done(); par ^= 1) {
    const Walk cur = w;
    kr.store(sm.k, tid, &sm.special[par]);
    vr.store(sm.v[par], tid, &sm.special[par]);
    sr.store(sm.t, sm.win, tid);
    __syncthreads();
    if (tid == 0) sm.special[par ^ 1] = 0;
    w.next(sm.seqs);
    if (!w.done()) load(w);
    const f32x4 s = dot_tile<DQK>(sm.k + 16 * wc * (DQK + 4), sm.q + 16 * wr * (DQK + 4), lane,
                                  f32x4{0.0f, 0.0f, 0.0f, 0.0f});
    const int i = (int)(my_r - cur.o);
    const int wbase = (N - 1) - bias_pos(i, cur.n_h) - cur.window_base(N);
    const bool row_ok = i >= 0 && i < cur.L;
    f32x4 p;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int x = 16 * wc + 4 * g + r, j = cur.x0 + x;
      float pv = 0.0f;
      if (row_ok && pair_valid(i, j, cur.n_h)) {
        const float b = sm.win[wbase + bias_pos(j, cur.n_h)] +
                        sm.tab[time_bucket64(ti - sm.t[x], ja.num_buckets)];
        const float sc = s[r] + b;
        pv = sc * sigmoid_fast(sc);
      }
      p[r] = pv;
    }
    *reinterpret_cast<f32x4*>(sm.p + (16 * wr + n) * kScoreLd + 16 * wc + 4 * g) = p;
    __syncthreads();
    const bool special = __builtin_amdgcn_readfirstlane(sm.special[par]) != 0;
    outer_tile<DV>(sm.p + 16 * wr * kScoreLd, sm.v[par], wc * (DV / 2), lane, special,
                   [&](int row, int x) {
                     const int ii = (int)(r0 + 16 * wr + row - cur.o);
                     return ii >= 0 && ii < cur.L && pair_valid(ii, cur.x0 + x, cur.n_h);
                   },
                   acc);
  }
  if (w.any_short) {
    __syncthreads();
    short_fwd<DQK, DV>(sm, ja, t, out, r0, head);
  }
  const float invN = 1.0f / (float)N;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int64_t row = r0 + 16 * wr + 4 * g + r;
    if (row < T && !(w.any_short && sm.seqs.short_row[16 * wr + 4 * g + r]))
#pragma unroll
      for (int nb = 0; nb < DV / 32; nb++)
        out[(row * H + head) * DV + wc * (DV / 2) + 16 * nb + n] = acc[nb][r] * invN;
  }
}

template <int DQK, int DV>
struct BwdLds {
  // Rows of the workgroup and of the tile: (q, dO) against (k, v).  Tiles
  // that the second contraction reads have two buffers.
  __align__(16) float own_qk[kRows * (DQK + 4)];
  __align__(16) float own_v[kRows * (DV + 4)];
  __align__(16) float tile_qk[2][kRows * (DQK + 4)];
  __align__(16) float tile_v[2][kRows * (DV + 4)];
  __align__(16) float p[kRows * kScoreLd];
  __align__(16) float ds[kRows * kScoreLd];
  int64_t t[kRows];
  float win[64];
  float tab[kBuckets];
  double time_acc[kBuckets];
  double short_pos[kShort];
  // Whether the tile of this parity holds an infinity or a NaN: set before a
  // tile's first barrier, read after its second, cleared between the next's.
  int special[2];
  Seqs seqs;
};

// Weight SiLU(s) and dS = dP SiLU'(s) of one pair (0, 0 if masked).
__device__ __forceinline__ void pair_grad(float s, float dp, float* p, float* ds) {
  const float sg = sigmoid_fast(s);
  *p = s * sg;
  *ds = dp * (sg + *p * (1.0f - sg));
}

// dQ and the bias gradients of short rows: position sums by distance into
// sm.short_pos, time sums as in the tile loop.
template <int DQK, int DV>
__device__ __forceinline__ void short_bwd_rows(BwdLds<DQK, DV>& sm, const JaggedArgs& ja,
                                               const Tensors& t, float* __restrict__ dq,
                                               int64_t r0, int head) {
  const ShortRow w(sm.seqs.short_row, r0);
  const int steps = rows_max(keys_of(w));
  if (!steps) return;
  constexpr int U = kShortStep<DQK, DV>;
  const int sub = threadIdx.x & 7, H = ja.num_heads, N = ja.max_seq_len;
  const float* kg = (const float*)t.k + head * DQK;
  const float* vg = (const float*)t.v + head * DV;
  f32x4 q[DQK / 32], g[DV / 32], acc[DQK / 32];
  load_slice<DQK>(sm.own_qk + (threadIdx.x >> 3) * (DQK + 4), sub, q);
  load_slice<DV>(sm.own_v + (threadIdx.x >> 3) * (DV + 4), sub, g);
#pragma unroll
  for (int e = 0; e < DQK / 32; e++) acc[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t ti = ja.timestamps[w.r];
  int run_b = -1;
  double run = 0.0;
  for (int d0 = 0; d0 < steps; d0 += U) {
    f32x4 k[U][DQK / 32], v[U][DV / 32];
    int64_t tj[U];
    float pos[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      ok[u] = d0 + u < keys_of(w);
      const int64_t r = ok[u] ? w.r + key_at(w, d0 + u) - w.i : w.r;
      load_slice<DQK>(kg + r * t.k_stride, sub, k[u]);
      load_slice<DV>(vg + r * t.v_stride, sub, v[u]);
      tj[u] = ja.timestamps[r];
      pos[u] = ja.rab_pos[max(N - 1 - d0 - u, 0)];
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int b = time_bucket64(ti - tj[u], ja.num_buckets);
      const float s = dot_slices<DQK>(q, k[u]) + (pos[u] + sm.tab[b]);
      const float dp = dot_slices<DV>(g, v[u]);
      double sum = 0.0;  // of the wave's rows
      if (ok[u]) {
        float p, ds;
        pair_grad(s, dp, &p, &ds);
        add_slice<DQK>(acc, ds, k[u]);
        sum = (double)ds;
        if (sub == 0) {
          if (b != run_b) {
            if (run_b >= 0) unsafeAtomicAdd(&sm.time_acc[run_b], run);
            run_b = b;
            run = 0.0;
          }
          run += sum;
        }
      }
#pragma unroll
      for (int off = 8; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
      if ((threadIdx.x & 63) == 0 && d0 + u < steps)
        unsafeAtomicAdd(&sm.short_pos[d0 + u], sum);
    }
  }
  if (run_b >= 0) unsafeAtomicAdd(&sm.time_acc[run_b], run);
  if (w.L) store_slice<DQK>(dq + (w.r * H + head) * DQK, sub, acc, 1.0f / (float)N);
}

// dK and dV of short rows (as keys).
template <int DQK, int DV>
__device__ __forceinline__ void short_bwd_keys(const BwdLds<DQK, DV>& sm, const JaggedArgs& ja,
                                               const Tensors& t, const float* __restrict__ dO,
                                               float* __restrict__ dk, float* __restrict__ dv,
                                               int64_t r0, int head) {
  const ShortRow w(sm.seqs.short_row, r0);
  const int count = !w.L ? 0 : w.i < w.n_h ? w.L - w.i : 1;  // rows that see the key
  const int steps = rows_max(count);
  if (!steps) return;
  constexpr int U = kShortStep<DQK, DV>;
  const int sub = threadIdx.x & 7, H = ja.num_heads, N = ja.max_seq_len;
  const float* qg = (const float*)t.q + head * DQK;
  const float* gg = dO + head * DV;
  const int64_t g_stride = (int64_t)H * DV;
  f32x4 k[DQK / 32], v[DV / 32], ak[DQK / 32], av[DV / 32];
  load_slice<DQK>(sm.own_qk + (threadIdx.x >> 3) * (DQK + 4), sub, k);
  load_slice<DV>(sm.own_v + (threadIdx.x >> 3) * (DV + 4), sub, v);
#pragma unroll
  for (int e = 0; e < DQK / 32; e++) ak[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int e = 0; e < DV / 32; e++) av[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t tj = ja.timestamps[w.r];
  for (int d0 = 0; d0 < steps; d0 += U) {
    f32x4 q[U][DQK / 32], g[U][DV / 32];
    int64_t ti[U];
    float pos[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      ok[u] = d0 + u < count;
      const int i = ok[u] ? w.i + d0 + u : w.i;
      const int64_t r = w.r + i - w.i;
      load_slice<DQK>(qg + r * t.q_stride, sub, q[u]);
      load_slice<DV>(gg + r * g_stride, sub, g[u]);
      ti[u] = ja.timestamps[r];
      pos[u] = ja.rab_pos[(N - 1) + bias_pos(w.i, w.n_h) - bias_pos(i, w.n_h)];
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const float s = dot_slices<DQK>(q[u], k) +
                      (pos[u] + sm.tab[time_bucket64(ti[u] - tj, ja.num_buckets)]);
      const float dp = dot_slices<DV>(g[u], v);
      if (ok[u]) {
        float p, ds;
        pair_grad(s, dp, &p, &ds);
        add_slice<DV>(av, p, g[u]);
        add_slice<DQK>(ak, ds, q[u]);
      }
    }
  }
  if (w.L) {
    store_slice<DQK>(dk + (w.r * H + head) * DQK, sub, ak, 1.0f / (float)N);
    store_slice<DV>(dv + (w.r * H + head) * DV, sub, av, 1.0f / (float)N);
  }
}

// Kind (a): dQ and the bias gradients of 32 query rows.
template <int DQK, int DV>
__device__ __forceinline__ void bwd_rows(BwdLds<DQK, DV>& sm, const JaggedArgs& ja,
                                         const Tensors& t, const float* __restrict__ dO,
                                         float* __restrict__ dq, double* __restrict__ pos_acc,
                                         double* __restrict__ time_acc, int64_t r0, int head) {
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
  const int64_t T = ja.total_tokens;
  const int H = ja.num_heads, N = ja.max_seq_len;
  const float* kg = (const float*)t.k + head * DQK;
  const float* vg = (const float*)t.v + head * DV;
  Walk w;
  w.start(ja, r0, false, sm.seqs);
  TileRegs<DQK> kr;
  TileRegs<DV> vr;
  SideRegs sr;
  auto load = [&](const Walk& x) {
    kr.load(kg + x.o * t.k_stride, t.k_stride, x.x0, x.L, tid);
    vr.load(vg + x.o * t.v_stride, t.v_stride, x.x0, x.L, tid);
    sr.load(ja, x, tid);
  };
  if (!w.done()) load(w);
  {
    const int rows = (int)min((int64_t)kRows, T - r0);
    TileRegs<DQK> qr;
    TileRegs<DV> gr;
    int ignored;
    qr.load((const float*)t.q + head * DQK + r0 * t.q_stride, t.q_stride, 0, rows, tid);
    gr.load(dO + (r0 * H + head) * DV, (int64_t)H * DV, 0, rows, tid);
    qr.store(sm.own_qk, tid, &ignored);
    gr.store(sm.own_v, tid, &ignored);
  }
  if (tid < min(ja.num_buckets, kBuckets)) sm.tab[tid] = ja.rab_time[tid];
  if (tid < kBuckets) sm.time_acc[tid] = 0.0;
  if (tid < kShort) sm.short_pos[tid] = 0.0;
  if (tid < 2) sm.special[tid] = 0;
  __syncthreads();
  const int64_t my_r = r0 + 16 * wr + n;
  const int64_t ti = ja.timestamps[min(my_r, T - 1)];
  f32x4 acc[DQK / 32];
#pragma unroll
  for (int nb = 0; nb < DQK / 32; nb++) acc[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  int run_b = -1;
  double run = 0.0;  // time-table sum of the thread's current bucket
  // Diagonals (wave 3): lane l % 32 = d owns offset i - j = (ra - x0) + d of
  // each tile, complete when the tile's d and the tile before's d - 32 are
  // added; the halves of the wave take 16 rows each.
  double carry = 0.0;
  const int dg = lane & 31;

  for (int par = 0; !w.done(); par ^= 1) {
    const Walk cur = w;
    kr.store(sm.tile_qk[par], tid, &sm.special[par]);
    vr.store(sm.tile_v[0], tid, &sm.special[par]);
    sr.store(sm.t, sm.win, tid);
    __syncthreads();
    if (tid == 0) sm.special[par ^ 1] = 0;
    w.next(sm.seqs);
    if (!w.done()) load(w);
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const f32x4 s = dot_tile<DQK>(sm.tile_qk[par] + 16 * wc * (DQK + 4),
                                  sm.own_qk + 16 * wr * (DQK + 4), lane, zero);
    const f32x4 dp = dot_tile<DV>(sm.tile_v[0] + 16 * wc * (DV + 4),
                                  sm.own_v + 16 * wr * (DV + 4), lane, zero);
    const int i = (int)(my_r - cur.o);
    const int wbase = (N - 1) - bias_pos(i, cur.n_h) - cur.window_base(N);
    const bool row_ok = i >= 0 && i < cur.L;
    f32x4 dsv;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int x = 16 * wc + 4 * g + r, j = cur.x0 + x;
      float ds = 0.0f;
      if (row_ok && pair_valid(i, j, cur.n_h)) {
        const int b = time_bucket64(ti - sm.t[x], ja.num_buckets);
        float p;
        pair_grad(s[r] + (sm.win[wbase + bias_pos(j, cur.n_h)] + sm.tab[b]), dp[r], &p, &ds);
        if (b != run_b) {
          if (run_b >= 0) unsafeAtomicAdd(&sm.time_acc[run_b], run);
          run_b = b;
          run = 0.0;
        }
        run += (double)ds;
      }
      dsv[r] = ds;
    }
    *reinterpret_cast<f32x4*>(sm.ds + (16 * wr + n) * kScoreLd + 16 * wc + 4 * g) = dsv;
    __syncthreads();
    const bool special = __builtin_amdgcn_readfirstlane(sm.special[par]) != 0;
    outer_tile<DQK>(sm.ds + 16 * wr * kScoreLd, sm.tile_qk[par], wc * (DQK / 2), lane, special,
                    [&](int row, int x) {
                      const int ii = (int)(r0 + 16 * wr + row - cur.o);
                      return ii >= 0 && ii < cur.L && pair_valid(ii, cur.x0 + x, cur.n_h);
                    },
                    acc);
    // Position table.  Tile row a (0..31) is row index ra' + a, ra' = r0 - o
    // (rows before the sequence hold zeros); only history rows and keys at
    // distinct positions enter the diagonals.
    const int base = (int)(r0 - cur.o);  // may be negative
    const int hist = min(max(cur.n_h - base, 0), kRows);  // rows a < hist are history
    if (wave == 3) {
      double now = 0.0, before = 0.0;
      for (int a = 16 * (lane >> 5); a < min(16 * (lane >> 5) + 16, hist); a++) {
        // offset (base + a) - (x0 + x) = (base - x0) + d, d = dg or dg - 32
        const int x = a - dg;
        if (x >= 0)
          now += (double)sm.ds[a * kScoreLd + x];
        else
          before += (double)sm.ds[a * kScoreLd + x + 32];
      }
      now += __shfl_xor(now, 32, 64);
      before += __shfl_xor(before, 32, 64);
      const double sum = now + carry;
      const int off = base - cur.x0 + dg;  // i - j
      if (lane < 32 && sum != 0.0 && off >= 0 && off < N)
        unsafeAtomicAdd(&pos_acc[(N - 1) - off], sum);
      // (sum may be NaN: it compares unequal to 0 and is added)
      carry = before;
      // The walk's last tile of this sequence: what was carried is complete.
      if (w.seq != cur.seq || w.x0 != cur.x0 + kRows) {
        const int last = off - 32;
        if (lane < 32 && carry != 0.0 && last >= 0 && last < N)
          unsafeAtomicAdd(&pos_acc[(N - 1) - last], carry);
        carry = 0.0;
      }
    } else if (wave == 2 && hist < kRows && cur.rb >= cur.n_h) {
      // Candidate rows: key x at offset n_h - p(x).
      double sum = 0.0;
      for (int a = max(hist, 0) + (lane >> 5); a < kRows; a += 2)
        sum += (double)sm.ds[a * kScoreLd + dg];
      sum += __shfl_xor(sum, 32, 64);
      const int off = cur.n_h - bias_pos(cur.x0 + dg, cur.n_h);
      if (lane < 32 && sum != 0.0) unsafeAtomicAdd(&pos_acc[(N - 1) - off], sum);
    }
  }
  if (run_b >= 0) unsafeAtomicAdd(&sm.time_acc[run_b], run);
  if (w.any_short) {
    __syncthreads();
    short_bwd_rows<DQK, DV>(sm, ja, t, dq, r0, head);
  }
  const float invN = 1.0f / (float)N;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int64_t row = r0 + 16 * wr + 4 * g + r;
    if (row < T && !(w.any_short && sm.seqs.short_row[16 * wr + 4 * g + r]))
#pragma unroll
      for (int nb = 0; nb < DQK / 32; nb++)
        dq[(row * H + head) * DQK + wc * (DQK / 2) + 16 * nb + n] = acc[nb][r] * invN;
  }
  __syncthreads();
  if (tid < kBuckets && sm.time_acc[tid] != 0.0)
    unsafeAtomicAdd(&time_acc[tid], sm.time_acc[tid]);
  if (tid < kShort && sm.short_pos[tid] != 0.0)
    unsafeAtomicAdd(&pos_acc[(N - 1) - tid], sm.short_pos[tid]);
}

// Kind (b): dK and dV of 32 key rows.
template <int DQK, int DV>
__device__ __forceinline__ void bwd_keys(BwdLds<DQK, DV>& sm, const JaggedArgs& ja,
                                         const Tensors& t, const float* __restrict__ dO,
                                         float* __restrict__ dk, float* __restrict__ dv,
                                         int64_t r0, int head) {
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave >> 1, wc = wave & 1;
  const int64_t T = ja.total_tokens;
  const int H = ja.num_heads, N = ja.max_seq_len;
  const float* qg = (const float*)t.q + head * DQK;
  const float* gg = dO + head * DV;
  const int64_t g_stride = (int64_t)H * DV;
  Walk w;
  w.start(ja, r0, true, sm.seqs);
  TileRegs<DQK> qr;
  TileRegs<DV> gr;
  SideRegs sr;
  auto load = [&](const Walk& x) {
    qr.load(qg + x.o * t.q_stride, t.q_stride, x.x0, x.L, tid);
    gr.load(gg + x.o * g_stride, g_stride, x.x0, x.L, tid);
    sr.load(ja, x, tid);
  };
  if (!w.done()) load(w);
  {
    const int rows = (int)min((int64_t)kRows, T - r0);
    TileRegs<DQK> kr;
    TileRegs<DV> vr;
    int ignored;
    kr.load((const float*)t.k + head * DQK + r0 * t.k_stride, t.k_stride, 0, rows, tid);
    vr.load((const float*)t.v + head * DV + r0 * t.v_stride, t.v_stride, 0, rows, tid);
    kr.store(sm.own_qk, tid, &ignored);
    vr.store(sm.own_v, tid, &ignored);
  }
  if (tid < min(ja.num_buckets, kBuckets)) sm.tab[tid] = ja.rab_time[tid];
  if (tid < 2) sm.special[tid] = 0;
  __syncthreads();
  const int64_t my_r = r0 + 16 * wr + n;  // the lane's key
  const int64_t tj = ja.timestamps[min(my_r, T - 1)];
  f32x4 ak[DQK / 32], av[DV / 32];
#pragma unroll
  for (int nb = 0; nb < DQK / 32; nb++) ak[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int nb = 0; nb < DV / 32; nb++) av[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  for (int par = 0; !w.done(); par ^= 1) {
    const Walk cur = w;
    qr.store(sm.tile_qk[par], tid, &sm.special[par]);
    gr.store(sm.tile_v[par], tid, &sm.special[par]);
    sr.store(sm.t, sm.win, tid);
    __syncthreads();
    if (tid == 0) sm.special[par ^ 1] = 0;
    w.next(sm.seqs);
    if (!w.done()) load(w);
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const f32x4 s = dot_tile<DQK>(sm.tile_qk[par] + 16 * wc * (DQK + 4),
                                  sm.own_qk + 16 * wr * (DQK + 4), lane, zero);
    const f32x4 dp = dot_tile<DV>(sm.tile_v[par] + 16 * wc * (DV + 4),
                                  sm.own_v + 16 * wr * (DV + 4), lane, zero);
    const int j = (int)(my_r - cur.o);
    const int wbase = (N - 1) + bias_pos(j, cur.n_h) - cur.window_base(N);
    const bool key_ok = j >= 0 && j < cur.L;
    f32x4 pv, dsv;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int x = 16 * wc + 4 * g + r, i = cur.x0 + x;
      float p = 0.0f, ds = 0.0f;
      if (key_ok && i < cur.L && pair_valid(i, j, cur.n_h)) {
        const int b = time_bucket64(sm.t[x] - tj, ja.num_buckets);
        pair_grad(s[r] + (sm.win[wbase - bias_pos(i, cur.n_h)] + sm.tab[b]), dp[r], &p, &ds);
      }
      pv[r] = p;
      dsv[r] = ds;
    }
    const int so = (16 * wr + n) * kScoreLd + 16 * wc + 4 * g;  // [key][row]
    *reinterpret_cast<f32x4*>(sm.p + so) = pv;
    *reinterpret_cast<f32x4*>(sm.ds + so) = dsv;
    __syncthreads();
    const bool special = __builtin_amdgcn_readfirstlane(sm.special[par]) != 0;
    auto keep = [&](int row, int x) {
      const int jj = (int)(r0 + 16 * wr + row - cur.o), i = cur.x0 + x;
      return jj >= 0 && i < cur.L && pair_valid(i, jj, cur.n_h);
    };
    outer_tile<DV>(sm.p + 16 * wr * kScoreLd, sm.tile_v[par], wc * (DV / 2), lane, special, keep,
                   av);
    outer_tile<DQK>(sm.ds + 16 * wr * kScoreLd, sm.tile_qk[par], wc * (DQK / 2), lane, special,
                    keep, ak);
  }
  if (w.any_short) {
    __syncthreads();
    short_bwd_keys<DQK, DV>(sm, ja, t, dO, dk, dv, r0, head);
  }
  const float invN = 1.0f / (float)N;
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int64_t row = r0 + 16 * wr + 4 * g + r;
    if (row < T && !(w.any_short && sm.seqs.short_row[16 * wr + 4 * g + r])) {
#pragma unroll
      for (int nb = 0; nb < DQK / 32; nb++)
        dk[(row * H + head) * DQK + wc * (DQK / 2) + 16 * nb + n] = ak[nb][r] * invN;
#pragma unroll
      for (int nb = 0; nb < DV / 32; nb++)
        dv[(row * H + head) * DV + wc * (DV / 2) + 16 * nb + n] = av[nb][r] * invN;
    }
  }
}

template <int DQK, int DV>
__global__ __launch_bounds__(kThreads) void bwd_f32_kernel(JaggedArgs ja, Tensors t,
                                                           const float* dO, float* dq, float* dk,
                                                           float* dv, double* pos_acc,
                                                           double* time_acc) {
  __shared__ BwdLds<DQK, DV> sm;
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  if (blockIdx.z == 0)
    bwd_rows<DQK, DV>(sm, ja, t, dO, dq, pos_acc, time_acc, r0, blockIdx.y);
  else
    bwd_keys<DQK, DV>(sm, ja, t, dO, dk, dv, r0, blockIdx.y);
}

__global__ __launch_bounds__(256) void f64_to_f32_kernel(const double* in, float* a, int64_t na,
                                                         float* b, int64_t nb, double scale) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < na + nb;
       i += (int64_t)gridDim.x * 256) {
    const float v = (float)(in[i] * scale);
    if (i < na)
      a[i] = v;
    else
      b[i - na] = v;
  }
}

}  // namespace

#define HSTU_F32_DISPATCH(CALL)      \
  if (dqk == 32 && dv == 32) CALL(32, 32)   \
  if (dqk == 32 && dv == 64) CALL(32, 64)   \
  if (dqk == 32 && dv == 128) CALL(32, 128) \
  if (dqk == 64 && dv == 32) CALL(64, 32)   \
  if (dqk == 64 && dv == 64) CALL(64, 64)   \
  if (dqk == 64 && dv == 128) CALL(64, 128) \
  if (dqk == 128 && dv == 32) CALL(128, 32) \
  if (dqk == 128 && dv == 64) CALL(128, 64) \
  if (dqk == 128 && dv == 128) CALL(128, 128)

hipError_t launch_attn_fwd_f32(const JaggedArgs& ja, const Tensors& t, int dqk, int dv, void* out,
                               hipStream_t s) {
  if (ja.total_tokens <= 0) return hipSuccess;
  const dim3 grid((unsigned)((ja.total_tokens + kRows - 1) / kRows), (unsigned)ja.num_heads);
#define CALL(A, B)                                                                           \
  {                                                                                          \
    hipLaunchKernelGGL((fwd_f32_kernel<A, B>), grid, dim3(kThreads), 0, s, ja, t,             \
                       (float*)out);                                                         \
    return hipGetLastError();                                                                \
  }
  HSTU_F32_DISPATCH(CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_f64_to_f32_scaled(const double* in, float* a, int64_t na, float* b, int64_t nb,
                                    double scale, hipStream_t s) {
  if (na + nb <= 0) return hipSuccess;
  const int64_t blocks = (na + nb + 255) / 256;
  hipLaunchKernelGGL(f64_to_f32_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256),
                     0, s, in, a, na, b, nb, scale);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const JaggedArgs& ja, const Tensors& t, int dqk, int dv,
                               const void* d_out, void* dq, void* dk, void* dv_out,
                               double* rab_pos_acc, double* rab_time_acc, hipStream_t s) {
  if (ja.total_tokens <= 0) return hipSuccess;
  const dim3 grid((unsigned)((ja.total_tokens + kRows - 1) / kRows), (unsigned)ja.num_heads, 2);
#define CALL(A, B)                                                                            \
  {                                                                                           \
    hipLaunchKernelGGL((bwd_f32_kernel<A, B>), grid, dim3(kThreads), 0, s, ja, t,              \
                       (const float*)d_out, (float*)dq, (float*)dk, (float*)dv_out,           \
                       rab_pos_acc, rab_time_acc);                                            \
    return hipGetLastError();                                                                 \
  }
  HSTU_F32_DISPATCH(CALL)
#undef CALL
  return hipErrorInvalidValue;
}

}  // namespace hstu
