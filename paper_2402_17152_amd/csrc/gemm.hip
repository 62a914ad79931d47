// Dense products of the layer's two linear maps: f_1 of Eq. 1 (with the
// SiLU of phi_1 and the bias in the epilogue, output split U|V|Q|K by
// columns) and f_2 of Eq. 3 (bias and the residual connection in the
// epilogue), with their input and weight gradients.
//
// All are C[m][n] = sum_k A(m, k) B(n, k) over bf16 operands with fp32
// accumulation on v_mfma_f32_32x32x16_bf16.  An operand is stored either
// k-contiguous (A[m][k], B[n][k]: activations and [out][in] weights in the
// forward) or k-major (A[k][m], B[k][n]: the transposed operands of the
// gradients).  A workgroup computes a 256 x 256 tile with 8 waves (the
// products without a SiLU), a 256 x 128 tile with 4 (f_1's forward), or, when
// those would not fill the chip, a 128 x 128 tile with 4; each wave 128 x 64
// (64 x 64), over k-steps of 32.  A k-contiguous tile gives a lane its 8
// contraction elements in one 16-byte LDS read; a k-major tile is read with
// two transposing reads (ds_read_b64_tr_b16) that return the same 8 elements
// in the same order.  The products are computed transposed (B's fragment as
// the matrix core's first operand), so a lane owns one output row and 4
// consecutive columns per register group.
//
// Staging: LDS DMA into a ring of three k-steps (four, 131 KB, for 256 x 256
// tiles), issued as many steps ahead less at most one, in a layout without
// padding whose 16-byte chunks are permuted so that every LDS read spreads
// over all banks.  The fragments of a half step are read while the matrix
// cores work on the half step before, across the one barrier per step, so
// neither the LDS nor the memory latency is in the chain.  Of the 4-wave
// tiles two workgroups share a CU and overlap one's epilogue with the
// other's products; a 256 x 256 tile has a CU to itself.
//
// Weight gradients split the contraction over the tokens; each split
// writes an fp32 slab and an ordered reduction sums the slabs, so results
// do not depend on scheduling.
#include "bias.h"
#include "kernels.h"

namespace hstu {

namespace {

constexpr int kGBK = 32;

// A workgroup of 2 x WN waves, each MB 32-row blocks by 64 columns: the tile
// is BM = 64 MB rows by BN = 64 WN columns; ring of S k-steps in LDS.
template <int MB, int WN, int S>
struct GemmShared {
  static constexpr int kA = 64 * MB * kGBK, kB = 64 * WN * kGBK;  // elements
  __align__(16) uint16_t t[S][kA + kB];
};

__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * -kLog2e));
}

// One operand tile in LDS: R rows of the m or n dimension x 32 of k, in
// 16-byte chunks.  k-contiguous: [row][4 chunks], chunk c of row r at
// position c ^ (r / 4 % 4).  k-major: [k][R / 8 chunks], chunk c of row k at
// c ^ 4 (k % 4).  Either way 16 (32) lanes of a 16-byte (transposing 8-byte)
// read meet all 64 banks.
template <bool KMAJOR, int R, int WAVES>
struct Operand {
  static constexpr int kOps = R * kGBK * 2 / 1024 / WAVES;  // 1 KB DMA operations per wave
  u32x4 rs;           // buffer resource words
  uint32_t ld_b;      // row stride in bytes
  uint32_t off[kOps]; // the lane's byte offsets at k = 0
  uint32_t rd[2];     // k-contiguous: LDS byte offsets of the two half steps
                      // k-major: [0] the lane's, without its 32-row block
  uint32_t x;         // k-major: the lane's k % 4

  __device__ __forceinline__ void init(const uint16_t* base, uint32_t bytes, int64_t ld, int wave,
                                       int lane) {
    rs = rsrc_words(base, bytes);
    ld_b = (uint32_t)ld * 2u;
    const int h = lane >> 5;
#pragma unroll
    for (int e = 0; e < kOps; e++) {
      const int op = wave * kOps + e;
      if constexpr (KMAJOR) {
        constexpr int kRowChunks = R / 8, kRowsPerOp = 64 / kRowChunks;
        const int k = op * kRowsPerOp + lane / kRowChunks;
        const int c = (lane % kRowChunks) ^ (4 * (k & 3));
        off[e] = (uint32_t)k * ld_b + 16u * (uint32_t)c;
      } else {
        const int row = 16 * op + (lane >> 2), c = (lane & 3) ^ ((row >> 2) & 3);
        off[e] = (uint32_t)row * ld_b + 16u * (uint32_t)c;
      }
    }
    if constexpr (KMAJOR) {
      x = (uint32_t)(lane >> 2) & 3u;
      rd[0] = (uint32_t)((8 * h + (int)x) * R * 2 + 32 * ((lane >> 4) & 1) + 8 * (lane & 3));
      rd[1] = 0;
    } else {
#pragma unroll
      for (int s = 0; s < 2; s++)
        rd[s] = (uint32_t)((lane & 31) * 64 + 16 * ((2 * s + h) ^ ((lane >> 2) & 3)));
      x = 0;
    }
  }
  // Issues the wave's share of the k-step starting at k0 into tile `t`.
  __device__ __forceinline__ void issue(uint16_t* t, int k0, int wave) const {
    const uint32_t kb = KMAJOR ? (uint32_t)k0 * ld_b : 2u * (uint32_t)k0;
    uint32_t l[kOps], o[kOps];
#pragma unroll
    for (int e = 0; e < kOps; e++) {
      l[e] = lds_addr(t + 512 * (wave * kOps + e));
      o[e] = off[e] + kb;
    }
    dma_to_lds16_asm(rs, l, o);
  }
  // MFMA operand of the 32 rows of block `blk` for the half step s: lane ->
  // row lane % 32, k = 16 s + 8 (lane / 32) .. +7.
  __device__ __forceinline__ u32x4 frag(const uint16_t* t, int blk, int s) const {
    const char* p = reinterpret_cast<const char*>(t);
    if constexpr (KMAJOR) {
      const char* q = p + rd[0] + 64u * ((uint32_t)blk ^ x) + 16 * s * R * 2;
      const uint2 lo = lds_read_tr16(reinterpret_cast<const uint16_t*>(q));
      const uint2 hi = lds_read_tr16(reinterpret_cast<const uint16_t*>(q + 4 * R * 2));
      return u32x4{lo.x, lo.y, hi.x, hi.y};
    } else {
      return *reinterpret_cast<const u32x4*>(p + rd[s] + blk * (32 * 64));
    }
  }
};

template <int MB, int WN, int S, bool A_KM, bool B_KM, int EPI, bool STREAM>
__global__ __launch_bounds__(128 * WN, 2) void gemm_bf16_kernel(GemmArgs g) {
  using Sh = GemmShared<MB, WN, S>;
  __shared__ Sh sm;
  constexpr int BM = 64 * MB, BN = 64 * WN;
  using OA = Operand<A_KM, BM, 2 * WN>;
  using OB = Operand<B_KM, BN, 2 * WN>;
  constexpr int kOps = OA::kOps + OB::kOps;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;  // wave tile: rows 32 MB wm .., columns 64 wn ..
  // Tile order: consecutive tiles (same row panel of A, n fastest) go to
  // one XCD (workgroup ids are dealt to the 8 XCDs round robin).
  const int tn = (g.N + BN - 1) / BN, nt = ((g.M + BM - 1) / BM) * tn;
  const int id = blockIdx.x, xcd = id & 7, per = nt >> 3, rem = nt & 7;
  const int tile = xcd * per + min(xcd, rem) + (id >> 3);
  const int m0 = (tile / tn) * BM, n0 = (tile % tn) * BN;
  const int kb = blockIdx.y * g.k_split;
  const int ke = min(g.K, kb + g.k_split);
  const int nk = (ke - kb + kGBK - 1) / kGBK;

  // Buffer ranges: rows past M / N (k-contiguous) and contraction rows at
  // or past ke (k-major) read as zeros; k-major columns past M / N read
  // neighbouring data that only reaches outputs that are not stored.
  OA oa;
  OB ob;
  if constexpr (A_KM)
    oa.init(g.a + m0, (uint32_t)(((int64_t)(ke - 1) * g.lda + (g.M - m0)) * 2), g.lda, wave, lane);
  else
    oa.init(g.a + (int64_t)m0 * g.lda,
            (uint32_t)(((int64_t)(min(g.M - m0, BM) - 1) * g.lda + g.K) * 2), g.lda, wave, lane);
  if constexpr (B_KM)
    ob.init(g.b + n0, (uint32_t)(((int64_t)(ke - 1) * g.ldb + (g.N - n0)) * 2), g.ldb, wave, lane);
  else
    ob.init(g.b + (int64_t)n0 * g.ldb,
            (uint32_t)(((int64_t)(min(g.N - n0, BN) - 1) * g.ldb + g.K) * 2), g.ldb, wave, lane);

  f32x16 acc[MB][2];
#pragma unroll
  for (int i = 0; i < MB; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int q = 0; q < 16; q++) acc[i][j][q] = 0.0f;

  // Steps go in ascending order in every tile and tile size: an output row of
  // the maps then has the same bits wherever it lies in a batch, as keys and
  // values cached from one batch and used with another need.
  int k_next = kb;
  auto issue = [&](int st) {
    oa.issue(sm.t[st], k_next, wave);
    ob.issue(sm.t[st] + Sh::kA, k_next, wave);
    k_next += kGBK;
  };

  u32x4 af[2][MB], bf[2][2];
  auto read = [&](int st, int s) {
    const uint16_t* ta = sm.t[st];
#pragma unroll
    for (int j = 0; j < 2; j++) bf[s][j] = ob.frag(ta + Sh::kA, 2 * wn + j, s);
#pragma unroll
    for (int i = 0; i < MB; i++) af[s][i] = oa.frag(ta, MB * wm + i, s);
  };
  auto product = [&](int s) {
#pragma unroll
    for (int i = 0; i < MB; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
        acc[i][j] = mfma32x32x16(as_bf16x8(bf[s][j]), as_bf16x8(af[s][i]), acc[i][j]);
  };
  // Every wave issues kOps operations per step, in step order, so a count
  // of outstanding ones tells which steps have landed.
  auto wait_all_but = [&](int steps) {  // until at most `steps` steps (< S) are in flight
    if (S > 3 && steps >= 3)
      wait_vmcnt_lgkmcnt0<3 * kOps>();
    else if (steps >= 2)
      wait_vmcnt_lgkmcnt0<2 * kOps>();
    else if (steps == 1)
      wait_vmcnt_lgkmcnt0<kOps>();
    else
      wait_vmcnt_lgkmcnt0<0>();
  };
  const int ahead = min(nk, S);
  for (int kt = 0; kt < ahead; kt++) issue(kt);
  wait_all_but(ahead - 1);
  barrier_no_fence();
  int st = 0;
  if (nk > 0) {
    read(0, 0);
    // (The last step stands outside the loop: on a path that joined it
    // without the wait below, product(1) would wait for the reads after it.)
    for (int kt = 0; kt + 1 < nk; kt++) {
      read(st, 1);
      product(0);
      // Step kt + 1 has landed (later ones may be in flight), and this wave
      // has its fragments of step kt; past the barrier every wave does, and
      // the step's place in the ring is free.
      if (kt + S <= nk)
        wait_vmcnt_lgkmcnt0<(S - 2) * kOps>();
      else
        wait_all_but(nk - kt - 2);
      barrier_no_fence();
      if (kt + S < nk) issue(st);
      st = st == S - 1 ? 0 : st + 1;
      read(st, 0);
      product(1);
    }
    read(st, 1);
    product(0);
    product(1);
  }
  // The epilogue's LDS overlays the ring: no wave may still read it.
  wait_vmcnt_lgkmcnt0<0>();
  barrier_no_fence();

  // Epilogue, per group of 32 rows: the wave writes its 32 x 64 fp32 block
  // to a private LDS region (acc[i][j] register 4 g4 + e is row lane % 32,
  // column 32 j + 8 g4 + 4 h + e), then each lane takes 8 consecutive
  // columns of a row back, applies bias / SiLU / residual and stores 16
  // bytes: a store instruction covers 8 rows x 128 contiguous bytes.  (LDS
  // operations of one wave complete in order.)
  constexpr int kEpLd = 64 + 4;
  float* ep = reinterpret_cast<float*>(&sm) + wave * (32 * kEpLd);
  const int h = lane >> 5;
  const int mr = m0 + 32 * MB * wm + (lane >> 3);  // the lane's first row
  const int cc = lane & 7, n = n0 + 64 * wn + 8 * cc;
  const bool n_ok = n < g.N;
  // The bias of the lane's columns, and the residual rows one 32-row block
  // ahead of their use (loads only: clamped into range).
  float bv[8] = {};
  u32x4 rv[2][4] = {};
  auto load_res = [&](int i) {
#pragma unroll
    for (int r = 0; r < 4; r++)
      rv[i & 1][r] = *reinterpret_cast<const u32x4*>(
          g.res + (int64_t)min(mr + 32 * i + 8 * r, g.M - 1) * g.ldr + min(n, g.N - 8));
  };
  const bool has_res = EPI == kEpiAdd && g.res;
  if constexpr (EPI != kEpiSlab) {
    if (has_res) load_res(0);
    if (g.bias) {
      const f32x4 b0 = *reinterpret_cast<const f32x4*>(g.bias + min(n, g.N - 8));
      const f32x4 b1 = *reinterpret_cast<const f32x4*>(g.bias + min(n, g.N - 8) + 4);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        bv[e] = b0[e];
        bv[4 + e] = b1[e];
      }
    }
  }
  auto store = [&](uint16_t* p, const float (&v)[8]) {
    const u32x4 o = pack_bf16x8(v);
    if constexpr (STREAM)
      __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(p));
    else
      *reinterpret_cast<u32x4*>(p) = o;
  };
#pragma unroll
  for (int i = 0; i < MB; i++) {
    if constexpr (EPI == kEpiAdd)
      if (has_res && i + 1 < MB) load_res(i + 1);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int g4 = 0; g4 < 4; g4++) {
        const f32x4 v = {acc[i][j][4 * g4], acc[i][j][4 * g4 + 1], acc[i][j][4 * g4 + 2],
                         acc[i][j][4 * g4 + 3]};
        *reinterpret_cast<f32x4*>(ep + (lane & 31) * kEpLd + 32 * j + 8 * g4 + 4 * h) = v;
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = (lane >> 3) + 8 * r, m = mr + 32 * i + 8 * r;
      const f32x4 lo = *reinterpret_cast<const f32x4*>(ep + row * kEpLd + 8 * cc);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(ep + row * kEpLd + 8 * cc + 4);
      if (m >= g.M || !n_ok) continue;
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      if constexpr (EPI == kEpiSlab) {
        float* o = g.slab + ((int64_t)blockIdx.y * g.M + m) * g.N + n;
        *reinterpret_cast<f32x4*>(o) = lo;
        *reinterpret_cast<f32x4*>(o + 4) = hi;
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] += bv[e];
        if constexpr (EPI == kEpiSilu) {
          if (g.c2) store(g.c2 + (int64_t)m * g.ldc2 + n, v);
#pragma unroll
          for (int e = 0; e < 8; e++) v[e] = silu_f(v[e]);
        } else if (has_res) {
#pragma unroll
          for (int e = 0; e < 4; e++) {
            v[2 * e] += __uint_as_float(rv[i & 1][r][e] << 16);
            v[2 * e + 1] += __uint_as_float(rv[i & 1][r][e] & 0xffff0000u);
          }
        }
        store(g.c + (int64_t)m * g.ldc + n, v);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// fp32 problems (small shapes): a plain tiled product on the vector ALUs,
// 64 x 64 tile per workgroup, 4 x 4 outputs per thread, any strides.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgsF32 g) {
  __shared__ float As[16][65], Bs[16][65];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < g.K; k0 += 16) {
    for (int x = tid; x < 16 * 64; x += 256) {
      const int kk = x >> 6, r = x & 63;
      const int k = k0 + kk, m = m0 + r, n = n0 + r;
      As[kk][r] = (k < g.K && m < g.M) ? g.a[(int64_t)m * g.sam + (int64_t)k * g.sak] : 0.0f;
      Bs[kk][r] = (k < g.K && n < g.N) ? g.b[(int64_t)n * g.sbn + (int64_t)k * g.sbk] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; kk++)
#pragma unroll
      for (int a = 0; a < 4; a++)
#pragma unroll
        for (int b = 0; b < 4; b++) acc[a][b] += As[kk][ty + 16 * a] * Bs[kk][tx + 16 * b];
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 4; a++)
#pragma unroll
    for (int b = 0; b < 4; b++) {
      const int m = m0 + ty + 16 * a, n = n0 + tx + 16 * b;
      if (m >= g.M || n >= g.N) continue;
      float v = acc[a][b];
      if constexpr (EPI == kEpiSlab) {
        g.c[(int64_t)m * g.ldc + n] = v;
      } else {
        if (g.bias) v += g.bias[n];
        if constexpr (EPI == kEpiSilu) {
          if (g.c2) g.c2[(int64_t)m * g.ldc2 + n] = v;
          v = v / (1.0f + expf(-v));
        } else if (g.res) {
          v += g.res[(int64_t)m * g.ldr + n];
        }
        g.c[(int64_t)m * g.ldc + n] = v;
      }
    }
}

// dpre = dZ * SiLU'(pre), dZ = [dU | dV | dQ | dK] from four dense
// [T][h][d] gradients, and partial column sums of the fp32 dpre for the
// bias gradient, one row of partials per block of kColRows token rows.
// HBM-bound.  A thread owns 8 consecutive columns (16-byte accesses in bf16;
// the four sources meet at multiples of 32 columns, so 8 columns never
// straddle two) of kColRows / 4 rows, all of whose loads are in flight at
// once; its workgroup's four row groups meet in LDS.  (One thread per 8
// columns and 32 rows: 27 us on 4.8 K tokens of 1024 columns, too few loads
// in flight.)
// NT: inputs of half the last-level cache and more are read past it, so that
// it keeps what the products read next.  The whole backward with ordinary
// against such reads (us; 1024, 2048, 4096 columns), by the inputs' MB, the
// same whether the gradients were just written or not:
//   96: 92 / 96, 114 / 116, 160 / 163     112: level
//   128: 116 / 111, 141 / 140, 203 / 200  192: 165 / 146, 205 / 189, 295 / 280
//   512: 355 / 342, 439 / 434, 646 / 636
constexpr int kColRows = 32;

template <bool BF16>
__device__ __forceinline__ void load8(const void* p, int64_t i, float (&v)[8]) {
  if constexpr (BF16) {
    const u32x4 r = *reinterpret_cast<const u32x4*>((const uint16_t*)p + i);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      v[2 * e] = __uint_as_float(r[e] << 16);
      v[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u);
    }
  } else {
    const f32x4 a = *reinterpret_cast<const f32x4*>((const float*)p + i);
    const f32x4 b = *reinterpret_cast<const f32x4*>((const float*)p + i + 4);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      v[e] = a[e];
      v[4 + e] = b[e];
    }
  }
}

template <bool BF16>
__device__ __forceinline__ void store8(void* p, int64_t i, const float (&v)[8]) {
  if constexpr (BF16) {
    const u32x4 r = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                     pack_bf16x2(v[6], v[7])};
    *reinterpret_cast<u32x4*>((uint16_t*)p + i) = r;
  } else {
    const f32x4 a = {v[0], v[1], v[2], v[3]}, b = {v[4], v[5], v[6], v[7]};
    *reinterpret_cast<f32x4*>((float*)p + i) = a;
    *reinterpret_cast<f32x4*>((float*)p + i + 4) = b;
  }
}

template <bool BF16, bool NT>
__device__ __forceinline__ void load8_once(const void* p, int64_t i, float (&v)[8]) {
  if constexpr (BF16 && NT) {
    const u32x4 r =
        __builtin_nontemporal_load(reinterpret_cast<const u32x4*>((const uint16_t*)p + i));
#pragma unroll
    for (int e = 0; e < 4; e++) {
      v[2 * e] = __uint_as_float(r[e] << 16);
      v[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u);
    }
  } else {
    load8<BF16>(p, i, v);
  }
}

// Sums over the workgroup's four row groups (waves) of each wave's 512
// columns, stored to one row of partials.
__device__ __forceinline__ void store_col_sums(float (*red)[512], const float (&sum)[8], int c0,
                                               int n, float* __restrict__ partial_row) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  store8<false>(red[wave], 8 * lane, sum);
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; e++) {
    const int x = threadIdx.x + 256 * e;
    if (c0 + x < n) partial_row[c0 + x] = (red[0][x] + red[1][x]) + (red[2][x] + red[3][x]);
  }
}

template <bool BF16, bool NT>
__global__ __launch_bounds__(256) void silu_bwd_kernel(int64_t T, int F, int hv, int hq,
                                                       const void* __restrict__ pre,
                                                       const void* __restrict__ du,
                                                       const void* __restrict__ dv,
                                                       const void* __restrict__ dq,
                                                       const void* __restrict__ dk,
                                                       void* __restrict__ dpre,
                                                       float* __restrict__ partial) {
  __shared__ __align__(16) float red[4][512];
  constexpr int kPer = kColRows / 4;
  const int c0 = 512 * blockIdx.x, c = c0 + 8 * (threadIdx.x & 63);
  float sum[8] = {};
  if (c < F) {
    const void* src;
    int w, cc;
    if (c < hv) {
      src = du, w = hv, cc = c;
    } else if (c < 2 * hv) {
      src = dv, w = hv, cc = c - hv;
    } else if (c < 2 * hv + hq) {
      src = dq, w = hq, cc = c - 2 * hv;
    } else {
      src = dk, w = hq, cc = c - 2 * hv - hq;
    }
    const int64_t r0 = (int64_t)blockIdx.y * kColRows + (threadIdx.x >> 6) * kPer;
    float x[kPer][8], d[kPer][8];
#pragma unroll
    for (int k = 0; k < kPer; k++) {
      const int64_t r = min(r0 + k, T - 1);
      load8_once<BF16, NT>(pre, r * F + c, x[k]);
      load8_once<BF16, NT>(src, r * w + cc, d[k]);
    }
#pragma unroll
    for (int k = 0; k < kPer; k++) {
      if (r0 + k >= T) break;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x[k][e] * -kLog2e));
        d[k][e] *= sg * (1.0f + x[k][e] * (1.0f - sg));
        sum[e] += d[k][e];
      }
      store8<BF16>(dpre, (r0 + k) * F + c, d[k]);
    }
  }
  store_col_sums(red, sum, c0, F, partial + (int64_t)blockIdx.y * F);
}

// Partial column sums of x [T][N] (row stride ld, N and ld multiples of 8)
// per block of kColRows rows.
template <bool BF16>
__global__ __launch_bounds__(256) void colsum_kernel(int64_t T, int N, int64_t ld,
                                                     const void* __restrict__ x,
                                                     float* __restrict__ partial) {
  __shared__ __align__(16) float red[4][512];
  constexpr int kPer = kColRows / 4;
  const int c0 = 512 * blockIdx.x, c = c0 + 8 * (threadIdx.x & 63);
  float sum[8] = {};
  if (c < N) {
    const int64_t r0 = (int64_t)blockIdx.y * kColRows + (threadIdx.x >> 6) * kPer;
    float v[kPer][8];
#pragma unroll
    for (int k = 0; k < kPer; k++) load8<BF16>(x, min(r0 + k, T - 1) * ld + c, v[k]);
#pragma unroll
    for (int k = 0; k < kPer; k++)
      if (r0 + k < T)
#pragma unroll
        for (int e = 0; e < 8; e++) sum[e] += v[k][e];
  }
  store_col_sums(red, sum, c0, N, partial + (int64_t)blockIdx.y * N);
}

// out[i] = sum over s of part[s][i], s in order (few rows, many columns:
// the split-K slabs), n a multiple of 4.  Four columns per thread and eight
// slabs' loads in flight: one column and one load at a time took 7 us for 19
// slabs of 1 MB.
__global__ __launch_bounds__(256) void reduce_slabs_kernel(int64_t n, int S,
                                                           const float* __restrict__ part,
                                                           float* __restrict__ out) {
  for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < n;
       i += 4 * (int64_t)gridDim.x * 256) {
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
    int k = 0;
    for (; k + 8 <= S; k += 8) {
      f32x4 v[8];
#pragma unroll
      for (int e = 0; e < 8; e++)
        v[e] = *reinterpret_cast<const f32x4*>(part + (int64_t)(k + e) * n + i);
#pragma unroll
      for (int e = 0; e < 8; e++) s += v[e];
    }
#pragma unroll 4
    for (; k < S; k++) s += *reinterpret_cast<const f32x4*>(part + (int64_t)k * n + i);
    *reinterpret_cast<f32x4*>(out + i) = s;
  }
}

// The same sum for many rows and few columns (bias partials): a block owns
// 16 columns; its 16 row groups each sum every 16th row, then the group
// sums are added in group order.  The order is fixed, so the result is.
__global__ __launch_bounds__(256) void reduce_cols_kernel(int n, int S,
                                                          const float* __restrict__ part,
                                                          float* __restrict__ out) {
  __shared__ float red[16][17];
  const int col = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + col;
  float s = 0.0f;
  if (i < n) {
#pragma unroll 8
    for (int k = grp; k < S; k += 16) s += part[(int64_t)k * n + i];
  }
  red[grp][col] = s;
  __syncthreads();
  if (grp == 0 && i < n) {
    float t = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; q++) t += red[q][col];
    out[i] = t;
  }
}

}  // namespace

int gemm_num_splits(int M, int N, int64_t K, int* k_split) {
  const int tiles = ((M + 255) / 256) * ((N + 255) / 256);
  int64_t want = (256 + tiles - 1) / tiles;
  // About 256 contraction rows per split at least (K = 257 makes splits of
  // 160 and 97), and at least one split.
  const int64_t max_splits = K > 256 ? (K + 255) / 256 : 1;
  want = want < 1 ? 1 : want > max_splits ? max_splits : want;
  int64_t ks = (K + want - 1) / want;
  ks = (ks + kGBK - 1) / kGBK * kGBK;
  if (ks < kGBK) ks = kGBK;
  *k_split = (int)ks;
  return (int)((K + ks - 1) / ks);
}

template <bool A_KM, bool B_KM, int EPI>
hipError_t gemm_case(const GemmArgs& g, int splits, hipStream_t s) {
  auto tiles = [&](int bm, int bn) {
    return (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn);
  };
  auto launch = [&](auto kernel, int bm, int bn) {
    const dim3 grid((unsigned)tiles(bm, bn), (unsigned)splits);
    hipLaunchKernelGGL(kernel, grid, dim3(2 * bn), 0, s, g);
    return hipGetLastError();
  };
  // Outputs past half of the 256 MB last-level cache bypass the caches; smaller
  // ones may be read from them by the next call.  f_1's forward at 2048 columns
  // with ordinary against bypassing stores (us), alone, then with a pass that
  // reads z after it, by the MB of z and z_pre:
  //   64: 30 / 29, 43 / 44      128: 55 / 53, 76 / 76    192: 81 / 80, 122 / 110
  //   256: 123 / 102, 164 / 162    512: 259 / 200, 344 / 337
  // f_2's y, alone: 64 MB 34 / 31, 160 MB 90 / 69, 384 MB 203 / 199.
  const bool stream =
      EPI != kEpiSlab && 2ll * g.M * g.N * (g.c2 ? 2 : 1) > (128ll << 20);
  constexpr bool kStream = EPI != kEpiSlab;
  // The largest tile that (nearly) fills the chip: one 256 x 256 workgroup per
  // CU, which reads a third less from the L2 per product than two of 256 x
  // 128 (f_1's backward at 60 K tokens 430 against 448 us); f_1's forward,
  // half of whose time is its stores, takes the two, one storing while the
  // other computes (194 against 199 us).
  if constexpr (EPI != kEpiSilu) {
    if (tiles(256, 256) * splits >= 224)
      return stream ? launch(gemm_bf16_kernel<4, 4, 4, A_KM, B_KM, EPI, kStream>, 256, 256)
                    : launch(gemm_bf16_kernel<4, 4, 4, A_KM, B_KM, EPI, false>, 256, 256);
  } else {
    if (tiles(256, 128) * splits >= 448)
      return stream ? launch(gemm_bf16_kernel<4, 2, 3, A_KM, B_KM, EPI, kStream>, 256, 128)
                    : launch(gemm_bf16_kernel<4, 2, 3, A_KM, B_KM, EPI, false>, 256, 128);
  }
  return launch(gemm_bf16_kernel<2, 2, 3, A_KM, B_KM, EPI, false>, 128, 128);
}

hipError_t launch_gemm_bf16(const GemmArgs& g, int a_kmajor, int b_kmajor, int epi, int splits,
                            hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (!a_kmajor && !b_kmajor && epi == kEpiSilu)
    return gemm_case<false, false, kEpiSilu>(g, splits, s);
  if (!a_kmajor && !b_kmajor && epi == kEpiAdd)
    return gemm_case<false, false, kEpiAdd>(g, splits, s);
  if (!a_kmajor && b_kmajor && epi == kEpiAdd)
    return gemm_case<false, true, kEpiAdd>(g, splits, s);
  if (a_kmajor && b_kmajor && epi == kEpiSlab)
    return gemm_case<true, true, kEpiSlab>(g, splits, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_f32(const GemmArgsF32& g, int epi, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const dim3 grid((unsigned)((g.M + 63) / 64), (unsigned)((g.N + 63) / 64));
  if (epi == kEpiSilu)
    hipLaunchKernelGGL(gemm_f32_kernel<kEpiSilu>, grid, dim3(256), 0, s, g);
  else if (epi == kEpiAdd)
    hipLaunchKernelGGL(gemm_f32_kernel<kEpiAdd>, grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL(gemm_f32_kernel<kEpiSlab>, grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

int64_t colsum_blocks(int64_t T) { return (T + kColRows - 1) / kColRows; }

hipError_t launch_silu_bwd(int is_bf16, int64_t T, int F, int hv, int hq, const void* pre,
                           const void* du, const void* dv, const void* dq, const void* dk,
                           void* dpre, float* partial, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const dim3 grid((unsigned)((F + 511) / 512), (unsigned)colsum_blocks(T));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, T, F, hv, hq, pre, du, dv, dq, dk, dpre,
                       partial);
  };
  if (!is_bf16)
    launch(silu_bwd_kernel<false, false>);
  else if (4 * T * F >= (128ll << 20))
    launch(silu_bwd_kernel<true, true>);
  else
    launch(silu_bwd_kernel<true, false>);
  return hipGetLastError();
}

hipError_t launch_colsum(int is_bf16, int64_t T, int N, int64_t ld, const void* x, float* partial,
                         hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const dim3 grid((unsigned)((N + 511) / 512), (unsigned)colsum_blocks(T));
  if (is_bf16)
    hipLaunchKernelGGL(colsum_kernel<true>, grid, dim3(256), 0, s, T, N, ld, x, partial);
  else
    hipLaunchKernelGGL(colsum_kernel<false>, grid, dim3(256), 0, s, T, N, ld, x, partial);
  return hipGetLastError();
}

hipError_t launch_reduce_cols(int n, int S, const float* part, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_cols_kernel, dim3((unsigned)((n + 15) / 16)), dim3(256), 0, s, n, S,
                     part, out);
  return hipGetLastError();
}

hipError_t launch_reduce_slabs(int64_t n, int S, const float* part, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 1023) / 1024;
  const dim3 grid((unsigned)(blocks < 4096 ? blocks : 4096));
  hipLaunchKernelGGL(reduce_slabs_kernel, grid, dim3(256), 0, s, n, S, part, out);
  return hipGetLastError();
}

}  // namespace hstu
