// Epilogue of the HSTU layer (Eq. 3): Y_pre = LayerNorm(A V) (.) U, and
// its backward.
// Layer norm over the D = h * d_v features of each token with biased
// variance and optional affine weight/bias; the result gates U
// elementwise.  Saves per-token mean and 1/sqrt(var + eps) for a backward.
//
// HBM-bound: one wave per token (several tokens per wave for D <= 256), each
// lane holds its 8-element chunks in registers (16-byte loads for bf16),
// two-pass mean/variance in fp32 with wave reductions, one pass of stores.
// The attention output x is read in fp32 for both dtypes: normalising divides
// by the row's spread, which can be far smaller than its magnitude, so a
// bf16-rounded x would carry errors of several percent into Y.
#include "kernels.h"

namespace hstu {

namespace {

template <bool BF16>
__device__ __forceinline__ void load8(const void* base, int64_t idx, float* out) {
  if constexpr (BF16) {
    u32x4 r = *reinterpret_cast<const u32x4*>((const uint16_t*)base + idx);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      out[2 * e] = __uint_as_float(r[e] << 16);
      out[2 * e + 1] = __uint_as_float(r[e] & 0xffff0000u);
    }
  } else {
    const f32x4* p = reinterpret_cast<const f32x4*>((const float*)base + idx);
    f32x4 a = p[0], b = p[1];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      out[e] = a[e];
      out[4 + e] = b[e];
    }
  }
}

template <bool BF16>
__device__ __forceinline__ void store8(void* base, int64_t idx, const float* v) {
  if constexpr (BF16) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; e++) r[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
    *reinterpret_cast<u32x4*>((uint16_t*)base + idx) = r;
  } else {
    f32x4 a, b;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      a[e] = v[e];
      b[e] = v[4 + e];
    }
    f32x4* p = reinterpret_cast<f32x4*>((float*)base + idx);
    p[0] = a;
    p[1] = b;
  }
}

// CH chunks of 8 elements per lane, LPR lanes per token row (64 / LPR rows
// per wave; LPR < 64 only with CH = 1): D <= 8 LPR CH.  Narrow rows share a
// wave, so its lanes are not idle past D.
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// The affine parameters of a lane's features, kept in registers over its
// rows where they fit (CH <= 2), else re-read (from cache) per row.  16-byte
// loads: read one by one per token they cost the forward 133 us instead of
// 40 us on 62 K tokens of 512 features.
template <int CH>
struct Affine {
  static constexpr bool kHeld = CH <= 2;
  const float* p;  // may be null: `fill` instead
  float fill;
  float v[kHeld ? CH : 1][8];
  __device__ __forceinline__ void read(int idx, float (&o)[8]) const {
    if (p) {
      // The caller's parameter arrays are only known to be 4-byte aligned.
      typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
      const f32x4u a = *reinterpret_cast<const f32x4u*>(p + idx);
      const f32x4u c = *reinterpret_cast<const f32x4u*>(p + idx + 4);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        o[e] = a[e];
        o[4 + e] = c[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = fill;
    }
  }
  __device__ __forceinline__ Affine(const float* ptr, float f, int D, int sub, int lpr)
      : p(ptr), fill(f) {
    if constexpr (kHeld) {
#pragma unroll
      for (int c = 0; c < CH; c++) {
        const int idx = (c * lpr + sub) * 8;
        if (idx < D) read(idx, v[c]);
      }
    }
  }
  __device__ __forceinline__ void get(int c, int idx, float (&o)[8]) const {
    if constexpr (kHeld) {
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = v[c][e];
    } else {
      read(idx, o);
    }
  }
};

template <bool BF16, int CH, int LPR>
__global__ __launch_bounds__(256) void ln_gate_kernel(int64_t T, int D, const void* __restrict__ x,
                                                      const void* __restrict__ u, int64_t u_stride,
                                                      const float* __restrict__ w,
                                                      const float* __restrict__ b, float eps,
                                                      void* __restrict__ y,
                                                      float* __restrict__ mean,
                                                      float* __restrict__ rstd) {
  constexpr int RPW = 64 / LPR;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int sub = lane % LPR, row = lane / LPR;
  const Affine<CH> aw(w, 1.0f, D, sub, LPR), ab(b, 0.0f, D, sub, LPR);
  const int64_t step = (int64_t)gridDim.x * (4 * RPW);
  for (int64_t t0 = ((int64_t)blockIdx.x * 4 + wave) * RPW; t0 < T; t0 += step) {
    const int64_t t = t0 + row;
    const bool ok = t < T;
    // u is loaded with x where both fit in registers, else when it is used.
    constexpr bool kEarly = CH <= 2;
    float v[CH][8], g[kEarly ? CH : 1][8];
    float sum = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int idx = (c * LPR + sub) * 8;
      if (ok && idx < D) {
        load8<false>(x, t * D + idx, v[c]);
        if constexpr (kEarly) load8<BF16>(u, t * u_stride + idx, g[c]);
#pragma unroll
        for (int e = 0; e < 8; e++) sum += v[c][e];
      }
    }
    const float mu = row_sum<LPR>(sum) / (float)D;
    float sq = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int idx = (c * LPR + sub) * 8;
      if (ok && idx < D) {
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float d = v[c][e] - mu;
          sq += d * d;
        }
      }
    }
    const float var = row_sum<LPR>(sq) / (float)D;
    const float rs = 1.0f / sqrtf(var + eps);
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int idx = (c * LPR + sub) * 8;
      if (ok && idx < D) {
        float ww[8], bb[8], out[8];
        aw.get(c, idx, ww);
        ab.get(c, idx, bb);
        const int gc = kEarly ? c : 0;
        if constexpr (!kEarly) load8<BF16>(u, t * u_stride + idx, g[gc]);
#pragma unroll
        for (int e = 0; e < 8; e++) out[e] = ((v[c][e] - mu) * rs * ww[e] + bb[e]) * g[gc][e];
        store8<BF16>(y, t * D + idx, out);
      }
    }
    if (ok && sub == 0) {
      if (mean) mean[t] = mu;
      if (rstd) rstd[t] = rs;
    }
  }
}

// Backward of the epilogue, per token: with z = (x - mean) * rstd (the
// forward's saved statistics) and zn = z * w + b,
//   du = zn (.) dy,  dzn = dy (.) u,  dw += dzn z,  db += dzn,
//   dz = dzn (.) w,  dx = rstd (dz - mean(dz) - z mean(dz z)).
// HBM-bound: 14 bytes per element in bf16.  A wave keeps the dw / db sums
// of its rows in registers; at the end a workgroup adds its waves' sums in
// LDS and stores one row of partials [2 D] (dw, then db), which the prep
// launch of the attention backward sums over the workgroups in a fixed
// order.  (One float atomic per feature and wave, 4096 waves on the same
// 2 D addresses, took 860 us on 62 K tokens of 512 features, of which the
// memory traffic is 75 us.)  A single workgroup stores the sums themselves.
template <bool BF16, int CH, int LPR>
__global__ __launch_bounds__(256) void ln_gate_bwd_kernel(
    int64_t T, int D, const void* __restrict__ x, const void* __restrict__ u, int64_t u_stride,
    const void* __restrict__ dy, const float* __restrict__ w, const float* __restrict__ b,
    const float* __restrict__ mean, const float* __restrict__ rstd, void* __restrict__ du,
    void* __restrict__ dx, void* __restrict__ dx_lo, float* __restrict__ dw_out,
    float* __restrict__ db_out) {
  constexpr int RPW = 64 / LPR, COLS = 8 * LPR;  // columns per chunk c
  __shared__ __align__(16) float red[4][2][COLS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int sub = lane % LPR, row = lane / LPR;
  const Affine<CH> aw(w, 1.0f, D, sub, LPR), ab(b, 0.0f, D, sub, LPR);
  float pw[CH][8], pb[CH][8];
#pragma unroll
  for (int c = 0; c < CH; c++)
#pragma unroll
    for (int e = 0; e < 8; e++) pw[c][e] = pb[c][e] = 0.0f;
  const int64_t step = (int64_t)gridDim.x * (4 * RPW);
  for (int64_t t0 = ((int64_t)blockIdx.x * 4 + wave) * RPW; t0 < T; t0 += step) {
    const int64_t t = t0 + row;
    const bool ok = t < T;
    const float mu = ok ? mean[t] : 0.0f, rs = ok ? rstd[t] : 0.0f;
    float z[CH][8], dz[CH][8];
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int idx = (c * LPR + sub) * 8;
      if (ok && idx < D) {
        float xv[8], uv[8], gv[8], ww[8], bb[8], o[8];
        load8<false>(x, t * D + idx, xv);
        load8<BF16>(u, t * u_stride + idx, uv);
        load8<BF16>(dy, t * D + idx, gv);
        aw.get(c, idx, ww);
        ab.get(c, idx, bb);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float zz = (xv[e] - mu) * rs;
          const float dzn = gv[e] * uv[e];
          z[c][e] = zz;
          o[e] = (zz * ww[e] + bb[e]) * gv[e];
          pw[c][e] += dzn * zz;
          pb[c][e] += dzn;
          dz[c][e] = dzn * ww[e];
          s1 += dz[c][e];
          s2 += dz[c][e] * zz;
        }
        store8<BF16>(du, t * D + idx, o);
      }
    }
    const float m1 = row_sum<LPR>(s1) / (float)D, m2 = row_sum<LPR>(s2) / (float)D;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int idx = (c * LPR + sub) * 8;
      if (ok && idx < D) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = rs * (dz[c][e] - m1 - z[c][e] * m2);
        store8<BF16>(dx, t * D + idx, o);
        if (BF16 && dx_lo) {
          // low terms: o - bf16(o), exact in fp32
          float r[8];
#pragma unroll
          for (int e = 0; e < 8; e++) r[e] = o[e] - bf16_bits_to_f32(f32_to_bf16_bits(o[e]));
          store8<BF16>(dx_lo, t * D + idx, r);
        }
      }
    }
  }
  if (!dw_out && !db_out) return;
  const int64_t out_row = gridDim.x > 1 ? (int64_t)blockIdx.x * 2 * D : 0;
#pragma unroll
  for (int c = 0; c < CH; c++) {
    // Rows of the wave, then (in wave order) the four waves.
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
      for (int e = 0; e < 8; e++) {
        pw[c][e] += __shfl_xor(pw[c][e], off, 64);
        pb[c][e] += __shfl_xor(pb[c][e], off, 64);
      }
    if (row == 0) {
      store8<false>(&red[wave][0][8 * sub], 0, pw[c]);
      store8<false>(&red[wave][1][8 * sub], 0, pb[c]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * COLS; i += 256) {
      const int which = i / COLS, col = i % COLS;
      const float s = red[0][which][col] + red[1][which][col] + red[2][which][col] +
                      red[3][which][col];
      float* o = which ? db_out : dw_out;
      if (o && c * COLS + col < D) o[out_row + c * COLS + col] = s;
    }
    __syncthreads();
  }
}

// The instance for D features: lanes per row for D <= 512, chunks above.
#define LN_DISPATCH(CALL)           \
  if (D <= 64) { CALL(1, 8) }       \
  if (D <= 128) { CALL(1, 16) }     \
  if (D <= 256) { CALL(1, 32) }     \
  if (D <= 512) { CALL(1, 64) }     \
  if (D <= 1024) { CALL(2, 64) }    \
  if (D <= 2048) { CALL(4, 64) }    \
  if (D <= 4096) { CALL(8, 64) }

int64_t rows_per_block(int32_t D) { return D <= 64 ? 32 : D <= 128 ? 16 : D <= 256 ? 8 : 4; }

template <bool BF16>
hipError_t ln_bwd_case(int64_t T, int32_t D, const void* x, const void* u, int64_t u_stride,
                       const void* dy, const float* w, const float* b, const float* mean,
                       const float* rstd, void* du, void* dx, void* dx_lo, float* dw,
                       float* db, int64_t blocks, hipStream_t s) {
  const dim3 grid((unsigned)blocks);
#define LN_BWD_CALL(C, LPR)                                                                   \
  hipLaunchKernelGGL((ln_gate_bwd_kernel<BF16, C, LPR>), grid, dim3(256), 0, s, T, D, x, u,    \
                     u_stride, dy, w, b, mean, rstd, du, dx, dx_lo, dw, db);                  \
  return hipGetLastError();
  LN_DISPATCH(LN_BWD_CALL)
#undef LN_BWD_CALL
  return hipErrorInvalidValue;
}

template <bool BF16>
hipError_t ln_case(int64_t T, int32_t D, const void* x, const void* u, int64_t u_stride,
                   const float* w, const float* b, float eps, void* y, float* mean, float* rstd,
                   hipStream_t s) {
  // At most the 8 workgroups a CU holds; each keeps the affine in registers.
  const int64_t rows = rows_per_block(D);
  dim3 grid((unsigned)min((T + rows - 1) / rows, (int64_t)2048));
#define LN_CALL(C, LPR)                                                                     \
  hipLaunchKernelGGL((ln_gate_kernel<BF16, C, LPR>), grid, dim3(256), 0, s, T, D, x, u,      \
                     u_stride, w, b, eps, y, mean, rstd);                                   \
  return hipGetLastError();
  LN_DISPATCH(LN_CALL)
#undef LN_CALL
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_ln_gate_bwd(int is_bf16, int64_t T, int32_t D, const void* x, const void* u,
                              int64_t u_stride, const void* dy, const float* w, const float* b,
                              const float* mean, const float* rstd, void* du, void* dx,
                              void* dx_lo, float* dw, float* db, float* part,
                              int64_t part_floats, ColSums* sums, hipStream_t s) {
  *sums = ColSums{};
  if (T <= 0) return hipSuccess;
  // Two passes of rows per workgroup before more workgroups only add
  // partials, and at most five workgroups on each of the 256 CUs.
  const int64_t rows = 2 * rows_per_block(D);
  int64_t blocks = min((T + rows - 1) / rows, (int64_t)1280);
  float *dw_out = dw, *db_out = db;
  if (dw || db) {
    blocks = max(min(blocks, part_floats / (2 * D)), (int64_t)1);
    if (blocks > 1) {
      *sums = ColSums{part, (int32_t)blocks, D, {dw, db}};
      dw_out = dw ? part : nullptr;
      db_out = db ? part + D : nullptr;
    }
  }
  if (is_bf16)
    return ln_bwd_case<true>(T, D, x, u, u_stride, dy, w, b, mean, rstd, du, dx, dx_lo, dw_out,
                             db_out, blocks, s);
  return ln_bwd_case<false>(T, D, x, u, u_stride, dy, w, b, mean, rstd, du, dx, nullptr, dw_out,
                            db_out, blocks, s);
}

hipError_t launch_ln_gate(int is_bf16, int64_t T, int32_t D, const void* x, const void* u,
                          int64_t u_stride, const float* w, const float* b, float eps, void* y,
                          float* mean, float* rstd, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  if (is_bf16) return ln_case<true>(T, D, x, u, u_stride, w, b, eps, y, mean, rstd, s);
  return ln_case<false>(T, D, x, u, u_stride, w, b, eps, y, mean, rstd, s);
}

}  // namespace hstu
