// Standalone timestamp bucketisation: materialises, for every sequence,
// the L x L matrix of time buckets bkt(t_i - t_j) (notation table, entry
// rab^{p,t}) as uint8, row-major, sequences concatenated at pair_offsets.
//
// HBM-write bound.  A workgroup of 8 waves owns 64 consecutive tokens of
// the batch (16 or 32 while those fill the chip), i.e. 64 rows of one
// sequence (or the rows of two or more sequences that meet inside the
// block), and walks the columns in slabs of 8192 (whole rows, for sequences
// up to that length) whose timestamps it stages in
// LDS.  When the
// timestamps of its rows and of the slab lie within 2^30 of the sequence's
// first one (always, for real event times), they are rebased to 32 bits
// and a pair costs v_sad_u32, v_ffbh_u32 and one saturating subtract that
// writes the bucket straight into its byte of the output dword (SDWA);
// otherwise the exact 64-bit form runs.
// A row segment is written as aligned 16-byte chunks, one per lane (a wave
// store covers 1 KB), plus at most 15 bytes at each end, written one byte
// per lane.  A chunk needs the timestamps of 16 consecutive columns: the
// slab is staged twice, shifted by 0 and 1 words, so that the copy
// matching the row's alignment holds them as four aligned 16-byte words
// (or, for half of the alignments, eight 8-byte words), and each copy
// inserts one padding word-quad every 64 entries, so that the lanes of a
// read (64 bytes apart) spread over the LDS banks.
// A wave takes four rows, 16 apart, together: their segments have one
// alignment (16 L is a multiple of 16), so one set of LDS reads and
// addresses serves all four.  Against one row at a time with 48 rows per
// workgroup of 4 waves: batches of 1 to 10 K tokens 10 against 16 us; 8
// sequences of 4096-8192 tokens (312 MB) 66 against 73 us into a buffer that
// the last-level cache holds part of, 76 us both into changing buffers,
// where the order of the writes binds (the stores alone, without reads or
// arithmetic, take 70 us; a plain fill 46).  More workgroups per CU only
// spread them further: two 83 us, five with 4096-column slabs 93.
#include "bias.h"
#include "kernels.h"

namespace hstu {

namespace {

constexpr int kBktThreads = 512;
constexpr int kBktWaves = kBktThreads / 64;
constexpr int kBktStep = 16;                // rows a wave takes together are this far apart
constexpr int kBktMaxRows = 4 * kBktStep;   // rows per workgroup, at most
constexpr int kBktCols = 8192;  // columns staged per slab
// Longest sequence that goes unstaged: a wave's lanes hold it (30000 sequences
// of 0 to 19 tokens 474 -> 143 us, 1000 of 30 55 -> 28, 300 of 64 30 -> 26).
constexpr int kBktShort = 64;
// Entry y of a copy sits at y + 4 (y >> kPadShift); y <= kBktCols.
constexpr int kPadShift = 6;
__device__ __forceinline__ int bkt_pidx(int y) { return y + 4 * (y >> kPadShift); }
constexpr int kBktLd = ((kBktCols + 2) + 4 * ((kBktCols + 2) / (1 << kPadShift) + 1) + 3) / 4 * 4;
// Entries 1024 further on (64 chunks of 16) sit this many words further.
constexpr int kChunkStep = 1024 + 4 * (1024 >> kPadShift);

struct __align__(16) BktShared {
  union {
    uint32_t t32[2][kBktLd];  // copy s holds column x at bkt_pidx(x + s)
    int64_t t64[kBktCols];
  };
  int64_t rowt[kBktMaxRows];    // the workgroup's row timestamps
};

// Leading-zero count of |ti - tj| < 2^31 (0xffffffff for 0), raised to
// zmin = 32 - nb when CLAMP (nb <= 31), so that the saturating 31 - z
// below is min(floor(log2 |dt|), nb - 1), and 0 for |dt| <= 1.
template <bool CLAMP>
__device__ __forceinline__ uint32_t lz32(uint32_t ti, uint32_t tj, uint32_t zmin) {
  uint32_t d, z;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(ti), "v"(tj));
  asm("v_ffbh_u32 %0, %1" : "=v"(z) : "v"(d));
  if constexpr (CLAMP) z = z > zmin ? z : zmin;  // 0xffffffff stays
  return z;
}

// Four buckets packed little-endian into one dword: byte 0 by a saturating
// subtract, bytes 1-3 by the same subtract writing its byte in place (SDWA).
template <bool CLAMP>
__device__ __forceinline__ uint32_t bkt4(uint32_t ti, uint32_t a, uint32_t b, uint32_t c,
                                         uint32_t d, uint32_t zmin, uint32_t c31) {
  const uint32_t z0 = lz32<CLAMP>(ti, a, zmin), z1 = lz32<CLAMP>(ti, b, zmin);
  const uint32_t z2 = lz32<CLAMP>(ti, c, zmin), z3 = lz32<CLAMP>(ti, d, zmin);
  uint32_t r;
  asm("v_sub_u32_e64 %0, 31, %1 clamp" : "=v"(r) : "v"(z0));
  asm("v_sub_u32_sdwa %0, %1, %2 clamp dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE "
      "src0_sel:DWORD src1_sel:DWORD"
      : "+v"(r) : "v"(c31), "v"(z1));
  asm("v_sub_u32_sdwa %0, %1, %2 clamp dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE "
      "src0_sel:DWORD src1_sel:DWORD"
      : "+v"(r) : "v"(c31), "v"(z2));
  asm("v_sub_u32_sdwa %0, %1, %2 clamp dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE "
      "src0_sel:DWORD src1_sel:DWORD"
      : "+v"(r) : "v"(c31), "v"(z3));
  return r;
}

// NR rows of the slab at once, 16 rows apart: 16 L is a multiple of 16, so
// their segments share one alignment, and with it the chunks' columns and
// every LDS read.  The first `nv` of them exist (nv >= 1).
template <bool CLAMP, int NR>
__device__ __forceinline__ void row_segments32(const BktShared& sm, const uint32_t (&ti)[NR],
                                               int nv, int nb, int64_t P, int64_t row_step,
                                               int ncols, uint8_t* __restrict__ out, int lane) {
  // Flat bytes [P, P + ncols) hold columns 0 .. ncols-1 of the slab in the
  // first row; relative to P: the head [0, hend), nch aligned 16-byte chunks
  // from h = (16 - P) mod 16, and the tail [tstart, ncols) (at most 15
  // bytes each).
  const uint32_t zmin = CLAMP ? (uint32_t)(32 - nb) : 0u;
  const uint32_t c31 = 31u;
  const int64_t cfirst = (P + 15) >> 4;
  const int h = (int)((cfirst << 4) - P);
  const int nch = max(0, (int)(((P + ncols) >> 4) - cfirst));
  const int hend = min(h, ncols), tstart = max(hend, h + 16 * nch);
  uint8_t* const row = out + P;
  // End bytes: lanes 0-15 the head, lanes 32-47 the tail (copy 0).
  {
    const int r = lane < 32 ? lane : tstart + (lane - 32);
    const bool on = lane < 32 ? lane < hend : (lane < 48 && r < ncols);
    if (on) {
      const uint32_t tj = sm.t32[0][bkt_pidx(r)];
#pragma unroll
      for (int k = 0; k < NR; k++)
        if (k < nv) {
          const uint32_t z = lz32<CLAMP>(ti[k], tj, zmin);
          uint32_t b;
          asm("v_sub_u32_e64 %0, 31, %1 clamp" : "=v"(b) : "v"(z));
          row[r + k * row_step] = (uint8_t)b;
        }
    }
  }
  if (lane >= nch) return;
  // Chunk a covers columns h + 16 a .. +15, entries y .. y + 15 of copy
  // s = P mod 2 with y = h + 16 a + s: a multiple of 4 when P mod 4 < 2
  // (16-byte reads), else 2 mod 4 (8-byte reads).  Moving 64 chunks on
  // adds 1024 entries, 16 whole pad periods: the offsets of the reads
  // from the first stay fixed and the first moves by 1088.
  const int k4 = (int)(P & 3), sc = k4 & 1;
  const int y = h + sc + 16 * lane;
  const int p0 = bkt_pidx(y);
  const uint32_t* src = sm.t32[sc] + p0;
  uint8_t* dst = row + h + 16 * lane;
  auto chunk = [&](const uint32_t (&t)[16]) {
#pragma unroll
    for (int k = 0; k < NR; k++)
      if (k < nv) {
        u32x4 v;
#pragma unroll
        for (int q = 0; q < 4; q++)
          v[q] = bkt4<CLAMP>(ti[k], t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3], zmin, c31);
        *reinterpret_cast<u32x4*>(dst + k * row_step) = v;
      }
    src += kChunkStep;
    dst += 64 * 16;
  };
  if (k4 < 2) {
    int dd[4];
#pragma unroll
    for (int m = 0; m < 4; m++) dd[m] = bkt_pidx(y + 4 * m) - p0;
    for (int a = lane; a < nch; a += 64) {
      uint32_t t[16];
#pragma unroll
      for (int m = 0; m < 4; m++) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(src + dd[m]);
#pragma unroll
        for (int e = 0; e < 4; e++) t[4 * m + e] = w[e];
      }
      chunk(t);
    }
  } else {
    int dd[8];
#pragma unroll
    for (int m = 0; m < 8; m++) dd[m] = bkt_pidx(y + 2 * m) - p0;
    for (int a = lane; a < nch; a += 64) {
      uint32_t t[16];
#pragma unroll
      for (int m = 0; m < 8; m++) {
        const uint2 w = *reinterpret_cast<const uint2*>(src + dd[m]);
        t[2 * m] = w.x;
        t[2 * m + 1] = w.y;
      }
      chunk(t);
    }
  }
}

__device__ __forceinline__ void row_segment64(const BktShared& sm, int64_t ti, int nb, int64_t P,
                                              int ncols, uint8_t* __restrict__ out, int lane) {
  for (int j = lane; j < ncols; j += 64) out[P + j] = (uint8_t)time_bucket64(ti - sm.t64[j], nb);
}

// Rows r0 .. r0 + rows - 1 of one sequence (timestamps t, length L, pairs
// from base), every column.
template <int NR>
__device__ __forceinline__ void bucketize_rows(BktShared& sm, int nb, const int64_t* __restrict__ t,
                                               int L, int64_t base, int r0, int rows,
                                               uint8_t* __restrict__ out, int tid, int wave,
                                               int lane) {
  // Short sequences: a wave holds every timestamp, a lane writes a byte of
  // each row; no staging and no barrier, of which a workgroup would otherwise
  // have three for each of its many sequences.
  if (L <= kBktShort) {
    const int64_t tj = t[min(lane, L - 1)];
    for (int x = wave; x < rows; x += kBktWaves) {
      const int64_t dt = readlane64(tj, r0 + x) - tj;
      if (lane < L) out[base + (int64_t)(r0 + x) * L + lane] = (uint8_t)time_bucket64(dt, nb);
    }
    return;
  }
  // 32-bit form: timestamps as offsets from t[0] - 2^30; it applies when
  // every offset the workgroup touches lies in [0, 2^31), so that two of
  // them differ by less than 2^31.  A slab's timestamps are loaded before
  // any output of that slab is stored: loads and stores share the wave's
  // memory counter, so a load issued after stores would wait for them.
  const int64_t t0 = t[0] - ((int64_t)1 << 30);
  auto in32 = [](int64_t d) { return d >= 0 && d < ((int64_t)1 << 31); };
  bool rows_ok = true;
  if (tid < rows) {
    const int64_t tr = t[r0 + tid];
    sm.rowt[tid] = tr;
    rows_ok = in32(tr - t0);
  }
  constexpr int kPer = kBktCols / kBktThreads;
  for (int c0 = 0; c0 < L; c0 += kBktCols) {
    const int ncols = min(kBktCols, L - c0);
    // Rebased low words, kept only if the whole workgroup passes (the
    // 64-bit form reloads the values).
    uint32_t cur[kPer];
    bool ok = rows_ok;
#pragma unroll
    for (int e = 0; e < kPer; e++) {
      const int x = tid + e * kBktThreads;
      const int64_t d = (x < ncols ? t[c0 + x] : t0) - t0;
      ok = ok && in32(d);
      cur[e] = (uint32_t)d;
    }
    const bool fast = __syncthreads_and(ok);  // also: previous slab fully consumed
    if (fast) {
      // (columns past the slab's are not read)
#pragma unroll
      for (int e = 0; e < kPer; e++) {
        if (e * kBktThreads >= ncols) break;
        const int x = tid + e * kBktThreads;
        sm.t32[0][bkt_pidx(x)] = cur[e];
        sm.t32[1][bkt_pidx(x + 1)] = cur[e];
      }
    } else {
      for (int x = tid; x < ncols; x += kBktThreads) sm.t64[x] = t[c0 + x];
    }
    __syncthreads();
    // A wave takes rows x, x + 16, ... for x = wave, wave + 8; row set-up is
    // wave-uniform (scalar unit).
    for (int x = wave; x < min(rows, kBktStep); x += kBktWaves) {
      const int nv = (rows - x + kBktStep - 1) / kBktStep;
      const int64_t P = base + (int64_t)(r0 + x) * L + c0, step = (int64_t)kBktStep * L;
      if (fast) {
        uint32_t ti[NR];
#pragma unroll
        for (int k = 0; k < NR; k++)
          ti[k] = (uint32_t)__builtin_amdgcn_readfirstlane(
              (int)(sm.rowt[min(x + k * kBktStep, rows - 1)] - t0));
        if (nb <= 31)
          row_segments32<true, NR>(sm, ti, nv, nb, P, step, ncols, out, lane);
        else
          row_segments32<false, NR>(sm, ti, nv, nb, P, step, ncols, out, lane);
      } else {
        for (int k = 0; k < nv; k++)
          row_segment64(sm, sm.rowt[x + k * kBktStep], nb, P + k * step, ncols, out, lane);
      }
    }
    __syncthreads();  // the slab (or the row timestamps) is restaged next
  }
}

// Workgroup g covers tokens [R g, R g + R), R = 16 NR, of the concatenated
// batch: the rows of the sequence(s) those tokens belong to, every column.
template <int NR>
__global__ __launch_bounds__(kBktThreads) void bucketize_kernel(
    int32_t num_seqs, int64_t total_tokens, int32_t nb, const int64_t* __restrict__ offs,
    const int64_t* __restrict__ ts, const int64_t* __restrict__ pair_offs,
    uint8_t* __restrict__ out) {
  __shared__ BktShared sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kRows = NR * kBktStep;
  for (int64_t g = blockIdx.x; g * kRows < total_tokens; g += gridDim.x) {
    int64_t R0 = g * kRows;
    const int64_t R1 = min(R0 + kRows, total_tokens);
    // b = the last sequence with offs[b] <= R0 (offsets are non-decreasing).
    int lo = 0, hi = num_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (offs[mid] <= R0) lo = mid; else hi = mid - 1;
    }
    for (int b = lo; b < num_seqs && R0 < R1; b++) {
      const int64_t o = offs[b], e = offs[b + 1];
      if (e <= R0) continue;  // empty sequence
      const int rows = (int)(min(e, R1) - R0);
      bucketize_rows<NR>(sm, nb, ts + o, (int)(e - o), pair_offs[b], (int)(R0 - o), rows, out, tid,
                     wave, lane);
      R0 += rows;
    }
  }
}

}  // namespace

hipError_t launch_bucketize(int32_t num_seqs, int64_t total_tokens, int32_t num_buckets,
                            const int64_t* seq_offsets, const int64_t* timestamps,
                            const int64_t* pair_offsets, int64_t total_pairs, uint8_t* out,
                            hipStream_t s) {
  if (total_pairs <= 0 || num_seqs <= 0 || total_tokens <= 0) return hipSuccess;
  // Fewer rows per workgroup while that fills the 512 workgroups the chip
  // holds.
  auto launch = [&](auto kernel, int rows) {
    const int64_t blocks = (total_tokens + rows - 1) / rows;
    hipLaunchKernelGGL(kernel, dim3((unsigned)min(blocks, (int64_t)1 << 30)), dim3(kBktThreads), 0,
                       s, num_seqs, total_tokens, num_buckets, seq_offsets, timestamps,
                       pair_offsets, out);
  };
  if (total_tokens <= 16 * 512)
    launch(bucketize_kernel<1>, kBktStep);
  else if (total_tokens <= 32 * 512)
    launch(bucketize_kernel<2>, 2 * kBktStep);
  else
    launch(bucketize_kernel<4>, 4 * kBktStep);
  return hipGetLastError();
}

}  // namespace hstu
