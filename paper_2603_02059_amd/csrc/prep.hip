// Centring, precision conversion and squared norms (the precomputed norms of
// Algorithm 1, stage 1; Eq. 4).
//
// Distances are translation invariant, so the fields are shifted per grid cell
// before the Gram product: with ~1e5 Pa offsets the uncentred inner products
// would cancel against the norms and lose every bit the reduced-precision
// paths carry. Any per-cell shift gives the same distances; the shift only has
// to remove the offset. It is the FP64 mean over an evenly strided sample of
// at most COLSTAT_SAMPLE rows (every row when T is at most that), which reads
// a small fraction of X and lies within about sigma / sqrt(COLSTAT_SAMPLE) of
// the full mean. Centred values are FP64. The squared norms are taken
// per chunk of GRAM_CHUNK elements, in FP64, of exactly the vector the Gram
// stage represents (FP32, FP16 or hi + lo), so that the Gram stage's
// N_i + N_j - 2G, assembled chunk by chunk, is a distance between the same two
// vectors up to the accumulation error (and, for BF16x3, the zero-mean lo.lo
// cross term).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "internal.h"
#include "topk_wave.h"

namespace traknn {
namespace {

// Partial column sums of the sampled rows (sample r is row r * stride) over
// blocks of COLSTAT_ROWS samples, one cell a thread (a wave reads 256 bytes of
// a row), COLSUM_BATCH rows in flight at a time, in a fixed order. The sample is
// at most 2048 rows, so latency bounds it on all but the widest grids: with
// four cells a thread and eight rows in flight the 128 rows of a block took 16
// round trips on a quarter of the waves (25 us for 1827 samples of 1961 cells,
// 7 us now).
constexpr int COLSUM_BATCH = 32;
__global__ __launch_bounds__(256) void colsum_partial_kernel(
    const float* __restrict__ X, int64_t ldx, int64_t nsamp, int64_t stride, int64_t D,
    double* __restrict__ part) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.y * COLSTAT_ROWS;
  if (c >= D) return;
  const int64_t r1 = r0 + COLSTAT_ROWS < nsamp ? r0 + COLSTAT_ROWS : nsamp;
  const int64_t step = stride * ldx;  // floats between sampled rows
  const float* p = X + r0 * step + c;
  double s = 0.0;
  int64_t r = r0;
  for (; r + COLSUM_BATCH <= r1; r += COLSUM_BATCH) {
    float v[COLSUM_BATCH];
#pragma unroll
    for (int u = 0; u < COLSUM_BATCH; ++u) v[u] = p[u * step];
#pragma unroll
    for (int u = 0; u < COLSUM_BATCH; ++u) s += (double)v[u];
    p += COLSUM_BATCH * step;
  }
  if (r < r1) {
    const int n = (int)(r1 - r);
    float v[COLSUM_BATCH];
#pragma unroll
    for (int u = 0; u < COLSUM_BATCH; ++u) v[u] = p[(u < n ? u : 0) * step];
#pragma unroll
    for (int u = 0; u < COLSUM_BATCH; ++u)
      if (u < n) s += (double)v[u];
  }
  part[(int64_t)blockIdx.y * D + c] = s;
}

// Fixed-order reduction of the partial sums -> per-cell sample mean.
__global__ __launch_bounds__(256) void colsum_reduce_kernel(
    const double* __restrict__ part, int64_t nsamp, int64_t D, int nchunks,
    double* __restrict__ mu) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= D) return;
  double s = 0.0;
#pragma unroll 8
  for (int q = 0; q < nchunks; ++q) s += part[(int64_t)q * D + c];
  mu[c] = s / (double)nsamp;
}

// Sum over the wave by a butterfly of strides 32, 16, ... 1 (every lane gets
// it), the exchanges of topk_wave.h.
template <int S = 32>
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_xor_d<S>(v);
  if constexpr (S > 1) return wave_sum<S / 2>(v);
  return v;
}

__device__ inline uint32_t bf16_bits_rne(float f) {
  // round-to-nearest-even of an FP32 value to BF16 (inputs are finite)
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ inline double bf16_bits_to_double(uint32_t b) {
  return (double)__uint_as_float(b << 16);
}

// Eight centred cells of a row, v, in the representation PREC emits: OUT / 16
// 16-byte chunks of the operand row. Returns the FP64 squared norm of the
// represented values.
template <int PREC>
constexpr int conv_bytes() { return PREC == TRAKNN_FP16 ? 16 : 32; }
template <int PREC>
__device__ __forceinline__ double convert8(const double (&v)[8], uint4 (&out)[conv_bytes<PREC>() / 16]) {
  double acc = 0.0;
  if constexpr (PREC == TRAKNN_FP32) {
    uint32_t f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float x = (float)v[u];
      acc += (double)x * (double)x;
      f[u] = __float_as_uint(x);
    }
    out[0] = make_uint4(f[0], f[1], f[2], f[3]);
    out[1] = make_uint4(f[4], f[5], f[6], f[7]);
  } else if constexpr (PREC == TRAKNN_FP16) {
    uint32_t packed[4];
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      const _Float16 h0 = (_Float16)(float)v[u], h1 = (_Float16)(float)v[u + 1];
      const double d0 = (double)(float)h0, d1 = (double)(float)h1;
      acc += d0 * d0;
      acc += d1 * d1;
      packed[u / 2] = (uint32_t)__builtin_bit_cast(uint16_t, h0) |
                      ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
    }
    out[0] = make_uint4(packed[0], packed[1], packed[2], packed[3]);
  } else {
    // BF16X3: the 16-byte chunk of 8 hi values is followed by the chunk of
    // the 8 matching lo values, so one 64-byte Gram slice row holds 16
    // (hi, lo) pairs.
    uint32_t hp[4], lp[4];
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      uint32_t hb[2], lb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        hb[t] = bf16_bits_rne((float)v[u + t]);
        const double hd = bf16_bits_to_double(hb[t]);
        lb[t] = bf16_bits_rne((float)(v[u + t] - hd));
        // norm of the represented value hi + lo (exact in FP64). The Gram
        // stage drops only the cross term lo_i.lo_j, which has zero mean;
        // a norm made of the three kept products alone would bias every
        // distance low by sum (lo_i - lo_j)^2 ~ 2.5e-6 (N_i + N_j).
        const double xv = hd + bf16_bits_to_double(lb[t]);
        acc += xv * xv;
      }
      hp[u / 2] = hb[0] | (hb[1] << 16);
      lp[u / 2] = lb[0] | (lb[1] << 16);
    }
    out[0] = make_uint4(hp[0], hp[1], hp[2], hp[3]);
    out[1] = make_uint4(lp[0], lp[1], lp[2], lp[3]);
  }
  return acc;
}

// Wave g of the grid owns norm chunk ch = g mod nch (GRAM_CHUNK elements; lane q
// the 8 consecutive elements 8q .. 8q+7) and converts it for nrows rows (a
// multiple of CONV_BATCH) starting at g / nch * nrows, keeping the chunk's
// means in registers. Bound by HBM (4 bytes read and 2 or 4 written per
// element): 0.35 ms for 27394 x 8192 fields in BF16x3, 5.2 TB/s, where a plain
// copy of this size moves 5.2 TB/s. CONV_BATCH rows are loaded together, and
// their converted chunk goes through LDS, because the operands lie slice by
// slice (internal.h): a lane's own cells are half a 64-byte row of one slice,
// so storing them directly writes 64-byte pieces Tpad * 64 bytes apart (0.50
// ms on the same fields), while the batch's rows of a slice are one 256-byte
// run. Each (row, chunk) squared norm (FP64 sum, stored FP32) goes to
// ncs[chunk * Tpad + row]. PREC selects the emitted representation.
constexpr int CONV_BATCH = 4;
template <int PREC>
__global__ __launch_bounds__(256) void centre_convert_kernel(
    const float* __restrict__ X, int64_t ldx, int64_t T, int64_t D,
    int64_t Tpad, int64_t Dpad, const double* __restrict__ mu, int parts, double nsamp,
    char* __restrict__ xc, float* __restrict__ ncs, int nrows) {
  static_assert(GRAM_CHUNK == 64 * 8, "a wave covers one norm chunk");
  constexpr int LB = conv_bytes<PREC>();  // bytes a lane emits per row
  constexpr int CB = 64 * LB;             // bytes of a row's chunk
  constexpr int PITCH = CB + GRAM_ROW_BYTES;
  constexpr int NSL = CB / GRAM_ROW_BYTES;  // slices of a chunk
  constexpr int CPR = GRAM_ROW_BYTES / 16;  // 16-byte chunks of a slice row
  static_assert(CONV_BATCH * CPR == 16, "16 lanes store a batch's rows of a slice");
  __shared__ __attribute__((aligned(16))) char stage[4][CONV_BATCH * PITCH];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t nch = norm_chunks(Dpad), g = (int64_t)blockIdx.x * 4 + w;
  const int64_t ch = g % nch, ib = g / nch * nrows;
  if (ib >= Tpad) return;  // no workgroup barrier below
  const int64_t e0 = ch * GRAM_CHUNK + 8 * lane;  // Dpad is a multiple of 8
  const bool in_pad = e0 < Dpad;
  const bool full = e0 + 8 <= D;
  const int64_t sl0 = ch * NSL, nsl = Dpad * LB / 8 / GRAM_ROW_BYTES;
  double m[8];
  if (parts == 0) {
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = e0 + u < D ? mu[e0 + u] : 0.0;
  } else {  // mu holds the partial sums: their reduction, as colsum_reduce_kernel's
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = 0.0;
    for (int q = 0; q < parts; ++q)
#pragma unroll
      for (int u = 0; u < 8; ++u) m[u] += e0 + u < D ? mu[q * D + e0 + u] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] /= nsamp;
  }
  for (int64_t i0 = ib; i0 < ib + nrows && i0 < Tpad; i0 += CONV_BATCH) {
    float x[CONV_BATCH][8];
#pragma unroll
    for (int r = 0; r < CONV_BATCH; ++r) {
      const float* xrow = X + (i0 + r) * ldx;
      const bool live = i0 + r < T;
      if (live && full) {
        const float4 a = *(const float4*)(xrow + e0);
        const float4 b = *(const float4*)(xrow + e0 + 4);
        x[r][0] = a.x, x[r][1] = a.y, x[r][2] = a.z, x[r][3] = a.w;
        x[r][4] = b.x, x[r][5] = b.y, x[r][6] = b.z, x[r][7] = b.w;
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) x[r][u] = live && e0 + u < D ? xrow[e0 + u] : 0.f;
      }
    }
    double acc[CONV_BATCH];
#pragma unroll
    for (int r = 0; r < CONV_BATCH; ++r) {
      const bool live = i0 + r < T;
      double v[8];
      uint4 out[LB / 16];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = live && e0 + u < D ? (double)x[r][u] - m[u] : 0.0;
      acc[r] = convert8<PREC>(v, out);
#pragma unroll
      for (int q = 0; q < LB / 16; ++q)
        *(uint4*)(stage[w] + r * PITCH + lane * LB + 16 * q) = out[q];
    }
    __builtin_amdgcn_wave_barrier();  // LDS accesses of a wave execute in order
    // 16 lanes per slice: row (lane / CPR) % CONV_BATCH, chunk lane % CPR
    const int row = lane / CPR % CONV_BATCH, c = lane % CPR;
#pragma unroll
    for (int t = 0; t < NSL / 4; ++t) {
      const int sl = 4 * t + (lane >> 4);
      const uint4 v = *(const uint4*)(stage[w] + row * PITCH + sl * GRAM_ROW_BYTES + 16 * c);
      if (sl0 + sl < nsl)
        *(uint4*)(xc + ((sl0 + sl) * Tpad + i0 + row) * GRAM_ROW_BYTES + 16 * c) = v;
    }
    __builtin_amdgcn_wave_barrier();
    float n = 0.f;
#pragma unroll
    for (int r = 0; r < CONV_BATCH; ++r) {
      const double s = wave_sum(in_pad ? acc[r] : 0.0);
      if (lane == r) n = i0 + r < T ? (float)s : 0.f;
    }
    if (lane < CONV_BATCH) ncs[ch * Tpad + i0 + lane] = n;
  }
}

}  // namespace

hipError_t launch_colstats(const float* X, int64_t ldx, int64_t T, int64_t D,
                           int tchunks, bool reduce, double* mu_part, double* mu,
                           hipStream_t s) {
  const int64_t stride = colstat_stride(T);
  const int64_t nsamp = (T + stride - 1) / stride;
  dim3 g1((unsigned)((D + 255) / 256), (unsigned)tchunks);
  hipLaunchKernelGGL(colsum_partial_kernel, g1, dim3(256), 0, s, X, ldx, nsamp, stride, D,
                     mu_part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !reduce) return e;
  hipLaunchKernelGGL(colsum_reduce_kernel, dim3((unsigned)((D + 255) / 256)),
                     dim3(256), 0, s, mu_part, nsamp, D, tchunks, mu);
  return hipGetLastError();
}

hipError_t launch_centre_convert(const float* X, int64_t ldx, int64_t T,
                                 int64_t D, int64_t Tpad, int64_t Dpad,
                                 int precision, int parts, const double* mu, void* xc,
                                 float* ncs, hipStream_t s) {
  const int64_t stride = colstat_stride(T);
  const double nsamp = (double)((T + stride - 1) / stride);
  // Rows per wave: 16 (the chunk's means are read once for them), fewer while
  // that leaves less than CONV_WAVES waves (16 per CU), so that a short series
  // is one memory latency deep instead of four: 18 -> 9 us on 512 x 1024 fields.
  constexpr int64_t CONV_WAVES = 4096;
  const int64_t nch = norm_chunks(Dpad);
  int nrows = 16;
  while (nrows > CONV_BATCH && nch * (Tpad / nrows) < CONV_WAVES) nrows /= 2;
  const dim3 g((unsigned)((nch * ((Tpad + nrows - 1) / nrows) + 3) / 4));
#define TRAKNN_CONVERT(P)                                                                        \
  hipLaunchKernelGGL(centre_convert_kernel<P>, g, dim3(256), 0, s, X, ldx, T, D, Tpad, Dpad, mu, \
                     parts, nsamp, (char*)xc, ncs, nrows)
  if (precision == TRAKNN_FP32) TRAKNN_CONVERT(TRAKNN_FP32);
  else if (precision == TRAKNN_BF16X3) TRAKNN_CONVERT(TRAKNN_BF16X3);
  else TRAKNN_CONVERT(TRAKNN_FP16);
#undef TRAKNN_CONVERT
  return hipGetLastError();
}

}  // namespace traknn
