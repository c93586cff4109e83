// Gradient of F = sum_t w_t s_t with the neighbour sets held fixed (Eq. 3 with
// Eq. 2 inside). Writing F = sum_{a,b} W_ab ||x_a - x_b||^2 with
//   W_ab = sum_t (w_t / k) sum_{j in N_t} sum_{m<L} [a = t+m][b = j+m],
// the gradient is a graph-Laplacian product
//   g_a = 2 sum_b (W_ab + W_ba) (x_a - x_b).
// Row a's W_ab terms come straight from the neighbour lists (t = a - m); its
// W_ba terms need the reverse lists (all t with j = a - m in N_t), which are
// built as a CSR: integer counting with atomics, a scan, an atomic fill and a
// per-bucket sort by t, so the reverse lists -- and hence every floating-point
// sum -- come out in the same order on every run. Each output row is then
// gathered in FP64 (field differences of FP32 inputs are exact in FP64) and
// rounded once to FP32; rows that no term touches are written as zeros by the
// same kernel. No distance value is needed: the
// derivative of a squared distance is the field difference itself.
#include <climits>

#include "internal.h"
#include "topk_wave.h"

namespace traknn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* p, int64_t n,
                                                       int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// Reverse-list counts, plus the rows any term touches: a = t + m (the rows
// of a weighted trajectory) and a = j + m (those of its neighbours), m < L.
// Flags are plain stores of 1, so concurrent writers agree.
__global__ __launch_bounds__(256) void rev_count_kernel(
    const int32_t* __restrict__ idx, const double* __restrict__ w, int np,
    int k, int L, int32_t* __restrict__ cnt, int32_t* __restrict__ touch) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= (int64_t)np * k) return;
  const int t = (int)(g / k);
  if (w[t] == 0.0) return;
  const int j = idx[g];
  if (j < 0 || j >= np) return;
  atomicAdd(&cnt[j], 1);
  for (int m = 0; m < L; ++m) {
    touch[t + m] = 1;
    touch[j + m] = 1;
  }
}

// Exclusive scan of cnt[0..n) into ptr[0..n], one workgroup of 1024 threads.
// Each thread sums its run of counts SCAN_BATCH loads at a time, the loads of
// a batch in flight together.
constexpr int SCAN_BATCH = 16;
__global__ __launch_bounds__(1024) void scan_kernel(const int32_t* __restrict__ cnt,
                                                    int n, int32_t* __restrict__ ptr) {
  __shared__ int32_t part[1024];
  const int tid = threadIdx.x;
  const int per = (n + 1023) / 1024;
  const int b = tid * per;
  const int e = b + per < n ? b + per : n;
  int32_t s = 0;
  for (int i0 = b; i0 < e; i0 += SCAN_BATCH) {
    int32_t v[SCAN_BATCH];
#pragma unroll
    for (int u = 0; u < SCAN_BATCH; ++u) v[u] = i0 + u < e ? cnt[i0 + u] : 0;
#pragma unroll
    for (int u = 0; u < SCAN_BATCH; ++u) s += v[u];
  }
  part[tid] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    int32_t v = tid >= off ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int32_t run = tid > 0 ? part[tid - 1] : 0;
  for (int i0 = b; i0 < e; i0 += SCAN_BATCH) {
    int32_t v[SCAN_BATCH];
#pragma unroll
    for (int u = 0; u < SCAN_BATCH; ++u) v[u] = i0 + u < e ? cnt[i0 + u] : 0;
#pragma unroll
    for (int u = 0; u < SCAN_BATCH; ++u) {
      if (i0 + u < e) ptr[i0 + u] = run;
      run += v[u];
    }
  }
  if (tid == 1023) ptr[n] = part[1023];
}

__global__ __launch_bounds__(256) void rev_fill_kernel(
    const int32_t* __restrict__ idx, const double* __restrict__ w, int np,
    int k, const int32_t* __restrict__ ptr, int32_t* __restrict__ fill,
    int32_t* __restrict__ rev) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= (int64_t)np * k) return;
  const int t = (int)(g / k);
  if (w[t] == 0.0) return;
  const int j = idx[g];
  if (j < 0 || j >= np) return;
  const int pos = atomicAdd(&fill[j], 1);
  rev[ptr[j] + pos] = t;
}

// Sort each reverse bucket by t, one wave per bucket: up to 64 entries in
// registers, up to SORT_LDS in the wave's LDS, longer ones where they are, by a
// bitonic network whose every exchange is ascending (the first step of a merge
// pairs an element with its mirror image), so that positions past the end act
// as +inf. Buckets hold k entries on average, but a trajectory near the centre
// of its data is a neighbour of hundreds: with one thread per bucket (insertion
// sort) the longest of T = 1461, k = 10 took 205 us, this 8 us.
constexpr int SORT_LDS = 1024;
__device__ __forceinline__ void sort_ints(int32_t* v, int n, int lane) {
  for (int size = 2; size < 2 * n; size <<= 1) {
    for (int s = size; s > 1; s >>= 1) {  // s == size: the mirror step
      const int half = s >> 1;
      for (int p = lane;; p += 64) {
        const int blk = p / half * s, off = p % half;
        const int i = blk + off, j = s == size ? blk + s - 1 - off : i + half;
        if (blk >= n) break;
        if (j < n) {
          const int32_t x = v[i], y = v[j];
          if (y < x) {
            v[i] = y;
            v[j] = x;
          }
        }
      }
      __threadfence_block();
      __builtin_amdgcn_wave_barrier();
    }
  }
}
__global__ __launch_bounds__(256) void rev_sort_kernel(const int32_t* __restrict__ ptr,
                                                       int np, int32_t* rev) {
  __shared__ int32_t lds[4][SORT_LDS];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = blockIdx.x * 4 + w;
  if (j >= np) return;
  const int b = ptr[j], n = ptr[j + 1] - b;
  if (n < 2) return;
  if (n <= 64) {
    double none = 0.0;
    int c = lane < n ? rev[b + lane] : INT_MAX;
    bitonic_sort64(none, c);  // equal distances: by the index alone
    if (lane < n) rev[b + lane] = c;
  } else if (n <= SORT_LDS) {
    for (int q = lane; q < n; q += 64) lds[w][q] = rev[b + q];
    __builtin_amdgcn_wave_barrier();
    sort_ints(lds[w], n, lane);
    for (int q = lane; q < n; q += 64) rev[b + q] = lds[w][q];
  } else {
    sort_ints(rev + b, n, lane);
  }
}

// A workgroup owns GB_COLS columns of one output row, 4 consecutive ones per
// thread (16-byte loads; strided rows fall back to scalar stores of the
// output). Rows that no term touches are written as zeros and nothing else. For
// the others the workgroup first lists the row's terms (source row, coefficient)
// in LDS, in a fixed order -- W_ab: a = t + m, b = j + m for j in N_t, by m and
// rank; W_ba: a = j + m with j in N_t, b = t + m, by m and t -- with the loads
// of weights, neighbours and reverse lists side by side instead of one behind
// the other; then each thread gathers its columns in FP64, GB_BATCH terms'
// source vectors in flight at once, rounded once to FP32. The first wave lists
// the forward terms and the first 64 reverse ones, the workgroup the others.
//
// What bounds it: with a few weighted trajectories HBM (the gradient's zeros and
// the source rows). One workgroup a row for the zero rows instead of one per
// GB_COLS columns: 139 against 105 us at T = 10957, D = 8192, 100 weighted.
// A gradient larger than the Infinity Cache is written with non-temporal stores
// (launch_backward). With all trajectories weighted the source rows, and among
// them the rows that many trajectories have as a neighbour, hundreds of terms
// long. T = 2000, D = 8192, L = 5, k = 10, all weighted, the whole backward:
// 663 us with the terms looked up one after the other and one-thread sorts, 581
// now; with one trajectory in every list 124 against 1.6 ms.
//
// A list costs a short row more than it saves. With one length offset (L = 1)
// a row's terms are few and lie in two runs, and up to GB_DIRECT of them are
// read where they are. L = 1, k = 1, all weighted, us looked up / listed /
// direct: T = 10957, D = 8192 264 / 276 / 243; T = 2000, D = 16384 85 / 89 / 84;
// T = 20000, D = 512 78 / 82 / 75 (listed by the whole workgroup; by the first
// wave 266, 90 and 80). 4, 8 and 16 direct terms are within 1% of each other.
constexpr int GB_BATCH = 4;    // terms whose source vectors are loaded together
constexpr int GB_DIRECT = 8;   // most terms of a row of L = 1 that are not listed
constexpr int GB_REV = 256;    // reverse terms listed at a time, at least 64
constexpr int GB_COLS = 256 * 4;
constexpr uint64_t INFINITY_CACHE_BYTES = (uint64_t)256 << 20;

// How the gradient is stored: by element where its rows are not 16-byte aligned,
// else 16 bytes a lane, through the caches or past them.
enum GradStore { GRAD_SCALAR, GRAD_VECTOR, GRAD_STREAM };

template <GradStore STORE>
__global__ __launch_bounds__(256) void grad_rows_kernel(
    const float* __restrict__ X, int64_t ldx, int T, int64_t D, int L, int k,
    const int32_t* __restrict__ idx, const double* __restrict__ w,
    const int32_t* __restrict__ ptr, const int32_t* __restrict__ rev,
    const int32_t* __restrict__ touch, float* __restrict__ g, int64_t ldg) {
  extern __shared__ __attribute__((aligned(16))) char terms[];
  double* const tc = (double*)terms;       // [L k + GB_REV]
  int* const tb = (int*)(tc + L * k + GB_REV);
  __shared__ int fwd, rv_b[TRAKNN_MAX_L], rv_e[TRAKNN_MAX_L + 1];  // reverse buckets, their ends
  const int a = blockIdx.x;
  const int np = T - L + 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t c = (int64_t)blockIdx.y * GB_COLS + 4 * tid;
  float* ga = g + (int64_t)a * ldg;
  auto store = [&](float4 v) __attribute__((always_inline)) {
    const f32x4 x = {v.x, v.y, v.z, v.w};
    if (STORE == GRAD_STREAM && c + 3 < D) {
      __builtin_nontemporal_store(x, (f32x4*)(ga + c));
    } else if (STORE == GRAD_VECTOR && c + 3 < D) {
      *(f32x4*)(ga + c) = x;
    } else {
      if (c < D) ga[c] = v.x;
      if (c + 1 < D) ga[c + 1] = v.y;
      if (c + 2 < D) ga[c + 2] = v.z;
      if (c + 3 < D) ga[c + 3] = v.w;
    }
  };
  if (!touch[a]) {
    store(make_float4(0.f, 0.f, 0.f, 0.f));
    return;
  }
  // FP32 source vector of row r at the thread's columns (zero past D)
  auto load = [&](int64_t r) __attribute__((always_inline)) {
    const float* p = X + r * ldx + c;
    if (c + 3 < D) return *(const float4*)p;
    return make_float4(c < D ? p[0] : 0.f, c + 1 < D ? p[1] : 0.f, c + 2 < D ? p[2] : 0.f,
                       c + 3 < D ? p[3] : 0.f);
  };
  const double invk = 1.0 / (double)k;
  const float4 x = load(a);
  const double xa[4] = {x.x, x.y, x.z, x.w};
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  // up to GB_BATCH terms, n of them: term(u, source row, coefficient). The others
  // read the row itself with weight 0 (an exact zero contribution).
  auto gather = [&](int n, auto term) __attribute__((always_inline)) {
    float4 xb[GB_BATCH];
    double cc[GB_BATCH];
#pragma unroll
    for (int u = 0; u < GB_BATCH; ++u) {
      int b = a;
      cc[u] = 0.0;
      if (u < n) term(u, b, cc[u]);
      xb[u] = load(b);
    }
#pragma unroll
    for (int u = 0; u < GB_BATCH; ++u) {
      acc[0] += cc[u] * (xa[0] - (double)xb[u].x);
      acc[1] += cc[u] * (xa[1] - (double)xb[u].y);
      acc[2] += cc[u] * (xa[2] - (double)xb[u].z);
      acc[3] += cc[u] * (xa[3] - (double)xb[u].w);
    }
  };
  auto finish = [&]() __attribute__((always_inline)) {
    store(make_float4((float)(2.0 * acc[0]), (float)(2.0 * acc[1]), (float)(2.0 * acc[2]),
                      (float)(2.0 * acc[3])));
  };
  if (L == 1) {
    const double wt = w[a];
    const int nf = wt != 0.0 ? k : 0, p0 = ptr[a], n = nf + ptr[a + 1] - p0;
    if (n <= GB_DIRECT) {
      for (int q = 0; q < n; q += GB_BATCH)
        gather(n - q, [&](int u, int& b, double& c) __attribute__((always_inline)) {
          const int e = q + u;
          const int r = e < nf ? idx[(int64_t)a * k + e] : rev[p0 + e - nf];
          if (e < nf && (r < 0 || r >= np)) return;
          b = r;
          c = (e < nf ? wt : w[r]) * invk;
        });
      finish();
      return;
    }
  }
  if (tid < 64) {  // the first wave lists the forward terms and the first reverse ones
    // the row's weights and reverse buckets, one length offset a lane
    const int ta = a - lane;
    const bool in = lane < L && ta >= 0 && ta < np;
    const double wt = in ? w[ta] : 0.0;
    const int p0 = in ? ptr[ta] : 0, p1 = in ? ptr[ta + 1] : 0;
    int sum = p1 - p0;
#pragma unroll
    for (int o = 1; o < TRAKNN_MAX_L; o <<= 1) {
      const int y = __shfl_up(sum, o, 64);
      if (lane >= o) sum += y;
    }
    if (lane < L) {
      rv_b[lane] = p0;
      rv_e[lane + 1] = sum;
    }
    if (lane == 0) rv_e[0] = 0;
    auto neighbour = [&](int m) __attribute__((always_inline)) {
      return lane < k ? idx[(int64_t)(a - m) * k + lane] : -1;
    };
    uint64_t ms = __ballot(wt != 0.0);
    int j = ms ? neighbour(__builtin_ctzll(ms)) : -1;
    // reverse term `lane`: its bucket rm, its place there
    int rm = 0;
    for (int m = 0; m < L; ++m) rm += lane >= __builtin_amdgcn_readlane(sum, m);
    const bool rev_in = rm < L;
    const int rp = __shfl(p1 - sum, rev_in ? rm : 0, 64) + lane;
    const int t = rev_in ? rev[rp] : 0;
    const double rw = rev_in ? w[t] : 0.0;
    int n = 0;
    while (ms) {
      const int m = __builtin_ctzll(ms);
      ms &= ms - 1;
      const int jn = ms ? neighbour(__builtin_ctzll(ms)) : -1;
      const double cm = readlane_d(wt, m) * invk;
      const uint64_t ok = __ballot(j >= 0 && j < np);
      if ((ok >> lane) & 1) {
        const int pos = n + mask_rank(ok);
        tb[pos] = j + m;
        tc[pos] = cm;
      }
      n += __builtin_popcountll(ok);
      j = jn;
    }
    if (rev_in) {
      tb[n + lane] = t + rm;
      tc[n + lane] = rw * invk;
    }
    if (lane == 0) fwd = n;
  }
  __syncthreads();
  const int nf = fwd, nr = rv_e[L];
  int done = 0;  // listed terms already gathered (the forward ones, after the first list)
  for (int r0 = 0; r0 == 0 || r0 < nr; r0 += GB_REV) {
    const int n = nf + (nr - r0 < GB_REV ? nr - r0 : GB_REV);
    if (r0 > 0) __syncthreads();  // the previous list is used
    if (nr > 64) {  // the first 64 are listed
      for (int e = r0 > 0 ? tid : tid + 64; e < n - nf; e += 256) {
        int m = 0;
        while (r0 + e >= rv_e[m + 1]) ++m;
        const int t = rev[rv_b[m] + (r0 + e - rv_e[m])];
        tb[nf + e] = t + m;
        tc[nf + e] = w[t] * invk;
      }
      __syncthreads();
    }
    for (int q = done; q < n; q += GB_BATCH)
      gather(n - q, [&](int u, int& b, double& c) __attribute__((always_inline)) {
        b = tb[q + u];
        c = tc[q + u];
      });
    done = nf;
  }
  finish();
}

}  // namespace

hipError_t launch_backward(const float* X, int64_t ldx, int64_t T, int64_t D,
                           int L, int k, const int32_t* idx, const double* w,
                           float* g, int64_t ldg, int32_t* zeroed, int32_t* ptr,
                           int32_t* rev, hipStream_t s) {
  // zeroed: the contiguous int32 arrays cnt [np], fill [np], touch [T]
  const int np = (int)(T - L + 1);
  int32_t* cnt = zeroed;
  int32_t* fill = zeroed + np;
  int32_t* touch = zeroed + 2 * (int64_t)np;
  const int64_t nz = 2 * (int64_t)np + T;
  const int64_t nk = (int64_t)np * k;
  const unsigned gk = (unsigned)((nk + 255) / 256);
  hipError_t e;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, s,
                     zeroed, nz, 0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(rev_count_kernel, dim3(gk), dim3(256), 0, s, idx, w, np, k, L, cnt, touch);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, cnt, np, ptr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(rev_fill_kernel, dim3(gk), dim3(256), 0, s, idx, w, np, k, ptr,
                     fill, rev);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(rev_sort_kernel, dim3((unsigned)((np + 3) / 4)), dim3(256), 0, s, ptr, np, rev);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 grid((unsigned)T, (unsigned)((D + GB_COLS - 1) / GB_COLS));
  const size_t lds = (size_t)(L * k + GB_REV) * (sizeof(double) + sizeof(int));  // at most 15 KB
  const bool vec_out = ldg % 4 == 0 && ((uintptr_t)g % 16) == 0;
  // Non-temporal stores for a gradient larger than the 256 MB Infinity Cache,
  // which no reader would find there. D = 8192, 100 trajectories weighted, us
  // non-temporal / plain. Calls back to back: 133 / 185 (359 MB), 124 / 159 (256
  // MB), 104 / 113 (192 MB), 72 / 74 (64 MB); one call on an idle GPU: 178 / 168
  // (359 MB). What counts is the call and a reader of the gradient behind it, on
  // caches full of other data: 815 / 837 (900 MB), 350 / 356 (300 MB), 328 / 317
  // (256 MB), 267 / 252 (192 MB), 147 / 128 (64 MB).
  const bool stream = (uint64_t)T * (uint64_t)D * 4 > INFINITY_CACHE_BYTES;
#define TRAKNN_GRAD_ROWS(S)                                                                     \
  hipLaunchKernelGGL(grad_rows_kernel<S>, grid, dim3(256), lds, s, X, ldx, (int)T, D, L, k, idx, \
                     w, ptr, rev, touch, g, ldg)
  if (!vec_out) TRAKNN_GRAD_ROWS(GRAD_SCALAR);
  else if (stream) TRAKNN_GRAD_ROWS(GRAD_STREAM);
  else TRAKNN_GRAD_ROWS(GRAD_VECTOR);
#undef TRAKNN_GRAD_ROWS
  return hipGetLastError();
}

}  // namespace traknn
