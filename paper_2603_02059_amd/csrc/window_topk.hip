// Trajectory distances by the diagonal window recurrence and exclusion-zone
// top-k (paper, Algorithm 1 stages 2-3; Eq. 5 and Eq. 3).
//
// D_L(i,j) = sum_{m<L} d(i+m, j+m) only ever walks along a diagonal of the
// distance matrix, so the natural gfx950 mapping puts one diagonal on each lane
// of a wave64: lane q of a wave follows the diagonal delta = j - i = delta_c + q.
// At step s the 64 lanes hold the 64 consecutive columns r + delta_c .. +63 of
// row r = r0 + s, i.e. one coalesced 256-byte segment of S per step, and each
// lane advances its own window with the recurrence
//   D <- (D - d(r, r+delta)) + d(r+L, r+L+delta)             (Eq. 5)
// in FP64. Every row block restarts its windows with a direct L-term sum, so
// rounding can never drift over more than a block's rows (and for FP32 inputs
// whose exponents span less than ~29 bits the FP64 recurrence is exact).
//
// The 64 candidates of a step all belong to the same row, so the top-k filter
// is one compare per lane against that row's bound and one ballot; the few
// candidates that pass are merged into the row's sorted list, held one entry
// per lane.
//
// A launch may cover part of the matrix (band mode, row-batched streaming):
// S then holds rows s0 .. s_end - 1, and column c of the matrix at column
// c - col0 of the buffer; the launch covers the trajectory rows row_lo ..
// row_cap - 1 against the candidate columns c_lo .. c_hi - 1 whose diagonal
// offset j - i lies in dmin .. dmax, reads values only in columns c_lo ..
// v_end - 1 (zero elsewhere, which leaves the windows of valid candidates
// exact). Only the diagonals of the offset range are visited, and only their
// values are relied on.
//
// A multi-length request (L = L_min .. L_max) runs the kernel on up to ten
// lengths at a time on the same distance matrix, each length with its own
// running sums, lists and exclusion zone |i - j| >= L. The result does not
// depend on the order in which the waves run, nor on how the lengths are
// grouped into passes.
#include <array>
#include <cfloat>
#include <climits>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "topk_wave.h"

namespace traknn {
namespace {

// ---------------------------------------------------------------------------
// Window + top-k kernel for the trajectory lengths L .. L + G - 1.
//
// What bounds it: one length at T = 27394 reads 4.7 GB of S (both triangles and
// the L - 1 halo rows of every eight) in 0.69 to 0.76 ms (L = 5, k = 10; 0.82 to
// 1.0 ms at k = 40; box to box, and under the clocks of the Gram before it), at
// the rate of a large read; short series, the latency of a few rounds (12 us at T
// = 512, 52 us at T = 5000); several lengths, vector issue. Before,
// every wave kept a list of its own for each of the eight rows and a merge
// kernel joined them, so that the work on lists grew with the waves: 0.84 and
// 1.39 ms plus 0.02 and 0.03 of merge at T = 27394, 28 + 14 us at T = 512, 125 +
// 28 us at T = 5000 (316 + 27 against 157 us at T = 10957).
//
// One workgroup of eight waves per block of eight rows. The block's diagonals
// go in chunks of 64, eight consecutive chunks (one per wave) a round: a round
// reads 2 KB runs of each of the 8 + L - 1 rows. A lane holds its diagonal's
// values of the current chunk and of the next one, which is on its way from
// memory meanwhile; a step is two FP64 adds, two readlanes of the row's bound,
// one compare and a ballot.
//
// The lists: wave w owns row w's sorted list, one entry per lane. Every wave
// filters its chunk's candidates against the rows' bounds (the lists' k-th
// distances, in LDS; candidates equal to the bound still reach the exact
// (distance, index) test) and appends the few that pass to the rows' buffers in
// LDS. After the round's barrier each owner merges its row's buffer into its
// list and lowers the bound, while the next round fills the other buffers: one
// barrier a round, and a bound read before its update is only looser. So a row
// has one list and one bound, as tight as a single scan's, whatever the number
// of waves, and the list goes straight to the output.
//
// Where a row's candidates of a round do not fit its buffer (a first round, when
// there is no bound yet; ties; distances that fall along the scan), the whole
// round is taken densely: the waves put all their sums in LDS, and each owner
// picks from its row's 512. It bounds them first by the k-th smallest of its
// lanes' minima (at least k are within it), so that one sort of at most 64 is
// the usual cost. Where distances fall along the scan every round is dense, and
// still cheaper than one insertion per candidate was: a ramp of T = 8000, D = 64,
// whole calls, L = 5, k = 10 1396 -> 711 us, L = 16, k = 64 5568 -> 2725; T = 5000,
// L = 1..10, k = 5 7660 -> 3135. Which rounds are dense changes nothing in the
// lists: they hold the k smallest of all candidates by (distance, index).
//
// A launch may start from lists that are already in the output (band mode's
// later passes): their rows have a bound from the first round on.
//
// The lengths of a multi-length sweep share one pass over S, as many as
// pass_lengths allows: the values of a chunk are read once for all of them, the
// lengths take turns with the lane's sums, and each length has its own lists
// (in LDS where there are several), bounds and exclusion zone. Each length's
// sums are started and slid exactly as in a pass of its own, so the results do
// not depend on the grouping.
// ---------------------------------------------------------------------------
constexpr int W1_ROWS = 8;         // rows per block
constexpr int W1_WAVES = W1_ROWS;  // wave w owns row w
constexpr int W1_CNT = 4;          // rotating counters of the buffers
constexpr int W1_MAX_G = 10;       // lengths per pass
// Entries of a row's buffer: a round passes k / r candidates of a row in
// expectation (r the round), and two sets of every length's buffers stay within
// the LDS that a dense round's sums take anyway.
constexpr int w1_cap(int G) { return G <= 2 ? 64 : G <= 5 ? 32 : 16; }

// LDS barrier that leaves the wave's vector loads in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  // vmcnt and expcnt at their maxima, lgkmcnt 0
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// A dense round's pick for one row: 512 distances dump[u * 64 * W1_ROWS +
// lane] (NaN: no candidate) of the columns col + 64 u + lane, u < 8, into the
// row's list.
__device__ __forceinline__ void dense_merge(const double* dump, int col, int k, double& ed, int& ei,
                                            double* sd, int* si, int lane) {
  constexpr int STEP = 64 * W1_ROWS;
  double tau = readlane_d(ed, k - 1);
  if (tau == __builtin_huge_val()) {
    double mn = tau;
#pragma unroll
    for (int u = 0; u < W1_WAVES; ++u) mn = __builtin_fmin(mn, dump[u * STEP + lane]);
    tau = readlane_d(sort_dist64(mn), k - 1);
  }
  tau = __builtin_fmin(tau, DBL_MAX);  // +inf is not listed
  int total = 0;  // entries in the scratch
  auto absorb = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_wave_barrier();
    double d = lane < total ? sd[lane] : __builtin_huge_val();
    int c = lane < total ? si[lane] : INT_MAX - 64 + lane;
    if (__builtin_amdgcn_readfirstlane(ei) == INT_MAX) {  // an empty list
      bitonic_sort64(d, c);
      const bool real = lane < (total < k ? total : k);
      ed = real ? d : __builtin_huge_val();
      ei = real ? c : INT_MAX;
    } else {
      const bool pass = lane < total && key_less(d, c, readlane_d(ed, k - 1),
                                                 __builtin_amdgcn_readlane(ei, k - 1));
      merge_batch(__ballot(pass), d, c, k, ed, ei, sd, si, lane);
    }
    __builtin_amdgcn_wave_barrier();
    total = 0;
  };
#pragma unroll 1
  for (int u = 0; u <= W1_WAVES; ++u) {
    if (u == W1_WAVES) {
      if (total) absorb();
      break;
    }
    const double d = dump[u * STEP + lane];
    const int c = col + 64 * u + lane;
    auto within = [&]() __attribute__((always_inline)) {
      return __ballot((d <= tau) & key_less(d, c, readlane_d(ed, k - 1),
                                            __builtin_amdgcn_readlane(ei, k - 1)));
    };
    uint64_t m = within();
    if (total + __builtin_popcountll(m) > 64) {
      absorb();
      m = within();
    }
    if ((m >> lane) & 1) {
      const int pos = total + mask_rank(m);
      sd[pos] = d;
      si[pos] = c;
    }
    total += __builtin_popcountll(m);
  }
}

template <int L, int G>
__global__ __launch_bounds__(64 * W1_WAVES, 4) void window1_kernel(
    const float* __restrict__ S, int64_t ldS, int T, int s0, int s_end, int col0, int c_lo,
    int c_hi, int v_end, int dmin, int dmax, int row_lo, int row_cap, int acc_end, int k,
    int np0, int32_t* __restrict__ idx, double* __restrict__ dist) {
  constexpr int R = W1_ROWS, W = W1_WAVES, CAP = w1_cap(G);
  constexpr int LG = L + G - 1;  // longest length of the pass
  constexpr int M = R + LG - 1;  // rows of values per chunk
  // the rows' buffers (two sets), under a dense round's sums
  constexpr int BUF = G * R * CAP;  // entries of a set
  constexpr int POOL_BYTES = W * R * 64 * 8;
  static_assert(2 * BUF * 12 <= POOL_BYTES && G <= W1_MAX_G && CAP <= 64, "buffers fit the pool");
  __shared__ __attribute__((aligned(16))) char pool[POOL_BYTES];
  __shared__ double scr_d[W][64];
  __shared__ int scr_i[W][64];
  __shared__ __attribute__((aligned(16))) double bnd[G * R];
  __shared__ int cnt[W1_CNT][G * R];
  extern __shared__ __attribute__((aligned(16))) char lists[];  // G > 1: [G][R][k]
  // An owner lowers a bound while other waves, already in the next round, read
  // it: relaxed atomics, so that a read sees the old value or the new one.
  auto bound_read = [&](int i) __attribute__((always_inline)) {
    return __hip_atomic_load(&bnd[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto bound_write = [&](int i, double v) __attribute__((always_inline)) {
    __hip_atomic_store(&bnd[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  double* const dump = (double*)pool;   // [W][R][64]
  double* const buf_d = (double*)pool;  // [2][G][R][CAP]
  int* const buf_i = (int*)(pool + 2 * BUF * 8);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r0 = row_lo + (int)blockIdx.x * R;
  const int t = r0 + w;  // the wave's own row
  // length L + g: candidate columns c_lo .. c_lo + ncand - 1, rows of this
  // block that exist
  auto chi = [&](int g) __attribute__((always_inline)) {
    const int npl = T - (L + g) + 1;
    return c_hi < npl ? c_hi : npl;
  };
  auto rows_of = [&](int g) __attribute__((always_inline)) {
    const int npl = T - (L + g) + 1;
    const int hi = row_cap < npl ? row_cap : npl;
    return hi - r0 < R ? (hi - r0 > 0 ? hi - r0 : 0) : R;
  };
  // diagonals of the block: every candidate column of some row, within the
  // offset range
  int64_t dlo = (int64_t)c_lo - (r0 + R - 1);
  if (dlo < dmin) dlo = dmin;
  int64_t dhi = (int64_t)chi(0) - 1 - r0;
  if (dhi > dmax) dhi = dmax;
  const int NC = chi(0) > c_lo && rows_of(0) > 0 && dhi >= dlo ? (int)((dhi - dlo + 1 + 63) / 64) : 0;

  // Values of diagonal delta at rows r0 + m (one 256-byte segment per row
  // for the wave), zero outside the held rows and the columns c_lo ..
  // v_end - 1. The pointer walks down the rows
  // with a stride the compiler treats as opaque, so no per-row address is
  // precomputed and held across chunks; chunks wholly inside the matrix skip
  // the bounds tests, the others read a safe element and discard it.
  float nxt[M];
  auto load = [&](int c) __attribute__((always_inline)) {
    const int64_t dc = dlo + 64 * (int64_t)c;
    int64_t stride = ldS + 1;
    asm volatile("" : "+s"(stride));
    const float* row = S + ((int64_t)(r0 - s0) * ldS + (r0 + dc - col0));  // wave-uniform
    const bool inb = r0 + dc >= c_lo && r0 + M - 1 < s_end && r0 + M - 1 + dc + 63 < v_end;
    if (inb) {
#pragma unroll
      for (int m = 0; m < M; ++m) {
        nxt[m] = row[lane];
        row += stride;
      }
    } else {
      const float* p = row + lane;
      int rows_in = s_end - r0;  // rows r0 + m with m < rows_in are held
      int64_t vlo = c_lo, vhi = v_end;
      asm volatile("" : "+s"(rows_in), "+s"(vlo), "+s"(vhi));
      int64_t col = r0 + dc + lane;  // column of row r0 + m, stepped with m
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const bool ok = (m < rows_in) & (col >= vlo) & (col < vhi);
        const float x = *(ok ? p : S);
        nxt[m] = ok ? x : 0.f;
        p += stride;
        col += 1;
      }
    }
  };
  if (w < NC) load(w);

  // The wave's own lists (row t, length L + g) and their bounds.
  double own_d = __builtin_huge_val();
  int own_i = INT_MAX;
  double* const list_d = (double*)lists + (size_t)w * k + lane;
  int* const list_i = (int*)((double*)lists + (size_t)G * R * k) + (size_t)w * k + lane;
  auto get = [&](int g, double& ed, int& ei) __attribute__((always_inline)) {
    if constexpr (G == 1) {
      ed = own_d;
      ei = own_i;
    } else {
      ed = lane < k ? list_d[g * R * k] : __builtin_huge_val();
      ei = lane < k ? list_i[g * R * k] : INT_MAX;
    }
  };
  auto put = [&](int g, double ed, int ei) __attribute__((always_inline)) {
    if constexpr (G == 1) {
      own_d = ed;
      own_i = ei;
    } else if (lane < k) {
      list_d[g * R * k] = ed;
      list_i[g * R * k] = ei;
    }
    const double kth = readlane_d(ed, k - 1);
    if (lane == 0) bound_write(g * R + w, kth);
  };
#pragma unroll 1
  for (int g = 0; g < G; ++g) {
    double ed = __builtin_huge_val();
    int ei = INT_MAX;
    const bool there = w < rows_of(g);
    if (there && t < acc_end && lane < k) {
      const int64_t o = ((int64_t)g * np0 + t) * k + lane;
      ed = dist[o];
      ei = idx[o] < 0 ? INT_MAX : idx[o];
    }
    put(g, ed, ei);
    if (!there && lane == 0) bound_write(g * R + w, -__builtin_huge_val());  // no such row: nothing passes
  }
  for (int q = threadIdx.x; q < W1_CNT * G * R; q += 64 * W) (&cnt[0][0])[q] = 0;
  lds_barrier();

  // interior chunks: every row exists for every length, and the columns and
  // the exclusion zone of the longest length (the strictest) are clear
  const bool full = rows_of(G - 1) == R;
  const int rounds = (NC + W - 1) / W;
#pragma unroll 1
  for (int r = 0; r < rounds; ++r) {
    const int c = r * W + w;
    const int64_t dc = dlo + 64 * (int64_t)c;
    const int delta = (int)dc + lane;
    const bool interior = full & (c < NC) & ((dc >= LG) | (dc + 63 <= -LG)) & (r0 + dc >= c_lo) &
                          (r0 + R - 1 + dc + 63 < chi(G - 1)) & (dc >= dmin) & (dc + 63 <= dmax);
    float cur[M];
#pragma unroll
    for (int m = 0; m < M; ++m) cur[m] = nxt[m];
    if (c + W < NC) load(c + W);
    // D_{L+g} of the block's rows on the lane's diagonal (NaN: no candidate),
    // D0 its first row's, a sum in increasing order
    auto sums = [&](int g, double D0, double (&Dj)[R]) __attribute__((always_inline)) {
      double D = D0;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        Dj[j] = D;
        if (j + 1 < R) D = (D - (double)cur[j]) + (double)cur[j + L + g];
      }
      if (!interior) {
        const bool okd = ((delta >= L + g) | (delta <= -(L + g))) & (delta >= dmin) &
                         (delta <= dmax) & (c < NC);
        const int nc = chi(g) - c_lo;
        int nr = rows_of(g);
        asm volatile("" : "+v"(nr));  // tested where it is used, not kept as masks
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const int col = r0 + j + delta;
          const bool ok = okd & ((unsigned)(col - c_lo) < (unsigned)(nc > 0 ? nc : 0)) & (j < nr);
          Dj[j] = ok ? Dj[j] : __builtin_nan("");
        }
      }
    };
    auto first_sum = [&]() __attribute__((always_inline)) {
      double D = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) D += (double)cur[l];
      return D;
    };
    const bool unbounded = r == 0 && r0 >= acc_end;  // no list yet: a dense round
    double D1[R];  // one length: its sums, kept for a dense round
    if constexpr (G == 1) sums(0, first_sum(), D1);
    if (!unbounded && c < NC) {
      double Dg = G == 1 ? 0.0 : first_sum();
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // the rows' bounds: with one length from a lane each, which keeps the
        // registers of seven waves per SIMD; else the same in every lane, which
        // saves the lane reads
        const double bl = G == 1 ? bound_read(lane & (R - 1)) : 0.0;
        double bound[R];
#pragma unroll
        for (int j = 0; j < R; ++j) bound[j] = G == 1 ? readlane_d(bl, j) : bound_read(g * R + j);
        double Dj[R];
        if constexpr (G == 1) {
#pragma unroll
          for (int j = 0; j < R; ++j) Dj[j] = D1[j];
        } else {
          sums(g, Dg, Dj);
          if (g + 1 < G) Dg += (double)cur[L + g];
        }
        uint64_t m[R];
        uint64_t any = 0;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          m[j] = __ballot(Dj[j] <= bound[j]);
          any |= m[j];
        }
        if (any) {
          // lane j reserves row j's entries, all rows at once
          int n = 0;
#pragma unroll
          for (int j = 0; j < R; ++j)
            n = lane_select((uint64_t)1 << j, (int)__builtin_popcountll(m[j]), n);
          int at = 0;
          if (n) at = __hip_atomic_fetch_add(&cnt[r & (W1_CNT - 1)][g * R + lane], n, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
          for (int j = 0; j < R; ++j)
            if (m[j]) {
              const int pos = __builtin_amdgcn_readlane(at, j) + mask_rank(m[j]);
              if (((m[j] >> lane) & 1) && pos < CAP) {
                const int o = (r & 1) * BUF + (g * R + j) * CAP + pos;
                buf_d[o] = Dj[j];
                buf_i[o] = r0 + j + delta;
              }
            }
        }
      }
    }
    lds_barrier();
    // every wave sees the same counts (they are cleared a round later): the
    // lengths whose buffers overflowed go densely
    uint32_t dense = unbounded ? (1u << G) - 1 : 0;
    if (!unbounded) {
      const int* const cr = cnt[r & (W1_CNT - 1)];
      const uint64_t o0 = __ballot(lane < G * R && cr[lane < G * R ? lane : 0] > CAP);
      uint64_t o1 = 0;
      if constexpr (G * R > 64) o1 = __ballot(lane + 64 < G * R && cr[lane + 64 < G * R ? lane + 64 : 0] > CAP);
      if (o0 | o1) {
        for (int g = 0; g < G; ++g)
          if (((g < 8 ? o0 >> (8 * g) : o1 >> (8 * (g - 8))) & 0xFF) != 0) dense |= 1u << g;
      }
      // the other lengths: merge the own row's buffers
      const int nq = lane < G ? cr[lane * R + w] : 0;
      uint64_t todo = __ballot(nq > 0) & ~(uint64_t)dense;
      while (todo) {
        const int g = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int n = __builtin_amdgcn_readlane(nq, g);
        const int o = (r & 1) * BUF + (g * R + w) * CAP + lane;
        const double d = lane < n ? buf_d[o] : __builtin_huge_val();
        const int ci = lane < n ? buf_i[o] : INT_MAX;
        double ed;
        int ei;
        get(g, ed, ei);
        // below +inf: not a lane past the entries, nor a distance that is +inf
        const uint64_t m = __ballot((d <= DBL_MAX) & key_less(d, ci, readlane_d(ed, k - 1),
                                                              __builtin_amdgcn_readlane(ei, k - 1)));
        if (!m) continue;
        merge_batch(m, d, ci, k, ed, ei, scr_d[w], scr_i[w], lane);
        put(g, ed, ei);
      }
    }
    if (dense) {
      lds_barrier();  // the buffers of this round are merged
#pragma unroll 1
      for (int g = 0; g < G; ++g) {
        if (!((dense >> g) & 1)) continue;
        if constexpr (G == 1) {
#pragma unroll
          for (int j = 0; j < R; ++j) dump[(w * R + j) * 64 + lane] = D1[j];
        } else {
          double Dg = first_sum();
#pragma unroll
          for (int q = 0; q < G; ++q) {
            if (q == g) {
              double Dj[R];
              sums(q, Dg, Dj);
#pragma unroll
              for (int j = 0; j < R; ++j) dump[(w * R + j) * 64 + lane] = Dj[j];
            }
            if (q + 1 < G) Dg += (double)cur[L + q];
          }
        }
        lds_barrier();
        if (w < rows_of(g)) {
          const int col = t + (int)(dlo + 64 * (int64_t)(r * W));
          double ed;
          int ei;
          get(g, ed, ei);
          dense_merge(dump + w * 64, col, k, ed, ei, scr_d[w], scr_i[w], lane);
          put(g, ed, ei);
        }
        lds_barrier();  // the sums are read before the pool is used again
      }
    }
    if (lane < G) cnt[(r + W1_CNT - 1) & (W1_CNT - 1)][lane * R + w] = 0;
  }
  // the row's lists; rows that do not exist for a length hold -1 and +inf
  if (t < row_cap) {
#pragma unroll 1
    for (int g = 0; g < G; ++g) {
      double ed;
      int ei;
      get(g, ed, ei);
      const bool there = w < rows_of(g);
      if (lane < k) {
        const int64_t o = ((int64_t)g * np0 + t) * k + lane;
        idx[o] = there && ei != INT_MAX ? ei : -1;
        dist[o] = there ? ed : __builtin_huge_val();
      }
    }
  }
}

// Lengths of a sweep's next pass when `left` remain: 10, 5, 2 or 1, as many as
// are left and hold at most 120 list entries a row between them: the first
// rounds pass about k candidates a row and length, which have to fit the
// buffers (w1_cap). Window stage, T = 27394, L = 1..10, k = 10: 4.6 ms with 10,
// 5.1 with 5, 6.1 with 2 a pass; T = 6000, L = 1..16, k = 20: 1.26, 1.10 and
// 1.12 ms. The lists' LDS (at most 12 KB) and the static 40 KB stay within 64.
inline int pass_lengths(int left, int k) {
  for (const int g : {10, 5, 2})
    if (left >= g && g * k <= 120) return g;
  return 1;
}

// Row blocks of rows row_lo .. row_cap - 1, the block of length L's lists at
// idx and dist.
template <int L, int G>
hipError_t launch_win1(const float* S, int64_t ldS, int T, const WindowRange& r, int row_lo,
                       int row_cap, int acc_end, int k, int np0, int32_t* idx, double* dist,
                       hipStream_t s) {
  const unsigned blocks = (unsigned)((row_cap - row_lo + W1_ROWS - 1) / W1_ROWS);
  const size_t lds = G > 1 ? (size_t)G * W1_ROWS * k * 12 : 0;
  hipLaunchKernelGGL((window1_kernel<L, G>), dim3(blocks), dim3(64 * W1_WAVES), lds, s, S, ldS, T,
                     (int)r.s0, (int)r.s_end, (int)r.col0, (int)r.c_lo, (int)r.c_hi, (int)r.v_end,
                     (int)r.dmin, (int)r.dmax, row_lo, row_cap, acc_end, k, np0, idx, dist);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void score_kernel(
    const double* __restrict__ dist, int T, int np0, int Lmin, int NL, int k,
    double* __restrict__ scores) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= (int64_t)NL * np0) return;
  const int li = (int)(g / np0);
  const int t = (int)(g % np0);
  const int npL = T - (Lmin + li) + 1;
  if (t >= npL) {
    scores[g] = __builtin_nan("");
    return;
  }
  double s = 0.0;
  for (int q = 0; q < k; ++q) s += dist[g * k + q];
  scores[g] = s / (double)k;
}

// Scores for every k' <= k from one neighbour list (the lists are sorted by
// (distance, index), so the k' nearest are its first k' entries): out[q] =
// mean of dist[0..q], summed in rank order -- out[k-1] is exactly s_t.
__global__ __launch_bounds__(256) void score_prefix_kernel(
    const double* __restrict__ dist, int T, int np0, int Lmin, int NL, int k,
    double* __restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= (int64_t)NL * np0) return;
  const int li = (int)(g / np0);
  const int t = (int)(g % np0);
  const int npL = T - (Lmin + li) + 1;
  double s = 0.0;
  for (int q = 0; q < k; ++q) {
    s += dist[g * k + q];
    out[g * k + q] = t < npL ? s / (double)(q + 1) : __builtin_nan("");
  }
}

// Local intrinsic dimension of every trajectory (the maximum-likelihood kNN
// estimator of Levina and Bickel that the paper applies with k in {20, 30,
// 40}, Section 5.1), for every prefix k' of its sorted list:
//   m_k' = 2 (k' - 1) / sum_{j<k'} ln(dist[k'-1] / dist[j]),
// the Euclidean log-ratio being half the log-ratio of the squared distances.
// out[0] (k' = 1, no ratio) and rows that do not exist are NaN; degenerate
// lists follow IEEE arithmetic (a zero below a positive k'-th distance gives
// 0, a zero k'-th distance NaN, k' equal distances +inf).
//
// Bound by the FP64 logarithms, k (k - 1) / 2 a row: the thread of (row, i)
// takes the ranks q = i and q = k - 1 - i, k - 1 logarithms in all, so that
// every lane has the same number. T = 27394, k = 40: 260 us with one thread per
// row (107 workgroups), 140 with one per (row, q), 82 now; k = 10: 18 and 9 us.
// With hundreds of thousands of rows and k up to 5 a thread per row was as fast
// (ten lengths, k = 3: 7.0 against 7.9 us, k = 5: 15.3 and 16.6, k = 7: 30.9 and
// 27.3).
__global__ __launch_bounds__(256) void local_dim_kernel(
    const double* __restrict__ dist, int T, int np0, int Lmin, int NL, int k,
    double* __restrict__ out) {
  // at most 16 lengths x 2^20 rows x 32 pairs of ranks: 32 bits hold them
  const unsigned half = (unsigned)(k + 1) / 2;
  const unsigned e = blockIdx.x * 256u + threadIdx.x;
  if (e >= (unsigned)NL * (unsigned)np0 * half) return;
  const unsigned row = e / half;
  const int lo = (int)(e - row * half), hi = k - 1 - lo;
  const int li = (int)(row / (unsigned)np0);
  const int t = (int)(row - (unsigned)li * (unsigned)np0);
  const bool exists = t < T - (Lmin + li) + 1;
  const int64_t g = row;
  const double* d = dist + g * k;
  const double d_lo = d[lo], d_hi = d[hi];
  double s_lo = 0.0, s_hi = 0.0;
  for (int it = 0; it < k - 1; ++it) {  // terms j < lo of lo, then j < hi of hi
    const bool first = it < lo;
    const double v = log((first ? d_lo : d_hi) / d[first ? it : it - lo]);
    s_lo = first ? s_lo + v : s_lo;
    s_hi = first ? s_hi : s_hi + v;
  }
  auto put = [&](int q, double s) {
    out[g * k + q] = q > 0 && exists ? 2.0 * (double)q / s : __builtin_nan("");
  };
  put(hi, s_hi);
  if (lo < hi) put(lo, s_lo);
}

}  // namespace

// Launchers of every compiled (L, G): one length, pairs from every L, and five
// or ten lengths from the starts that a sweep's passes reach.
using WinLaunch = hipError_t (*)(const float*, int64_t, int, const WindowRange&, int, int, int,
                                 int, int, int32_t*, double*, hipStream_t);
template <int G, int... Ls>
constexpr std::array<WinLaunch, sizeof...(Ls)> win_table(std::integer_sequence<int, Ls...>) {
  return {&launch_win1<Ls + 1, G>...};
}
constexpr auto kWin1 = win_table<1>(std::make_integer_sequence<int, TRAKNN_MAX_L>{});
constexpr auto kWin2 = win_table<2>(std::make_integer_sequence<int, TRAKNN_MAX_L - 1>{});
static WinLaunch window_launcher(int L, int G) {
  if (L < 1 || L + G - 1 > TRAKNN_MAX_L) return nullptr;
  if (G == 1) return kWin1[L - 1];
  if (G == 2) return kWin2[L - 1];
  if (G == 5) return L == 1 ? &launch_win1<1, 5> : L == 6 ? &launch_win1<6, 5> : L == 11 ? &launch_win1<11, 5> : nullptr;
  return G == 10 && L == 1 ? &launch_win1<1, 10> : nullptr;
}

hipError_t launch_window(const float* S, int64_t ldS, int64_t T, int L_min, int L_max, int k,
                         const WindowRange& r, int64_t t0, int64_t nt, int64_t acc_end,
                         int32_t* idx, double* dist, hipStream_t s) {
  const int64_t np0 = T - L_min + 1;
  for (int L = L_min; L <= L_max;) {
    const int G = pass_lengths(L_max - L + 1, k);
    const WinLaunch f = window_launcher(L, G);
    if (!f) return hipErrorInvalidValue;
    const int64_t off = (int64_t)(L - L_min) * np0 * k;
    const hipError_t e = f(S, ldS, (int)T, r, (int)t0, (int)(t0 + nt), (int)acc_end, k, (int)np0,
                           idx + off, dist + off, s);
    if (e != hipSuccess) return e;
    L += G;
  }
  return hipSuccess;
}

hipError_t launch_score(const double* dist, int64_t T, int L_min, int L_max,
                        int k, double* scores, hipStream_t s) {
  const int np0 = (int)(T - L_min + 1);
  const int NL = L_max - L_min + 1;
  const int64_t n = (int64_t)NL * np0;
  hipLaunchKernelGGL(score_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256),
                     0, s, dist, (int)T, np0, L_min, NL, k, scores);
  return hipGetLastError();
}

hipError_t launch_score_prefix(const double* dist, int64_t T, int L_min, int L_max,
                               int k, double* out, hipStream_t s) {
  const int np0 = (int)(T - L_min + 1);
  const int NL = L_max - L_min + 1;
  const int64_t n = (int64_t)NL * np0;
  hipLaunchKernelGGL(score_prefix_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256),
                     0, s, dist, (int)T, np0, L_min, NL, k, out);
  return hipGetLastError();
}

hipError_t launch_local_dim(const double* dist, int64_t T, int L_min, int L_max, int k,
                            double* out, hipStream_t s) {
  const int np0 = (int)(T - L_min + 1);
  const int NL = L_max - L_min + 1;
  const int64_t n = (int64_t)NL * np0 * ((k + 1) / 2);
  hipLaunchKernelGGL(local_dim_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     dist, (int)T, np0, L_min, NL, k, out);
  return hipGetLastError();
}

}  // namespace traknn
