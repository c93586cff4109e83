// Wave-level (distance, index) top-k helpers shared by the window kernels and
// the fused tile kernels: a sorted list of up to 64 entries is held one entry
// per lane (lane q holds entry q), candidates arrive 64 at a time (one per
// lane), and keys compare lexicographically by (distance, index) so every
// list is unique (paper, Eq. 3 with ties broken by the smaller index).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

namespace traknn {

__device__ __forceinline__ double readlane_d(double v, int l) {
  int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
// (ad, ai) < (bd, bi) lexicographically; bitwise, so it compiles to three
// compares and two mask operations instead of short-circuit branches.
__device__ __forceinline__ bool key_less(double ad, int ai, double bd, int bi) {
  return (ad < bd) | ((ad == bd) & (ai < bi));
}

__device__ __forceinline__ double dpp_shr1_d(double v, double old) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), 0x138, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), 0x138, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ int dpp_shr1_i(int v, int old) {
  return __builtin_amdgcn_update_dpp(old, v, 0x138, 0xF, 0xF, false);
}

// Insert the masked lanes' candidates (D, col), in lane order, into a sorted
// list held in registers (lane q < k holds entry q; lanes from k on are
// don't-care): each insertion that beats the k-th entry shifts the tail of
// the list one lane up with DPP wave_shr:1.
__device__ __forceinline__ void insert_reg(uint64_t mask, double D, int col, int k,
                                           double& ed, int& ei) {
  while (mask) {
    const int src = __builtin_ctzll(mask);
    mask &= mask - 1;
    const double cd = readlane_d(D, src);
    const int ci = __builtin_amdgcn_readlane(col, src);
    const double kd = readlane_d(ed, k - 1);
    const int ki = __builtin_amdgcn_readlane(ei, k - 1);
    if (!key_less(cd, ci, kd, ki)) continue;
    const double pd = dpp_shr1_d(ed, -__builtin_huge_val());  // lane 0: -inf
    const int pi = dpp_shr1_i(ei, INT_MIN);
    const bool lt_prev = key_less(cd, ci, pd, pi);
    const bool lt_self = key_less(cd, ci, ed, ei);
    ed = lt_prev ? pd : (lt_self ? cd : ed);
    ei = lt_prev ? pi : (lt_self ? ci : ei);
  }
}

// The lanes whose number has bit BIT (a power of two) clear; for 64, every lane.
constexpr uint64_t lanes_clear(int bit) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l)
    if (!(l & bit)) m |= (uint64_t)1 << l;
  return m;
}
// a in the lanes of the mask, b elsewhere.
template <typename T>
__device__ __forceinline__ T lane_select(uint64_t mask, T a, T b) {
  return __builtin_amdgcn_inverse_ballot_w64(mask) ? a : b;
}

// The value v of lane (lane ^ S), S a power of two up to 32, by vector ALU
// moves alone (an LDS permute's latency would be paid at every step of a
// sorting network). Strides up to 8 stay inside rows of 16 lanes and use DPP:
// quad permutes for 1 and 2; row rotations for 8 (by 8) and for 4 (by 12 where
// bit 2 of the lane is clear, giving lane + 4, else by 4, giving lane - 4).
// 16 and 32 swap rows and half-waves of two copies of v. Every lane of the wave
// must be active.
template <int S>
__device__ __forceinline__ int lane_xor(int v) {
  static_assert(S == 1 || S == 2 || S == 4 || S == 8 || S == 16 || S == 32, "stride");
  if constexpr (S == 1) {
    return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  } else if constexpr (S == 2) {
    return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  } else if constexpr (S == 4) {
    const int up = __builtin_amdgcn_mov_dpp(v, 0x12C, 0xF, 0xF, false);  // row_ror:12
    const int dn = __builtin_amdgcn_mov_dpp(v, 0x124, 0xF, 0xF, false);  // row_ror:4
    return lane_select(lanes_clear(4), up, dn);
  } else if constexpr (S == 8) {
    return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, false);  // row_ror:8
  } else if constexpr (S == 16) {
    // the first result holds the even rows' values in both rows of a pair, the
    // second the odd rows'
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    return lane_select(lanes_clear(16), (int)r[1], (int)r[0]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return lane_select(lanes_clear(32), (int)r[1], (int)r[0]);
  }
}
template <int S>
__device__ __forceinline__ double lane_xor_d(double v) {
  return __hiloint2double(lane_xor<S>(__double2hiint(v)), lane_xor<S>(__double2loint(v)));
}

// The lanes of a bitonic merge step that keep the smaller of a pair: blocks of
// SIZE lanes end ascending where bit SIZE of the lane is clear, descending
// elsewhere; S is the step's stride. Compile-time masks: a network costs no
// register and no compare for them.
template <int SIZE, int S>
constexpr uint64_t keep_min_lanes() {
  return ~(lanes_clear(S) ^ lanes_clear(SIZE));
}

// One merge of a bitonic network over the wave: compare-exchange with the
// lane S apart, then S / 2, ... 1. SELECT exchanges by lane masks, without
// branches; otherwise under the execution mask, skipped where no lane
// exchanges. The window and FP64 kernels, with five to seven waves per SIMD,
// take the first (the window at k = 40: 816 against 865 us), the MFMA-fused
// consumer, with two, the second (call at D = 32, k = 10: 1313 against 1364 us).
template <bool SELECT, int SIZE, int S>
__device__ __forceinline__ void bitonic_merge64(double& d, int& c) {
  const double pd = lane_xor_d<S>(d);
  const int pc = lane_xor<S>(c);
  if constexpr (SELECT) {
    const uint64_t less = __ballot(pd < d) | (__ballot(pd == d) & __ballot(pc < c));
    const uint64_t take = less ^ ~keep_min_lanes<SIZE, S>();
    d = lane_select(take, pd, d);
    c = lane_select(take, pc, c);
  } else if (__builtin_amdgcn_inverse_ballot_w64(keep_min_lanes<SIZE, S>()) ==
             key_less(pd, pc, d, c)) {
    d = pd;
    c = pc;
  }
  if constexpr (S > 1) bitonic_merge64<SELECT, SIZE, S / 2>(d, c);
}

// Sort the wave's 64 keys (d, c) ascending by (distance, index) across the
// lanes: afterwards lane r holds the r-th smallest (bitonic network of lane
// exchanges, unrolled so that every stride is a compile-time constant). Keys
// must be distinct for a unique result; every lane must be active.
template <bool SELECT = true, int SIZE = 2>
__device__ __forceinline__ void bitonic_sort64(double& d, int& c) {
  bitonic_merge64<SELECT, SIZE, SIZE / 2>(d, c);
  if constexpr (SIZE < 64) bitonic_sort64<SELECT, SIZE * 2>(d, c);
}

// The wave's 64 distances (NaN-free) ascending across the lanes, by the same
// network on the keys alone.
template <typename T, int SIZE, int S>
__device__ __forceinline__ T sort_dist_merge64(T d) {
  if constexpr (sizeof(T) == 8) {
    const T p = lane_xor_d<S>(d);
    d = lane_select(keep_min_lanes<SIZE, S>(), __builtin_fmin(d, p), __builtin_fmax(d, p));
  } else {
    const T p = __builtin_bit_cast(T, lane_xor<S>(__builtin_bit_cast(int, d)));
    d = lane_select(keep_min_lanes<SIZE, S>(), __builtin_fminf(d, p), __builtin_fmaxf(d, p));
  }
  if constexpr (S > 1) return sort_dist_merge64<T, SIZE, S / 2>(d);
  return d;
}
template <typename T, int SIZE = 2>
__device__ __forceinline__ T sort_dist64(T d) {
  d = sort_dist_merge64<T, SIZE, SIZE / 2>(d);
  if constexpr (SIZE < 64) return sort_dist64<T, SIZE * 2>(d);
  return d;
}

// A batch with at least this many entries to take into a sorted list is merged
// by sorts rather than by one insertion each.
constexpr int LIST_SORT_MIN = 6;

// Position of a lane's entry among those of the mask.
__device__ __forceinline__ int mask_rank(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Merge the masked lanes' entries (d, c), each below the list's k-th, into the
// sorted list (ed, ei) in registers (lane q < k holds entry q). Many entries:
// compacted in the wave's scratch (64 entries) they go in with the list (lanes
// < k) up to 64 - k at a time (lanes k ..), one sort each, whose first k lanes
// are the new list. Few: by insertion. Every lane must be active.
__device__ __forceinline__ void merge_batch(uint64_t m, double d, int c, int k, double& ed,
                                            int& ei, double* sd, int* si, int lane) {
  const int cnt = __builtin_popcountll(m);
  const int room = 64 - k;  // entries one sort takes beside the list
  if (cnt >= LIST_SORT_MIN && room >= LIST_SORT_MIN) {
    const int pos = mask_rank(m);
    __builtin_amdgcn_wave_barrier();
    if ((m >> lane) & 1) {
      sd[pos] = d;
      si[pos] = c;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int c0 = 0; c0 < cnt; c0 += room) {
      const int src = lane - k + c0;
      double md = lane < k ? ed : __builtin_huge_val();
      int mi = lane < k ? ei : INT_MAX - 64 + lane;
      if (lane >= k && src < cnt) {
        md = sd[src];
        mi = si[src];
      }
      bitonic_sort64(md, mi);
      const bool real = mi < INT_MAX - 64;
      ed = real ? md : __builtin_huge_val();
      ei = real ? mi : INT_MAX;
    }
    __builtin_amdgcn_wave_barrier();
  } else if (m) {
    insert_reg(m, d, c, k, ed, ei);
  }
}

}  // namespace traknn
