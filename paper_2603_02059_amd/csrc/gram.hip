// Symmetric Gram product and distance epilogue (paper, Algorithm 1 stage 1 and
// Eq. 4): for every tile pair I <= J of 256 (128, 64) fields,
//   d(i,j) = N_i + N_j - 2 <x_i, x_j>   (MFMA, FP32 accumulation),
// stored FP32 at (i,j) and (j,i). Only the upper triangle of tile pairs is
// computed, which halves the contraction as the paper's symmetric batching
// does.
//
// Distance-form accumulation: K runs in chunks of GRAM_CHUNK elements, and once
// a chunk's products are in the accumulators, one extra FP32 MFMA of depth 2
// adds -(N_i^c + N_j^c)/2, the chunk's squared norms (FP64 sums rounded to
// FP32, from the centring pass). The accumulators then hold -d/2 over the
// finished chunks, so they never grow much beyond the distance itself: their
// FP32 rounding errors scale with d + N/(number of chunks) instead of with the
// norms N, which for near neighbours are several times larger than d. The
// epilogue only scales by -2.
//
// Tiling for gfx950, large problems (pick_tile gives short series smaller
// tiles of the same form): 512 threads = 8 wave64s in a 2x4 arrangement, each
// wave owning a 128x64 block = 4x2 MFMA 32x32 blocks held in accumulation
// registers. K runs in slices of 64 bytes of each of the 512 operand rows
// (2 x 16 KB of LDS), four slice buffers deep. Rows are stored with their four
// 16-byte chunks XOR-swizzled by the row index so that the ds_read_b128
// fragment loads of 32 consecutive rows spread over all banks.
//
// What bounds it: with every operand zero (so that the clock is not held down
// by power) the main loop is bound by the arrival of the operands, not by the
// MFMAs. Two buffers of 128 bytes per row with one barrier each gave a load one
// step to land and issued its loads in one burst after the barrier; four
// buffers of 64 bytes give it three of the shorter steps, and the loads are
// spread between the MFMAs. At T = 27394, D = 8192 that took FP16 from 5.06 to
// 4.23 ms with zero operands (5.77 to 5.20 ms with Gaussian ones) and BF16x3
// from 11.08 to 10.14 ms (13.73 to 12.80 ms), all on one box; FP32, MFMA-bound,
// is unchanged. Warming the L2 with touches four to six stages ahead changed
// nothing.
//
// Workgroups are mapped XCD-aware: the hardware deals consecutive workgroup
// ids round-robin to the 8 XCDs, so each XCD is handed a contiguous run of a
// grouped tile order (4 block-rows x successive block-columns). The ~32 tiles
// an XCD runs at once then share 4 A panels and ~8 B panels in its L2.
//
// Band mode (row-batched streaming, for T whose T x T matrix does not fit):
// the kernel fills a band of rows a_row0 .. a_row0 + rows_out - 1 against the
// columns from a_row0's block-column on (the columns before it belong to
// earlier bands), every tile (I, J) of the rectangle that holds an entry above
// the diagonal computed directly. It is stored twice: as rows, into a buffer
// whose row 0 is field a_row0 and column 0 field c0, and transposed, so
// that the later fields' rows of the band's columns are contiguous too.
#include <type_traits>

#include "dist_clamp.h"
#include "fused_walk.h"
#include "internal.h"

namespace traknn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int RB = GRAM_ROW_BYTES;  // bytes per row per slice
// Shape of a workgroup: a TILE x TILE block of the matrix by THREADS / 64 waves
// in a WAVES_M x WAVES_N grid, each owning a WT_M x WT_N block in 32x32 MFMA
// blocks, with BUFFERS slices of both operands in LDS.
template <int TILE_, int THREADS_, int BUFFERS_>
struct GramShape {
  static constexpr int TILE = TILE_, THREADS = THREADS_, BUFFERS = BUFFERS_;
  static constexpr int NWAVES = THREADS / 64;
  static constexpr int WAVES_M = 2, WAVES_N = NWAVES / WAVES_M;
  static constexpr int WT_M = TILE / WAVES_M, WT_N = TILE / WAVES_N;
  static constexpr int BM = WT_M / 32, BN = WT_N / 32;  // MFMA blocks per wave
  static constexpr int OPER_BYTES = TILE * RB;           // one operand of a slice
  static constexpr int SLICE_BYTES = 2 * OPER_BYTES;     // both operands
  static constexpr int BLK_PER_WAVE = OPER_BYTES / 1024 / NWAVES;  // 1 KB loads
  static constexpr int PART_LOADS = 2 * BLK_PER_WAVE;    // a wave's loads of a slice
  static constexpr int PART_READS = 2 * (BM + BN);       // a wave's fragment reads
  static constexpr int NORM_LDS = 2 * 2 * TILE * 4;      // two chunks' norms, I and J rows
  static constexpr int LDS_BYTES = BUFFERS * SLICE_BYTES + NORM_LDS;
  static constexpr int MIN_WAVES = TILE == 256 ? 1 : 2;  // register budget (waves per SIMD)
  static_assert(BM >= 1 && BN >= 1 && BLK_PER_WAVE >= 1, "a wave owns a block and a load");
  static_assert((BUFFERS & (BUFFERS - 1)) == 0 && BUFFERS >= 4, "buffers: a power of two");
};
// 256: large problems and the fused mode. 128 and 64: launches that would leave
// CUs idle (pick_tile); two workgroups of either share a CU (66 KB of LDS each),
// and the 64-field tile, whose steps are the shortest, keeps eight slices in
// flight.
using Shape256 = GramShape<GRAM_TILE, GRAM_THREADS, 4>;
using Shape128 = GramShape<128, 256, 4>;
using Shape64 = GramShape<64, 256, 8>;
// s_waitcnt immediate for vmcnt <= n and lgkmcnt == 0 (expcnt at max)
constexpr int vmcnt_le(int n) { return (n & 15) | (7 << 4) | ((n >> 4) << 14); }
// Workgroup barrier that leaves this wave's N youngest vector loads in flight
// (the direct loads of later slices), where __syncthreads waits for all.
template <int N>
__device__ __forceinline__ void barrier_keeping() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(vmcnt_le(N));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
constexpr int EPI_PITCH = 36;  // floats per parked accumulator column (32 + 4)
// Physical 16-byte slot of logical chunk `chunk` in LDS row `row` (64 bytes,
// four chunks). XORing the row's bits 2-3 gives any 8 or 16 aligned
// consecutive rows distinct slots modulo 256 bytes (and the same for any 32
// rows modulo 512), so ds_read_b128 of 32 consecutive rows is conflict-free.
// It ignores row bits 4 and up, so rows 16 apart share a key.
__device__ __forceinline__ int swz_key(int row) { return (row >> 2) & 3; }

// Tile id -> (I, J), I <= J < nb, I < nrows (<= nb), in the XCD-aware
// grouped order described above; ntiles = nrows nb - nrows (nrows - 1) / 2.
__device__ __forceinline__ bool decode_tile(int64_t wg, int nb, int nrows, int64_t ntiles,
                                            int& I, int& J) {
  const int64_t per = (ntiles + NUM_XCD - 1) / NUM_XCD;
  const int64_t lin = (wg % NUM_XCD) * per + wg / NUM_XCD;
  if (lin >= ntiles) return false;
  int64_t u = lin;
  for (int I0 = 0; I0 < nrows; I0 += GRAM_GROUP_ROWS) {
    const int gm = nrows - I0 < GRAM_GROUP_ROWS ? nrows - I0 : GRAM_GROUP_ROWS;
    const int64_t cnt = (int64_t)gm * nb - ((int64_t)gm * I0 + (int64_t)gm * (gm - 1) / 2);
    if (u < cnt) {
      const int64_t head = (int64_t)gm * (gm - 1) / 2;
      if (u < head) {
        // head columns J = I0 + m hold m + 1 rows each
        int m = 0;
        while ((int64_t)(m + 1) * (m + 2) / 2 <= u) ++m;
        J = I0 + m;
        I = I0 + (int)(u - (int64_t)m * (m + 1) / 2);
      } else {
        const int64_t v = u - head;
        J = I0 + gm - 1 + (int)(v / gm);
        I = I0 + (int)(v % gm);
      }
      return true;
    }
    u -= cnt;
  }
  return false;
}

// Operand fragments of a slice for one wave: two 16-byte chunks of each of the
// wave's 128 A rows and 64 B rows. Lane half h (lanes 32h .. 32h+31) supplies
// k-group h of every MFMA; A and B use the same assignment, so which elements
// a group holds does not matter. A slice holds
//   BF16x3: 16 (hi, lo) pairs: x0/y0 = hi (chunk 2h), x1/y1 = lo (chunk
//           2h + 1); MFMAs hi.hi', hi.lo', lo.hi'.
//   FP16:   32 values, two k-slices (chunks h and 2 + h), one MFMA each.
//   FP32:   16 values, chunks h and 2 + h, four depth-2 MFMAs each.
template <int PREC, class G>
struct Part {
  using V = typename std::conditional<PREC == TRAKNN_BF16X3, bf16x8,
            typename std::conditional<PREC == TRAKNN_FP16, f16x8, f32x4>::type>::type;
  V x0[G::BM], x1[G::BM], y0[G::BN], y1[G::BN];
};
template <int PREC, class G>
constexpr int part_mfmas() {
  return (PREC == TRAKNN_BF16X3 ? 3 : PREC == TRAKNN_FP16 ? 2 : 8) * G::BM * G::BN;
}

// Lane offsets of the two chunks in the A and B tiles of a slice buffer. The
// wave's rows wm*WT_M + q*32 + r32 (A) and wn*WT_N + q*32 + r32 (B) share the
// swizzle key of r32, so q is an immediate offset of q * 32 rows.
struct PartOffsets {
  int a0, a1, b0, b1;
};
template <int PREC, class G>
__device__ __forceinline__ PartOffsets part_offsets(int wm, int wn, int lane) {
  const int r32 = lane & 31, h = lane >> 5;
  const int key = swz_key(r32);
  const int c0 = PREC == TRAKNN_BF16X3 ? 2 * h : h;
  const int c1 = c0 + (PREC == TRAKNN_BF16X3 ? 1 : 2);
  PartOffsets o;
  o.a0 = (wm * G::WT_M + r32) * RB + ((c0 ^ key) << 4);
  o.a1 = (wm * G::WT_M + r32) * RB + ((c1 ^ key) << 4);
  o.b0 = G::OPER_BYTES + (wn * G::WT_N + r32) * RB + ((c0 ^ key) << 4);
  o.b1 = G::OPER_BYTES + (wn * G::WT_N + r32) * RB + ((c1 ^ key) << 4);
  return o;
}

// MFMA number I of a part. Per accumulator the order of the products is fixed
// (hi.hi', hi.lo', lo.hi' of a slice; slice by slice), whatever else a
// schedule interleaves.
template <int PREC, class G, int I>
__device__ __forceinline__ void mfma_step(const Part<PREC, G>& P, f32x16 (&acc)[G::BM][G::BN]) {
  if constexpr (PREC == TRAKNN_BF16X3) {
    constexpr int bm = I / (3 * G::BN), bn = I / 3 % G::BN, t = I % 3;
    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
        t == 2 ? P.x1[bm] : P.x0[bm], t == 1 ? P.y1[bn] : P.y0[bn], acc[bm][bn], 0, 0, 0);
  } else if constexpr (PREC == TRAKNN_FP16) {
    constexpr int c = I / (G::BM * G::BN), bm = I / G::BN % G::BM, bn = I % G::BN;
    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c ? P.x1[bm] : P.x0[bm],
                                                         c ? P.y1[bn] : P.y0[bn], acc[bm][bn], 0, 0, 0);
  } else {
    constexpr int c = I / (4 * G::BM * G::BN), e = I / (G::BM * G::BN) % 4, bm = I / G::BN % G::BM, bn = I % G::BN;
    acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(
        c ? P.x1[bm][e] : P.x0[bm][e], c ? P.y1[bn][e] : P.y0[bn][e], acc[bm][bn], 0, 0, 0);
  }
}
template <int PREC, class G, int I = 0>
__device__ __forceinline__ void mfma_part(const Part<PREC, G>& P, f32x16 (&acc)[G::BM][G::BN]) {
  if constexpr (I < part_mfmas<PREC, G>()) {
    mfma_step<PREC, G, I>(P, acc);
    mfma_part<PREC, G, I + 1>(P, acc);
  }
}

// Fragment read number R of a part (A chunks of each block, then B chunks).
template <int PREC, class G, int R>
__device__ __forceinline__ void read_step(const char* __restrict__ buf, const PartOffsets& o,
                                          Part<PREC, G>& P) {
  using V = typename Part<PREC, G>::V;
  constexpr bool b = R >= 2 * G::BM;
  constexpr int q = (b ? R - 2 * G::BM : R) / 2;
  const V v = *(const V*)(buf + (b ? (R % 2 ? o.b1 : o.b0) : (R % 2 ? o.a1 : o.a0)) + q * 32 * RB);
  if constexpr (b) {
    if constexpr (R % 2) P.y1[q] = v;
    else P.y0[q] = v;
  } else {
    if constexpr (R % 2) P.x1[q] = v;
    else P.x0[q] = v;
  }
}

template <int PREC, class G, int R = 0>
__device__ __forceinline__ void read_part(const char* __restrict__ buf, const PartOffsets& o,
                                          Part<PREC, G>& P) {
  if constexpr (R < G::PART_READS) {
    read_step<PREC, G, R>(buf, o, P);
    read_part<PREC, G, R + 1>(buf, o, P);
  }
}

// The MFMAs of part P with the reads of part N and PART_LOADS direct loads
// (LOAD) placed between them: two reads after each of the first MFMAs, a load after
// every load_every()-th. All loads at once hold the wave's MFMAs back behind
// the CU's address unit, which takes 64 bytes per clock: spreading them alone
// took the BF16x3 Gram from 14.23 to 13.85 ms (T = 27394, D = 8192).
template <int PREC, class G>
constexpr int load_every() {
  return part_mfmas<PREC, G>() / G::PART_LOADS;
}
template <int PREC, class G, bool LOAD, int I = 0, typename LOADF>
__device__ __forceinline__ void mfma_read_load(const Part<PREC, G>& P, f32x16 (&acc)[G::BM][G::BN],
                                               const char* __restrict__ buf,
                                               const PartOffsets& o, Part<PREC, G>& N, LOADF load) {
  if constexpr (I < part_mfmas<PREC, G>()) {
    mfma_step<PREC, G, I>(P, acc);
    if constexpr (2 * I < G::PART_READS) {
      read_step<PREC, G, 2 * I>(buf, o, N);
      read_step<PREC, G, 2 * I + 1>(buf, o, N);
    }
    constexpr int E = load_every<PREC, G>();
    if constexpr (LOAD && I % E == E - 1 && I / E < G::PART_LOADS) load(I / E);
    __builtin_amdgcn_sched_barrier(0);
    mfma_read_load<PREC, G, LOAD, I + 1>(P, acc, buf, o, N, load);
  }
}

// Fused mode (FUSE 1: the first round's launch, 2: a later round's): the tile's
// trajectory stride is fg.B = 256 - (L - 1) rounded down to a multiple of 4,
// so consecutive tiles overlap by L - 1 fields and hold every term of Eq. 2
// of their trajectory pairs. After the main loop nothing is stored: the
// distances are staged in LDS in four parts -- the rows of the first and
// second half of the tile's trajectory rows, then (transposed) the columns of
// either half of its trajectory columns, each with its L - 1 halo -- and the
// tile consumer (fused_walk.h) of each part offers every pair to its row (row
// parts) or to its column (column parts) and writes their slots. The distances are formed exactly as
// the matrix mode forms them (same operands, same order, the smaller field on
// the A side), so the two modes agree bit for bit wherever the FP64 window
// sums are exact.
constexpr int FPITCH = GRAM_TILE + 1;  // floats per staged row (odd: transposed reads)
constexpr int FUSED_MAX_STAGED = (GRAM_TILE - 16) / 2 + 15;  // rows of a part, L <= 16
constexpr int FUSED_VAL_BYTES = FUSED_MAX_STAGED * FPITCH * 4;
// the staged part, then each wave's first-round scratch
constexpr int FUSED_EST_OFFSET = (FUSED_VAL_BYTES + 15) / 16 * 16;
constexpr int FUSED_EST_BYTES = FUSED_EST_OFFSET + (GRAM_THREADS / 64) * EST_SCRATCH_BYTES;
constexpr int FUSED_LDS = FUSED_EST_BYTES > Shape256::LDS_BYTES ? FUSED_EST_BYTES : Shape256::LDS_BYTES;
static_assert(FUSED_LDS <= 160 * 1024, "a fused part must fit in the LDS of a CU");

template <int PREC, bool BAND, class G = Shape256, int FUSE = 0>
__global__ __launch_bounds__(G::THREADS, G::MIN_WAVES) void gram_kernel(
    const char* __restrict__ xc, int64_t slice_bytes, int nsl,
    const float* __restrict__ ncs, int64_t T, int64_t Tpad, int nb, int64_t ntiles,
    int64_t a_row0, int nbi, int64_t rows_out, int64_t c0, float* __restrict__ S, int64_t ldS,
    float* __restrict__ ST, int64_t ldST, FusedGeom fg, const double* __restrict__ fbound,
    FusedSlots fout) {
  constexpr int TILE = G::TILE, WT_M = G::WT_M, WT_N = G::WT_N, BM = G::BM, BN = G::BN;
  constexpr int WAVES_M = G::WAVES_M, WAVES_N = G::WAVES_N, NWAVES = G::NWAVES;
  __shared__ __attribute__((aligned(16))) char lds[FUSE ? FUSED_LDS : G::LDS_BYTES];
  float* const nrm = (float*)(lds + G::BUFFERS * G::SLICE_BYTES);  // [2][I TILE | J TILE]
  int I, J;
  if constexpr (FUSE != 0) {
    // the round's tiles, each XCD a contiguous run of them (as decode_tile)
    const int64_t per = (ntiles + NUM_XCD - 1) / NUM_XCD;
    const int64_t lin = (int64_t)(blockIdx.x % NUM_XCD) * per + blockIdx.x / NUM_XCD;
    if (lin >= ntiles || !fused_band_tile(lin, fg, I, J)) return;
  } else if constexpr (BAND) {
    // the band's tiles that hold entries above the diagonal: J >= J0 + I,
    // the upper triangle of the columns from J0 on, cut to the band's rows
    const int J0 = (int)(a_row0 / TILE);
    if (!decode_tile(blockIdx.x, nb - J0, nbi, ntiles, I, J)) return;
    J += J0;
  } else {
    if (!decode_tile(blockIdx.x, nb, nb, ntiles, I, J)) return;
  }
  // first fields of the tile's A and B panels
  const int64_t arow = FUSE ? (int64_t)I * fg.B : (BAND ? a_row0 : 0) + (int64_t)I * TILE;
  const int64_t brow = FUSE ? (int64_t)J * fg.B : (int64_t)J * TILE;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int wm = w / WAVES_N, wn = w % WAVES_N;
  const char* Ag = xc + arow * RB;
  const char* Bg = xc + brow * RB;

  // Direct buffer -> LDS loads (buffer_load_dwordx4 ... lds): lane q of a load
  // lands at byte 16*q of the wave's 1 KB destination block (16 rows), so each
  // lane fetches the logical chunk whose swizzled slot is that destination.
  // Each wave moves BLK_PER_WAVE blocks of A and of B per slice and no VGPR
  // stages the data. The operands lie slice by slice (internal.h), so a panel's rows
  // of a slice are one contiguous 16 KB block: a buffer resource per slice and
  // panel, and one lane offset shared by every block.
  constexpr int BLK_PER_WAVE = G::BLK_PER_WAVE, BUFFERS = G::BUFFERS;
  constexpr int RSRC_WORD3 = 0x00020000;  // raw 32-bit buffer, gfx9 family
  const uint32_t voff = (uint32_t)((lane >> 2) * RB + (((lane & 3) ^ swz_key(lane >> 2)) << 4));
  // load v of a slice: block v / 2 of the wave, of A (v even) or B
  auto issue_one = [&](int sl, int v) __attribute__((always_inline)) {
    char* dst = lds + (sl & (BUFFERS - 1)) * G::SLICE_BYTES + (v & 1) * G::OPER_BYTES;
    const int blk = w * BLK_PER_WAVE + v / 2;  // 1 KB block
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((v & 1 ? Bg : Ag) + sl * slice_bytes), 0, G::OPER_BYTES, RSRC_WORD3);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rs, (__attribute__((address_space(3))) void*)(dst + blk * 1024), 16, voff, blk * 1024, 0, 0);
  };
  auto issue = [&](int sl) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 2 * BLK_PER_WAVE; ++v) issue_one(sl, v);
  };

  f32x16 acc[BM][BN];
#pragma unroll
  for (int a = 0; a < BM; ++a)
#pragma unroll
    for (int b = 0; b < BN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  // Chunk norms: each wave fetches 64 of the chunk's TILE N_i^c or TILE N_j^c
  // (a direct load) into the chunk's LDS slot, as far as they go.
  auto issue_norms = [&](int ch) __attribute__((always_inline)) {
    constexpr int PER = TILE / 64;  // waves per operand
    if (NWAVES == 2 * PER || w < 2 * PER) {
      const float* src = ncs + (int64_t)ch * Tpad + (w < PER ? arow : brow) + (w % PER) * 64 + lane;
      __builtin_amdgcn_global_load_lds(src, nrm + (ch & 1) * 2 * TILE + w * 64, 4, 0, 0);
    }
  };
  // acc += -(N_i^c + N_j^c)/2 as a depth-2 FP32 MFMA: lanes 0-31 supply
  // k = 0 (A: N_i^c, B: -1/2), lanes 32-63 k = 1 (A: 1, B: -N_j^c/2); all
  // products are exact.
  const int r32 = lane & 31;
  const bool khi = lane >= 32;
  auto correct = [&](int ch) {
    const float* nA = nrm + (ch & 1) * 2 * TILE;
    const float* nB = nA + TILE;
    float av[BM], bv[BN];
#pragma unroll
    for (int bm = 0; bm < BM; ++bm) {
      const float x = nA[wm * WT_M + bm * 32 + r32];
      av[bm] = khi ? 1.0f : x;
    }
#pragma unroll
    for (int bn = 0; bn < BN; ++bn) {
      const float y = nB[wn * WT_N + bn * 32 + r32];
      bv[bn] = khi ? -0.5f * y : -0.5f;
    }
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
      for (int bn = 0; bn < BN; ++bn)
        acc[bm][bn] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[bm], bv[bn], acc[bm][bn], 0, 0, 0);
  };
  constexpr int SPC = GRAM_CHUNK / (PREC == TRAKNN_FP16 ? 32 : 16);  // slices per chunk (even)

  // Slice sl lives in buffer sl % BUFFERS. Step sl runs the MFMAs of slice sl
  // from registers, reads slice sl + 1's fragments (the barrier before the step
  // made it visible) and issues slice sl + BUFFERS's loads into the buffer that
  // slice sl left in the step before. So a load has BUFFERS - 1 steps to land,
  // LDS read latency hides behind MFMAs, and a wait leaves the loads of the
  // BUFFERS - 2 youngest slices in flight.
  constexpr int KEEP = (BUFFERS - 2) * G::PART_LOADS;
  const PartOffsets o = part_offsets<PREC, G>(wm, wn, lane);
  auto buffer = [&](int sl) __attribute__((always_inline)) {
    return lds + (sl & (BUFFERS - 1)) * G::SLICE_BYTES;
  };
  Part<PREC, G> P0, P1;
  issue_norms(0);
  issue(0);
  issue(1);
  if (nsl >= BUFFERS) {
#pragma unroll
    for (int b = 2; b < BUFFERS; ++b) issue(b);
    barrier_keeping<KEEP>();
  } else {
    for (int b = 2; b < nsl; ++b) issue(b);
    barrier_keeping<0>();
  }
  read_part<PREC, G>(buffer(0), o, P0);
  barrier_keeping<KEEP>();  // slice 0's buffer is read before step 0 refills it
  auto step = [&](int sl, const Part<PREC, G>& P, Part<PREC, G>& N, auto load_c)
                  __attribute__((always_inline)) {
    constexpr bool LOAD = decltype(load_c)::value;  // slice sl + BUFFERS exists
    mfma_read_load<PREC, G, LOAD>(P, acc, buffer(sl + 1), o, N,
                                  [&](int v) __attribute__((always_inline)) { issue_one(sl + BUFFERS, v); });
    barrier_keeping<LOAD ? KEEP : 0>();
  };
  // after the second step of a pair: the chunk's norms once it is done, and
  // the next chunk's on their way (their slot was last read a chunk ago; they
  // land before that chunk ends, which is BUFFERS - 2 steps or the tail's
  // first wait away)
  static_assert(BUFFERS - 2 < SPC, "a chunk's norms land within the chunk");
  auto chunk = [&](int sl) __attribute__((always_inline)) {
    if ((sl + 1) % SPC == 0) {
      correct(sl / SPC);
      issue_norms(sl / SPC + 1);
    }
  };
  int sl = 0;
  for (; sl + 1 + BUFFERS < nsl; sl += 2) {
    step(sl, P0, P1, std::true_type{});
    step(sl + 1, P1, P0, std::true_type{});
    chunk(sl + 1);
  }
#pragma unroll 1
  for (; sl + 2 < nsl; sl += 2) {
    step(sl, P0, P1, std::false_type{});
    step(sl + 1, P1, P0, std::false_type{});
    chunk(sl + 1);
  }
  step(sl, P0, P1, std::false_type{});
  mfma_part<PREC, G>(P1, acc);
  correct(sl / SPC);
  __syncthreads();  // every wave is done with the operand buffers

  if constexpr (FUSE != 0) {
    float* V = (float*)lds;  // [staged][FPITCH]
    const int hs = fg.B / 2;                           // recipients per part
    const int Rs = hs + fg.L - 1;                      // staged rows (columns)
    // the snapshot distances, once: d = -2 acc, clamped
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
      for (int bn = 0; bn < BN; ++bn)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[bm][bn][r] = clamp_distance(-2.f * acc[bm][bn][r]);
    // accumulator r of a 32x32 block holds row 8 (r / 4) + 4 (lane / 32) + r % 4
    // of the block, column lane % 32
    const int lrow = 4 * (lane >> 5), lcol = lane & 31;
#pragma unroll 1
    for (int part = 0; part < 4; ++part) {
      const bool cols = part >= 2;
      const int off = (part & 1) * hs;  // first staged tile row (column)
      if (!cols) {
        // rows off .. off + Rs - 1 of the tile, as staged rows
#pragma unroll
        for (int bm = 0; bm < BM; ++bm) {
          const int rb = wm * WT_M + bm * 32;
          if (rb + 32 <= off || rb >= off + Rs) continue;
          const bool whole = rb >= off && rb + 32 <= off + Rs;  // every row of the block
#pragma unroll
          for (int bn = 0; bn < BN; ++bn) {
            float* base = V + (rb - off + lrow) * FPITCH + wn * WT_N + bn * 32 + lcol;
            if (whole) {
#pragma unroll
              for (int r = 0; r < 16; ++r) base[(8 * (r >> 2) + (r & 3)) * FPITCH] = acc[bm][bn][r];
            } else {
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const int dr = 8 * (r >> 2) + (r & 3);
                const int rel = rb - off + lrow + dr;
                if (rel >= 0 && rel < Rs) base[dr * FPITCH] = acc[bm][bn][r];
              }
            }
          }
        }
      } else {
        // columns off .. off + Rs - 1 of the tile, as staged rows (transposed)
#pragma unroll
        for (int bn = 0; bn < BN; ++bn) {
          const int cb = wn * WT_N + bn * 32;
          if (cb + 32 <= off || cb >= off + Rs) continue;
          const int rel = cb + lcol - off;
          if (rel >= 0 && rel < Rs) {
#pragma unroll
            for (int bm = 0; bm < BM; ++bm) {
              float* base = V + rel * FPITCH + wm * WT_M + bm * 32 + lrow;
#pragma unroll
              for (int r = 0; r < 16; ++r) base[8 * (r >> 2) + (r & 3)] = acc[bm][bn][r];
            }
          }
        }
      }
      __syncthreads();
      // row parts: recipients are the tile's rows (slot J + 1); column parts:
      // its columns (slot I)
      const int p0 = (cols ? J : I) * fg.B + off, q0 = (cols ? I : J) * fg.B;
      char* est = lds + FUSED_EST_OFFSET + w * EST_SCRATCH_BYTES;
      const EstScratch sc{(double*)est, (int*)(est + 64 * sizeof(double))};
      side_topk_len<TILE / 64, FUSE == 1>(fg.L, V, FPITCH, 1, fg.B, hs, p0, q0, cols ? -1 : 1,
                                          cols ? I : J + 1, fg.np, w, GRAM_THREADS / 64, lane,
                                          fbound, fout, sc);
      __syncthreads();
    }
    return;
  }

  // Epilogue through LDS (the operand buffers are free now): d = -2 acc.
  // Accumulator r of
  // lane l in a 32x32 block holds row 8*(r/4) + 4*(l/32) + r%4, column l%32;
  // each 32-row band (bm) of every wave is parked column-major in LDS with
  // compile-time accumulator indices, then all threads write the band's
  // distances coalesced: rows of S for (i, j), and 128-byte runs of S rows for
  // the mirrored (j, i). The whole-matrix mode writes them non-temporally: S is
  // read back only after the Gram, far too large for the caches.
  static_assert(NWAVES * WT_N * EPI_PITCH * 4 <= G::LDS_BYTES, "epilogue staging must fit");
  constexpr int CGROUPS = G::THREADS / TILE;          // threads per tile column
  constexpr int RPT = WAVES_M * 32 / CGROUPS;         // band rows each of them writes
  static_assert(RPT > 0 && 32 % RPT == 0, "a thread's rows lie in one 32-row band");
  float* stg = (float*)lds;  // [NWAVES][WT_N][EPI_PITCH]
  const bool diag = !BAND && I == J;
  const int64_t i_base = (int64_t)I * TILE, j_base = (int64_t)J * TILE;
#pragma unroll
  for (int bm = 0; bm < BM; ++bm) {
    float* mine = stg + w * WT_N * EPI_PITCH;
#pragma unroll
    for (int bn = 0; bn < BN; ++bn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = bn * 32 + (lane & 31);
        const int row = 8 * q + 4 * (lane >> 5);
        *(f32x4*)(mine + col * EPI_PITCH + row) =
            f32x4{acc[bm][bn][4 * q + 0], acc[bm][bn][4 * q + 1],
                  acc[bm][bn][4 * q + 2], acc[bm][bn][4 * q + 3]};
      }
    __syncthreads();
    // (i, j): thread tid owns tile column jl = tid % TILE and RPT rows from
    // r0 of the band of wave row wm_ (rows wm_*WT_M + bm*32 + r)
    {
      const int jl = tid & (TILE - 1);
      const int wm_ = tid / TILE * RPT / 32, r0 = tid / TILE * RPT % 32;
      const int wn_ = jl / WT_N, c = jl % WT_N;
      const int64_t j = j_base + jl;
      if (j < T) {
        const float* src = stg + (wm_ * WAVES_N + wn_) * WT_N * EPI_PITCH + c * EPI_PITCH + r0;
        const int il0 = wm_ * WT_M + bm * 32 + r0;
        const int64_t i0 = i_base + il0;
        // rows written: those below rows_out and, on a diagonal tile, above
        // the diagonal (il < jl); the row pointer steps by ldS
        int64_t nr = rows_out - i0;
        if (diag && jl - il0 < nr) nr = jl - il0;
        const int n = nr < RPT ? (int)nr : RPT;
        float* dst = S + i0 * ldS + (j - c0);
        // band mode: a field's distance to itself is stored as 0, as the
        // mirrored pass stores it in the symmetric mode
        const int64_t dz = BAND ? j - (a_row0 + i0) : -1;
        for (int r = 0; r < n; ++r, dst += ldS) {
          const float v = clamp_distance(-2.f * src[r]);
          if constexpr (BAND)
            *dst = r == dz ? 0.f : v;
          else  // the whole matrix is read back only after the Gram: stream it
            __builtin_nontemporal_store(v, dst);
        }
      }
    }
    // (j, i): 8 threads per (column, row half) write 32 consecutive i, into S
    // itself or, in band mode, into the transposed band
    {
      for (int run = tid >> 3; run < WAVES_M * TILE; run += G::THREADS / 8) {
        const int jl = run / WAVES_M, wm_ = run % WAVES_M;
        const int wn_ = jl / WT_N, c = jl % WT_N;
        const int64_t j = j_base + jl;
        if (j >= T) continue;
        const int q = tid & 7;
        const int il0 = wm_ * WT_M + bm * 32 + 4 * q;
        const int64_t i0 = i_base + il0;
        const f32x4 g = *(const f32x4*)(stg + (wm_ * WAVES_N + wn_) * WT_N * EPI_PITCH +
                                         c * EPI_PITCH + 4 * q);
        float f[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f[e] = clamp_distance(-2.f * g[e]);
        }
        if constexpr (BAND) {
          // i0 is a band row: field a_row0 + i0
          float* dst = ST + (j - c0) * ldST + i0;
          const int64_t dj = j - (a_row0 + i0);  // field j's position in the run, if any
          if (i0 + 3 < rows_out && (dj < 0 || dj > 3)) {
            *(f32x4*)dst = f32x4{f[0], f[1], f[2], f[3]};
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (i0 + e < rows_out) dst[e] = dj == e ? 0.f : f[e];
          }
        } else {
          float* dst = S + j * ldS + i0;
          if (!diag && i0 + 3 < T) {
            __builtin_nontemporal_store(f32x4{f[0], f[1], f[2], f[3]}, (f32x4*)dst);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int il = il0 + e;
              if (i0 + e >= T) continue;
              if (!diag || il < jl) dst[e] = f[e];
              else if (il == jl) dst[e] = 0.f;
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace

// Tiles of one shape over the whole matrix (a_row0 < 0) or a band of it:
// block-rows, block-columns and the tiles (I, J) with an entry above the
// diagonal.
struct TileCount {
  int nb, nbi;
  int64_t ntiles;
};
static TileCount count_tiles(int tile, int64_t T, int64_t a_row0, int64_t rows_out) {
  TileCount c;
  c.nb = (int)((T + tile - 1) / tile);
  c.nbi = a_row0 >= 0 ? (int)((rows_out + tile - 1) / tile) : c.nb;
  const int64_t nbc = c.nb - (a_row0 >= 0 ? a_row0 / tile : 0);
  c.ntiles = c.nbi * nbc - (int64_t)c.nbi * (c.nbi - 1) / 2;
  return c;
}

// Which tile a launch takes. Smaller tiles give a short series more
// workgroups than CUs; larger ones move fewer operand bytes per product. The
// cost of a shape is its tiles per CU, rounded up, times the time a CU takes
// per tile, measured at D = 8192 on full launches, in units of a 16th of a
// 256-field tile of the same precision: the MFMA-bound FP32 loses little to
// smaller tiles, FP16, bound by its operands, the most. Measured at D = 8192,
// 256 / 128 / 64 fields, us: T = 512 387 / 121 / 68 (BF16x3), 1811 / 479 / 142
// (FP32), 152 / 58 / 40 (FP16); T = 2048 387 / 133 / 173, 1812 / 484 / 387,
// 153 / 63 / 89; T = 6000 940 / 742 / 979, 3786 / 2349 / 2246, 375 / 319 / 468;
// T = 16000 4481 / 4893 / 8153, 14653 / 14419 / 16151, 1815 / 2034 / 3581. At
// D = 32 and 1024 the same choices win or are within 3%. Every shape forms each
// distance from the same products in the same order.
static int pick_tile(int precision, int64_t T, int64_t a_row0, int64_t rows_out) {
  constexpr int tiles[3] = {256, 128, 64};
  const double cost[3][3] = {{16.0, 4.2, 1.12}, {16.0, 5.0, 1.9}, {16.0, 5.4, 2.3}};
  static_assert(TRAKNN_FP32 == 0 && TRAKNN_BF16X3 == 1 && TRAKNN_FP16 == 2, "rows of cost");
  int best = 0;
  double least = 0.0;
  for (int i = 0; i < 3; ++i) {
    const int64_t n = count_tiles(tiles[i], T, a_row0, rows_out).ntiles;
    const double c = (double)((n + NUM_CU - 1) / NUM_CU) * cost[precision][i];
    if (i == 0 || c < least) best = i, least = c;
  }
  return tiles[best];
}

// Launch of one shape over the whole matrix (a_row0 < 0) or a band of it.
template <int PREC, class G>
static hipError_t launch_shape(const char* x, const float* ncs, int64_t T, int64_t Tpad, int nsl,
                               int64_t a_row0, int64_t rows_out, int64_t c0, float* S, int64_t ldS,
                               float* ST, int64_t ldST, hipStream_t s) {
  const TileCount t = count_tiles(G::TILE, T, a_row0, rows_out);
  const dim3 grid((unsigned)((t.ntiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD));
  const int64_t slice_bytes = Tpad * GRAM_ROW_BYTES;
  const FusedGeom fg{};
  const FusedSlots fo{};
#define TRAKNN_GRAM_LAUNCH(B)                                                             \
  hipLaunchKernelGGL((gram_kernel<PREC, B, G>), grid, dim3(G::THREADS), 0, s, x, slice_bytes, \
                     nsl, ncs, T, Tpad, t.nb, t.ntiles, a_row0, t.nbi, rows_out, c0, S, ldS, ST, \
                     ldST, fg, nullptr, fo)
  if (a_row0 >= 0) TRAKNN_GRAM_LAUNCH(true);
  else TRAKNN_GRAM_LAUNCH(false);
#undef TRAKNN_GRAM_LAUNCH
  return hipGetLastError();
}

template <int PREC>
static hipError_t launch_prec(const char* x, const float* ncs, int64_t T, int64_t Tpad, int nsl,
                              int64_t a_row0, int64_t rows_out, int64_t c0, float* S, int64_t ldS,
                              float* ST, int64_t ldST, hipStream_t s) {
  switch (pick_tile(PREC, T, a_row0, rows_out)) {
    case 64:
      return launch_shape<PREC, Shape64>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
    case 128:
      return launch_shape<PREC, Shape128>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
    default:
      return launch_shape<PREC, Shape256>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
  }
}

hipError_t launch_gram_band(const void* xc, const float* ncs, int64_t T, int64_t Tpad,
                            int64_t Dpad, int precision, int64_t a_row0, int64_t rows_out,
                            int64_t c0, float* S, int64_t ldS, float* ST, int64_t ldST,
                            hipStream_t s) {
  const int nsl = (int)(Dpad / stage_k(precision)) * 2;
  const char* x = (const char*)xc;
  if (precision == TRAKNN_FP32)
    return launch_prec<TRAKNN_FP32>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
  if (precision == TRAKNN_BF16X3)
    return launch_prec<TRAKNN_BF16X3>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
  return launch_prec<TRAKNN_FP16>(x, ncs, T, Tpad, nsl, a_row0, rows_out, c0, S, ldS, ST, ldST, s);
}

hipError_t launch_gram(const void* xc, const float* ncs, int64_t T, int64_t Tpad,
                       int64_t Dpad, int precision, float* S, int64_t ldS, hipStream_t s) {
  return launch_gram_band(xc, ncs, T, Tpad, Dpad, precision, -1, T, 0, S, ldS, nullptr, 0, s);
}

hipError_t launch_gram_fused(const void* xc, const float* ncs, int64_t T, int64_t Tpad,
                             int64_t Dpad, int precision, const FusedGeom& g, bool establish,
                             const double* bound, const FusedSlots& out, hipStream_t s) {
  const int64_t slice_bytes = Tpad * GRAM_ROW_BYTES;
  const int nsl = (int)(Dpad / stage_k(precision)) * 2;
  const int64_t ntiles = fused_band_tiles(g);
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid((unsigned)((ntiles + NUM_XCD - 1) / NUM_XCD * NUM_XCD));
  const char* x = (const char*)xc;
#define TRAKNN_GRAM_FUSED(P, F)                                                           \
  hipLaunchKernelGGL((gram_kernel<P, false, Shape256, F>), grid, dim3(GRAM_THREADS), 0, s, x, slice_bytes, \
                     nsl, ncs, T, Tpad, 0, ntiles, (int64_t)0, 0, T, (int64_t)0, nullptr, \
                     (int64_t)0, nullptr, (int64_t)0, g, bound, out)
  switch (precision) {
    case TRAKNN_FP32:
      if (establish) TRAKNN_GRAM_FUSED(TRAKNN_FP32, 1);
      else TRAKNN_GRAM_FUSED(TRAKNN_FP32, 2);
      break;
    case TRAKNN_BF16X3:
      if (establish) TRAKNN_GRAM_FUSED(TRAKNN_BF16X3, 1);
      else TRAKNN_GRAM_FUSED(TRAKNN_BF16X3, 2);
      break;
    default:
      if (establish) TRAKNN_GRAM_FUSED(TRAKNN_FP16, 1);
      else TRAKNN_GRAM_FUSED(TRAKNN_FP16, 2);
      break;
  }
#undef TRAKNN_GRAM_FUSED
  return hipGetLastError();
}

}  // namespace traknn
