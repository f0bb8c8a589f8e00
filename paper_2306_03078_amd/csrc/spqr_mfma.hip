// Batches of 4 to 16 vectors on the matrix cores: one kernel for the dense part and the outliers, one that adds the
// partial results; launchers, launch plan and scratch of that path.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <mutex>

#include "../../include/spqr.h"
#include "spqr_batch.h"
#include "spqr_kernels.h"

namespace spqr {

// ---------------------------------------------------------------------------
// P[split][b][rows] = X[b][columns of the split] . W_hat[rows][columns of the split]^T in binary32, outliers included.
//
// Dense part.  A lane owns one whole tile (256 codes in registers, the layout's own unit) and an MFMA's A operand wants
// 16 different rows of the same columns across 16 lanes.  Lanes 16g .. 16g+15 therefore hold the SAME tile column of 16
// consecutive strips: row r of the 16 strips is one A operand of v_mfma_f32_16x16x32_f16 straight from the registers
// the lane dequantised it into (K index = tile column g of 4 and 8 columns inside the tile), and D[r] holds row r of
// the 16 strips for the 16 vectors of the batch.  No weight passes through LDS, the wavefronts of a workgroup meet
// only for the outliers and at the end.  Weights are dequantised as in Sec. 4.2's kernel, s_hat * (q - z_hat) in one
// binary32 FMA, rounded once to binary16; a B operand is 8 consecutive columns of one batch row, 16 bytes from X.
//
// A workgroup of 4 wavefronts owns a group of 16 strips and a range of columns, in units of 16 tile columns (4 per
// wavefront).  Few rows x many columns would leave CUs idle, so gridDim.y splits the columns; every split writes its
// own partial result (see sum_groups_kernel).
//
// Outliers.  The workgroup's piece of the batch passes through LDS transposed, XT[column][16 vectors], at most 1536
// columns (SH::COLS) at a time, so an outlier meets its 16 activations in two 16-byte LDS reads.  (From L2 the same
// 32-byte line costs an L1 look-up per entry, about 10 clocks per entry and CU.)  Where a row's entries begin and end
// inside the columns of the piece is interpolated (lower_columns), 4 lanes take a row's entries in turn, rows of more than
// kLongRow entries in the piece are shared out among the wavefronts, 64 lanes each.  One writer per sum, fixed orders
// everywhere: results are deterministic.  Where the launch leaves CUs over, they are a workgroup's own (APART, plan_batch).
//
// What bounds it (17920 x 6656, 4-bit, Zipf outliers, 16 vectors, weights streamed, 39 us with the sums; 43.5 before the weights
// were rounded in pairs, 41.2 before the first workgroups of the CUs had more units, batch_shares): vector issue for a half of it (5.5 instructions per weight with the outliers) beside the stream of the
// weights (14 us at the rate of a copy); the rest is the start (row bounds, XT) and the memory latency that two workgroups per CU
// leave.  Without outliers 30 us.  Before (weights transposed through LDS quarter tile by quarter tile, outliers in a
// kernel of their own that gathered from L2): 55 us; 8192 x 22016, 3-bit, 75 -> 63 us; 22016 x 8192 77 -> 66 us; three of
// 6656^2 at 4 vectors 57 -> 49 us.
// ---------------------------------------------------------------------------
constexpr int kLongRow = 64;                 // entries of a row inside a piece beyond which a whole wavefront takes it

template <int TR, int TC> struct BatchShape {
  static constexpr int ROWS = 16 * lane_rows(TR);                    // rows of a group of 16 strips
  static constexpr int CHUNK = 1536 / (kUnitTiles * TC);             // units per piece of XT
  static constexpr int COLS = CHUNK * kUnitTiles * TC;
  static constexpr int SUM = ROWS + 4;                               // floats per vector of a buffer of sums (the 4: banks)
  static constexpr int XT = (COLS + COLS / 8) * 32;                  // a column's line of 32 bytes, one line free in nine (banks)
  static constexpr int SLICE = 16 * 20;                              // floats of one row of 16 strips, 16 vectors (20: banks)
  static constexpr int SUMS = 3 * lane_rows(TR) * SLICE * 4;         // each wavefront sums a quarter of the rows, from three others
  static constexpr int SHARED = XT > SUMS ? XT : SUMS;               // XT, then the wavefronts' sums
  static constexpr int LDS = SHARED + SUM * 64 + ROWS * 8;           // + sums of the outliers + row bounds
  static_assert(2 * LDS <= 160 * 1024, "two workgroups share a CU");
};

// Reduces 16 values per lane over the aligned group of 4 lanes: lane l of the group ends with values 4l .. 4l+3 in v[0..3].
__device__ __forceinline__ void quad_scatter(float (&v)[16], int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float send = lane & 2 ? v[i] : v[i + 8], keep = lane & 2 ? v[i + 8] : v[i];
    v[i] = keep + stage_partner<4>(send, lane);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float send = lane & 1 ? v[i] : v[i + 4], keep = lane & 1 ? v[i + 4] : v[i];
    v[i] = keep + stage_partner<5>(send, lane);
  }
}

// p[s]: the first index in [a, z) whose column is >= c[s], or z (columns increase; on a broken row some index in
// [a, z]); a < z.  Both at once.  A look-up is a lane's own cache line and a round a trip to memory (a microsecond while
// the weights stream), so both are kept few: the columns of a row are spread over [0, n) as a rule, so a granule of 8
// entries is read where the column is expected, and again as far off as its columns say; from the fourth round on the
// bracket is halved.  (Binary search: 14 look-ups in 7 rounds for a row of 67; seven probes a round: 42 in 3, and
// slower than that.)
__device__ __forceinline__ void lower_columns(const uint16_t* __restrict__ col, int n, int a, int z, const int (&c)[2],
                                              int (&p)[2]) {
  const u32x4* col8 = reinterpret_cast<const u32x4*>(col);
  const float density = (float)(z - a) / (float)n;
  int hi[2], at[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) { p[s] = a; hi[s] = z; at[s] = a + (int)((float)c[s] * density); }
  for (int round = 0; p[0] < hi[0] || p[1] < hi[1]; ++round) {
    int q[2];
    u32x4 g[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (round >= 3) at[s] = p[s] + ((hi[s] - p[s]) >> 1);
      q[s] = max(min(at[s], hi[s] - 1), min(p[s], z - 1)) >> 3;   // (a bracket that is closed: some granule of the row)
      g[s] = col8[(uint32_t)q[s]];
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int first = max(p[s], 8 * q[s]), last = min(hi[s], 8 * q[s] + 8);
      if (first >= last) continue;             // closed
      const uint32_t w[4] = {g[s].x, g[s].y, g[s].z, g[s].w};
      int below = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int v = (int)(k & 1 ? w[k / 2] >> 16 : w[k / 2] & 0xFFFFu), e = 8 * q[s] + k;
        below += e >= first && e < last && v < c[s];
      }
      if (below == last - first) {             // all left of c: on to the right
        p[s] = last;
        at[s] = last + (int)((float)max(c[s] - (int)(w[3] >> 16), 0) * density);
      } else if (below == 0) {                 // none: to the left
        hi[s] = first;
        at[s] = first - 1 - (int)((float)max((int)(w[0] & 0xFFFFu) - c[s], 0) * density);
      } else {
        p[s] = hi[s] = first + below;
      }
    }
  }
}

// The sums of one workgroup: group `group` of matrix A, units [u_lo, u_hi) of its columns.  X: the batch in the
// matrix's column order.  P: this split's partial results of the matrix (b * m floats).  APART: the workgroup takes only
// the dense part or only the outliers of the sets [set_lo, set_hi) of 64 rows (and writes those rows), else both.
template <int W, int TR, int TC, int AXIS, bool APART>
__device__ __forceinline__ void batch_group_body(const DevMatrix& A, const uint16_t* __restrict__ X, int batch,
                                                 float* __restrict__ P, int group, int u_lo, int u_hi, int set_lo, int set_hi,
                                                 uint8_t* smem) {
  using SH = BatchShape<TR, TC>;
  using DQ = Dequant<W, TR, TC, AXIS>;
  using B = BatchTile<W, TR, TC, AXIS>;
  using T = typename B::T;
  constexpr int TILE_BYTES = 16 * T::KW + 4 * T::SD, ROWS = SH::ROWS, LR = DQ::LR, NSUB = DQ::NSUB, KG = DQ::KG, SUM = SH::SUM;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int n = A.g.n, ntc = A.g.ntc, ntr = A.g.ntr * NSUB, m = A.g.m;
  const bool dense = !APART || set_lo >= set_hi, sparse = A.nnz > 0 && (!APART || !dense);
  const int outliers_first = sparse ? (int)((blockIdx.x + gridDim.x * blockIdx.y) / kCUs) & 1 : 0;
  uint16_t* xt = reinterpret_cast<uint16_t*>(smem);                       // XT[COLS][16]
  float* red = reinterpret_cast<float*>(smem);                            // afterwards: slices of [16][20]
  float* osum = reinterpret_cast<float*>(smem + SH::SHARED);              // [16][SUM]: outlier sums
  int* row_lo = reinterpret_cast<int*>(smem + SH::SHARED + SUM * 64);     // [ROWS] entries of the piece, by row
  int* row_hi = row_lo + ROWS;

  constexpr int STRIPS = 16 / NSUB;          // strips of tiles of a group
  const uint8_t* base = A.packed + (int64_t)group * STRIPS * ntc * TILE_BYTES;
  const int my_strip = min(group * 16 + i16, ntr - 1) - group * 16, half = NSUB == 2 ? my_strip & 1 : 0;
  const uint32_t strip_off = (uint32_t)(my_strip / NSUB) * (uint32_t)ntc * TILE_BYTES;
  const uint32_t xrow = (uint32_t)min(i16, batch - 1) * (uint32_t)n * 2u;
  DQ dq(half);

  float4_t D[LR];
#pragma unroll
  for (int r = 0; r < LR; ++r) D[r] = float4_t{0.f, 0.f, 0.f, 0.f};
  // the first free line of XT stays zero: it is what an entry of another row meets (its own column may hold an infinity)
  if (sparse && tid < 8) reinterpret_cast<uint32_t*>(xt + 8 * 16)[tid] = 0;

  const int nst = (ntc + 3) >> 2;              // steps of 4 tile columns
  // the wavefront's step of unit u (a step behind the last one loads the last one and counts nothing)
  auto issue = [&](B& t, u32x4 (&x)[KG], int u) {
    const int st = min(4 * u + wave, nst - 1);
    const int blk = st >> 4, L = min(64, ntc - 64 * blk), tl = min(4 * st + g4, ntc - 1);
    const bool real = u < u_hi;                // uniform; behind the range every lane reads the group's first tile
    const uint32_t l = real ? (uint32_t)(tl - 64 * blk) : 0u;
    load_batch_tile(t, base + (real ? (int64_t)64 * blk * TILE_BYTES : 0), real ? L : 1, real ? strip_off : 0u, l, half);
    const uint8_t* xs = reinterpret_cast<const uint8_t*>(X);
#pragma unroll
    for (int j = 0; j < KG; ++j) x[j] = *reinterpret_cast<const u32x4*>(xs + (real ? xrow + (uint32_t)tl * (TC * 2) + 16 * j : 0u));
    __builtin_amdgcn_sched_barrier(0);         // the requests go out here, not between the multiplies of the tile before
  };
  auto multiply = [&](const B& t, const u32x4 (&x)[KG], int u) {
    const bool live = 16 * u + 4 * wave + g4 < ntc;
    dq.begin(t, live);
    // 8 columns at a time, so that few groups' constants are alive (the two tiles and the sums leave room for no more)
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      dq.columns(t, j);
      const uint32_t xv[4] = {live ? x[j].x : 0u, live ? x[j].y : 0u, live ? x[j].z : 0u, live ? x[j].w : 0u};
#pragma unroll
      for (int r = 0; r < LR; ++r) {
        D[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dq.operand(t, r, j), __builtin_bit_cast(half8_t, xv), D[r], 0, 0, 0);
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  for (int c_lo = u_lo; c_lo < u_hi; c_lo += SH::CHUNK) {   // pieces of the column range, workgroup-uniform
    const int c_hi = min(u_hi, c_lo + SH::CHUNK);
    const int k0 = c_lo * kUnitTiles * TC, k1 = min(n, c_hi * kUnitTiles * TC);
    B t0, t1;
    u32x4 x0[KG], x1[KG];
    if (dense) issue(t0, x0, c_lo);
    if (sparse) {
      if (c_lo > u_lo) __syncthreads();        // everyone is done with the previous piece
      int bounds[2] = {0, 0};                  // of the row's entries, then of those in the piece; requested ahead of X
      const int row = group * ROWS + tid;
      if ((APART ? tid >= 64 * set_lo && tid < 64 * set_hi : tid < ROWS) && row < m) {
        bounds[0] = A.row_ptr[row];
        bounds[1] = A.row_ptr[row + 1];
      }
      // the piece of X, transposed: thread = 8 columns of 2 vectors; the 8 pairs of vectors of 8 neighbouring blocks of
      // columns are a wavefront's, which write all 64 banks (the free line after every 8)
      const int units8 = (k1 - k0) >> 3;       // n and the units are multiples of 8
      for (int q = tid; q < 8 * units8; q += 256) {
        const int c8 = q >> 3, v = 2 * (q & 7);
        const u32x4 z = {0u, 0u, 0u, 0u};
        const u32x4 lo = v < batch ? *reinterpret_cast<const u32x4*>(X + (int64_t)v * n + k0 + 8 * c8) : z;
        const u32x4 hi = v + 1 < batch ? *reinterpret_cast<const u32x4*>(X + (int64_t)(v + 1) * n + k0 + 8 * c8) : z;
        uint32_t* d = reinterpret_cast<uint32_t*>(xt + (9 * c8) * 16 + v);
        const uint32_t a4[4] = {lo.x, lo.y, lo.z, lo.w}, b4[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          d[(2 * k) * 8] = (a4[k] & 0xFFFFu) | (b4[k] << 16);
          d[(2 * k + 1) * 8] = (a4[k] >> 16) | (b4[k] & 0xFFFF0000u);
        }
      }
      if (tid < ROWS) {
        const int a = bounds[0], z = bounds[1], c[2] = {k0, k1};
        if (a < z && (k0 > 0 || k1 < n)) lower_columns(A.col, n, a, z, c, bounds);
        row_lo[tid] = bounds[0];
        row_hi[tid] = max(bounds[0], bounds[1]);
      }
    }
    // the dense part of the piece: two units per trip, the next one's loads ahead of the arithmetic
    auto dense_part = [&]() {
      int u = c_lo;
      while (u + 1 < c_hi) {
        issue(t1, x1, u + 1);
        multiply(t0, x0, u);
        issue(t0, x0, u + 2);                  // behind the last unit: a dummy
        multiply(t1, x1, u + 1);
        u += 2;
      }
      if (u < c_hi) multiply(t0, x0, u);
    };
    auto outlier_part = [&]() {
      __syncthreads();                           // XT and the row bounds are complete
      const bool first = c_lo == u_lo;
      const int width = k1 - k0;
      // acc += two entries' values (binary16 pair) times their 16 activations, x the index of the first, those of them that
      // lie in [lo, lo + len): one v_perm pairs the two activations of a vector, one v_dot2 takes them (products exact,
      // binary32 sums, the same bits as two v_fma_mix; half the issue)
      auto add_pair = [&](uint32_t cols, uint32_t vals, int x, int lo, uint32_t len, float (&acc)[16]) {
        const bool in0 = (uint32_t)(x - lo) < len, in1 = (uint32_t)(x + 1 - lo) < len;
        // a column outside the piece (a broken row) stays inside XT
        const int c0 = min(max((int)(cols & 0xFFFFu) - k0, 0), width - 1), c1 = min(max((int)(cols >> 16) - k0, 0), width - 1);
        const u32x4* l0 = reinterpret_cast<const u32x4*>(xt + (in0 ? c0 + (c0 >> 3) : 8) * 16);
        const u32x4* l1 = reinterpret_cast<const u32x4*>(xt + (in1 ? c1 + (c1 >> 3) : 8) * 16);
        const u32x4 a0 = l0[0], a1 = l0[1], b0 = l1[0], b1 = l1[1];
        const uint32_t a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w}, b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
        const half2_t w = as_half2((in0 ? vals & 0xFFFFu : 0u) | (in1 ? vals & 0xFFFF0000u : 0u));
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const half2_t lo16 = as_half2(__builtin_amdgcn_perm(b[q], a[q], 0x05040100u));   // a.lo, b.lo
          const half2_t hi16 = as_half2(__builtin_amdgcn_perm(b[q], a[q], 0x07060302u));   // a.hi, b.hi
          acc[2 * q] = __builtin_amdgcn_fdot2(w, lo16, acc[2 * q], false);
          acc[2 * q + 1] = __builtin_amdgcn_fdot2(w, hi16, acc[2 * q + 1], false);
        }
      };
      auto put = [&](int lr, int v, float s) {   // row lr = LR * strip + r lives at r * 16 + strip
        float* d = osum + v * SUM + (lr % LR) * 16 + lr / LR;
        *d = first ? s : *d + s;
      };
      const uint32_t* col2 = reinterpret_cast<const uint32_t*>(A.col);    // aligned pairs of entries; the last entry's
      const uint32_t* val2 = reinterpret_cast<const uint32_t*>(A.val);    // pair is inside its granule of 16 bytes
      const int last2 = (int)((A.nnz - 1) >> 1);
      // Rows of up to kLongRow entries: 4 lanes each, 16 rows per wavefront at a time, a lane takes every 4th pair.  The
      // first pairs of all of the wavefront's rows are requested together.
      constexpr int SETS = ROWS / 64, PRE = 8 / SETS;
      uint32_t cw[SETS][PRE], vw[SETS][PRE];
      int lo[SETS], hi[SETS];
      bool mine[SETS];                           // not a long row: its sums are written below
#pragma unroll
      for (int k = 0; k < SETS; ++k) {
        if (APART && (k < set_lo || k >= set_hi)) continue;   // workgroup-uniform
        const int lr = 16 * (wave + 4 * k) + (lane >> 2);
        lo[k] = row_lo[lr];
        hi[k] = row_hi[lr];
        mine[k] = hi[k] - lo[k] <= kLongRow;
        hi[k] = mine[k] ? hi[k] : lo[k];
#pragma unroll
        for (int h = 0; h < PRE; ++h) {
          const uint32_t at = (uint32_t)min((lo[k] >> 1) + (lane & 3) + 4 * h, last2);
          cw[k][h] = col2[at];
          vw[k][h] = val2[at];
        }
      }
#pragma unroll
      for (int k = 0; k < SETS; ++k) {
        if (APART && (k < set_lo || k >= set_hi)) continue;
        float acc[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const int x0 = (lo[k] & ~1) + 2 * (lane & 3);
#pragma unroll
        for (int h = 0; h < PRE; ++h)
          if (__builtin_amdgcn_ballot_w64(x0 + 8 * h < hi[k]) != 0)
            add_pair(cw[k][h], vw[k][h], x0 + 8 * h, lo[k], (uint32_t)(hi[k] - lo[k]), acc);
        for (int x = x0 + 8 * PRE; __builtin_amdgcn_ballot_w64(x < hi[k]) != 0; x += 32) {   // 32 more entries at a time
          uint32_t cm[4], vm[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const uint32_t at = (uint32_t)min((x >> 1) + 4 * h, last2);
            cm[h] = col2[at];
            vm[h] = val2[at];
          }
#pragma unroll
          for (int h = 0; h < 4; ++h)
            if (__builtin_amdgcn_ballot_w64(x + 8 * h < hi[k]) != 0)
              add_pair(cm[h], vm[h], x + 8 * h, lo[k], (uint32_t)(hi[k] - lo[k]), acc);
        }
        quad_scatter(acc, lane);
        if (mine[k]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) put(16 * (wave + 4 * k) + (lane >> 2), 4 * (lane & 3) + i, acc[i]);
        }
      }
      // Long rows, dealt to the wavefronts in turn: aligned granules of 8 entries (16 bytes of columns, 16 of values), two
      // per lane at a time; a row's first ones are requested while the row before is added up.
      const u32x4* col8 = reinterpret_cast<const u32x4*>(A.col);
      const u32x4* val8 = reinterpret_cast<const u32x4*>(A.val);
      int taken = 0, r0 = -64;
      uint64_t mask = 0;
      auto next_long = [&]() {                   // this wavefront's next long row, -1 behind the last (wave-uniform)
        for (;;) {
          while (mask == 0) {
            r0 += 64;
            if (r0 >= ROWS) return -1;
            mask = __builtin_amdgcn_ballot_w64(row_hi[r0 + lane] - row_lo[r0 + lane] > kLongRow);
          }
          const int lr = r0 + __builtin_ctzll(mask);
          mask &= mask - 1;
          if ((taken++ & 3) == wave) return lr;
        }
      };
      auto fetch = [&](int g0, int g_hi, u32x4 (&c8)[2], u32x4 (&v8)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t at = (uint32_t)min(g0 + lane + 64 * h, g_hi);
          c8[h] = col8[at];
          v8[h] = val8[at];
        }
      };
      u32x4 c8[2], v8[2], nc8[2], nv8[2];
      int lr = next_long();
      if (lr >= 0) fetch(row_lo[lr] >> 3, (row_hi[lr] - 1) >> 3, c8, v8);
      while (lr >= 0) {                          // wave-uniform
        const int next = next_long();
        if (next >= 0) fetch(row_lo[next] >> 3, (row_hi[next] - 1) >> 3, nc8, nv8);
        const int rlo = row_lo[lr], rhi = row_hi[lr], g_hi = (rhi - 1) >> 3;
        float acc[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        for (int g0 = rlo >> 3;;) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int e = 8 * (g0 + lane + 64 * h);
            if (h > 0 && __builtin_amdgcn_ballot_w64(e < rhi) == 0) break;
            const uint32_t c4[4] = {c8[h].x, c8[h].y, c8[h].z, c8[h].w}, v4[4] = {v8[h].x, v8[h].y, v8[h].z, v8[h].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) add_pair(c4[k], v4[k], e + 2 * k, rlo, (uint32_t)(rhi - rlo), acc);
          }
          if ((g0 += 128) > g_hi) break;
          fetch(g0, g_hi, c8, v8);
        }
        int v;
        const float s = wave_reduce_rows<16>(acc, lane, &v);
        if ((lane & 3) == 0) put(lr, v, s);      // 4 lanes hold each sum
        lr = next;
#pragma unroll
        for (int h = 0; h < 2; ++h) { c8[h] = nc8[h]; v8[h] = nv8[h]; }
      }
    };
    // Every second workgroup of a CU takes the outliers first: one of a pair is at its look-ups while the other's
    // weights stream.
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {
      if (part == outliers_first) {
        if (dense) dense_part();
      } else if (sparse) {
        outlier_part();
      }
    }
  }

  // The wavefronts' sums meet in LDS (over XT): every wavefront adds up a quarter of the rows, in the order of the
  // wavefronts, and writes them.  Slice (3 q + k) holds row q of the wavefront that is number k of the other three.
  __syncthreads();
  constexpr int QR = LR / 4;
  const int at = i16 * 20 + 4 * g4;
  if (dense) {                                 // workgroup-uniform
#pragma unroll
    for (int r = 0; r < LR; ++r) {
      const int q = r / QR;                    // the wavefront that adds up row r
      if (q != wave) *reinterpret_cast<float4_t*>(red + (3 * r + (wave < q ? wave : wave - 1)) * SH::SLICE + at) = D[r];
    }
    __syncthreads();
  } else if (4 * g4 * LR < 64 * set_lo || 4 * g4 * LR >= 64 * set_hi) {
    return;                                    // another workgroup's rows
  }
  if (i16 >= batch) return;
  // partial results of a group: [vector][row of the strip][strip], `strips` of them (16, fewer in the last group)
  const int strips = min(16, ntr - group * 16);
  float* out = P + (int64_t)batch * group * ROWS + i16 * (strips * LR);
#pragma unroll
  for (int r = 0; r < LR; ++r) {
    if (r / QR != wave) continue;              // wave-uniform
    float4_t sum = float4_t{0.f, 0.f, 0.f, 0.f};
    if (dense) {
#pragma unroll
      for (int w = 0; w < 4; ++w)
        sum += w == r / QR ? D[r] : *reinterpret_cast<const float4_t*>(red + (3 * r + (w < r / QR ? w : w - 1)) * SH::SLICE + at);
    }
    if (sparse) sum += *reinterpret_cast<const float4_t*>(osum + i16 * SUM + 16 * r + 4 * g4);
    if (strips == 16) {
      *reinterpret_cast<float4_t*>(out + 16 * r + 4 * g4) = sum;       // 16-byte stores: m is a multiple of 8
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (4 * g4 + k < strips) out[strips * r + 4 * g4 + k] = sum[k];
    }
  }
}

// The units of a split: `per`, `more` more for the first `lead` of them.
struct Shares {
  int per, lead, more;
  __host__ __device__ int first(int y) const { return y * per + (y < lead ? y : lead) * more; }
};

// APART: z == 0 is the dense part, the other z share the sets of 64 rows of the outliers, whose sums are partial results of
// their own (gridDim.y of them, behind the dense ones).
template <int W, int TR, int TC, int AXIS, bool APART>
__device__ __forceinline__ void batch_group_share(const DevMatrix& A, const uint16_t* __restrict__ X, int batch,
                                                  float* __restrict__ P, int group, Shares shares, uint8_t* smem) {
  const int units = (A.g.ntc + kUnitTiles - 1) / kUnitTiles, y = blockIdx.y, u_lo = shares.first(y);   // never empty (host)
  const int z = APART ? blockIdx.z : 0, sets = APART ? BatchShape<TR, TC>::ROWS / 64 / (gridDim.z - 1) : 0;
  const int split = y + (z > 0 ? gridDim.y : 0);
  batch_group_body<W, TR, TC, AXIS, APART>(A, X, batch, P + (int64_t)split * batch * A.g.m, group, u_lo,
                                           min(units, shares.first(y + 1)), z > 0 ? (z - 1) * sets : 0, z * sets, smem);
}

template <int W, int TR, int TC, int AXIS, bool APART>
__global__ void __launch_bounds__(256, 2)
batch_group_kernel(DevMatrix A, const uint16_t* __restrict__ X, int batch, float* __restrict__ P, Shares shares) {
  extern __shared__ __align__(16) uint8_t smem[];
  batch_group_share<W, TR, TC, AXIS, APART>(A, X, batch, P, blockIdx.x, shares, smem);
}

// Several matrices that share the batch X and the format (q/k/v, gate/up of a decoder block) in one grid: blockIdx.x
// counts the groups of all matrices.  Every workgroup does exactly what it would do in a launch of its own matrix.
struct BatchFusedItem {
  DevMatrix A;
  float* P;                                  // partial results
  void* Y;
  int groups;
};
struct BatchFused {
  int count;
  BatchFusedItem it[SPQR_MAX_FUSED];
};

template <int W, int TR, int TC, int AXIS, bool APART>
__global__ void __launch_bounds__(256, 2)
batch_group_fused_kernel(BatchFused F, const uint16_t* __restrict__ X, int batch, Shares shares) {
  extern __shared__ __align__(16) uint8_t smem[];
  int bx = blockIdx.x, i = 0;
  for (; i < F.count - 1; ++i) {             // workgroup-uniform
    if (bx < F.it[i].groups) break;
    bx -= F.it[i].groups;
  }
  batch_group_share<W, TR, TC, AXIS, APART>(F.it[i].A, X, batch, F.it[i].P, bx, shares, smem);
}

// Y[v][row] = sum over the splits of P, in their order, rounded once to the output type.  One workgroup per group of
// 16 strips and vector, a thread per row of the group: the splits are read in the order they were
// written, the rows leave in their own.
__device__ __forceinline__ void sum_groups_body(const Geometry& g, const float* __restrict__ P, int splits, int batch,
                                                void* __restrict__ Y, int y_dtype, int group) {
  __shared__ float rows[256];
  const int TR = lane_rows(g.tile_rows), strips = min(16, g.m / TR - group * 16), live = strips * TR;
  const int t = threadIdx.x, v = blockIdx.y;
  if (t < live) {
    const float* p = P + (int64_t)batch * group * 16 * TR + v * live + t;
    const int64_t stride = (int64_t)batch * g.m;
    float s = p[0];
#pragma unroll 4
    for (int k = 1; k < splits; ++k) s += p[k * stride];
    rows[(t % strips) * TR + t / strips] = s;
  }
  __syncthreads();
  if (t < live) {
    const int64_t at = (int64_t)v * g.m + group * 16 * TR + t;
    if (y_dtype == SPQR_F32) static_cast<float*>(Y)[at] = rows[t];
    else static_cast<uint16_t*>(Y)[at] = f2h_rne(rows[t]);
  }
}
__global__ void __launch_bounds__(256)
sum_groups_kernel(Geometry g, const float* __restrict__ P, int splits, int batch, void* __restrict__ Y, int y_dtype) {
  sum_groups_body(g, P, splits, batch, Y, y_dtype, blockIdx.x);
}
__global__ void __launch_bounds__(256) sum_groups_fused_kernel(BatchFused F, int splits, int batch, int y_dtype) {
  int bx = blockIdx.x, i = 0;
  for (; i < F.count - 1; ++i) {             // workgroup-uniform
    if (bx < F.it[i].groups) break;
    bx -= F.it[i].groups;
  }
  sum_groups_body(F.it[i].A.g, F.it[i].P, splits, batch, F.it[i].Y, y_dtype, bx);
}

static hipError_t launch_sum_groups(const Geometry& g, const float* P, int splits, int b, void* Y, int y_dtype, hipStream_t stream) {
  const int rows = 16 * lane_rows(g.tile_rows);
  hipLaunchKernelGGL(sum_groups_kernel, dim3((g.m + rows - 1) / rows, b), dim3(rows), 0, stream, g, P, splits, b, Y, y_dtype);
  return hipGetLastError();
}

// Scratch of the batch path.  A call on a stream that is not being captured takes the buffer the library keeps for
// that stream: work on one stream runs in order, so its calls can share one buffer, and nothing is allocated or
// freed per call (on this runtime a stream-ordered allocation waits on the host until the stream's earlier work is
// done, which keeps the next call's launches from being queued behind the running one: about 5 us per call).  The
// buffer grows when a call needs more (the stream is synchronised first) and is kept until the process ends; up to
// kScratchStreams streams per device have one; further streams allocate stream-ordered from a memory pool of the
// library's own (one per device, unlimited release threshold), captured calls from the device's default pool, which
// the capture turns into allocation nodes of the graph (graphs of many such calls replay correctly with it; with the
// library's own pool the allocations of all but the first call of a capture failed).  A buffer's lock is held while its call is enqueued: calls from several host
// threads on one stream do not interleave their kernels.
constexpr int kScratchStreams = 8;
struct ScratchSlot {
  std::mutex lock;                           // held while a call that uses the buffer is enqueued
  hipStream_t stream = nullptr;
  uint8_t* buf = nullptr;
  size_t size = 0;
  bool taken = false;
};
struct Scratch {
  uint8_t* p = nullptr;
  bool pooled = false;                       // stream-ordered allocation, to be freed on the stream
  std::unique_lock<std::mutex> hold;
};

static hipMemPool_t scratch_pool(int dev) {
  static std::mutex lock;
  static hipMemPool_t pools[kMaxDevices];
  static bool tried[kMaxDevices];
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> hold(lock);
  if (!tried[dev]) {
    tried[dev] = true;
    hipMemPoolProps props = {};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool = nullptr;
    if (hipMemPoolCreate(&pool, &props) == hipSuccess) {
      uint64_t keep = UINT64_MAX;
      if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess) pools[dev] = pool;
      else (void)hipMemPoolDestroy(pool);
    }
    if (pools[dev] == nullptr) (void)hipGetLastError();
  }
  return pools[dev];
}

// hipErrorNotSupported: no scratch to be had (the caller takes the vector path).
static hipError_t scratch_get(Scratch* sc, size_t bytes, int dev, hipStream_t stream, bool allow_stream_ordered = true) {
  static std::mutex table_lock;
  static ScratchSlot slots[kMaxDevices][kScratchStreams];
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(stream, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone;
  ScratchSlot* slot = nullptr;
  if (!capturing && dev >= 0 && dev < kMaxDevices) {
    std::lock_guard<std::mutex> hold(table_lock);
    for (int i = 0; i < kScratchStreams && slot == nullptr; ++i)
      if (slots[dev][i].taken && slots[dev][i].stream == stream) slot = &slots[dev][i];
    for (int i = 0; i < kScratchStreams && slot == nullptr; ++i)
      if (!slots[dev][i].taken) {
        slot = &slots[dev][i];
        slot->taken = true;
        slot->stream = stream;
      }
  }
  if (slot != nullptr) {
    sc->hold = std::unique_lock<std::mutex>(slot->lock);
    if (slot->size < bytes) {
      // the stream's earlier calls may still read the old buffer
      if (slot->buf != nullptr && (hipStreamSynchronize(stream) != hipSuccess || hipFree(slot->buf) != hipSuccess)) {
        (void)hipGetLastError();
        sc->hold.unlock();
        return hipErrorNotSupported;
      }
      slot->buf = nullptr;
      slot->size = 0;
      const size_t want = (bytes + bytes / 4 + 0xFFFFF) & ~(size_t)0xFFFFF;   // some room, whole megabytes
      if (hipMalloc(reinterpret_cast<void**>(&slot->buf), want) != hipSuccess) {
        (void)hipGetLastError();
        slot->buf = nullptr;
        sc->hold.unlock();
        return hipErrorNotSupported;
      }
      slot->size = want;
    }
    sc->p = slot->buf;
    sc->pooled = false;
    return hipSuccess;
  }
  // The fused launch set never runs on a stream-ordered allocation: that is the kind of scratch the one memory
  // fault seen on this path had (a captured graph of fused calls, cause unknown); its caller falls back to one
  // call per matrix.
  if (!allow_stream_ordered) return hipErrorNotSupported;
  // captured: the device's default pool (allocation nodes of the graph); else the library's own pool
  hipMemPool_t pool = capturing ? nullptr : scratch_pool(dev);
  const hipError_t e = pool != nullptr ? hipMallocFromPoolAsync(reinterpret_cast<void**>(&sc->p), bytes, pool, stream)
                                       : hipMallocAsync(reinterpret_cast<void**>(&sc->p), bytes, stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    sc->p = nullptr;
    return hipErrorNotSupported;
  }
  sc->pooled = true;
  return hipSuccess;
}
// after the call's last kernel is enqueued
static hipError_t scratch_put(Scratch* sc, hipStream_t stream) {
  hipError_t e = hipSuccess;
  if (sc->pooled && sc->p != nullptr) e = hipFreeAsync(sc->p, stream);
  if (sc->hold.owns_lock()) sc->hold.unlock();
  sc->p = nullptr;
  return e;
}

// Groups of 16 strips of a matrix, and the units of its columns the splits are made of.
static int batch_groups(const Geometry& g) { return (g.m / lane_rows(g.tile_rows) + 15) / 16; }
static int batch_sets(const Geometry& g) { return lane_rows(g.tile_rows) / 4; }      // of 64 rows
static int batch_units(const Geometry& g) { return (g.ntc + kUnitTiles - 1) / kUnitTiles; }

// Plan of a launch for the groups of one matrix or of several: units per split and how many workgroups share the outliers
// of a split of a group beside its dense one (0: the dense workgroup takes them too), by a model of the launch in
// microseconds.  The chip's 256 CUs take the workgroups in grid order, each the CU with the least work; the launch lasts
// `start` and the longest CU.  A workgroup that does both costs both + both_unit per unit of 16 tile columns, for every further
// piece of XT (with outliers) `piece`, and for its outliers (thousands of entries, rows far longer than the mean); a
// dense one and one of outliers less each, but all of them together more.  So outliers go apart where the chip has CUs left
// over (small layers: the outliers' trips to memory run beside the weights' instead of behind them, and heavy rows are
// shared out further), and wide pieces of XT pay on large ones.
// Fitted to every split and share of 173 layers and sets of layers (1024^2 to two of 22016 x 8192, 16 vectors; uniform, full
// columns, full rows, Zipf rows): the choice is 1.5 % off the best on average, 14 % at most, and 11 % faster than the
// model before, which knew no shares and priced a piece at 4.5: 22016 x 8192 with 8 x 32 tiles 80 -> 63 us (3 units), 5120^2
// 4-bit with Zipf rows 24.9 -> 18.3, 1024^2 with them 16.9 -> 11.1, two of 22016 x 8192 with 16 x 16 tiles 118 -> 98; 17920
// x 6656 as before.  The worst against that model is 11008 x 4096, 3-bit, with 8 full rows: 23.9 -> 25.7 (6 units and the
// outliers in 4 shares where 3 units and none or 4 units and 2 shares give 23.9).
struct BatchCosts {
  float start_both, both, both_unit, both_entry, both_heavy, both_heavy_unit;              // workgroups that do both
  float start_apart, dense, dense_unit, outliers, outlier_unit, entry, heavy, heavy_unit;  // (entry, heavy: shared)
};
constexpr float kPieceBoth = 7.f, kPieceApart = 6.f;
static const BatchCosts kCosts16x16 = {13.72f, 3.05f, 1.93f, 0.05f, 4.81f, 1.22f, 7.54f, 1.51f, 1.75f, 2.47f, 0.03f, 1.49f, 9.33f, 0.54f};
static const BatchCosts kCosts8x32 = {8.55f, 4.1f, 2.86f, 0.63f, 1.8f, 0.f, 6.83f, 0.93f, 2.34f, 3.21f, 0.26f, 1.15f, 3.12f, 0.f};
static const BatchCosts kCosts32x8 = {7.98f, 6.48f, 1.29f, 0.32f, 3.f, 0.f, 5.08f, 1.55f, 1.15f, 5.37f, 0.f, 1.04f, 3.f, 0.f};

// The chip's CUs by the work they have been given.
class CuLoads {
  struct Level { float load; int64_t cus; };
  Level l_[16];                              // rising loads
  int n_ = 1;
  void put(float load, int64_t cus) {
    int k = n_;
    while (k > 0 && l_[k - 1].load > load) --k;
    if (k > 0 && load - l_[k - 1].load < 1e-3f) { l_[k - 1].cus += cus; return; }
    if (n_ == 16) { l_[n_ - 1].cus += cus; return; }   // (never seen; the longest CU stays right to a level)
    for (int i = n_++; i > k; --i) l_[i] = l_[i - 1];
    l_[k] = {load, cus};
  }

 public:
  CuLoads() { l_[0] = {0.f, kCUs}; }
  void add(int64_t workgroups, float cost) {
    if (workgroups <= 0 || cost <= 0.f) return;
    while (workgroups > 0) {
      if (n_ == 1 && workgroups >= kCUs) {
        l_[0].load += cost * (float)(workgroups / kCUs);
        workgroups %= kCUs;
        continue;
      }
      const int64_t k = workgroups < l_[0].cus ? workgroups : l_[0].cus;
      const float load = l_[0].load + cost;
      if ((l_[0].cus -= k) == 0) {
        --n_;
        for (int i = 0; i < n_; ++i) l_[i] = l_[i + 1];
      }
      put(load, k);
      workgroups -= k;
    }
  }
  float longest() const { return l_[n_ - 1].load; }
};

struct BatchPlan { int groups, per, splits, shares, parts; };  // parts: partial results, dense and of the outliers

// Partial results stay below 24 MB where there is more than one: beyond that the columns are not split (so many rows fill
// the chip by themselves).
static BatchPlan plan_batch(const DevMatrix* As, int count, int b) {
  const Geometry& g = As[0].g;
  const int units = batch_units(g), chunk = 1536 / (kUnitTiles * g.tile_cols), sets = batch_sets(g);
  int groups = 0;
  int64_t rows = 0, nnz = 0;
  bool heavy = false;                        // rows far longer than the mean, by the descriptor's hint
  for (int i = 0; i < count; ++i) {
    groups += batch_groups(As[i].g);
    rows += As[i].g.m;
    nnz += As[i].nnz;
    heavy = heavy || (double)As[i].max_row_nnz > kLongRow + 8.0 * (double)As[i].nnz / As[i].g.m;
  }
  const bool sparse = nnz > 0;
  const BatchCosts& c = g.tile_cols == 16 ? kCosts16x16 : (g.tile_cols == 32 ? kCosts8x32 : kCosts32x8);
  const float entries = (float)((double)nnz / (double)rows * 16 * lane_rows(g.tile_rows) / units / 1000.0);   // per unit
  const int64_t values = (int64_t)b * rows, most = values > 0 ? ((int64_t)6 << 20) / values : 1;
  const int pin_per = option(SPQR_OPT_BATCH_STEPS), pin_shares = option(SPQR_OPT_BATCH_SHARES);
  auto cost = [&](int per, int splits, int shares) {
    const int last = units - (splits - 1) * per;
    auto pieces = [&](int p, float price) { return sparse ? price * (float)((p + chunk - 1) / chunk - 1) : 0.f; };
    auto both = [&](int p) {
      return c.both + c.both_unit * (float)p + pieces(p, kPieceBoth) + c.both_entry * entries * (float)p +
             (heavy ? c.both_heavy + c.both_heavy_unit * (float)p : 0.f);
    };
    auto dense = [&](int p) { return c.dense + c.dense_unit * (float)p; };
    auto outliers = [&](int p) {
      return c.outliers + pieces(p, kPieceApart) + c.outlier_unit * (float)p +
             (c.entry * entries * (float)p + (heavy ? c.heavy + c.heavy_unit * (float)p : 0.f)) / (float)shares;
    };
    CuLoads cu;
    const bool apart = shares > 0 || !sparse;
    cu.add((int64_t)groups * (splits - 1), apart ? dense(per) : both(per));
    cu.add(groups, apart ? dense(last) : both(last));
    if (shares > 0) {
      cu.add((int64_t)groups * (splits - 1) * shares, outliers(per));
      cu.add((int64_t)groups * shares, outliers(last));
    }
    return (apart ? c.start_apart : c.start_both) + cu.longest();
  };
  BatchPlan best = {groups, units, 1, 0, 1};
  float best_cost = 1e30f;
  auto consider = [&](int per) {
    const int splits = (units + per - 1) / per;
    if (pin_per < 1 && per != (units + splits - 1) / splits) return;       // the same splits in more even pieces exist
    for (int shares = 0; shares <= (sparse ? sets : 0); shares = shares == 0 ? 1 : 2 * shares) {
      const int parts = splits * (shares > 0 ? 2 : 1);
      if (pin_shares >= 1 && shares != (pin_shares - 1 < sets ? pin_shares - 1 : sets) && sparse) continue;
      if (parts > 1 && parts > most && !(pin_per >= 1 && shares == 0)) continue;
      const float t = cost(per, splits, shares);
      if (t < best_cost - 1e-3f) { best_cost = t; best = {groups, per, splits, shares, parts}; }
    }
  };
  if (pin_per >= 1) {                        // pinned (tuning, tests)
    best.per = pin_per < units ? pin_per : units;
    best.parts = best.splits = (units + best.per - 1) / best.per;
    consider(best.per);
    return best;
  }
  for (int per = chunk < units ? chunk : units; per >= 1; --per) consider(per);
  for (int per = chunk + 1; per <= units && best_cost > 1e29f; ++per) consider(per);   // few parts allowed: more pieces each
  return best;
}

// The units of a plan's splits.  Where every CU gets two workgroups that do both parts, the first takes the dense part first and the
// second the outliers (batch_group_body), and the second of a CU lives longer: us of a workgroup by its units, of 17920 x 6656 and
// three of 6656^2, 16 x 16 tiles, Zipf rows, 4 and 16 vectors: 9.4 + 4.2 u and 12.2 + 5.2 u; a unit of 32 x 8 tiles is half as wide.  So the
// splits whose workgroups come first get more where that shortens the longest life by 2 us (less is not seen: 3 3 3 3 3 -> 5 5 2 2 1
// cost up to 9 %, 2 of 8 x 32 tiles -> 3 and 1 3 to 8 %; those have no more than 3 units a piece of XT and stay even).
// Three of 6656^2, 4 vectors, units 5 5 5 5 5 1 -> 5 5 5 4 4 3: 44.5 -> 41.2 us; 17920 x 6656, 16 vectors, 4 4 4 4 4 4 2 -> 5 5 5 3 3 3 2:
// 41.2 -> 39.3.  262 layers and sets of layers against even splits: 7.5 % faster to 2 % slower, on average 2.4, 2.1 and 2.4 % faster (16 x 16
// along the columns and the rows, 32 x 8) where the widths differ.
static Shares batch_shares(const BatchPlan& p, const DevMatrix* As, int count) {
  const Geometry& g = As[0].g;
  const int units = batch_units(g), chunk = 1536 / (kUnitTiles * g.tile_cols), wgs = p.groups * p.splits, lead = kCUs / p.groups;
  Shares best = {p.per, 0, 0};
  int64_t nnz = 0;
  for (int i = 0; i < count; ++i) nnz += As[i].nnz;
  if (nnz == 0 || p.shares > 0 || wgs <= kCUs || wgs > 2 * kCUs || lead < 1 || lead >= p.splits || g.tile_cols == 32 || option(SPQR_OPT_BATCH_STEPS) >= 1)
    return best;
  const float wide = (float)g.tile_cols / 16.f;
  auto longest = [&](const Shares& s) {      // of a first one and of the widest that comes second
    return std::max(9.4f + 4.2f * wide * (float)(s.per + s.more), 12.2f + 5.2f * wide * (float)std::min(s.per, units - s.first(lead)));
  };
  float least = longest(best) - 2.f;
  for (int per = p.per; per >= 1; --per) {
    const Shares s = {per, lead, std::max(0, (units - p.splits * per + lead - 1) / lead)};
    const bool covered = s.first(p.splits) >= units && s.first(p.splits - 1) < units;      // all of them, no split empty
    if (!covered || per + s.more > std::max(chunk, p.per) || longest(s) >= least) continue;   // (one piece of XT more would cost more)
    best = s;
    least = longest(s);
  }
  return best;
}

int plan_batch_hook(const DevMatrix* As, int count, int b, int* plan) {
  const BatchPlan p = plan_batch(As, count, b);
  const Shares s = batch_shares(p, As, count);
  plan[0] = p.per; plan[1] = p.splits; plan[2] = p.shares;
  plan[3] = s.per; plan[4] = s.lead; plan[5] = s.more;
  return batch_units(As[0].g);
}

static size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

template <typename Kernel>
static hipError_t allow_lds(Kernel k, int bytes, PerDevice& ready) {
  const int dev = current_device();
  if (ready.get(dev)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) ready.set(dev, 1);
  return e;
}

// Takes `bytes` of scratch from the caller's workspace or the library.
static hipError_t batch_scratch(const Workspace& ws, size_t bytes, hipStream_t stream, bool allow_stream_ordered, Scratch* sc,
                                uint8_t** p) {
  if (ws.from_caller) {                      // nothing is allocated, freed or waited for
    if (ws.p == nullptr || ws.bytes < bytes) return hipErrorOutOfMemory;
    *p = ws.p;
    return hipSuccess;
  }
  if (scratch_get(sc, bytes, current_device(), stream, allow_stream_ordered) != hipSuccess) return hipErrorNotSupported;
  *p = sc->p;
  return hipSuccess;
}

// Scratch: the partial results and, with a permutation, the batch in the matrix's column order: see scratch_get.
// hipErrorNotSupported = no scratch to be had; the caller takes the vector path.
template <int W, int TR, int TC, int AXIS>
static hipError_t launch_mfma_t(const DevMatrix& A, const uint16_t* X, int b, void* Y, int y_dtype, hipStream_t stream,
                                const Workspace& ws) {
  using SH = BatchShape<TR, TC>;
  const Geometry& g = A.g;
  const BatchPlan p = plan_batch(&A, 1, b);
  const size_t xp_bytes = A.perm != nullptr ? up256((size_t)b * g.n * 2) : 0;
  static PerDevice ready[2];
  const auto kernel = p.shares > 0 ? &batch_group_kernel<W, TR, TC, AXIS, true> : &batch_group_kernel<W, TR, TC, AXIS, false>;
  hipError_t e = allow_lds(kernel, SH::LDS, ready[p.shares > 0]);
  if (e != hipSuccess) return e;
  Scratch sc;
  uint8_t* scratch = nullptr;
  e = batch_scratch(ws, xp_bytes + (size_t)p.parts * b * g.m * sizeof(float), stream, true, &sc, &scratch);
  if (e != hipSuccess) return e;
  float* P = reinterpret_cast<float*>(scratch + xp_bytes);
  const uint16_t* Xin = X;
  if (A.perm != nullptr) {
    uint16_t* xp = reinterpret_cast<uint16_t*>(scratch);
    e = launch_gather_x(X, A.perm, xp, g.n, b, stream);
    Xin = xp;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(kernel, dim3(p.groups, p.splits, 1 + p.shares), dim3(256), SH::LDS, stream, A, Xin, b, P, batch_shares(p, &A, 1));
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = launch_sum_groups(g, P, p.parts, b, Y, y_dtype, stream);
  const hipError_t ef = scratch_put(&sc, stream);
  return e == hipSuccess ? ef : e;
}

// Whether a batch of b >= 4 vectors takes the matrix-core path.  Its time hardly depends on b, the vector path re-reads
// the weights once per 4 vectors.  Measured with eager calls (b = 4..16 over the layers of the 7B, 33B and 65B shapes, both
// paths forced) the matrix cores win from 5 vectors on for any layer (4096^2 at b = 4 / 5 / 6 / 7: 16.5 us against 12.0 /
// 17.8 / 19.7 / 25.8) and from 4 on for layers of 30 M weights or more (17920x6656 at b = 4: 43 us against 57; 11008x4096
// 24.9 against 22.9).  The line for smaller layers stays at 7: with group_axis 0 the vector path keeps its weights in
// binary32, and 5 or 6 vectors have always had that.  `alloc_nodes`: the call's scratch would be
// allocation nodes of a graph under capture (library-owned scratch on a capturing stream), about 10 us more
// per call: then from 13 vectors on for any layer, from 8 on for layers of 40 M weights and from 5 on for
// layers of 100 M.  The option SPQR_OPT_BATCH_PATH forces one or the other wherever both apply (tests
// compare the two).
bool mfma_wanted(const Geometry& g, int b, bool alloc_nodes) {
  const int forced = option(SPQR_OPT_BATCH_PATH);
  if (forced == SPQR_BATCH_PATH_VECTOR) return false;
  if (forced == SPQR_BATCH_PATH_MATRIX) return true;   // (_DENSE: the rule below, for calls the dense copy cannot take)
  const double weights = (double)g.m * (double)g.n;
  if (alloc_nodes) return b >= 13 || (b >= 8 && weights >= 40e6) || weights >= 100e6;
  return b >= 7 || weights >= 30e6;
}

bool stream_is_capturing(hipStream_t stream) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) != hipSuccess) { (void)hipGetLastError(); return true; }
  return cs != hipStreamCaptureStatusNone;
}

template <int W, int TR, int TC, int AXIS>
static hipError_t launch_mfma_fused_t(const DevMatrix* As, int count, const uint16_t* X, int b, void* const* Ys, int y_dtype,
                                      hipStream_t stream, const Workspace& ws) {
  using SH = BatchShape<TR, TC>;
  const Geometry& g0 = As[0].g;
  BatchFused F;
  F.count = count;
  for (int i = 0; i < count; ++i) {
    F.it[i].A = As[i];
    F.it[i].Y = Ys[i];
    F.it[i].groups = batch_groups(As[i].g);
  }
  const BatchPlan p = plan_batch(As, count, b);
  size_t total = As[0].perm != nullptr ? up256((size_t)b * g0.n * 2) : 0, at[SPQR_MAX_FUSED];
  for (int i = 0; i < count; ++i) {
    at[i] = total;
    total += up256((size_t)p.parts * b * As[i].g.m * sizeof(float));
  }
  static PerDevice ready[2];
  const auto kernel = p.shares > 0 ? &batch_group_fused_kernel<W, TR, TC, AXIS, true> : &batch_group_fused_kernel<W, TR, TC, AXIS, false>;
  hipError_t e = allow_lds(kernel, SH::LDS, ready[p.shares > 0]);
  if (e != hipSuccess) return e;
  Scratch sc;
  uint8_t* scratch = nullptr;
  e = batch_scratch(ws, total, stream, false, &sc, &scratch);
  if (e != hipSuccess) return e;
  for (int i = 0; i < count; ++i) F.it[i].P = reinterpret_cast<float*>(scratch + at[i]);
  const uint16_t* Xin = X;
  if (As[0].perm != nullptr) {
    uint16_t* xp = reinterpret_cast<uint16_t*>(scratch);
    e = launch_gather_x(X, As[0].perm, xp, g0.n, b, stream);
    Xin = xp;
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(kernel, dim3(p.groups, p.splits, 1 + p.shares), dim3(256), SH::LDS, stream, F, Xin, b, batch_shares(p, As, count));
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(sum_groups_fused_kernel, dim3(p.groups, b), dim3(SH::ROWS), 0, stream, F, p.parts, b, y_dtype);
    e = hipGetLastError();
  }
  const hipError_t ef = scratch_put(&sc, stream);
  return e == hipSuccess ? ef : e;
}


#define SPQR_MFMA_INSTANCES(CASE) \
  CASE(3, 16, 16, 1) CASE(3, 16, 16, 0) CASE(4, 16, 16, 1) CASE(4, 16, 16, 0) \
  CASE(3, 8, 32, 1) CASE(4, 8, 32, 1) CASE(3, 32, 8, 0) CASE(4, 32, 8, 0)

// Scratch a batch of b <= 16 vectors needs on this path: for the matrices one at a time and, if `fused`, all of them in
// one launch set.
size_t mfma_workspace_bound(const DevMatrix* As, int count, int b, bool fused) {
  const size_t xp = As[0].perm != nullptr ? up256((size_t)b * As[0].g.n * 2) : 0;
  size_t worst = 0;
  for (int i = 0; i < count; ++i) {
    const size_t need = xp + up256((size_t)plan_batch(&As[i], 1, b).parts * b * As[i].g.m * sizeof(float));
    if (need > worst) worst = need;
  }
  if (!fused) return worst;
  const BatchPlan p = plan_batch(As, count, b);
  size_t total = xp;
  for (int i = 0; i < count; ++i) total += up256((size_t)p.parts * b * As[i].g.m * sizeof(float));
  return total > worst ? total : worst;
}

// Runs `launch` on `need` bytes of the caller's workspace or of the library's buffer for the stream.
template <typename Launch>
static hipError_t on_scratch(const Workspace& ws, size_t need, hipStream_t stream, Launch launch) {
  if (ws.from_caller) {
    if (ws.p == nullptr || ws.bytes < need) return hipErrorNotSupported;
    return launch(ws.p);
  }
  // far too large for allocation nodes of a graph, and stream-ordered allocations wait on the host
  Scratch sc;
  if (scratch_get(&sc, need, current_device(), stream, false) != hipSuccess) return hipErrorNotSupported;
  const hipError_t e = launch(sc.p);
  const hipError_t ef = scratch_put(&sc, stream);
  return e == hipSuccess ? ef : e;
}

hipError_t launch_prompt_scratch(const DevMatrix* As, int count, const uint16_t* X, int b, void* const* Ys, int y_dtype,
                                 hipStream_t stream, const Workspace& ws) {
  const int most = prompt_fit(As, count, b, ws);
  if (most < 0) return hipErrorNotSupported;
  return on_scratch(ws, prompt_workspace_bytes(As, count, b, most), stream,
                    [&](uint8_t* p) { return launch_prompt(As, count, X, b, Ys, y_dtype, stream, p, most); });
}

hipError_t launch_prefill_scratch(const DevMatrix& A, const uint16_t* X, int b, void* Y, int y_dtype, hipStream_t stream,
                                  const Workspace& ws) {
  return on_scratch(ws, prefill_workspace_bytes(A, b), stream,
                    [&](uint8_t* p) { return launch_prefill(A, X, b, Y, y_dtype, stream, p); });
}

// ---- scratch for callers that cannot allocate ------------------------------------------------------------
// One array per device, resident from the moment the library's code is loaded on it until the process ends.
// In host code its name stands for the symbol, not for a device address: the address is asked per device
// (each GPU holds its own copy) and only that pointer is ever handed to kernels.  All calls on a device that
// use it share it: calls that overlap on one GPU (different streams) race.  Nothing in it has to start at
// zero: every word a call reads (the batch in column order, the partial results, the sorted outliers and their ranges, the
// dense copy) is written earlier in the same call.
static __device__ __align__(256) uint8_t scratch[SPQR_STATIC_SCRATCH_BYTES];

hipError_t static_workspace(Workspace* ws) {
  static std::mutex lock;
  static uint8_t* ptr[kMaxDevices];          // the array's address on each device, nullptr = not asked yet
  const int dev = current_device();
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> hold(lock);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    ptr[dev] = static_cast<uint8_t*>(p);
  }
  ws->from_caller = true;
  ws->fixed = true;
  ws->p = ptr[dev];
  ws->bytes = SPQR_STATIC_SCRATCH_BYTES;
  return hipSuccess;
}

// Tile shapes the matrix-core kernel is built for: the ones the vector kernel is tuned for.
bool mfma_has_instance(const Geometry& g) {
  const bool shape16 = g.tile_rows == 16 && g.tile_cols == 16;
  const bool shape8x32 = g.tile_rows == 8 && g.tile_cols == 32 && g.axis == 1;
  const bool shape32x8 = g.tile_rows == 32 && g.tile_cols == 8 && g.axis == 0;
  return g.layout == kBilevel && (g.w_bits == 3 || g.w_bits == 4) && (shape16 || shape8x32 || shape32x8);
}

hipError_t launch_mfma(const DevMatrix& A, const uint16_t* X, int b, void* Y, int y_dtype, hipStream_t stream,
                       const Workspace& ws) {
  const Geometry& g = A.g;
#define SPQR_MFMA_CASE(W_, TR_, TC_, AX_) \
  if (g.w_bits == W_ && g.tile_rows == TR_ && g.tile_cols == TC_ && g.axis == AX_) \
    return launch_mfma_t<W_, TR_, TC_, AX_>(A, X, b, Y, y_dtype, stream, ws);
  SPQR_MFMA_INSTANCES(SPQR_MFMA_CASE)
#undef SPQR_MFMA_CASE
  return hipErrorNotSupported;
}

hipError_t launch_mfma_fused(const DevMatrix* As, int count, const uint16_t* X, int b, void* const* Ys, int y_dtype,
                             hipStream_t stream, const Workspace& ws) {
  const Geometry& g = As[0].g;
#define SPQR_MFMA_CASE(W_, TR_, TC_, AX_) \
  if (g.w_bits == W_ && g.tile_rows == TR_ && g.tile_cols == TC_ && g.axis == AX_) \
    return launch_mfma_fused_t<W_, TR_, TC_, AX_>(As, count, X, b, Ys, y_dtype, stream, ws);
  SPQR_MFMA_INSTANCES(SPQR_MFMA_CASE)
#undef SPQR_MFMA_CASE
  return hipErrorNotSupported;
}

}  // namespace spqr
