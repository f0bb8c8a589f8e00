// Prompt-sized batches (the prompt phase of Sec. 5, "Inference Time"): one kernel from the compressed weights to the
// products of up to 256 vectors.  Sec. 4.2 makes 16-bit weights first and then multiplies; here the 16-bit weights exist
// only in LDS, a workgroup's block of columns at a time, outliers added, and the matrix cores read them from there, for 64 to
// 192 vectors; more vectors than that read and dequantise the weights once per that many.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <numeric>

#include "../../include/spqr.h"
#include "spqr_batch.h"
#include "spqr_kernels.h"
#include "spqr_sort.h"

namespace spqr {

// A lane of the multiplying kernel takes 8 rows of a tile, of any height; a group is 16 such strips.
constexpr int kLaneRows = 8, kGroupRows = 16 * kLaneRows;

// Several matrices that share the batch X and the format in one grid (one: a set of one); blockIdx.x counts the groups of all
// matrices.  Every workgroup does what it would do in a launch of its own matrix.
struct PromptItem {
  DevMatrix A;
  void* Y;
  uint32_t* counts;
  int32_t* offs;                             // ranges of the sorted outliers
  int entries0;                              // where the matrix's outliers begin in `entries`
  int groups;
};
struct PromptSet {
  uint32_t* entries;                         // sorted outliers of all matrices
  float* P;                                  // partial results [slot][vector][128 places of a group, by group]
  int count, groups;                         // matrices, groups of all of them
  PromptItem it[SPQR_MAX_FUSED];
};
// The address of a pointer that the compiler can't see to be global memory (else its loads count as LDS operations too).
template <typename V> __device__ __forceinline__ V* global_pointer(uint64_t address) {
  return (V*)reinterpret_cast<__attribute__((address_space(1))) V*>(address);
}
__device__ __forceinline__ int find_item(const PromptSet& S, int& group) {   // workgroup-uniform
  int i = 0;
  for (; i < S.count - 1; ++i) {
    if (group < S.it[i].groups) break;
    group -= S.it[i].groups;
  }
  return i;
}

// ---------------------------------------------------------------------------
// The outliers of a group of 16 strips, sorted by the wavefront that dequantises them and by when it does: a phase is 8
// columns of each of the 16 tile columns of a unit, a bin the 4 tile columns of it that one wavefront takes.  The group's
// range of `entries` becomes offs[group][bin] .. offs[group][bin + 1], each entry its place in the phase's block of operands
// (16 bits) and its value.  A counting sort in two kernels over chunks of kSortChunk entries, each with a slot of `counts`
// (spqr_sort.h).
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 512, kSortPer = kSortChunk / kSortThreads, kSortMaxPhases = 512, kSortMaxBins = 4 * kSortMaxPhases;
// The kernels are trips to memory one after the other, so the entries of a thread are few (512 threads: 11008 x 4096 twice, 5.8
// and 10.2 us; 256: 5.2 and 12; 1024: 6.4 and 13) and the chunks of a group side by side, see sort_workgroups.

// Bin of a column: a unit of 16 tile columns (1 << unit_shift columns) has kg phases of 4 bins.
__device__ __forceinline__ int bin_of(int col, int unit_shift, int kg) {
  const int tt = (col >> (unit_shift - 4)) & 15;
  return ((col >> unit_shift) * kg + ((col >> 3) & (kg - 1))) * 4 + (tt >> 2);
}

// The batch as operands: XS[phase][wavefront of the tile column][16 vectors][lane], 16 bytes a lane (8 columns of a vector:
// lane 16 g4 + i holds vector i and tile column g4 of the wavefront's four), zeros behind the last tile column and vector.
// A load of an operand is then one run of 1 KB, 16 clocks of the vector cache; from X itself it is a line per lane, 64 of them.
__device__ __forceinline__ void order_x(const uint16_t* __restrict__ X, int batch, int n, int tile_cols, int kg, int blocks16, int at,
                                        u32x4* __restrict__ XS) {
  const int lane = at & 63, i16 = lane & 15, g4 = lane >> 4;
  int k = at >> 6;
  const int v = 16 * (k % blocks16) + i16;
  k /= blocks16;
  const int s = k & 3, ph = k >> 2, u = ph / kg, j = ph % kg, col = (kUnitTiles * u + 4 * s + g4) * tile_cols + 8 * j;
  XS[at] = v < batch && col < n ? *reinterpret_cast<const u32x4*>(X + (int64_t)v * n + col) : u32x4{0u, 0u, 0u, 0u};
}

// Workgroups of groups * wgs and more order the batch, the others count, `wgs` to a group: each takes every wgs-th chunk.  (The first
// chunks of all groups side by side: workgroups go to the XCDs in turn, and with the chunks of a group side by side and 32 of them
// the only ones that most groups have were all one XCD's, 9.1 us against 5.6 at 4096^2 with Zipf rows.)
__global__ void __launch_bounds__(kSortThreads)
count_phases_kernel(PromptSet S, int groups, int wgs, int unit_shift, int kg, int bins, const uint16_t* __restrict__ X, int batch,
                    int blocks16, u32x4* __restrict__ XS) {
  __shared__ uint32_t hist[kSortMaxBins];
  if ((int)blockIdx.x >= groups * wgs) {
    const int at = ((int)blockIdx.x - groups * wgs) * kSortThreads + (int)threadIdx.x;
    if (at < bins * blocks16 * 64) order_x(X, batch, S.it[0].A.g.n, S.it[0].A.g.tile_cols, kg, blocks16, at, XS);
    return;
  }
  int group = blockIdx.x % groups;
  const PromptItem& it = S.it[find_item(S, group)];
  const DevMatrix& A = it.A;
  if (A.nnz == 0) return;                    // workgroup-uniform
  const int tid = threadIdx.x;
  const GroupRange range = group_range(A.row_ptr, group, kGroupRows, A.g.m, (int)A.nnz);
  const int s = range.s, z = range.z;
  for (int k = blockIdx.x / groups; s + kSortChunk * k < z; k += wgs) {          // workgroup-uniform
    for (int u = tid; u < bins; u += kSortThreads) hist[u] = 0;
    __syncthreads();
    uint16_t c[kSortPer];
#pragma unroll
    for (int i = 0; i < kSortPer; ++i) c[i] = A.col[(uint32_t)min(s + kSortChunk * k + tid + kSortThreads * i, z - 1)];
#pragma unroll
    for (int i = 0; i < kSortPer; ++i)
      if (s + kSortChunk * k + tid + kSortThreads * i < z) atomicAdd(&hist[bin_of(min((int)c[i], A.g.n - 1), unit_shift, kg)], 1u);
    __syncthreads();
    uint32_t* out = it.counts + count_slot(range, group, k) * bins;
    for (int u = tid; u < bins; u += kSortThreads) out[u] = hist[u];
    __syncthreads();
  }
}

// PB: bins a thread adds up.
template <int PB>
__global__ void __launch_bounds__(kSortThreads)
sort_phases_kernel(PromptSet S, int unit_shift, int kg, int bins) {
  constexpr int LR = kLaneRows, ROWS = kGroupRows;
  __shared__ int rp[ROWS + 1];
  __shared__ int start[kSortThreads * PB];            // this chunk's next free place, by bin
  __shared__ int wave_sum[kSortThreads / 64];
  int group = blockIdx.x;
  const PromptItem& it = S.it[find_item(S, group)];
  const DevMatrix& A = it.A;
  if (A.nnz == 0) return;                    // workgroup-uniform
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = A.g.m;
  const GroupRange range = group_range(A.row_ptr, group, ROWS, m, (int)A.nnz);
  const int s = range.s, z = range.z, chunks = sort_chunks(range);
  const uint32_t* in = it.counts + count_slot(range, group, 0) * bins;
  int32_t* offs = it.offs + (int64_t)group * (bins + 1);
  for (int k = blockIdx.y; k < max(chunks, 1); k += gridDim.y) {             // workgroup-uniform
    // the chunk's entries and the row pointers are on their way while the places are worked out
    uint16_t c[kSortPer], v[kSortPer];
    if (chunks > 0) {
#pragma unroll
      for (int i = 0; i < kSortPer; ++i) {
        const uint32_t e = (uint32_t)min(s + kSortChunk * k + tid + kSortThreads * i, z - 1);
        c[i] = A.col[e];
        v[i] = A.val[e];
      }
    }
    if (k == (int)blockIdx.y)
      for (int r = tid; r <= ROWS; r += kSortThreads) rp[r] = A.row_ptr[min(group * ROWS + r, m)];
    // entries of the group in the thread's bins, and how many of them earlier chunks hold
    int total[PB], before[PB], sum = 0;
#pragma unroll
    for (int h = 0; h < PB; ++h) {
      const int u = PB * tid + h;
      total[h] = before[h] = 0;
      if (u < bins) {
#pragma unroll 4
        for (int q = 0; q < chunks; ++q) {
          const int n = (int)in[(int64_t)q * bins + u];
          total[h] += n;
          before[h] += q < k ? n : 0;
        }
      }
      sum += total[h];
    }
    const int own = sum;                     // inclusive sum over the threads
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(sum, off, 64);
      sum += lane >= off ? up : 0;
    }
    if (lane == 63) wave_sum[wave] = sum;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSortThreads / 64 - 1; ++w) sum += w < wave ? wave_sum[w] : 0;
    int first = s + sum - own;
#pragma unroll
    for (int h = 0; h < PB; ++h) {
      const int u = PB * tid + h, at = min(first, z);      // (no further than z, also where broken row pointers let groups share slots)
      start[u] = at + before[h];
      if (k == 0 && u < bins) offs[u] = at;
      first += total[h];
    }
    if (k == 0 && tid == 0) offs[bins] = z;
    __syncthreads();
    if (chunks > 0) {
#pragma unroll
      for (int i = 0; i < kSortPer; ++i) {
        const int e = s + kSortChunk * k + tid + kSortThreads * i;
        if (e >= z) continue;
        int lo = 0;                          // the last row that starts at or before e
#pragma unroll
        for (int step = ROWS / 2; step > 0; step >>= 1) lo += rp[lo + step] <= e ? step : 0;
        const int col = min((int)c[i], A.g.n - 1);
        const int at = atomicAdd(&start[bin_of(col, unit_shift, kg)], 1);
        // tile column of the unit 4 s + g4, place ((s * LR + row) * 64 + g4 * 16 + strip) * 8 + column of the 8
        const int tt = (col & ((1 << unit_shift) - 1)) >> (unit_shift - 4);
        const uint32_t pos = (uint32_t)((((tt >> 2) * LR + lo % LR) * 64 + (tt & 3) * 16 + lo / LR) * 8 + (col & 7));
        S.entries[it.entries0 + min(max(at, s), z - 1)] = pos | ((uint32_t)v[i] << 16);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// P = X . W_hat^T for 16 * NVB * 4 / RW vectors per blockIdx.y (see the batch kernel for the layout of the operands: a lane
// holds 8 rows of a tile, 16 lanes the same tile column of 16 strips, row r of the strips is an operand).  The units of all
// groups of 16 strips stand in one row, group by group, and a workgroup of 4 wavefronts takes `run` of them, whatever groups
// they belong to: as many workgroups as the chip holds, all of one length.  A phase is 8 columns of each of the 16 tile columns
// of a unit.  Wavefront w dequantises 4 of the tile columns, leaves its operands in LDS, in the order they will be read (16
// bytes per lane, no bank conflict), and adds its outliers there; meanwhile all 4 multiply the phase before, each 8 / RW rows
// of every strip with its own 16 * NVB vectors.  Two buffers, one barrier a phase, two workgroups on a CU.
//
// Why so.  Vector instructions and matrix ones share a SIMD's issue (one of 16 x 16 x 32 costs 8 clocks of it and the matrix
// core 16, a vector one 4 to 5): a phase of 128 rows and 128 vectors is 64 and 215 of them per wavefront, 1.5 k clocks a SIMD,
// so the dequantisation and the multiplications are spread between each other, and 8 rows a lane instead of 16 leave the
// registers and the LDS (65 KB) for a second workgroup, whose wavefronts run where this one's wait at the barrier.  A whole
// row of units instead of a grid of groups times splits: 17920 x 6656 is 140 groups of 26 units, which no number of splits
// deals evenly to 256 CUs.
// Measured (the whole call with the sort, 20 and 15 us, and the sums, 11 and 5; before: groups of 256 rows, one workgroup of one
// wavefront per SIMD, a matrix at a time): 17920 x 6656, 4-bit, 256 vectors 162 -> 118 us; gate and up 11008 x 4096, 3-bit, 77
// vectors 101 -> 59; 4096^2 at 128 vectors, which the dense copy took, 39 -> 34.  Slower than that kernel: 8 x 32 tiles with 4 to 16 M
// weights, 1 to 2 of some 25 us (a workgroup's start is that much longer; at most 4 % when calls follow one another closely, 7 %
// faster alone), and the same tiles without any outliers, where ordering the batch is a launch more and 256 vectors are two passes
// instead of one (48 .. 256 vectors, 2048^2 11 .. 13 -> 15 .. 20, 4096^2 13 .. 25 -> 18 .. 36; from 45 M weights on as fast or faster).
// ---------------------------------------------------------------------------
template <int W, int TR, int TC, int AXIS, int RW, int NVB>
__global__ void __launch_bounds__(256, 2)
prompt_group_kernel(PromptSet S, const u32x4* __restrict__ XS, int batch, int blocks16, int run) {
  constexpr int LR = kLaneRows, ROWS = kGroupRows;
  using DQ = Dequant<W, TR, TC, AXIS, LR>;
  using B = BatchTile<W, TR, TC, AXIS, LR>;
  using T = typename B::T;
  constexpr int TILE_BYTES = 16 * T::KW + 4 * T::SD, NSUB = DQ::NSUB, KG = DQ::KG;
  constexpr int STRIPS = 16 / NSUB, PHASE = 4 * LR * 1024, AHEAD = 2, LAST = KG - 1, PAIRS = 4 * LR;
  constexpr int VW = 4 / RW, RB = LR / RW, N = 4 * RB, DQN = 3 * N / 4, RING = 3;
  constexpr int XD = NVB >= 3 ? 2 : 4;       // buffers of operands of X
  extern __shared__ __align__(16) uint8_t smem[];            // two buffers of PHASE bytes
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave / VW, vw = wave % VW, i16 = lane & 15, g4 = lane >> 4;
  const int ntc = S.it[0].A.g.ntc, units = (ntc + kUnitTiles - 1) / kUnitTiles;
  const int lo = blockIdx.x * run, hi = min(S.groups * units, lo + run);   // never empty (host)
  DQ dq(i16 % NSUB);

  // The unit whose tiles are loaded next: its group there and what the matrix is, all of it workgroup-uniform.  The matrices
  // wait in LDS: a scalar load in the loop, even one that is hardly ever taken, makes every wait for LDS one for all of it.
  int4* items = reinterpret_cast<int4*>(smem + 2 * PHASE + 512);
  if (tid < SPQR_MAX_FUSED) {
    const PromptItem& it = S.it[min(tid, S.count - 1)];
    const uint64_t packed = reinterpret_cast<uint64_t>(it.A.packed);
    items[tid] = make_int4((int)(uint32_t)packed, (int)(uint32_t)(packed >> 32), it.A.g.ntr, it.groups);
  }
  __syncthreads();
  int ld_group = lo / units, ld_unit = lo % units, ld_left = hi - lo;
  int ld_item = find_item(S, ld_group);
  const uint32_t row_bytes = (uint32_t)ntc * TILE_BYTES;
  B t;
  auto load_unit = [&]() {                   // rows and columns behind the matrix: its last ones
    const int4 item = items[ld_item];
    const uint64_t packed = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(item.x) | ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(item.y) << 32);
    const int strips = __builtin_amdgcn_readfirstlane(item.z) - ld_group * STRIPS;
    const int t0 = min(kUnitTiles * ld_unit + 4 * wave, (ntc - 1) & ~3), blk = t0 >> 6, L = min(64, ntc - 64 * blk);
    const uint8_t* base = global_pointer<const uint8_t>(packed) + (int64_t)ld_group * STRIPS * row_bytes + (int64_t)64 * blk * TILE_BYTES;
    load_batch_tile(t, base, L, (uint32_t)min(i16 / NSUB, strips - 1) * row_bytes, (uint32_t)(min(t0 + g4, ntc - 1) - 64 * blk), i16 % NSUB);
    --ld_left;                               // behind the last unit of the run: that one again, which nobody multiplies
    const int unit = ld_unit + (ld_left > 0 ? 1 : 0), group = ld_group + (unit == units ? 1 : 0);
    const bool last = group == __builtin_amdgcn_readfirstlane(item.w);
    ld_unit = unit == units ? 0 : unit;
    ld_group = last ? 0 : group;
    ld_item += last ? 1 : 0;
  };
  u32x4 xb[XD][NVB];                         // operands of X by the wavefront that dequantised the tiles, XD - 1 steps ahead
  auto load_x = [&](int ph, int s) {         // ph: phase of the matrix, s its wavefront
    const u32x4* from = XS + ((int64_t)(4 * ph + s) * blocks16 + (blockIdx.y * VW + vw) * NVB) * 64;   // uniform
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb) xb[s % XD][vb] = from[64 * vb + lane];
  };
  // The wavefront's outliers of a phase: the first AHEAD per lane are requested a phase ahead, whether there are any or not
  // (the compiler waits for what the longest path to a place may have requested, so no load of the loop is behind a branch;
  // the ranges wait in LDS for the same reason).
  const int phases = (hi - lo) * KG;
  int2* ranges = reinterpret_cast<int2*>(smem + 2 * PHASE + 512 + 16 * SPQR_MAX_FUSED);          // of this workgroup's bins, and an empty one
  int o0 = 0, o1 = 0;
  uint32_t ent[AHEAD];
  auto fetch_outliers = [&](int from) {
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) ent[k] = S.entries[(uint32_t)max(min(from + lane + 64 * k, o1 - 1), 0)];
  };
  auto load_outliers = [&](int ph) {         // behind the last phase: none
    const int2 r = ranges[min(ph * 4 + wave, phases * 4)];
    o0 = __builtin_amdgcn_readfirstlane(r.x);
    o1 = __builtin_amdgcn_readfirstlane(r.y);
    fetch_outliers(o0);
  };
  uint32_t at[AHEAD];
  uint16_t w16[AHEAD];
  const uint32_t spare = 2 * PHASE + 2 * tid;                // where a lane without an outlier reads and writes
  auto read_places = [&](uint32_t buf, int from) {           // every position at most once: no two lanes meet
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      at[k] = from + 64 * k + lane < o1 ? buf + 2 * (ent[k] & (PHASE / 2 - 1)) : spare;   // (a place is below PHASE / 2)
      w16[k] = *reinterpret_cast<const uint16_t*>(smem + at[k]);
    }
  };
  auto write_places = [&]() {
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) *reinterpret_cast<uint16_t*>(smem + at[k]) = f2h_rne(h2f(w16[k]) + h2f((uint16_t)(ent[k] >> 16)));
  };
  auto add_rest = [&](uint32_t buf) {        // those behind the first 64 * AHEAD
    for (int from = o0 + 64 * AHEAD; from < o1; from += 64 * AHEAD) {
      fetch_outliers(from);
      read_places(buf, from);
      write_places();
    }
  };
  // (a lane's address in a buffer and constants: the LDS instructions hold those)
  const uint32_t to_write = (uint32_t)(wave * LR * 64 + lane) * 16, to_read = (uint32_t)(rw * RB * 64 + lane) * 16;

  int gg = lo / units, u = lo % units;       // group of all and unit of it that is multiplied
  load_unit();
#pragma unroll
  for (int s = 0; s < XD - 1; ++s) load_x(u * KG, s);
  if (tid < 64) reinterpret_cast<uint64_t*>(smem + 2 * PHASE)[tid] = 0;
  for (int k = tid; k <= 4 * phases; k += 256) {
    int2 r = {0, 0};
    int group = (lo + k / (4 * KG)) / units;
    const int bin = (lo + k / (4 * KG)) % units * (4 * KG) + k % (4 * KG);
    if (k < 4 * phases) {
      int i = 0;
      for (; i < S.count - 1 && group >= S.it[i].groups; ++i) group -= S.it[i].groups;
      const PromptItem& it = S.it[i];
      if (it.A.nnz > 0) {
        const int32_t* off = it.offs + (int64_t)group * (units * KG * 4 + 1) + bin;
        r = make_int2(it.entries0 + off[0], it.entries0 + off[1]);
      }
    }
    ranges[k] = r;
  }
  uint32_t cur = 0;                          // which buffer is read
  dq.begin(t, kUnitTiles * u + 4 * wave + g4 < ntc);
  dq.columns(t, 0);
#pragma unroll
  for (int r = 0; r < LR; ++r) *reinterpret_cast<half8_t*>(smem + to_write + 1024 * r) = dq.operand(t, r, 0);
  __syncthreads();                           // the ranges
  load_outliers(0);
  read_places(0, o0);
  write_places();
  add_rest(0);
  if (LAST == 0) load_unit();
  load_outliers(1);
  __syncthreads();

  for (int at_unit = lo; at_unit < hi; ++gg) {               // groups; workgroup-uniform
  float4_t D[RB][NVB];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb) D[r][vb] = float4_t{0.f, 0.f, 0.f, 0.f};
  const int end = min(hi, (gg + 1) * units);
  for (; at_unit < end; ++at_unit) {
    const int next_u = u + 1 < units ? u + 1 : 0;
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      const int nj = j == LAST ? 0 : j + 1, next_ph = j == LAST ? next_u * KG : u * KG + nj;
      if (nj == 0) dq.begin(t, kUnitTiles * next_u + 4 * wave + g4 < ntc);   // on to the next unit's tile
      dq.columns(t, nj);
      // Operand i of the phase: row i % RB of the wavefront's rows, tiles of wavefront i / RB.
      const uint8_t* from = smem + cur + to_read;
      const uint32_t nxt = cur ^ PHASE;
      uint8_t* to = smem + nxt + to_write;
      auto read_operand = [&](int i) { return *reinterpret_cast<const u32x4*>(from + ((i / RB) * LR + i % RB) * 1024); };
      u32x4 a[RING], w = {};
#pragma unroll
      for (int i = 0; i < RING - 1; ++i) a[i] = read_operand(i);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int s = i / RB, r = i % RB;
        if (i + RING - 1 < N) a[(i + RING - 1) % RING] = read_operand(i + RING - 1);
        if (r == 0) {
          if (s + XD - 1 < 4) load_x(u * KG + j, s + XD - 1);
          else load_x(next_ph, s + XD - 5);
        }
        if (i < DQN) {                       // the next phase's weights, a few beside each multiplication
#pragma unroll
          for (int q = PAIRS * i / DQN; q < PAIRS * (i + 1) / DQN; ++q) {
            w[q % 4] = dq.pair(t, q / 4, nj, q % 4);
            if (q % 4 == 3) *reinterpret_cast<u32x4*>(to + 1024 * (q / 4)) = w;
          }
        }
        if (i == DQN) read_places(nxt, o0);
        if (i == DQN + 1 && nj == LAST) load_unit();
        if (i == DQN + 2) write_places();
#pragma unroll
        for (int vb = 0; vb < NVB; ++vb)
          D[r][vb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a[i % RING]),
                                                            __builtin_bit_cast(half8_t, xb[s % XD][vb]), D[r][vb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      add_rest(nxt);
      load_outliers((at_unit - lo) * KG + j + 2);
      __syncthreads();
      cur = nxt;
    }
    u = next_u;
  }
  // the end of a group or of the run: partial results, place 16 r + strip of the group, see sum_phases_kernel
  const int slot = blockIdx.x - (uint32_t)(gg * units) / (uint32_t)run;
  const int64_t mp = (int64_t)S.groups * ROWS;
  int l = lane;
  asm volatile("" : "+v"(l));                // (the addresses are made here, not kept in registers throughout)
#pragma unroll
  for (int vb = 0; vb < NVB; ++vb) {
    const int v = ((blockIdx.y * VW + vw) * NVB + vb) * 16 + (l & 15);
    float* out = S.P + ((int64_t)slot * batch + v) * mp + (int64_t)gg * ROWS + 4 * (l >> 4);
    if (v < batch) {
#pragma unroll
      for (int r = 0; r < RB; ++r) *reinterpret_cast<float4_t*>(out + 16 * (rw * RB + r)) = D[r][vb];
    }
  }
  }
}

// Y[v][row] = sum over the runs that a group is part of, in their order, rounded once to the output type: 4 places a thread, ROWS / 4
// threads a vector; the rows turn round in LDS (16-byte reads; the stride against bank conflicts).
__global__ void __launch_bounds__(256) sum_phases_kernel(PromptSet S, int units, int run, int batch, int y_dtype) {
  constexpr int LR = kLaneRows, ROWS = kGroupRows, TV = ROWS / 4, VECS = 256 / TV, STRIDE = LR + 4;
  __shared__ __align__(16) float rows[VECS][16 * STRIDE];
  int group = blockIdx.x;
  const int splits = (group * units + units - 1) / run - group * units / run + 1;
  const int q = threadIdx.x % TV, w = threadIdx.x / TV, v = VECS * blockIdx.y + w;
  const int64_t mp = (int64_t)S.groups * ROWS, stride = (int64_t)batch * mp;
  const float* p = S.P + (int64_t)v * mp + (int64_t)group * ROWS + 4 * q;
  const PromptItem& it = S.it[find_item(S, group)];
  const int m = it.A.g.m;
  if (v < batch) {
    float4_t s = *reinterpret_cast<const float4_t*>(p);
#pragma unroll 4
    for (int k = 1; k < splits; ++k) s += *reinterpret_cast<const float4_t*>(p + k * stride);
#pragma unroll
    for (int k = 0; k < 4; ++k) rows[w][(4 * (q % 4) + k) * STRIDE + q / 4] = s[k];
  }
  __syncthreads();
  const int row = group * ROWS + 4 * q;      // (m is a multiple of 8)
  if (v >= batch || row >= m) return;
  const float4_t s = *reinterpret_cast<const float4_t*>(&rows[w][(4 * q / LR) * STRIDE + 4 * q % LR]);
  const int64_t at = (int64_t)v * m + row;
  if (y_dtype == SPQR_F32) {
    *reinterpret_cast<float4_t*>(static_cast<float*>(it.Y) + at) = s;
  } else {
    uint32_t h[2] = {(uint32_t)f2h_rne(s[0]) | ((uint32_t)f2h_rne(s[1]) << 16), (uint32_t)f2h_rne(s[2]) | ((uint32_t)f2h_rne(s[3]) << 16)};
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(it.Y) + at) = make_uint2(h[0], h[1]);
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// Vectors per workgroup: 16 * NVB * 4 / RW, and what a phase takes (us) of a workgroup alone on its CU and of two that share
// it.  (Measured over eight layers of 4 M to 119 M weights and all formats; a workgroup's start is 3 us and 0.04 a vector, 5
// more where two start at once, a partial result its way to memory and back at 4 TB/s.  256 vectors a workgroup would be 128
// sums a lane: the compiler spills, 140 us against 95 for 17920 x 6656, 4-bit, 256 vectors.)
struct PromptWidth { int rw, nvb, vectors; double one_us, two_us; };
constexpr PromptWidth kWidths[] = {{2, 2, 64, 1.6, 2.2}, {2, 3, 96, 1.7, 2.4}, {1, 2, 128, 2.05, 2.9}, {1, 3, 192, 2.25, 3.5}};
constexpr double kSortUs = 15;                // the counting and the sorting of the outliers and the launches of a call
constexpr int kMostRunPhases = 2048;          // their ranges of outliers lie in LDS: 32 bytes each
constexpr int kWidthCount = sizeof(kWidths) / sizeof(kWidths[0]);

struct PromptPlan { int groups, units, unit_shift, kg, bins, width, vblocks, run, runs, slots; double us; };
static int prompt_groups(const Geometry& g) { return (g.m + kGroupRows - 1) / kGroupRows; }
// Partial results of a group: the most runs that a group can be part of.  Groups begin at multiples of gcd(units, run) behind a
// run's beginning, at run - gcd at the latest.
static int prompt_slots(int units, int run) { return (run - std::gcd(units, run) + units - 1) / run + 1; }
// most_slots > 0: no more partial results than that.
static PromptPlan plan_prompt(const DevMatrix* As, int count, int b, int most_slots) {
  const Geometry& g = As[0].g;
  PromptPlan p;
  p.groups = 0;
  for (int i = 0; i < count; ++i) p.groups += prompt_groups(As[i].g);
  p.units = (g.ntc + kUnitTiles - 1) / kUnitTiles;
  p.unit_shift = g.tile_cols == 8 ? 7 : (g.tile_cols == 16 ? 8 : 9);
  p.kg = g.tile_cols / 8;
  p.bins = p.units * p.kg * 4;
  const int total = p.groups * p.units, most_run = kMostRunPhases / p.kg;
  const int64_t places = (int64_t)p.groups * kGroupRows;
  int64_t most = std::max<int64_t>(((int64_t)16 << 20) / ((int64_t)b * places), 1);   // 64 MB of them
  if (most_slots > 0) most = std::min<int64_t>(most, most_slots);
  const int pin = option(SPQR_OPT_PROMPT_PLAN), pin_units = pin % 1024;   // (tuning, tests)
  const int widest = kWidths[kWidthCount - 1].vectors;
  const int pin_vectors = 64 * (pin / 1024) < widest ? 64 * (pin / 1024) : widest;
  p.us = 1e30;
  for (int w = 0; w < kWidthCount; ++w) {
    const PromptWidth& c = kWidths[w];
    if (pin_vectors > 0 && c.vectors != pin_vectors && !(c.vectors < pin_vectors && 2 * c.vectors > pin_vectors && b <= c.vectors)) continue;
    const int vblocks = (b + c.vectors - 1) / c.vectors;
    for (int k = 1; k <= 2; ++k) {           // workgroups per CU
      const int wgs = k * kCUs / vblocks > 0 ? k * kCUs / vblocks : 1, even = std::min((total + wgs - 1) / wgs, most_run);
      auto consider = [&](int run) {
        if (run > most_run || prompt_slots(p.units, run) > most) return false;
        const int runs = (total + run - 1) / run, rest = runs % wgs;
        const double one = run * p.kg * c.one_us + 3.0 + 0.04 * c.vectors, all = k == 1 ? one : run * p.kg * c.two_us + 8.0 + 0.04 * c.vectors;
        const double parts_us = (double)b * kGroupRows * 8 / 4e6 * (runs + p.groups);
        // full rounds of workgroups, then one that may have the CUs to themselves
        const double last = rest == 0 ? 0.0 : runs > wgs && rest * vblocks <= kCUs ? one : all;
        const double cost = runs / wgs * all + last + parts_us;
        if (cost < p.us - 1e-9) { p.us = cost; p.width = w; p.vblocks = vblocks; p.run = run; }
        return true;
      };
      // Even shares; where those are more partial results of a group than there may be, the next longer runs that are not, and
      // whole groups, one result each (a run may hold one at least: kSortMaxPhases).
      if (consider(even)) continue;
      if (most > 1) consider(std::max<int>(even, (int)((p.units - 1 + most - 2) / (most - 1))));
      consider(p.units);
      consider(std::min((even + p.units - 1) / p.units, most_run / p.units) * p.units);
    }
  }
  if (pin_units >= 1) p.run = std::min(pin_units, std::min(total, most_run));
  p.runs = (total + p.run - 1) / p.run;
  p.slots = prompt_slots(p.units, p.run);
  return p;
}

// The formats the batch kernel has; more outliers than one weight in four go through the dense copy instead.
bool prompt_has_instance(const DevMatrix& A) {
  return mfma_has_instance(A.g) && A.nnz <= (int64_t)A.g.m * A.g.n / 4 && A.nnz < 0x7FFF0000ll && (int64_t)A.g.m * A.g.n < ((int64_t)1 << 44) &&
         (A.g.ntc + kUnitTiles - 1) / kUnitTiles * (A.g.tile_cols / 8) <= kSortMaxPhases;
}

// Where the dense copy pays against slices of 16 (prefill_wanted: from 48 vectors on, later on larger layers) and this kernel
// is faster than the copy: from 4 M weights and 512 columns on.  Times in us, the copy -> here, 48 to 256 vectors, 1 % of outliers,
// uniform and with Zipf rows: 2048^2 25 .. 31 -> 21 .. 27 and 24 .. 31 -> 23 .. 29, 4096^2 35 .. 45 -> 28 .. 43 and 33 .. 44 -> 29 .. 44,
// 1024 x 17920 58 .. 65 -> 32 .. 47 and 57 .. 63 -> 36 .. 49, 17920 x 1536 44 .. 65 -> 33 .. 52 and 42 .. 62 -> 35 .. 57; 1024^2 21 .. 24
// against 22 .. 24; 17920 x 256 23 .. 32 against 27 .. 36 (too few phases to a group).  The one size above the line that loses
// is 2048 x 4096 and its like above 192 vectors with uneven rows, 31 .. 33 against 32 .. 36, where the copy's multiply fills the chip.
// Tiles of 8 columns: from 18 M on (17920 x 1024, Zipf rows, 34 .. 48 against 33 .. 49; 3072 x 6144 37 .. 48 against 36 .. 47); from 12 M
// on below 96 vectors, with fewer than 2048 rows (the copy's multiply has few workgroups there: 512 x 24576, Zipf rows, 65 .. 70 -> 37 .. 45)
// or where the rows hold much the same number of outliers (a unit is one phase, and a group with heavy rows makes every one of its
// phases longer: 4096^2 from 96 vectors on 35 .. 43 against 35 .. 43 uniform, 35 .. 42 against 37 .. 47 with Zipf rows).
// From 17 vectors on this kernel would beat the slices, but they add the outliers in binary32 and here weight + outlier is rounded to
// binary16, so no batch that took the slices moves here.  With a pinned plan (SPQR_OPT_PROMPT_PLAN) the size is no matter.
static bool prompt_pays(const DevMatrix& A, int b) {
  const double weights = (double)A.g.m * A.g.n, mean = (double)A.nnz / A.g.m;
  if (A.g.n < 512 || weights < 4e6) return false;
  const bool even = A.nnz == 0 || (A.max_row_nnz > 0 && A.max_row_nnz <= 64 + 8 * mean);     // by the descriptor's hint
  return A.g.tile_cols != 8 || weights >= 18e6 || (weights >= 12e6 && (b < 96 || A.g.m < 2048 || even));
}

bool prompt_wanted(const DevMatrix& A, int b) {
  return option(SPQR_OPT_BATCH_PATH) == SPQR_BATCH_PATH_AUTO && prompt_has_instance(A) && prefill_wanted(A, b) &&
         (prompt_pays(A, b) || option(SPQR_OPT_PROMPT_PLAN) >= 1);
}

// Scratch of one call: the batch as operands, in column order before that if there is a permutation, per matrix the sorted outliers, their ranges,
// the counts, the partial results.
static int prompt_blocks16(const PromptPlan& p) { return p.vblocks * kWidths[p.width].vectors / 16; }
static size_t prompt_offsets(const DevMatrix* As, int count, int b, const PromptPlan& p, uint8_t* scratch, PromptSet* S) {
  size_t total = 0;
  auto take = [&](size_t bytes) { uint8_t* at = scratch + total; total += up256(bytes); return at; };
  take((size_t)p.bins * prompt_blocks16(p) * 1024);
  if (As[0].perm != nullptr) take((size_t)b * As[0].g.n * 2);
  int64_t nnz = 0;
  for (int i = 0; i < count; ++i) nnz += As[i].nnz;
  uint8_t* entries = take((size_t)nnz * 4);
  nnz = 0;
  for (int i = 0; i < count; ++i) {
    const DevMatrix& A = As[i];
    const int groups = prompt_groups(A.g);
    uint8_t* offs = take(A.nnz > 0 ? (size_t)groups * (p.bins + 1) * 4 : 0);
    uint8_t* counts = take(A.nnz > 0 ? (size_t)count_slots(A.nnz, groups) * p.bins * 4 : 0);
    if (S != nullptr) S->it[i] = {A, nullptr, reinterpret_cast<uint32_t*>(counts), reinterpret_cast<int32_t*>(offs), (int)nnz, groups};
    nnz += A.nnz;
  }
  uint8_t* P = take((size_t)p.slots * b * p.groups * kGroupRows * sizeof(float));
  if (S != nullptr) {
    S->entries = reinterpret_cast<uint32_t*>(entries);
    S->P = reinterpret_cast<float*>(P);
    S->count = count;
    S->groups = p.groups;
  }
  return total;
}

// Workgroups per group of the sort: as many as the group with the most outliers may have chunks, by what the descriptors say of the
// longest row (nothing: any row may be full): a chunk behind another one waits for all of its trips to memory.  In all no more
// than the chip takes about at once (but 4 a group), for most find no chunk where a few rows hold the outliers.  128 vectors, whole
// call in us, 4 a group -> this: 512 x 24576 with 8 full rows 74 .. 103 -> 40 .. 45, 1024 x 17920 with Zipf rows 63 .. 70 -> 42 .. 48,
// 8192 x 22016 with them 120 .. 143 -> 105 .. 117 (counting and sorting 12 + 31 -> 9.4 + 17.4; with 512 in all 10 + 22, with 2048 9.4 +
// 17.6); 4096^2 and 17920 x 6656 as before.
constexpr int kMostSortWgs = 1024;
static int sort_workgroups(const DevMatrix* As, int count, int groups) {
  int64_t most = 0;
  for (int i = 0; i < count; ++i) {
    const int64_t row = As[i].max_row_nnz > 0 ? As[i].max_row_nnz : As[i].g.n;
    most = std::max(most, std::min(As[i].nnz, row * kGroupRows));
  }
  const int64_t chunks = (most + kSortChunk - 1) / kSortChunk;
  return (int)std::max<int64_t>(1, std::min<int64_t>(chunks, std::max(4, kMostSortWgs / groups)));
}

double prompt_us(const DevMatrix* As, int count, int b) { return plan_prompt(As, count, b, 0).us + kSortUs; }

int plan_prompt_hook(const DevMatrix* As, int count, int b, int most_slots, int32_t* plan, double* us) {
  const PromptPlan p = plan_prompt(As, count, b, most_slots);
  *us = p.us;
  plan[0] = kWidths[p.width].vectors; plan[1] = p.run; plan[2] = p.runs; plan[3] = p.slots;
  plan[4] = sort_workgroups(As, count, p.groups);
  return p.units;
}

size_t prompt_workspace_bytes(const DevMatrix* As, int count, int b, int most_slots) {
  return prompt_offsets(As, count, b, plan_prompt(As, count, b, most_slots), nullptr, nullptr);
}

// Scratch of a given size, a caller's workspace or the static array: with less than this the call takes the slices of 16, which
// add the outliers in binary32, where this kernel and the dense copy round weight + outlier to binary16.  A call's rounding is not to
// depend on what a plan of this kernel happens to need, so the line does not move with the plans: it is the room of the dense copy for
// the layers that are this kernel's only because it is faster than the copy, and for those that it always took the room of the
// plan it began with, groups of 16 strips of 8 or 16 rows and equal splits of the columns, one workgroup per CU.
size_t prompt_line_bytes(const DevMatrix& A, int b) {
  const Geometry& g = A.g;
  const double weights = (double)g.m * g.n;
  if (option(SPQR_OPT_PROMPT_PLAN) >= 1) return 0;             // a pinned plan takes layers of any size
  if (g.tile_rows != 8 && (weights < 24e6 || (b > 192 && g.n <= 2048))) return prefill_workspace_bytes(A, b);
  const int rows = 16 * lane_rows(g.tile_rows), groups = (g.m + rows - 1) / rows, units = (g.ntc + kUnitTiles - 1) / kUnitTiles;
  const int kg = g.tile_cols / 8, phases = units * kg;
  const int64_t values = (int64_t)b * g.m, most = ((int64_t)16 << 20) / values;               // 64 MB of partial results
  int splits = 1;
  double best = 1e30;
  for (int nvb = 1; nvb <= (rows == 256 ? 2 : 4); nvb *= 2) {  // 64 * nvb vectors a workgroup: us of a phase, 5 of its start
    const double phase_us = rows == 256 ? (nvb == 1 ? 1.8 : 2.3) : (nvb == 1 ? 1.0 : nvb == 2 ? 1.2 : 1.8);
    const int64_t wgs = (int64_t)groups * ((b + 64 * nvb - 1) / (64 * nvb));
    for (int s = 1; s <= units && (s == 1 || s <= most); ++s) {
      const int per = (units + s - 1) / s, even = (units + per - 1) / per;
      const double cost = (double)((wgs * even + kCUs - 1) / kCUs) * (per * kg * phase_us + 5.0) + even * ((double)b * g.m * 8 / 4e6);
      if (cost < best - 1e-9) { best = cost; splits = even; }
    }
  }
  size_t total = up256((size_t)splits * values * sizeof(float)) + (A.perm != nullptr ? up256((size_t)b * g.n * 2) : 0);
  if (A.nnz > 0)                             // the sorted outliers, their ranges, the counts
    total += up256((size_t)A.nnz * 4) + up256((size_t)groups * (phases + 1) * 4) + up256((size_t)count_slots(A.nnz, groups) * phases * 4);
  return total;
}

int prompt_fit(const DevMatrix* As, int count, int b, const Workspace& ws) {
  if (!ws.from_caller) return 0;
  for (int i = 0; i < count; ++i)
    if (ws.bytes < prompt_line_bytes(As[i], b)) return -1;
  if (prompt_workspace_bytes(As, count, b) <= ws.bytes) return 0;
  for (int slots = 3; ws.fixed && slots >= 1; --slots)         // fewer partial results
    if (prompt_workspace_bytes(As, count, b, slots) <= ws.bytes) return slots;
  return -1;
}

template <int W, int TR, int TC, int AXIS, int RW, int NVB>
static hipError_t launch_prompt_t(const PromptSet& S, const u32x4* XS, int b, const PromptPlan& p, hipStream_t stream) {
  constexpr int PHASES = 2 * 4 * kLaneRows * 1024 + 512 + 16 * SPQR_MAX_FUSED, MOST = 160 * 1024;
  static PerDevice ready;                    // more than 64 KB of LDS per workgroup is an opt-in per kernel and device
  const int dev = current_device();
  if (!ready.get(dev)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prompt_group_kernel<W, TR, TC, AXIS, RW, NVB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, MOST);
    if (e != hipSuccess) return e;
    ready.set(dev, 1);
  }
  hipLaunchKernelGGL((prompt_group_kernel<W, TR, TC, AXIS, RW, NVB>), dim3(p.runs, p.vblocks), dim3(256),
                     PHASES + (4 * p.run * p.kg + 1) * 8, stream, S, XS, b, prompt_blocks16(p), p.run);
  return hipGetLastError();
}
template <int W, int TR, int TC, int AXIS>
static hipError_t launch_prompt_width(const PromptSet& S, const u32x4* XS, int b, const PromptPlan& p, hipStream_t stream) {
  switch (p.width) {
    case 0: return launch_prompt_t<W, TR, TC, AXIS, kWidths[0].rw, kWidths[0].nvb>(S, XS, b, p, stream);
    case 1: return launch_prompt_t<W, TR, TC, AXIS, kWidths[1].rw, kWidths[1].nvb>(S, XS, b, p, stream);
    case 2: return launch_prompt_t<W, TR, TC, AXIS, kWidths[2].rw, kWidths[2].nvb>(S, XS, b, p, stream);
    default: return launch_prompt_t<W, TR, TC, AXIS, kWidths[3].rw, kWidths[3].nvb>(S, XS, b, p, stream);
  }
}

// Y_i[b][m_i] = X[b][n] . W_hat_i^T for matrices of one format, width and permutation.  `scratch`:
// prompt_workspace_bytes(As, count, b, most_slots) bytes, 256-byte aligned.
hipError_t launch_prompt(const DevMatrix* As, int count, const uint16_t* X, int b, void* const* Ys, int y_dtype, hipStream_t stream,
                         uint8_t* scratch, int most_slots) {
  if (scratch == nullptr || b < 1 || b > 256 || count < 1 || count > SPQR_MAX_FUSED) return hipErrorInvalidValue;
  const Geometry& g = As[0].g;
  int64_t nnz = 0;
  for (int i = 0; i < count; ++i) {
    const Geometry& h = As[i].g;
    if (!prompt_has_instance(As[i]) || h.n != g.n || h.w_bits != g.w_bits || h.tile_rows != g.tile_rows || h.axis != g.axis) return hipErrorInvalidValue;
    nnz += As[i].nnz;
  }
  const PromptPlan p = plan_prompt(As, count, b, most_slots);
  if (p.vblocks * kWidths[p.width].vectors < b || p.run < 1 || (int64_t)p.runs * p.run < (int64_t)p.groups * p.units ||
      (int64_t)(p.runs - 1) * p.run >= (int64_t)p.groups * p.units)
    return hipErrorInvalidValue;
  PromptSet S;
  prompt_offsets(As, count, b, p, scratch, &S);
  for (int i = 0; i < count; ++i) S.it[i].Y = Ys[i];
  hipError_t e = hipSuccess;
  const uint16_t* Xin = X;
  const int blocks16 = prompt_blocks16(p);
  u32x4* XS = reinterpret_cast<u32x4*>(scratch);
  if (As[0].perm != nullptr) {
    uint16_t* xp = reinterpret_cast<uint16_t*>(scratch + up256((size_t)p.bins * blocks16 * 1024));
    e = launch_gather_x(X, As[0].perm, xp, g.n, b, stream);
    if (e != hipSuccess) return e;
    Xin = xp;
  }
  const int wgs = sort_workgroups(As, count, p.groups);
  hipLaunchKernelGGL(count_phases_kernel, dim3(p.groups * wgs + (p.bins * blocks16 * 64 + kSortThreads - 1) / kSortThreads), dim3(kSortThreads), 0, stream, S, p.groups,
                     wgs, p.unit_shift, p.kg, p.bins, Xin, b, blocks16, XS);
  if (nnz > 0) {
    const auto sort = p.bins <= kSortThreads ? &sort_phases_kernel<1> : p.bins <= 2 * kSortThreads ? &sort_phases_kernel<2> : &sort_phases_kernel<4>;
    hipLaunchKernelGGL(sort, dim3(p.groups, wgs), dim3(kSortThreads), 0, stream, S, p.unit_shift, p.kg, p.bins);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = hipErrorInvalidValue;
#define SPQR_CASE(W_, TR_, TC_, AX_)                                                     \
  if (g.w_bits == W_ && g.tile_rows == TR_ && g.tile_cols == TC_ && g.axis == AX_)       \
    e = launch_prompt_width<W_, TR_, TC_, AX_>(S, XS, b, p, stream);
  SPQR_CASE(3, 16, 16, 1) SPQR_CASE(4, 16, 16, 1) SPQR_CASE(3, 8, 32, 1) SPQR_CASE(4, 8, 32, 1)
  SPQR_CASE(3, 16, 16, 0) SPQR_CASE(4, 16, 16, 0) SPQR_CASE(3, 32, 8, 0) SPQR_CASE(4, 32, 8, 0)
#undef SPQR_CASE
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sum_phases_kernel, dim3(p.groups, (b + 7) / 8), dim3(256), 0, stream, S, p.units, p.run, b, y_dtype);
  return hipGetLastError();
}

}  // namespace spqr
