// Prompt-sized batches (the prompt phase of Sec. 5, "Inference Time"): one kernel from the compressed weights to the
// products of up to 256 vectors.  Sec. 4.2 makes 16-bit weights first and then multiplies; here the 16-bit weights exist
// only in LDS, a workgroup's block of columns at a time, outliers added, and the matrix cores read them from there, for 64,
// 128 or (strips of 8 rows) 256 vectors; more vectors than that read and dequantise the weights once per that many.
#include <hip/hip_runtime.h>
#include <cstdint>

#include "../../include/spqr.h"
#include "spqr_batch.h"
#include "spqr_kernels.h"
#include "spqr_sort.h"

namespace spqr {

// ---------------------------------------------------------------------------
// The outliers of a group of 16 strips, sorted by phase (8 columns of each of 16 tile columns, the block the multiplying
// kernel has in LDS at a time): the group's range of `entries` becomes offs[group][phase] .. offs[group][phase + 1], each
// entry its place in the block (16 bits) and its value.  A counting sort in two kernels over chunks of kSortChunk entries,
// each with a slot of `counts` (spqr_sort.h).
// ---------------------------------------------------------------------------
constexpr int kSortPer = kSortChunk / 256, kSortMaxPhases = 512;
constexpr int kSortWgs = 8;                  // workgroups per group; each takes every 8th chunk

// Phase of a column: a unit of 16 tile columns (1 << unit_shift columns) has kg of them.
__device__ __forceinline__ int phase_of(int col, int unit_shift, int kg) { return (col >> unit_shift) * kg + ((col >> 3) & (kg - 1)); }

__global__ void __launch_bounds__(256)
count_phases_kernel(DevMatrix A, int rows, int unit_shift, int kg, int phases, uint32_t* __restrict__ counts) {
  __shared__ uint32_t hist[kSortMaxPhases];
  const int tid = threadIdx.x, group = blockIdx.x;
  const GroupRange range = group_range(A.row_ptr, group, rows, A.g.m, (int)A.nnz);
  const int s = range.s, z = range.z;
  for (int k = blockIdx.y; s + kSortChunk * k < z; k += kSortWgs) {          // workgroup-uniform
    for (int u = tid; u < phases; u += 256) hist[u] = 0;
    __syncthreads();
    uint16_t c[kSortPer];
#pragma unroll
    for (int i = 0; i < kSortPer; ++i) c[i] = A.col[(uint32_t)min(s + kSortChunk * k + tid + 256 * i, z - 1)];
#pragma unroll
    for (int i = 0; i < kSortPer; ++i)
      if (s + kSortChunk * k + tid + 256 * i < z) atomicAdd(&hist[phase_of(min((int)c[i], A.g.n - 1), unit_shift, kg)], 1u);
    __syncthreads();
    uint32_t* out = counts + count_slot(range, group, k) * phases;
    for (int u = tid; u < phases; u += 256) out[u] = hist[u];
    __syncthreads();
  }
}

// LR: rows per strip of the multiplying kernel.
template <int LR>
__global__ void __launch_bounds__(256)
sort_phases_kernel(DevMatrix A, int unit_shift, int kg, int phases, const uint32_t* __restrict__ counts, int32_t* __restrict__ offs,
                  uint32_t* __restrict__ entries) {
  constexpr int ROWS = 16 * LR;
  __shared__ int rp[ROWS + 1];
  __shared__ int start[kSortMaxPhases];      // this chunk's next free place, by phase
  __shared__ int wave_sum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, group = blockIdx.x, m = A.g.m;
  const GroupRange range = group_range(A.row_ptr, group, ROWS, m, (int)A.nnz);
  const int s = range.s, z = range.z, chunks = sort_chunks(range);
  const uint32_t* in = counts + count_slot(range, group, 0) * phases;
  for (int k = blockIdx.y; k < max(chunks, 1); k += kSortWgs) {              // workgroup-uniform
    // the chunk's entries and the row pointers are on their way while the places are worked out
    uint16_t c[kSortPer], v[kSortPer];
    if (chunks > 0) {
#pragma unroll
      for (int i = 0; i < kSortPer; ++i) {
        const uint32_t e = (uint32_t)min(s + kSortChunk * k + tid + 256 * i, z - 1);
        c[i] = A.col[e];
        v[i] = A.val[e];
      }
    }
    if (k == (int)blockIdx.y)
      for (int r = tid; r <= ROWS; r += 256) rp[r] = A.row_ptr[min(group * ROWS + r, m)];
    // entries of the group per phase (2 tid, 2 tid + 1), and how many of them earlier chunks hold
    int total[2] = {0, 0}, before[2] = {0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int u = 2 * tid + h;
      if (u < phases) {
#pragma unroll 4
        for (int q = 0; q < chunks; ++q) {
          const int n = (int)in[(int64_t)q * phases + u];
          total[h] += n;
          before[h] += q < k ? n : 0;
        }
      }
    }
    int sum = total[0] + total[1];           // inclusive sum over the threads
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(sum, off, 64);
      sum += lane >= off ? up : 0;
    }
    if (lane == 63) wave_sum[wave] = sum;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 3; ++w) sum += w < wave ? wave_sum[w] : 0;
    // (no further than z, also where broken row pointers let groups share slots)
    const int first[2] = {min(s + sum - total[0] - total[1], z), min(s + sum - total[1], z)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int u = 2 * tid + h;
      start[u] = first[h] + before[h];
      if (k == 0) {
        if (u < phases) offs[(int64_t)group * (phases + 1) + u] = first[h];
        if (u == 0) offs[(int64_t)group * (phases + 1) + phases] = z;
      }
    }
    __syncthreads();
    if (chunks > 0) {
#pragma unroll
      for (int i = 0; i < kSortPer; ++i) {
        const int e = s + kSortChunk * k + tid + 256 * i;
        if (e >= z) continue;
        int lo = 0;                          // the last row that starts at or before e
#pragma unroll
        for (int step = ROWS / 2; step > 0; step >>= 1) lo += rp[lo + step] <= e ? step : 0;
        const int col = min((int)c[i], A.g.n - 1);
        const int at = atomicAdd(&start[phase_of(col, unit_shift, kg)], 1);
        // tile column of the unit 4 s + g4, place ((s * LR + row) * 64 + g4 * 16 + strip) * 8 + column of the 8
        const int tt = (col & ((1 << unit_shift) - 1)) >> (unit_shift - 4);
        const uint32_t pos = (uint32_t)((((tt >> 2) * LR + lo % LR) * 64 + (tt & 3) * 16 + lo / LR) * 8 + (col & 7));
        entries[min(max(at, s), z - 1)] = pos | ((uint32_t)v[i] << 16);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// P[split][vector][rows] = X . W_hat^T for 64 * NVB vectors per blockIdx.z (see the batch kernel for the layout of the operands: a lane
// holds a tile, 16 lanes the same tile column of 16 strips, row r of the strips is an operand).  A workgroup of 4
// wavefronts owns a group of 16 strips (256 or 128 rows) and 64 * NVB vectors; a phase is 8 columns of each of the 16 tile
// columns of a unit.  Wavefront w dequantises 4 of the tile columns and leaves its operands in LDS, in the order they
// will be read (16 bytes per lane, no bank conflict); the outliers of the phase are added there; then every wavefront
// multiplies all of them with its own 16 * NVB vectors, whose operands come from X (L2) one phase ahead.  Two buffers: the
// next phase is dequantised between the multiplications of this one, so vector issue hides behind the matrix cores.
// One wavefront per SIMD and one workgroup per CU (64 x NVB sums a lane with strips of 16 rows, 128.5 KB of LDS; half of
// both with strips of 8): a dequantised weight is used for 64 * NVB vectors, an operand read from LDS for NVB
// multiplications.
//
// What bounds it: issue and LDS.  A phase with strips of 16 rows and 128 vectors is 128 matrix instructions (2048
// clocks), 530 vector ones and 90 LDS operations per wavefront with its outliers, 256 KB read from LDS per workgroup (2048
// clocks), and takes 2.3 us, of which the outliers' two barriers and round trip are a part (17920 x 6656, 256 vectors:
// vector issue 35 % of a wavefront's time, the matrix cores 26 %).  Measured (with the sort and the sums, 19 and 17 us of
// the 161): 17920 x 6656, 4-bit, 256 vectors 240 -> 161 us (380 TFLOP/s), 128 vectors 173 -> 95 us; gate and up 11008 x
// 4096, 3-bit, 77 vectors 149 -> 101 us.  Before, the weights went through a dense binary16 copy in memory (70 us of writing it, 30 us
// of adding the outliers there, 137 us of multiplying at 256 vectors).
// ---------------------------------------------------------------------------
template <int W, int TR, int TC, int AXIS, int NVB>
__global__ void __launch_bounds__(256, 1)
prompt_group_kernel(DevMatrix A, const uint16_t* __restrict__ X, int batch, float* __restrict__ P, int units_per_split,
                    const uint32_t* __restrict__ entries, const int32_t* __restrict__ offs) {
  using DQ = Dequant<W, TR, TC, AXIS>;
  using B = BatchTile<W, TR, TC, AXIS>;
  using T = typename B::T;
  constexpr int TILE_BYTES = 16 * T::KW + 4 * T::SD, LR = DQ::LR, NSUB = DQ::NSUB, KG = DQ::KG, ROWS = 16 * LR;
  constexpr int STRIPS = 16 / NSUB, PHASE = 4 * LR * 1024, AHEAD = 4, LAST = KG - 1;
  extern __shared__ __align__(16) uint8_t smem[];            // two buffers of PHASE bytes, 2 bytes nobody reads per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4, group = blockIdx.x;
  const int n = A.g.n, ntc = A.g.ntc, ntr = A.g.ntr * NSUB, m = A.g.m;
  const int units = (ntc + kUnitTiles - 1) / kUnitTiles;
  const int u_lo = blockIdx.y * units_per_split, u_hi = min(units, u_lo + units_per_split);   // never empty (host)
  const bool sparse = A.nnz > 0;
  const int32_t* off = offs + (int64_t)group * (units * KG + 1);

  const uint8_t* base = A.packed + (int64_t)group * STRIPS * ntc * TILE_BYTES;
  const int my_strip = min(group * 16 + i16, ntr - 1) - group * 16, half = NSUB == 2 ? my_strip & 1 : 0;
  const uint32_t strip_off = (uint32_t)(my_strip / NSUB) * (uint32_t)ntc * TILE_BYTES;
  const int vec0 = (blockIdx.z * 4 + wave) * 16 * NVB;
  uint32_t xrow[NVB];
#pragma unroll
  for (int vb = 0; vb < NVB; ++vb) xrow[vb] = (uint32_t)min(vec0 + 16 * vb + i16, batch - 1) * (uint32_t)n * 2u;
  DQ dq(half);

  float4_t D[LR][NVB];
#pragma unroll
  for (int r = 0; r < LR; ++r)
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb) D[r][vb] = float4_t{0.f, 0.f, 0.f, 0.f};

  auto load_unit = [&](B& t, int u) {        // behind the range every lane reads the group's first tile
    const bool real = u < u_hi;
    const int t0 = min(kUnitTiles * u + 4 * wave, (ntc - 1) & ~3), blk = t0 >> 6, L = min(64, ntc - 64 * blk);
    const uint32_t l = real ? (uint32_t)(min(t0 + g4, ntc - 1) - 64 * blk) : 0u;
    load_batch_tile(t, base + (real ? (int64_t)64 * blk * TILE_BYTES : 0), real ? L : 1, real ? strip_off : 0u, l, half);
  };
  u32x4 xb[4][NVB];                          // the operands of X of a phase, by the wavefront that dequantised the tiles
  auto load_x = [&](int u, int j, int s) {
    const int tl = min(kUnitTiles * u + 4 * s + g4, ntc - 1);
    const uint32_t at = (uint32_t)tl * (TC * 2) + 16u * j;
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb) xb[s][vb] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(X) + (xrow[vb] + at));
  };
  // The outliers of the phase being dequantised: the first AHEAD per thread are requested a phase ahead.  They are added
  // AHEAD at a time, reads first; one that does not exist goes to the thread's own spare place.
  int o0 = 0, o1 = 0;
  uint32_t ent[AHEAD];
  const uint32_t spare = PHASE + tid;        // in halves, from the start of the LDS
  auto fetch_outliers = [&](int from) {
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) ent[k] = entries[(uint32_t)min(from + tid + 256 * k, o1 - 1)];
  };
  int off_v = 0;                             // lane l: where phase l of the current 32 begins
  auto load_outliers = [&](int u, int j) {
    o0 = o1 = 0;
    if (sparse && u < u_hi) {                // workgroup-uniform
      const int ph = (u - u_lo) * KG + j;
      if ((ph & 31) == 0) off_v = off[min(u * KG + j + lane, units * KG)];
      o0 = __builtin_amdgcn_readlane(off_v, ph & 31);
      o1 = __builtin_amdgcn_readlane(off_v, (ph & 31) + 1);
      if (o0 < o1) fetch_outliers(o0);
    }
  };
  auto add_outliers = [&](uint8_t* buf) {    // every position at most once: no two threads meet
    __syncthreads();
    if (o0 >= o1) return;                    // workgroup-uniform
    uint16_t* all = reinterpret_cast<uint16_t*>(smem);
    const uint32_t at0 = (uint32_t)(buf - smem) / 2;
    for (int from = o0;;) {
      uint32_t at[AHEAD];
      uint16_t w[AHEAD];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        at[k] = from + tid + 256 * k < o1 ? at0 + (ent[k] & (PHASE / 2 - 1)) : spare;   // (a place is below PHASE / 2)
        w[k] = all[at[k]];
      }
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) all[at[k]] = f2h_rne(h2f(w[k]) + h2f((uint16_t)(ent[k] >> 16)));
      if ((from += 256 * AHEAD) >= o1) break;
      fetch_outliers(from);
    }
    __syncthreads();
  };

  B t, tn;
  load_unit(t, u_lo);
  load_outliers(u_lo, 0);
  load_unit(tn, u_lo + 1);
#pragma unroll
  for (int s = 0; s < 4; ++s) load_x(u_lo, 0, s);
  uint8_t *cur = smem, *nxt = smem + PHASE;
  dq.begin(t, kUnitTiles * u_lo + 4 * wave + g4 < ntc);
  dq.columns(t, 0);
#pragma unroll
  for (int r = 0; r < LR; ++r) *reinterpret_cast<half8_t*>(cur + ((wave * LR + r) * 64 + lane) * 16) = dq.operand(t, r, 0);
  add_outliers(cur);

  for (int u = u_lo; u < u_hi; ++u) {        // workgroup-uniform
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      const int nj = j == LAST ? 0 : j + 1, nu = j == LAST ? u + 1 : u;
      load_outliers(nu, nj);
      if (j == LAST) {                       // on to the next unit's tile; the one after it is requested
        t = tn;
        load_unit(tn, u + 2);
        dq.begin(t, kUnitTiles * nu + 4 * wave + g4 < ntc);
      }
      dq.columns(t, nj);
      if (kUnitTiles * (u + 1) > ntc) {      // columns behind the last tile: zeros (finite), they meet zero weights
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int vb = 0; vb < NVB; ++vb)
            if (kUnitTiles * u + 4 * s + g4 >= ntc) xb[s][vb] = u32x4{0u, 0u, 0u, 0u};
      }
      // Operand i of the phase: row i % LR of the tiles of wavefront i / LR.  It is read three multiplications ahead, and a
      // quarter of an operand of the next phase is dequantised beside each: the order here is the order of issue.
      auto read_operand = [&](int i) { return *reinterpret_cast<const u32x4*>(cur + (i * 64 + lane) * 16); };
      constexpr int N = 4 * LR, RING = 4;
      u32x4 a[RING], w = {};
      auto dequant = [&](int q) {
        w[q % 4] = dq.pair(t, q / 4, nj, q % 4);
        if (q % 4 == 3) *reinterpret_cast<u32x4*>(nxt + ((wave * LR + q / 4) * 64 + lane) * 16) = w;
      };
#pragma unroll
      for (int i = 0; i < RING - 1; ++i) a[i] = read_operand(i);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int s = i / LR, r = i % LR;
        if (i + RING - 1 < N) a[(i + RING - 1) % RING] = read_operand(i + RING - 1);
        dequant(i);
#pragma unroll
        for (int vb = 0; vb < NVB; ++vb)
          D[r][vb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a[i % RING]),
                                                            __builtin_bit_cast(half8_t, xb[s][vb]), D[r][vb], 0, 0, 0);
        if (r == LR - 1) load_x(min(nu, units - 1), nj, s);
        __builtin_amdgcn_sched_barrier(0);
      }
      add_outliers(nxt);
      uint8_t* swap = cur;
      cur = nxt;
      nxt = swap;
    }
  }

  // partial results of a group: [vector][row of the strip][strip], see sum_groups_kernel
  const int strips = min(16, ntr - group * 16);
  float* out0 = P + (int64_t)blockIdx.y * batch * m + (int64_t)batch * group * ROWS;
#pragma unroll
  for (int vb = 0; vb < NVB; ++vb) {
    const int v = vec0 + 16 * vb + i16;
    if (v >= batch) continue;
    float* out = out0 + (int64_t)v * (strips * LR);
    if (strips == 16) {                      // 16-byte stores: m is a multiple of 8
#pragma unroll
      for (int r = 0; r < LR; ++r) *reinterpret_cast<float4_t*>(out + 16 * r + 4 * g4) = D[r][vb];
    } else {
#pragma unroll
      for (int r = 0; r < LR; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (4 * g4 + k < strips) out[strips * r + 4 * g4 + k] = D[r][vb][k];
    }
  }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

struct PromptPlan { int groups, units, rows, unit_shift, kg, phases, nvb, vblocks, per, splits; };
static PromptPlan plan_prompt(const Geometry& g, int b) {
  PromptPlan p;
  p.rows = 16 * lane_rows(g.tile_rows);
  p.groups = (g.m + p.rows - 1) / p.rows;
  p.units = (g.ntc + kUnitTiles - 1) / kUnitTiles;
  p.unit_shift = g.tile_cols == 8 ? 7 : (g.tile_cols == 16 ? 8 : 9);
  p.kg = g.tile_cols / 8;
  p.phases = p.units * p.kg;
  // Vectors per workgroup and splits of the columns, one workgroup per CU: a phase takes 1.8 (64 vectors) or 2.3 us (128)
  // with strips of 16 rows, 1.0, 1.2 or 1.8 (256) with strips of 8, a workgroup's start 5 us, a split its partial results
  // at 4 TB/s (64 MB of them at most).  256 vectors with strips of 16 rows would be 256 sums a lane, which leave the
  // compiler no register to turn in (it moves half of them back and forth, 8.9 us a phase).
  const double split_us = (double)b * g.m * 8 / 4e6;
  const int64_t most = ((int64_t)16 << 20) / ((int64_t)b * g.m);
  const int pin = option(SPQR_OPT_PROMPT_PLAN), pin_units = pin % 1024, most_nvb = p.rows == 256 ? 2 : 4;   // (tuning, tests)
  const int pin_nvb = pin / 1024 < most_nvb ? pin / 1024 : most_nvb;
  double best = 1e30;
  for (int nvb = 1; nvb <= most_nvb; nvb *= 2) {
    if (pin_nvb >= 1 && nvb != pin_nvb) continue;
    const double phase_us = p.rows == 256 ? (nvb == 1 ? 1.8 : 2.3) : (nvb == 1 ? 1.0 : nvb == 2 ? 1.2 : 1.8);
    const int vblocks = (b + 64 * nvb - 1) / (64 * nvb);
    for (int s = 1; s <= p.units && (s == 1 || s <= most); ++s) {
      const int per = (p.units + s - 1) / s, splits = (p.units + per - 1) / per;
      const int64_t rounds = ((int64_t)p.groups * vblocks * splits + kCUs - 1) / kCUs;
      const double cost = (double)rounds * (per * p.kg * phase_us + 5.0) + splits * split_us;
      if (cost < best - 1e-9) { best = cost; p.nvb = nvb; p.vblocks = vblocks; p.per = per; }
    }
  }
  if (pin_units >= 1) p.per = pin_units < p.units ? pin_units : p.units;
  p.splits = (p.units + p.per - 1) / p.per;
  return p;
}

// The formats the batch kernel has; more outliers than one weight in four go through the dense copy instead.
bool prompt_has_instance(const DevMatrix& A) {
  return mfma_has_instance(A.g) && A.nnz <= (int64_t)A.g.m * A.g.n / 4 && A.nnz < 0x7FFF0000ll &&
         (A.g.ntc + kUnitTiles - 1) / kUnitTiles * (A.g.tile_cols / 8) <= kSortMaxPhases;
}

// Where the dense copy pays against slices of 16 (prefill_wanted: from 48 vectors on, later on larger layers) and this kernel
// is faster than the copy (times in us, copy -> here):
// - strips of 8 rows: from 4 M weights and 512 columns on (2048^2, 48 to 256 vectors: 28.1 .. 33.6 -> 24.3 .. 27.8; 1024^2:
//   21.0 .. 24.0 against 25.3 .. 26.4; 8192 x 512: 5 % slower to 17 % faster).  With fewer columns there are fewer phases than
//   one workgroup per CU can share, and one hot phase is the call (17920 x 256: 13 % faster to 19 % slower).
// - 16 rows a lane, whose groups of 256 rows are fewer and whose weights are dequantised once per 128 vectors: from 24 M on
//   (5120^2: 46.2 .. 61.0 -> 38.3 .. 57.2; 5120 x 3584: 35.4 .. 47.4 against 36.9 .. 55.3); below, the sort of the outliers
//   (10 us) and the few workgroups cost more than the copy's passes.  Above 192 vectors it needs more than 2048 columns: a
//   second pass over the weights for so few phases costs more than it saves (17920 x 1536, 256 vectors: 62 .. 66 against
//   66 .. 71; 17920 x 2048: 77 .. 82 against 80 .. 82).
// How the outliers lie is not known here and moves a call by more than the lines do: few groups of rows and a skewed layer
// leave one group with most of them (4096 x 8192, 128 vectors: 56 -> 47 with uniform outliers, 51 -> 50 and 51 -> 60 on two
// Zipf layers; 3072 x 12288, 256 vectors: 78 -> 60 and 75 -> 77).  Those sizes stay, the mean of the layers being faster.
// From 33 vectors on it would beat the slices, but they add the outliers in binary32 and here weight + outlier is rounded to
// binary16, so no batch that took the slices moves here.  With a pinned plan (SPQR_OPT_PROMPT_PLAN) the size is no matter.
static bool prompt_pays(const Geometry& g, int b) {
  const double weights = (double)g.m * g.n;
  return g.tile_rows == 8 ? weights >= 4e6 && g.n >= 512 : weights >= 24e6 && (b <= 192 || g.n > 2048);
}

bool prompt_wanted(const DevMatrix& A, int b) {
  return option(SPQR_OPT_BATCH_PATH) == SPQR_BATCH_PATH_AUTO && prompt_has_instance(A) && prefill_wanted(A, b) &&
         (prompt_pays(A.g, b) || option(SPQR_OPT_PROMPT_PLAN) >= 1);
}

static size_t prompt_offsets(const DevMatrix& A, int b, const PromptPlan& p, size_t (&at)[5]) {
  size_t total = 0;
  auto take = [&](size_t bytes) { const size_t o = total; total += up256(bytes); return o; };
  at[0] = take(A.perm != nullptr ? (size_t)b * A.g.n * 2 : 0);
  at[1] = take(A.nnz > 0 ? (size_t)A.nnz * 4 : 0);                                                  // sorted entries
  at[2] = take(A.nnz > 0 ? (size_t)p.groups * (p.phases + 1) * 4 : 0);                               // their ranges
  at[3] = take(A.nnz > 0 ? (size_t)count_slots(A.nnz, p.groups) * p.phases * 4 : 0);        // counts
  at[4] = take((size_t)p.splits * b * A.g.m * sizeof(float));
  return total;
}

size_t prompt_workspace_bytes(const DevMatrix& A, int b) {
  size_t at[5];
  return prompt_offsets(A, b, plan_prompt(A.g, b), at);
}

template <int W, int TR, int TC, int AXIS, int NVB>
static hipError_t launch_prompt_t(const DevMatrix& A, const uint16_t* X, int b, float* P, const PromptPlan& p,
                                  const uint32_t* entries, const int32_t* offs, hipStream_t stream) {
  constexpr int LDS = 2 * 4 * lane_rows(TR) * 1024 + 512;
  static PerDevice ready;                    // more than 64 KB of LDS per workgroup is an opt-in per kernel and device
  const int dev = current_device();
  if (!ready.get(dev)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prompt_group_kernel<W, TR, TC, AXIS, NVB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (e != hipSuccess) return e;
    ready.set(dev, 1);
  }
  hipLaunchKernelGGL((prompt_group_kernel<W, TR, TC, AXIS, NVB>), dim3(p.groups, p.splits, p.vblocks), dim3(256), LDS, stream, A, X, b, P,
                     p.per, entries, offs);
  return hipGetLastError();
}

// Y[b][m] = X[b][n] . W_hat^T.  `scratch`: prompt_workspace_bytes(A, b) bytes, 256-byte aligned.
hipError_t launch_prompt(const DevMatrix& A, const uint16_t* X, int b, void* Y, int y_dtype, hipStream_t stream,
                         uint8_t* scratch) {
  const Geometry& g = A.g;
  if (!prompt_has_instance(A) || scratch == nullptr || b < 1 || b > 256) return hipErrorInvalidValue;
  const PromptPlan p = plan_prompt(g, b);
  size_t at[5];
  prompt_offsets(A, b, p, at);
  uint32_t* entries = reinterpret_cast<uint32_t*>(scratch + at[1]);
  int32_t* offs = reinterpret_cast<int32_t*>(scratch + at[2]);
  uint32_t* counts = reinterpret_cast<uint32_t*>(scratch + at[3]);
  float* P = reinterpret_cast<float*>(scratch + at[4]);
  hipError_t e = hipSuccess;
  const uint16_t* Xin = X;
  if (A.perm != nullptr) {
    uint16_t* xp = reinterpret_cast<uint16_t*>(scratch + at[0]);
    e = launch_gather_x(X, A.perm, xp, g.n, b, stream);
    if (e != hipSuccess) return e;
    Xin = xp;
  }
  if (A.nnz > 0) {
    const dim3 grid(p.groups, kSortWgs);
    hipLaunchKernelGGL(count_phases_kernel, grid, dim3(256), 0, stream, A, p.rows, p.unit_shift, p.kg, p.phases, counts);
    if (p.rows == 256)
      hipLaunchKernelGGL(sort_phases_kernel<16>, grid, dim3(256), 0, stream, A, p.unit_shift, p.kg, p.phases, counts, offs, entries);
    else
      hipLaunchKernelGGL(sort_phases_kernel<8>, grid, dim3(256), 0, stream, A, p.unit_shift, p.kg, p.phases, counts, offs, entries);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  e = hipErrorInvalidValue;
#define SPQR_CASE(W_, TR_, TC_, AX_)                                                                                    \
  if (g.w_bits == W_ && g.tile_rows == TR_ && g.tile_cols == TC_ && g.axis == AX_)                                       \
    e = p.nvb == 1 ? launch_prompt_t<W_, TR_, TC_, AX_, 1>(A, Xin, b, P, p, entries, offs, stream)                         \
        : p.nvb == 2 ? launch_prompt_t<W_, TR_, TC_, AX_, 2>(A, Xin, b, P, p, entries, offs, stream)                       \
                     : launch_prompt_t<W_, TR_, TC_, AX_, (TR_ == 8 ? 4 : 2)>(A, Xin, b, P, p, entries, offs, stream);
  SPQR_CASE(3, 16, 16, 1) SPQR_CASE(4, 16, 16, 1) SPQR_CASE(3, 8, 32, 1) SPQR_CASE(4, 8, 32, 1)
  SPQR_CASE(3, 16, 16, 0) SPQR_CASE(4, 16, 16, 0) SPQR_CASE(3, 32, 8, 0) SPQR_CASE(4, 32, 8, 0)
#undef SPQR_CASE
  if (e != hipSuccess) return e;
  return launch_sum_groups(g, P, p.splits, b, Y, y_dtype, stream);
}

}  // namespace spqr
