// The sweep (Alg. 1, lines 4-20) with 16 rows per workgroup, for beta2 <= 16.  Included by spqr_encode.hip, contraction off.
//
// A workgroup of 8 wavefronts owns 16 rows and goes through super-blocks of 128 columns, whose weights and corner of H^ic stay in
// LDS.  The steps inside a block of beta1 columns depend on one another, the columns right of the super-block (line 16, the
// O(m n^2) part) only on its errors, so the two run side by side:
//   front   wavefronts 0-3 (one on each SIMD): per block, all four bring its columns up to date and test for outliers, 4 rows
//           each; then wavefront 0 fits the second level and takes the columns in order, while 1 gives the block before it to the rest
//           of the super-block and writes its results and 2 and 3 keep the next super-block's columns in registers and give them
//           the errors of this one and of the one before.  They meet at a barrier of their own.
//   far     wavefronts 4-7, and the front's when they are through with the super-block: the errors of the super-block BEFORE
//           applied to everything right of the next one, in tasks out of a queue.
// Same operations in the same order on every weight as sweep_kernel, hence the same bits.
//
// 4096^2, blocks of 16, 1.3 % outliers: 3.5 ms (6.6 with the far columns after the chain instead of beside it, true divisions
// everywhere and B1 + 1 fits a test).  Clocks of a workgroup, of 7.4 M when they were taken (3.65 ms): the front has 4.6 (a block of 16 columns: tests 4400, chain
// with the second level 7300, the meetings and what wavefronts 2 and 3 are late 4300), the far columns alone after it 2.2, the end of
// a super-block 0.4.  Bound: binary64 issue.  The products and differences of the feedback are 3.6 M clocks of a SIMD at 3.7 ns a pair
// (two wavefronts, 256 CUs), the tests 0.9, chain or near columns 1.1: three quarters of the time; what is left is the chain
// where the far columns are few, and the last task of every super-block.
#pragma once

namespace spqr_enc {

typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kRows16 = 16, kWaves16 = 8, kFront16 = 4, kSuper16 = 128;

// ---------------------------------------------------------------------------
// a / b correctly rounded with a prepared divisor: Markstein's final step (IBM J. Res. Dev. 34, 1990) on a quotient that the
// reciprocal in two parts makes faithful (Brisebarre, Muller, Raina, IEEE Trans. Comput. 53, 2004).  Four dependent operations
// where the division instruction sequence has a dozen; holds while nothing under- or overflows: |b| in [2^-100, 2^100], |a| in
// [2^-300, 2^300], or a zero (whose sign may be lost).  Callers check and fall back on a / b.
// ---------------------------------------------------------------------------
struct Divisor { double b, hi, lo; };
__device__ __forceinline__ Divisor divisor_of(double b) {
  const double hi = 1.0 / b;
  return {b, hi, __builtin_fma(-hi, b, 1.0) * hi};
}
__device__ __forceinline__ double divide(double a, const Divisor& d) {
  const double q = __builtin_fma(a, d.hi, a * d.lo);
  return __builtin_fma(__builtin_fma(-q, d.b, a), d.hi, q);
}
__device__ __forceinline__ bool divisor_in_range(double b) { return __builtin_fabs(b) >= 0x1p-100 && __builtin_fabs(b) <= 0x1p100; }
constexpr double kDivTop = 0x1p300, kDivLow = 0x1p-300;
// fit_from_range(): the scale, true where the range allows divide() (a range of 0 gives the scale 1 either way).
__device__ __forceinline__ bool scale_of_range(double lo, double hi, const Divisor& levels, double* s) {
  const double range = hi - lo, sc = divide(range, levels);
  *s = sc == 0.0 ? 1.0 : sc;
  return range <= kDivTop && (range >= kDivLow || range == 0.0);
}

// Values the compiler may not derive anything from before this point: what a phase computes from them (addresses above all) is not
// kept in registers through the others (which spilled 130 registers).
__device__ __forceinline__ int fresh_s(int v) { asm volatile("" : "+s"(v)); return v; }
__device__ __forceinline__ int fresh_v(int v) { asm volatile("" : "+v"(v)); return v; }

// Doubles by a uniform base and row and a lane's offset in bytes (no addresses in vector registers).  The row's offset is not part of a
// buffer's bounds check: rows and columns that may lie behind the last ones are held back by the callers.
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer_of(const double* base, size_t count) {
  const size_t bytes = count * sizeof(double);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(base), 0, (int)(uint32_t)(bytes < 0xFFFFFFF8u ? bytes : 0xFFFFFFF8u), 0x00027000);
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double buffer_f64(Buffer b, int off, int row_off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, off, row_off, 0));
}
__device__ __forceinline__ void buffer_put_f64(double v, Buffer b, int off, int row_off) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, off, row_off, 0);
}

template <int... I, class F> __device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }

// A double of another lane of the same 16 (DPP).
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kDppRor = 0x120, kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int dpp_quad(int k) { return k * 0x55; }

// Minimum and maximum over the row's 16 lanes.
__device__ __forceinline__ double row_min(double v) {
  v = fmin(v, dpp_f64<kDppRor + 8>(v)); v = fmin(v, dpp_f64<kDppRor + 4>(v));
  v = fmin(v, dpp_f64<kDppRor + 2>(v)); return fmin(v, dpp_f64<kDppRor + 1>(v));
}
__device__ __forceinline__ double row_max(double v) {
  v = fmax(v, dpp_f64<kDppRor + 8>(v)); v = fmax(v, dpp_f64<kDppRor + 4>(v));
  v = fmax(v, dpp_f64<kDppRor + 2>(v)); return fmax(v, dpp_f64<kDppRor + 1>(v));
}
// ... over the 15 others: runs of 1, 2, 4 and 8 lanes, then two of eight that overlap.
__device__ __forceinline__ double others_min(double v) {
  v = dpp_f64<kDppRor + 1>(v);
  v = fmin(v, dpp_f64<kDppRor + 1>(v)); v = fmin(v, dpp_f64<kDppRor + 2>(v));
  v = fmin(v, dpp_f64<kDppRor + 4>(v)); return fmin(v, dpp_f64<kDppRor + 7>(v));
}
__device__ __forceinline__ double others_max(double v) {
  v = dpp_f64<kDppRor + 1>(v);
  v = fmax(v, dpp_f64<kDppRor + 1>(v)); v = fmax(v, dpp_f64<kDppRor + 2>(v));
  v = fmax(v, dpp_f64<kDppRor + 4>(v)); return fmax(v, dpp_f64<kDppRor + 7>(v));
}

// second_level() on 16 lanes, beta2 of them a tile.
__device__ __forceinline__ void second_level16(double v, int beta2, double levels, double* hat, uint8_t* code, uint16_t* s2_bits,
                                               uint16_t* z2_bits) {
  double lo = v, hi = v;
  lo = fmin(lo, dpp_f64<kDppXor1>(lo)); hi = fmax(hi, dpp_f64<kDppXor1>(hi));
  if (beta2 > 2) { lo = fmin(lo, dpp_f64<kDppXor2>(lo)); hi = fmax(hi, dpp_f64<kDppXor2>(hi)); }
  if (beta2 > 4) { lo = fmin(lo, dpp_f64<kDppHalfMirror>(lo)); hi = fmax(hi, dpp_f64<kDppHalfMirror>(hi)); }
  if (beta2 > 8) { lo = fmin(lo, dpp_f64<kDppMirror>(lo)); hi = fmax(hi, dpp_f64<kDppMirror>(hi)); }
  second_level_of_range(v, lo, hi, levels, hat, code, s2_bits, z2_bits);
}

// ---------------------------------------------------------------------------
// LDS.
// ---------------------------------------------------------------------------
// The corner of H^ic: for each block of B1 rows the columns from its own diagonal on, block after block.
template <int B1> struct Sweep16Lds {
  double esb[2][kSuper16][kRows16];                      // errors E of this super-block's columns and of the one before
  double wsb[kSuper16][kRows16 + 1];                     // this one's weights (the 1: banks)
  double corner[(kSuper16 / B1 + 1) * kSuper16 * B1 / 2];
  f64x2 diag[kSuper16];                                  // its diagonal as divisors: hi, lo
  double t[3][kRows16][B1 + 1];                          // squared errors of the tests: whole group, without its minimum, without its maximum
  double s1[kRows16], z1[kRows16];                       // first-level statistics of the current block
  double s_hat[2][kRows16], z_hat[2][kRows16];           // de-quantised ones, of this block and the one before
  uint32_t om[2][kRows16];                               // outliers
  uint32_t q[2][kRows16][B1 / 4];                        // codes, four to a word
  uint32_t met, ready, task[2], diag_bad[2];             // the last two by the parity of the super-block
};
template <int B1> constexpr int corner_at(int g) { return B1 * (g * kSuper16 - B1 * (g * (g - 1) / 2)); }   // block g's rows of kSuper16 - g B1
static_assert(corner_at<16>(kSuper16 / 16) == (kSuper16 / 16 + 1) * kSuper16 * 16 / 2, "all of the blocks");

__device__ __forceinline__ void wait_for(uint32_t* count, uint32_t target) {
  while ((int32_t)(__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - target) < 0) __builtin_amdgcn_s_sleep(0);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// The front's wavefronts meet.  All kFront16 of them are resident and come here equally often, so every wait ends.
__device__ __forceinline__ void meet(uint32_t* met, uint32_t* target, int lane) {
  *target += kFront16;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane == 0) __hip_atomic_fetch_add(met, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  wait_for(met, *target);
}

// ---------------------------------------------------------------------------
// Far: line 16 for C runs of 64 columns from k0 on, ROWS of the workgroup's rows from r0 on: W[:, k] = src[:, k] - E[:, j] * H^ic[ub + j, k] for
// the kSuper16 columns j of a super-block, in order.  A lane holds ROWS rows of C columns; the errors are LDS broadcasts (for 16
// rows eight reads of 16 bytes per column j whatever C is: with one column a lane they are what the pass waits for, two are even with
// the arithmetic), three reads ahead; H^ic comes straight from memory, four j ahead.
// ---------------------------------------------------------------------------
template <int C, int ROWS>
__device__ __forceinline__ void far_feedback(const double* src, double* W, const double* __restrict__ U, int n, int row0, int rows, int lane,
                                             int ub, int k0, int r0, const double (*esb)[kRows16]) {
  constexpr int PF = 4;                                  // (kSuper16 is a multiple of 2 PF)
  const int off = (k0 + lane) * 8, pitch = n * 8;        // columns behind the last one: the next row's of H^ic (there is one), the last one's of W
  double cur[C][ROWS], u[2][PF][C];
  const size_t u_end = (size_t)n * n;
  auto fetch = [&](int buf, int j) {                     // rows ub + j .. + PF - 1 of H^ic
    const size_t first = (size_t)(ub + j) * n;
    const auto rows_j = buffer_of(U + first, u_end - first);
#pragma unroll
    for (int q = 0; q < PF; ++q)
#pragma unroll
      for (int c = 0; c < C; ++c) u[buf][q][c] = buffer_f64(rows_j, off + 512 * c, q * pitch);
  };
  fetch(0, 0);
  const size_t w_first = (size_t)row0 * n;
  const auto w_rows = buffer_of(src + w_first, (size_t)rows * n);
#pragma unroll
  for (int r = 0; r < ROWS; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) cur[c][r] = buffer_f64(w_rows, min(off + 512 * c, pitch - 8), min(r0 + r, rows - 1) * pitch);
  constexpr int AHEAD = 3, PAIRS = ROWS / 2;             // the last ones read behind the errors, into what follows them in LDS
  const double* pe = &esb[0][r0];
  auto pair = [&](int t) { return *reinterpret_cast<const f64x2*>(pe + t / PAIRS * kRows16 + t % PAIRS * 2); };
  f64x2 e[AHEAD + 1];
#pragma unroll
  for (int t = 0; t < AHEAD; ++t) e[t] = pair(t);
#pragma unroll 1
  for (int j = 0; j < kSuper16; j += 2 * PF) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      fetch(half ^ 1, min(j + PF * (half + 1), kSuper16 - PF));      // behind the last four: the same ones again, unused
#pragma unroll
      for (int t = 0; t < PF * PAIRS; ++t) {
        const int h = t % PAIRS, q = t / PAIRS;
        e[(t + AHEAD) % (AHEAD + 1)] = pair(t + AHEAD);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          cur[c][2 * h] = cur[c][2 * h] - e[t % (AHEAD + 1)].x * u[half][q][c];
          cur[c][2 * h + 1] = cur[c][2 * h + 1] - e[t % (AHEAD + 1)].y * u[half][q][c];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      pe += PF * kRows16;
    }
  }
  rows = fresh_s(rows);
  const auto w_out = buffer_of(W + w_first, (size_t)rows * n);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    if (k0 + 64 * c + lane < n) {
#pragma unroll
      for (int r = 0; r < ROWS; ++r)
        if (r0 + r < rows) buffer_put_f64(cur[c][r], w_out, off + 512 * c, (r0 + r) * pitch);
    }
  }
}

template <int ROWS>
__device__ __forceinline__ void far_task(int runs, const double* src, double* W, const double* __restrict__ U, int n, int row0, int rows,
                                         int lane, int ub, int k0, int r0, const double (*esb)[kRows16]) {
  switch (runs) {
    case 1: far_feedback<1, ROWS>(src, W, U, n, row0, rows, lane, ub, k0, r0, esb); break;
    case 2: far_feedback<2, ROWS>(src, W, U, n, row0, rows, lane, ub, k0, r0, esb); break;
    case 3: far_feedback<3, ROWS>(src, W, U, n, row0, rows, lane, ub, k0, r0, esb); break;
    default: far_feedback<4, ROWS>(src, W, U, n, row0, rows, lane, ub, k0, r0, esb); break;
  }
}

// ---------------------------------------------------------------------------
// Front.
// ---------------------------------------------------------------------------
// The block at column ib of the super-block: the block before it gives its feedback to these columns; outliers() (line 8); fit_statistics()'
// first level (line 9).  A wavefront has rows 4 wave .. 4 wave + 3, 16 lanes each, a lane the columns c0 + 16 k.
//
// A group without one of its weights has another range only if that weight alone is the minimum or the maximum: of the B1 + 1 fits
// of a row at most three differ, and the errors under them are each computed once, by the lane of their column (B1 times fewer
// divisions).  The sums add them in column order, without the left-out one, as ever.
template <int B1>
__device__ __forceinline__ void block_tests(Sweep16Lds<B1>& S, const SweepArgs& a, const Divisor& levels, int ib, int par, int p, int wave, int lane, const double (*esb)[kRows16]) {
  constexpr int LC = B1 < 16 ? B1 : 16, K = B1 / LC;
  const int row = lane >> 4, r = 4 * wave + row, cl = lane & 15, c0 = min(cl, LC - 1);
  const bool valid = cl < LC;
  const int width = kSuper16 - ib;
  const double* ublk = S.corner + corner_at<B1>(ib / B1);
  double v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = S.wsb[ib + c0 + 16 * k][r];
  if (ib > 0) {
    const double* up = S.corner + corner_at<B1>(ib / B1 - 1) + B1 + c0;
#pragma unroll
    for (int j = 0; j < B1; ++j) {
      const double e = esb[ib - B1 + j][r];
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = v[k] - e * up[j * (width + B1) + 16 * k];
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (valid) S.wsb[ib + c0 + 16 * k][r] = v[k];
  }
  uint32_t om = 0;
  if (a.tau < INFINITY) {
    double pmin = INFINITY, pmax = -INFINITY;            // of this lane's columns
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (valid) { pmin = fmin(pmin, v[k]); pmax = fmax(pmax, v[k]); }
    const double omin = others_min(pmin), omax = others_max(pmax), lo = fmin(omin, pmin), hi = fmax(omax, pmax);
    double lo_x[K], hi_x[K], lo2 = lo, hi2 = hi;         // without column c0 + 16 k; the second smallest and largest
#pragma unroll
    for (int k = 0; k < K; ++k) {
      lo_x[k] = omin; hi_x[k] = omax;
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (j != k) { lo_x[k] = fmin(lo_x[k], v[j]); hi_x[k] = fmax(hi_x[k], v[j]); }
      if (valid) { lo2 = fmax(lo2, lo_x[k]); hi2 = fmin(hi2, hi_x[k]); }
    }
    lo2 = row_max(lo2); hi2 = row_min(hi2);
    // lane 4 i + f of a row fits range f, and hands it to its neighbours
    const double flo = (lane & 3) == 1 ? lo2 : lo;
    double s;
    bool bad = !scale_of_range(flo, (lane & 3) == 2 ? hi2 : hi, levels, &s) || !divisor_in_range(s);
    const Divisor ds = divisor_of(s);
    const double z = divide(-flo, ds);
    double e[3][K];
    auto errors = [&](auto F) {
      constexpr int f = decltype(F)::value;
      const Divisor d = {dpp_f64<dpp_quad(f)>(ds.b), dpp_f64<dpp_quad(f)>(ds.hi), dpp_f64<dpp_quad(f)>(ds.lo)};
      const double zf = dpp_f64<dpp_quad(f)>(z);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int c = c0 + 16 * k;
        const double q = fmin(fmax(floor(divide(v[k], d) + zf + 0.5), 0.0), a.w_top);
        const double x = v[k] - d.b * (q - zf), ax = __builtin_fabs(x);
        bad = bad || !(__builtin_fabs(v[k]) <= kDivTop) || !(ax <= kDivTop) || (ax < kDivLow && x != 0.0);
        const double y = divide(x, {ublk[c * width + c], S.diag[ib + c].x, S.diag[ib + c].y});
        e[f][k] = y * y;
      }
    };
    auto share = [&](int f) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (valid) S.t[f][r][c0 + 16 * k] = e[f][k];
    };
    double base = 0.0, own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) own[k] = 0.0;
    errors(std::integral_constant<int, 0>{});
    bool exact = __any(bad) || S.diag_bad[p];            // wave-uniform, as what follows
    if (!exact) {
      share(0);
#pragma unroll
      for (int c = 0; c < B1; ++c) base = base + S.t[0][r][c];
      if (__any(!(base <= a.tau))) {                     // otherwise no difference exceeds tau: the errors left are not negative
        errors(std::integral_constant<int, 1>{});
        errors(std::integral_constant<int, 2>{});
        exact = __any(bad);
        share(1); share(2);
        const double* mine[K];
#pragma unroll
        for (int k = 0; k < K; ++k) mine[k] = S.t[lo_x[k] != lo ? 1 : hi_x[k] != hi ? 2 : 0][r];
#pragma unroll
        for (int c = 0; c < B1; ++c)
#pragma unroll
          for (int k = 0; k < K; ++k) own[k] = own[k] + (c != c0 + 16 * k ? mine[k][c] : 0.0);   // sums of squares: + 0 changes none
      }
    }
    if (exact) {                                         // out of the range of divide(): each test as the algorithm says it
      auto group_error = [&](int x) {
        double l = INFINITY, h = -INFINITY;
        for (int c = 0; c < B1; ++c) {
          const double w = S.wsb[ib + c][r];
          if (c != x) { l = fmin(l, w); h = fmax(h, w); }
        }
        double sx, zx, t = 0.0;
        fit_from_range(l, h, a.w_top, &sx, &zx);
        for (int c = 0; c < B1; ++c) {
          const double w = S.wsb[ib + c][r];
          const double y = (w - sx * (quantize(w, sx, zx, a.w_top) - zx)) / ublk[c * width + c];
          t = c != x ? t + y * y : t;
        }
        return t;
      };
      base = group_error(-1);
#pragma unroll
      for (int k = 0; k < K; ++k) own[k] = group_error(c0 + 16 * k);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint64_t vote = __ballot(valid && (base - own[k]) > a.tau);
      om |= ((uint32_t)(vote >> (16 * row)) & 0xFFFFu) << (16 * k);
    }
  }
  double lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (valid && !((om >> (c0 + 16 * k)) & 1u)) { lo = fmin(lo, v[k]); hi = fmax(hi, v[k]); }
  lo = row_min(lo); hi = row_max(hi);
  if (lo > hi) { lo = 0.0; hi = 0.0; }                   // nothing left
  double s1, z1;
  if (__all(scale_of_range(lo, hi, levels, &s1))) z1 = -lo / s1;
  else fit_from_range(lo, hi, a.w_top, &s1, &z1);
  if (cl == 0) { S.s1[r] = s1; S.z1[r] = z1; S.om[par][r] = om; }
}

// Lines 10-15 for HB columns from h0 of the block on, one after the other, by one wavefront: a lane per row, the four groups of 16
// lanes do the same.  16 columns in registers at a time (32 of them spill): a second half first takes the errors of the first, in
// the order of the columns, which is the order line 14 gives it.  False where divide() does not hold: wsb, where the columns start
// from, is only written at the end, and the block is taken again by block_columns_exact().
//
// What bounds it is the chain of 19 dependent operations a column, and the wavefront is alone on it: the order of the instructions
// is fixed by hand.  Between a column's steps stand the updates that the column before owes to the later ones (its own successor
// got its update at once), and the LDS reads of the next column's row of H^ic.  (As the compiler orders it, every column first takes
// the updates of all columns before it, one after the other, and then waits for its reads: 11200 clocks a block of 16 columns
// with the second level, 7300 so.)
//
// An error of exactly 0, of a row of zeros or of weights that their codes meet, stays on this path, its sign set by hand: 4096^2 with a
// row of zeros in every workgroup 3.5 ms, as without, 5.1 when zeros were taken again with true divisions.
template <int B1>
__device__ __forceinline__ bool block_columns(Sweep16Lds<B1>& S, double w_top, int ib, int h0, int par, int lane, double s_hat, double z_hat,
                                              double (*esb)[kRows16]) {
  constexpr int HB = B1 < 16 ? B1 : 16;
  const int r = lane & 15, width = kSuper16 - ib;
  const double* ublk = S.corner + corner_at<B1>(ib / B1) + h0;
  const f64x2* diag = S.diag + ib + h0;
  const int kept = (int)~(S.om[par][r] >> h0);
  const Divisor ds = divisor_of(s_hat);
  // of |x|: its high word, the lowest bit set where the low word is not 0, less 1: a zero is -1, the largest unsigned and the least signed
  uint32_t lowest = divisor_in_range(s_hat) ? ~0u : 0u;
  int highest = -1;
  const uint32_t one = (uint32_t)fresh_s(1);             // (min with a constant 1 becomes a comparison, a wait and a selection)
  constexpr uint32_t kLow = (1023u - 300u) << 20, kHigh = (1023u + 299u) << 20;      // 2^299: then v is below 2^300 too (s_hat (q - z_hat) is small)
  double w[HB];
#pragma unroll
  for (int c = 0; c < HB; ++c) w[c] = S.wsb[ib + h0 + c][r];
#pragma unroll 1
  for (int j = 0; j < h0; ++j) {
    const double ej = esb[ib + j][r];
#pragma unroll
    for (int k = 0; k < HB; ++k) w[k] = w[k] - ej * ublk[j * width + k];
  }
  ublk += h0 * width;
  f64x2 u[3][HB / 2], div[2];                            // rows c - 1, c, c + 1 of H^ic, their columns from the diagonal on; hi, lo
  auto read_row = [&](int c, int h) {                     // (no half that nobody uses: its registers would be given away with the read in flight)
    if (2 * h >= c) u[c % 3][h] = *reinterpret_cast<const f64x2*>(ublk + c * width + 2 * h);
    else if (2 * h + 1 >= c) u[c % 3][h].y = ublk[c * width + 2 * h + 1];
  };
  auto at = [&](int c, int k) { return u[c % 3][k / 2][k % 2]; };      // (c + 2 for c - 1)
#pragma unroll
  for (int h = 0; h < HB / 2; ++h) read_row(0, h);
  div[0] = diag[0];
  uint32_t qs[HB / 4];
#pragma unroll
  for (int k = 0; k < HB / 4; ++k) qs[k] = 0;
  double before = 0.0, prod[2];                          // E of the column before
  __builtin_amdgcn_sched_barrier(0);
  unrolled(std::make_integer_sequence<int, HB>{}, [&](auto column) __attribute__((always_inline)) {
    constexpr int c = decltype(column)::value;
    // the updates column c - 1 owes: to itself (its final weight) and to the columns from c + 1 on; products one ahead of differences
    constexpr int owed = c == 0 ? 0 : HB - c;
    int op = 0, next = c / 2;
    auto column_of = [&](int i) { return i == 0 ? c - 1 : c + i; };
    auto fill = [&]() {
      if (op < 2 * owed) {
        if (op == 0 || (op % 2 == 1 && op < 2 * owed - 1)) {
          const int i = (op + 1) / 2;
          prod[i % 2] = before * at(c + 2, column_of(i));
        } else {
          const int i = op == 2 * owed - 1 ? owed - 1 : op / 2 - 1;
          w[column_of(i)] = w[column_of(i)] - prod[i % 2];
        }
        ++op;
      }
    };
    auto read_next = [&]() {
      if (c + 1 < HB && next < HB / 2) read_row(c + 1, next++);
    };
#define SPQR_STEP(...) __VA_ARGS__; read_next(); fill(); fill(); __builtin_amdgcn_sched_barrier(0)
    if (c + 1 < HB) div[(c + 1) % 2] = diag[c + 1];
    const double v = w[c], hi = div[c % 2].x, lo = div[c % 2].y;
    SPQR_STEP(double t = v * ds.lo);
    SPQR_STEP(t = __builtin_fma(v, ds.hi, t));
    SPQR_STEP(double d = __builtin_fma(-t, ds.b, v));
    SPQR_STEP(t = __builtin_fma(d, ds.hi, t));
    SPQR_STEP(t = t + z_hat);
    SPQR_STEP(t = t + 0.5);
    SPQR_STEP(t = floor(t));
    SPQR_STEP(t = fmax(t, 0.0));
    SPQR_STEP(const double q = fmin(t, w_top));
    SPQR_STEP(d = q - z_hat);
    SPQR_STEP(d = s_hat * d);
    SPQR_STEP(const double x = v - d);
    SPQR_STEP(t = x * lo);
    SPQR_STEP(t = __builtin_fma(x, hi, t));
    const uint32_t high = (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32), low = (uint32_t)__builtin_bit_cast(uint64_t, x);
    const uint32_t size = ((high & 0x7FFFFFFFu) | min(low, one)) - 1u;
    const uint32_t sign = (high ^ (uint32_t)(__builtin_bit_cast(uint64_t, hi) >> 32)) & 0x80000000u;    // (divide() may lose a zero's)
    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe(kept, c, 1);
    SPQR_STEP(d = __builtin_fma(-t, at(c, c), x));
    SPQR_STEP(t = __builtin_fma(d, hi, t));
    lowest = min(lowest, size);
    highest = max(highest, (int)size);
    qs[c / 4] |= (uint32_t)q << (8 * (c % 4));
    const uint64_t tb = __builtin_bit_cast(uint64_t, t);
    const uint32_t ec_low = (uint32_t)tb & keep, ec_high = ((uint32_t)(tb >> 32) & keep & 0x7FFFFFFFu) | sign;
    SPQR_STEP(const double ec = __builtin_bit_cast(double, (uint64_t)ec_high << 32 | ec_low));
    esb[ib + h0 + c][r] = ec;                            // (the same from all four groups)
#pragma unroll
    for (int rest = 0; rest < 2 * owed; ++rest) fill();
    if constexpr (c + 1 < HB) { SPQR_STEP(d = ec * at(c, c + 1)); SPQR_STEP(w[c + 1] = w[c + 1] - d); }
    else w[c] = w[c] - ec * at(c, c);
    before = ec;
#undef SPQR_STEP
  });
  if (__any(lowest < kLow || highest > (int)kHigh)) return false;
  if (lane < kRows16) {
#pragma unroll
    for (int k = 0; k < HB / 4; ++k) S.q[par][r][h0 / 4 + k] = qs[k];
#pragma unroll
    for (int c = 0; c < HB; ++c) S.wsb[ib + h0 + c][r] = w[c];
  }
  return true;
}
// The same with true divisions, in LDS.
template <int B1>
__device__ __forceinline__ void block_columns_exact(Sweep16Lds<B1>& S, double w_top, int ib, int h0, int par, int lane, double s_hat, double z_hat,
                                                    double (*esb)[kRows16]) {
  const int r = lane & 15, width = kSuper16 - ib, end = min(B1, h0 + 16);
  const double* ublk = S.corner + corner_at<B1>(ib / B1);
  const uint32_t om = S.om[par][r];
  if (lane >= kRows16) return;
#pragma unroll 1
  for (int j = 0; j < h0; ++j)
#pragma unroll 1
    for (int k = h0; k < end; ++k) S.wsb[ib + k][r] = S.wsb[ib + k][r] - esb[ib + j][r] * ublk[j * width + k];
  uint32_t qs = 0;
#pragma unroll 1
  for (int c = h0; c < end; ++c) {
    const double v = S.wsb[ib + c][r];
    const double q = quantize(v, s_hat, z_hat, w_top);
    const double ec = (v - s_hat * (q - z_hat)) / ublk[c * width + c] * ((om >> c) & 1u ? 0.0 : 1.0);
    esb[ib + c][r] = ec;
#pragma unroll 1
    for (int k = c; k < end; ++k) S.wsb[ib + k][r] = S.wsb[ib + k][r] - ec * ublk[c * width + k];
    qs |= (uint32_t)(uint8_t)q << (8 * (c % 4));
    if (c % 4 == 3) { S.q[par][r][c / 4] = qs; qs = 0; }
  }
}

// fit_statistics()' second level, both statistics at once (16 lanes each), and the block's columns.
template <int B1>
__device__ __forceinline__ void block_chain(Sweep16Lds<B1>& S, const SweepArgs& a, int ib, int g, int par, int p, int lane, int row0, int rows,
                                            double (*esb)[kRows16]) {
  const int r = lane & 15;
  const bool zero = lane & 16;
  double hat;
  uint8_t code;
  uint16_t s2, z2;
  second_level16(zero ? S.z1[r] : S.s1[r], a.beta2, zero ? a.z_top : a.s_top, &hat, &code, &s2, &z2);
  if (lane < 32 && r < rows) {
    const int row = row0 + r, ng = a.n / B1;
    (zero ? a.out.z_q : a.out.s_q)[(size_t)row * ng + g] = code;
    if (row % a.beta2 == 0) {
      const size_t t = (size_t)(row / a.beta2) * ng + g;
      (zero ? a.out.s_z : a.out.s_s)[t] = s2;
      (zero ? a.out.z_z : a.out.z_s)[t] = z2;
    }
  }
  if (lane < 32) (zero ? S.z_hat : S.s_hat)[par][r] = hat;
  const double s_hat = S.s_hat[par][r], z_hat = S.z_hat[par][r];
#pragma unroll 1
  for (int h0 = 0; h0 < B1; h0 += 16)
    if (S.diag_bad[p] || !block_columns<B1>(S, a.w_top, ib, h0, par, lane, s_hat, z_hat, esb))
      block_columns_exact<B1>(S, a.w_top, ib, h0, par, lane, s_hat, z_hat, esb);
}

// The block at ib, whose columns are done: its feedback to the super-block's columns behind the block after it (that one takes it in its
// own tests), a thread per pair of columns of a row.  Threads t of `threads`.
template <int B1>
__device__ __forceinline__ void block_feedback(Sweep16Lds<B1>& S, int ib, int sbw, int t, int threads, const double (*esb)[kRows16]) {
  const int r = t & 15, width = kSuper16 - ib;
  const double* ublk = S.corner + corner_at<B1>(ib / B1) - ib;
  constexpr int HB = B1 < 16 ? B1 : 16;
#pragma unroll 1
  for (int h = 0; h < B1; h += HB) {
    double e[HB];
#pragma unroll
    for (int j = 0; j < HB; ++j) e[j] = esb[ib + h + j][r];
#pragma unroll 1
    for (int k = ib + 2 * B1 + 2 * (t >> 4); k < sbw; k += threads / 8) {
      double w0 = S.wsb[k][r], w1 = S.wsb[k + 1][r];
#pragma unroll
      for (int j = 0; j < HB; ++j) {
        const f64x2 u = *reinterpret_cast<const f64x2*>(&ublk[(h + j) * width + k]);
        w0 = w0 - e[j] * u.x;
        w1 = w1 - e[j] * u.y;
      }
      S.wsb[k][r] = w0;
      S.wsb[k + 1][r] = w1;
    }
  }
}
// Wavefronts 1 to 3 for many columns, 2 and 3 have nothing else to do then; 1 alone for few.
__device__ __forceinline__ int feedback_threads(int columns) { return columns > 48 ? 64 * 3 : 64; }
// Its codes, outliers and their values, by one wavefront.
template <int B1>
__device__ __forceinline__ void block_results(const Sweep16Lds<B1>& S, const SweepArgs& a, int ib, int sb, int par, int lane, int row0, int rows) {
  const int r = lane & 15;
  const double s_hat = S.s_hat[par][r], z_hat = S.z_hat[par][r];
  const uint32_t om = S.om[par][r];
  for (int c = 4 * (lane >> 4); c < B1; c += 16) {
    if (r >= rows) continue;
    const uint32_t q = S.q[par][r][c / 4];
    uint32_t mask = 0, val[2] = {0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if ((om >> (c + k)) & 1u) {
        mask |= 1u << (8 * k);
        val[k / 2] |= (uint32_t)f64_to_f16_bits(S.wsb[ib + c + k][r] - s_hat * ((double)((q >> (8 * k)) & 0xFFu) - z_hat)) << (16 * (k % 2));
      }
    }
    const size_t at = (size_t)(row0 + r) * a.n + sb + ib + c;
    *reinterpret_cast<uint32_t*>(a.out.Q + at) = q;
    *reinterpret_cast<uint32_t*>(a.out.outlier_mask + at) = mask;
    reinterpret_cast<uint32_t*>(a.out.outlier_val + at)[0] = val[0];
    reinterpret_cast<uint32_t*>(a.out.outlier_val + at)[1] = val[1];
  }
}

// The next super-block's columns on their way: a wavefront has 64 of them, a lane one, all 16 rows; they take this super-block's errors,
// steps 0 .. 127, as its blocks are done.
struct Near {
  static constexpr int PF = 8;
  double cur[kRows16], u[PF];
  int done;
};
__device__ __forceinline__ void near_fetch(double (&u)[Near::PF], const double* __restrict__ U, int n, int row, int off) {
  const size_t first = (size_t)row * n;
  const Buffer b = buffer_of(U + first, (size_t)n * n - first);
#pragma unroll
  for (int q = 0; q < Near::PF; ++q) u[q] = buffer_f64(b, off, q * n * 8);
}
__device__ __forceinline__ void near_steps(Near& N, const double* __restrict__ U, int n, int sb, int off, int limit, const double (*esb)[kRows16]) {
#pragma unroll 1
  for (; N.done < limit; N.done += Near::PF) {
    double un[Near::PF];
    near_fetch(un, U, n, sb + min(N.done + Near::PF, kSuper16 - Near::PF), off);
    const double* pe = &esb[N.done][0];
    constexpr int AHEAD = 7, PAIRS = kRows16 / 2;        // (one wavefront a SIMD: nobody else hides the reads)
    f64x2 e[AHEAD + 1];
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) e[t] = *reinterpret_cast<const f64x2*>(pe + 2 * t);
#pragma unroll
    for (int t = 0; t < Near::PF * PAIRS; ++t) {
      const int h = t % PAIRS;
      if (t + AHEAD < Near::PF * PAIRS) e[(t + AHEAD) % (AHEAD + 1)] = *reinterpret_cast<const f64x2*>(pe + 2 * (t + AHEAD));
      N.cur[2 * h] = N.cur[2 * h] - e[t % (AHEAD + 1)].x * N.u[t / PAIRS];
      N.cur[2 * h + 1] = N.cur[2 * h + 1] - e[t % (AHEAD + 1)].y * N.u[t / PAIRS];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < Near::PF; ++q) N.u[q] = un[q];
  }
}

// The next super-block's columns of the weights, as the passes before left them.
__device__ __forceinline__ void near_weights(Near& N, const double* src, int n, int row0, int rows, int off) {
  const Buffer b = buffer_of(src + (size_t)row0 * n, (size_t)rows * n);
  off = min(off, (n - 1) * 8);
#pragma unroll
  for (int r = 0; r < kRows16; ++r) N.cur[r] = buffer_f64(b, off, min(r, rows - 1) * n * 8);
}

// ROWS rows j0, j0 + step, .. of the corner of H^ic at column `at`, on their way into LDS (behind the last row and column: the last
// ones, never used).
template <int ROWS> struct CornerRows { double v[ROWS][2]; };
template <int ROWS>
__device__ __forceinline__ void fetch_corner(CornerRows<ROWS>& c, const double* __restrict__ U, int n, int at, int j0, int step, int lane) {
  const int left = n - 1 - at, first = at + min(j0, left);
  const Buffer b = buffer_of(U + (size_t)first * n, (size_t)(n - first) * n);
  const int col = at + min(lane, left), col64 = at + min(64 + lane, left);
#pragma unroll
  for (int t = 0; t < ROWS; ++t) {
    const int row_off = (min(at + j0 + step * t, n - 1) - first) * n * 8;
    c.v[t][0] = buffer_f64(b, col * 8, row_off);
    c.v[t][1] = buffer_f64(b, col64 * 8, row_off);
  }
}
template <int B1, int ROWS>
__device__ __forceinline__ void put_corner(Sweep16Lds<B1>& S, const CornerRows<ROWS>& c, int j0, int step, int lane) {
#pragma unroll
  for (int t = 0; t < ROWS; ++t) {
    const int j = j0 + step * t, g = j / B1;
    double* to = S.corner + corner_at<B1>(g) + (j % B1) * (kSuper16 - g * B1) - g * B1;
    if (lane >= g * B1) to[lane] = c.v[t][0];
    if (64 + lane >= g * B1) to[64 + lane] = c.v[t][1];
  }
}

// The super-block's weights as the sweep leaves them, 8 rows for each of two wavefronts.
template <int B1>
__device__ __forceinline__ void store_final(const Sweep16Lds<B1>& S, double* W, int n, int sb, int sbw, int wave, int row0, int rows, int lane) {
  for (int r = 8 * wave; r < min(8 * wave + 8, rows); ++r)
    for (int k = lane; k < sbw; k += 64) W[(size_t)(row0 + r) * n + sb + k] = S.wsb[k][r];
}

template <int B1>
__global__ void __launch_bounds__(64 * kWaves16, 2) sweep16_kernel(SweepArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  Sweep16Lds<B1>& S = *reinterpret_cast<Sweep16Lds<B1>*>(lds);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = a.n, row0 = blockIdx.x * kRows16, rows = min(kRows16, a.m - row0);   // a tile is inside or outside
  const double* __restrict__ U = a.U;
  // Row-major here, written as the super-blocks and their far columns are through; what no far pass has been over yet is read where
  // the caller left it (a copy of 4096^2 before the sweep took 41 us, of 11008 x 4096 118).
  double* W = a.Wt;
  const Divisor levels = divisor_of(a.w_top);
  uint32_t target = 0;

  // the first super-block (rows behind the last one shadow it)
  if (tid < 2) S.task[tid] = 0;
  if (tid == 0) S.met = S.ready = 0;
  for (int r = 2 * wave; r < 2 * wave + 2; ++r)
#pragma unroll
    for (int k = lane; k < kSuper16; k += 64) S.wsb[k][r] = a.W[(size_t)(row0 + min(r, rows - 1)) * n + min(k, n - 1)];
  {
    bool ok = true;
    if (tid < kSuper16) {
      const Divisor d = divisor_of(tid < n ? U[(size_t)tid * n + tid] : 1.0);
      S.diag[tid] = f64x2{d.hi, d.lo};
      ok = divisor_in_range(d.b);
    }
    CornerRows<kSuper16 / kWaves16> c;
    fetch_corner(c, U, n, 0, wave, kWaves16, lane);
    put_corner<B1>(S, c, wave, kWaves16, lane);
    const int out_of_range = __syncthreads_or(!ok);
    if (tid < 2) S.diag_bad[tid] = out_of_range && tid == 0;
    __syncthreads();
  }

  for (int sb = 0; sb < n; sb += kSuper16) {
    const int next = sb + kSuper16, p = (sb / kSuper16) & 1, sbw = min(kSuper16, n - sb);
    if (wave < kFront16) {
      __builtin_amdgcn_s_setprio(2);
      const int blocks = sbw / B1;
      // (a loop for each kind of wavefront: what the near ones keep in registers does not weigh on the chain)
      if (wave < 2) {
        for (int b = 0; b < blocks; ++b) {
          block_tests<B1>(S, a, levels, fresh_s(b * B1), b & 1, p, wave, fresh_v(lane), S.esb[p]);
          meet(&S.met, &target, lane);
          if (wave == 0) block_chain<B1>(S, a, fresh_s(b * B1), sb / B1 + b, b & 1, p, fresh_v(lane), row0, rows, S.esb[p]);
          else if (b > 0) {
            block_feedback<B1>(S, fresh_s(b * B1) - B1, sbw, fresh_v(lane), feedback_threads(sbw - (b + 1) * B1), S.esb[p]);
            block_results<B1>(S, a, fresh_s(b * B1) - B1, sb, (b & 1) ^ 1, fresh_v(lane), row0, rows);
          }
          meet(&S.met, &target, lane);
        }
        if (wave == 1) block_results<B1>(S, a, fresh_s(sbw) - B1, sb, (blocks - 1) & 1, fresh_v(lane), row0, rows);
        store_final<B1>(S, W, n, sb, sbw, wave, row0, rows, fresh_v(lane));
        if (tid == 0) { S.diag_bad[p ^ 1] = 0; S.task[p ^ 1] = 0; }
        meet(&S.met, &target, lane);
      } else {
        // near: a block's rows of the corner are free when the block after the next one is begun, the next super-block's take their place
        const bool near = next < n;
        const int half = wave & 1, ncol = 64 * half + lane, noff = (next + ncol) * 8;
        Near N = {};                                     // (set in every case: otherwise the registers are carried round the whole loop)
        Divisor diag = {1.0, 1.0, 0.0};
        if (near) {
          N.done = 0;
          near_fetch(N.u, U, n, sb, noff);
          if (next + ncol < n) diag = divisor_of(U[(size_t)(next + ncol) * n + next + ncol]);
        }
        for (int b = 0; b < blocks; ++b) {
          block_tests<B1>(S, a, levels, fresh_s(b * B1), b & 1, p, wave, fresh_v(lane), S.esb[p]);
          meet(&S.met, &target, lane);
          CornerRows<B1 / 2> c = {};
          if (near && b >= 2) fetch_corner(c, U, n, next, (b - 2) * B1 + half, 2, fresh_v(lane));
          if (b > 0 && feedback_threads(sbw - (b + 1) * B1) > 64) block_feedback<B1>(S, fresh_s(b * B1) - B1, sbw, fresh_v(tid) - 64, 64 * 3, S.esb[p]);
          if (near) {                                    // (128 columns: at least four blocks)
            const int start = blocks / 4;
            if (b == start) {                            // the far wavefronts have been over these columns
              if (sb > 0) wait_for(&S.ready, 4 * (uint32_t)(sb / kSuper16));
              near_weights(N, sb > 0 ? W : a.W, n, row0, rows, fresh_v(noff));
            }
            if (b >= start) near_steps(N, U, n, sb, noff, min(b * B1, kSuper16 * (b + 1 - start) / (blocks - start)) & -Near::PF, S.esb[p]);
            if (b >= 2) put_corner<B1>(S, c, (b - 2) * B1 + half, 2, lane);
          }
          meet(&S.met, &target, lane);
        }
        if (near) near_steps(N, U, n, sb, noff, kSuper16, S.esb[p]);
        meet(&S.met, &target, lane);
        if (near) {
#pragma unroll
          for (int r = 0; r < kRows16; ++r) S.wsb[ncol][r] = N.cur[r];
#pragma unroll 1
          for (int j = kSuper16 - 2 * B1 + half; j < kSuper16; j += B1 < 8 ? 2 * B1 : 16) {
            CornerRows<B1 < 8 ? B1 : 8> c;
            fetch_corner(c, U, n, next, j, 2, fresh_v(lane));
            put_corner<B1>(S, c, j, 2, lane);
          }
          S.diag[ncol] = f64x2{diag.hi, diag.lo};
          if (!divisor_in_range(diag.b)) S.diag_bad[p ^ 1] = 1;
        }
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (sb > 0 && next < n) {
      // the errors of the super-block before, first to the columns the near wavefronts wait for, 4 rows each
      far_feedback<2, 4>(sb == kSuper16 ? a.W : W, W, U, n, row0, rows, lane, sb - kSuper16, next, 4 * (wave - kFront16), S.esb[p ^ 1]);
      __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the stores are done
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) __hip_atomic_fetch_add(&S.ready, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // The errors of the super-block before, to the runs of 64 columns right of the next one: four runs a task, of the last 14 runs
    // four in two halves of 8 rows, of the last 6 two (a task takes 64 us at most, alone on its SIMD half of that).
    const int from = next + kSuper16, runs = sb > 0 && from < n ? (n - from + 63) / 64 : 0;
    const int fine = min(runs, 6), medium = min(runs - fine, 8), wide = runs - fine - medium;
    const int wides = (wide + 3) / 4, mediums = (medium + 3) / 4 * 2, tasks = wides + mediums + (fine + 1) / 2 * 2;
    const double* src = sb == kSuper16 ? a.W : W;
    while (runs > 0) {
      uint32_t got = 0;
      if (lane == 0) got = __hip_atomic_fetch_add(&S.task[p], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const int task = __builtin_amdgcn_readfirstlane((int)got);
      if (task >= tasks) break;                          // wave-uniform; the count only grows
      const int n = fresh_s(a.n), row0 = fresh_s(blockIdx.x * kRows16), rows = fresh_s(min(kRows16, a.m - row0)), lane = fresh_v(tid & 63);
      if (task < wides) {
        far_task<16>(min(4, wide - 4 * task), src, W, U, n, row0, rows, lane, sb - kSuper16, from + 256 * task, 0, S.esb[p ^ 1]);
      } else {
        const bool last = task >= wides + mediums;
        const int t = last ? task - wides - mediums : task - wides, first = last ? wide + medium + t / 2 * 2 : wide + t / 2 * 4;
        far_task<8>(last ? min(2, runs - first) : min(4, wide + medium - first), src, W, U, n, row0, rows, lane, sb - kSuper16,
                    from + 64 * first, 8 * (t & 1), S.esb[p ^ 1]);
      }
    }
    __syncthreads();
  }
}

}  // namespace spqr_enc
