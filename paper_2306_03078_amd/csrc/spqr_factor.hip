// Lines 2 and 3 of Alg. 1 (SpQRQuantize): H = 2 X X^T and H^ic = Cholesky((H + lambda I)^-1), binary64.
//
// The factor the sweep needs is the upper triangular U with U^T U = (H + lambda I)^-1.  With A = H + lambda I
// and J the index reversal, a lower Cholesky factor L of J A J gives A = R R^T with R = J L J upper triangular,
// so A^-1 = R^-T R^-1 and U = R^-1 = J L^-1 J: one Cholesky factorisation and one triangular inverse, both in the
// reversed index space, no product of two triangular matrices and no second factorisation.
//
//   init      L <- lower triangle of J A J, padded with an identity to a multiple of 64 (nothing right of the diagonal blocks)
//   per block column k (64 wide): potrf of the diagonal block and its inverse (one workgroup, in LDS);
//             the panel below times that inverse (transposed); the trailing lower triangle minus panel x panel^T
//   trtri     X = L^-1 by doubling: with L = [[A, 0], [C, B]], L^-1 = [[A^-1, 0], [-B^-1 C A^-1, B^-1]].  Level s joins
//             neighbouring diagonal blocks of 64 * 2^s: two launches of 64 x 64 tile products per level (T = C A^-1,
//             then -B^-1 T written over C), every tile of every pair in parallel.  The inverse ends up where L was.
//   final     U[i][j] = X[n-1-i][n-1-j] for j >= i
//
// Every tile product runs on the matrix cores (v_mfma_f64_16x16x4_f64), at the vector ALU's rate, but an operand of one
// 8-byte half of an LDS read per lane feeds two instructions of 64 clocks.  n = d = 4096, Hessian and factor together 4.77 -> 3.26 ms:
// Hessian 1.48 -> 1.19 (after idle 1.6 -> 1.3: no vector instructions in the inner loop, see tile_product); block columns 33 -> 22 us on
// average (the diagonal block's chain, potrf_diag); the triangular inverse 0.92 -> 0.55 (the same loop, and tiles dealt so that CUs have
// equal work).  What is left: a block column's two launches, of 12 us (the 64 dependent steps 4 of them, the product before them 3, the blocks
// between the panels 3) and of 5 (start, end and one product), and in the early ones the tiles beside them, up to 30 (update_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "../../include/spqr_encode.h"

namespace spqr_fac {

constexpr int NB = 64;                       // block size of the factorisation
constexpr int KC = 16;                       // depth of one LDS stage of a tile product
// Padded row of a staged operand: Hessian of 4096 inputs with 2, 4, 8 and 12 more than KC 1.20, 1.19, 1.22 and 1.30 ms (warm).
constexpr int LP = KC + 4;

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x2_8 __attribute__((ext_vector_type(2), aligned(8)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// D += A B for one 16 x 16 block: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16], D[r] is row l / 16 + 4 r, column l % 16.
__device__ __forceinline__ f64x4 mfma4(double a, double b, f64x4 d) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0); }

// A tile of 64 x 64 of four wavefronts, 32 x 32 each; two LDS buffers of KC steps, the next one's values in registers while this one is
// multiplied.  Both operands are staged by rows, k innermost: a lane's 16-byte read is two steps of k for one row, so a product of 8
// steps takes 4 reads for 8 instructions of 64 clocks.  (One step a read, the rows innermost: as many clocks of LDS as of the matrix
// cores, with bank conflicts on top.)
//
// A binary64 matrix instruction keeps the vector unit from any other: the inner loop has none.  A stage is fetched by a uniform base,
// which the scalar unit moves on, and offsets that stay as they are; the buffers' places are constants of the instructions.  (A dozen
// address and select instructions a stage and thread: the Hessian of 4096 inputs and samples 1.39 ms instead of 1.19, 58 of 68 TFLOP/s.)
struct Tile { f64x4 d[2][2]; };
struct alignas(16) Stage { double a[2][NB][LP], b[2][NB][LP]; };     // (without the alignment an LDS read is two of 8 bytes)

typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer_of(const double* base) {    // (no bound: everything read lies in the matrix)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(base), 0, -1, 0x00027000);
}

// What a thread stages of an operand of 64 rows: the pairs (k, k + 1) of rows row(0) and row(1).
struct ByRows {                              // k innermost in memory: consecutive threads fetch consecutive k
  const double* base;
  uint32_t off[2];
  __device__ __forceinline__ ByRows(const double* first, int pitch) : base(first) {        // pitch: of the rows
#pragma unroll
    for (int q = 0; q < 2; ++q) off[q] = ((uint32_t)row(q) * (uint32_t)pitch + (uint32_t)k(q)) * 8u;
  }
  static __device__ __forceinline__ int row(int q) { return ((int)threadIdx.x + 256 * q) / (KC / 2); }
  static __device__ __forceinline__ int k(int) { return 2 * ((int)threadIdx.x % (KC / 2)); }
  __device__ __forceinline__ void fetch(f64x2 (&v)[2]) const {
    const Buffer b = buffer_of(base);
#pragma unroll
    for (int q = 0; q < 2; ++q) v[q] = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(b, off[q], 0, 0));
  }
  __device__ __forceinline__ void advance(int stages) { base += stages * KC; }
};
struct ByFarRows : ByRows {                  // ... of rows that a 32-bit offset does not reach: a pointer each (two additions a stage and row more)
  const f64x2_8* at[2];
  __device__ __forceinline__ ByFarRows(const double* first, int pitch, int last) : ByRows(first, 0) {      // rows behind `last`: the last
#pragma unroll
    for (int q = 0; q < 2; ++q) at[q] = reinterpret_cast<const f64x2_8*>(first + (size_t)min(row(q), last) * pitch + k(q));
  }
  __device__ __forceinline__ void fetch(f64x2 (&v)[2]) const {
#pragma unroll
    for (int q = 0; q < 2; ++q) v[q] = *at[q];
  }
  __device__ __forceinline__ void advance(int stages) {
#pragma unroll
    for (int q = 0; q < 2; ++q) at[q] += stages * (KC / 2);
  }
};
struct ByColumns {                           // the rows innermost: consecutive threads fetch consecutive rows
  const double* base;
  uint32_t off[2], pitch;                    // pitch: of k
  __device__ __forceinline__ ByColumns(const double* first, int pitch_) : base(first), pitch(pitch_) {
#pragma unroll
    for (int q = 0; q < 2; ++q) off[q] = ((uint32_t)k(q) * pitch + (uint32_t)row(q)) * 8u;
  }
  static __device__ __forceinline__ int row(int) { return (int)threadIdx.x % NB; }
  static __device__ __forceinline__ int k(int q) { return 2 * (((int)threadIdx.x + 256 * q) / NB); }
  __device__ __forceinline__ void fetch(f64x2 (&v)[2]) const {
    const Buffer b = buffer_of(base);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      v[q] = f64x2{__builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, off[q], 0, 0)),
                   __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, off[q], pitch * 8u, 0))};
  }
  __device__ __forceinline__ void advance(int stages) { base += (size_t)(stages * KC) * pitch; }
};

template <class A, class B> __device__ __forceinline__ void stash(Stage& S, int buf, const f64x2 (&pa)[2], const f64x2 (&pb)[2]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    *reinterpret_cast<f64x2*>(&S.a[buf][A::row(q)][A::k(q)]) = pa[q];
    *reinterpret_cast<f64x2*>(&S.b[buf][B::row(q)][B::k(q)]) = pb[q];
  }
}
__device__ __forceinline__ void multiply(Tile& acc, const Stage& S, int buf) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, g4 = lane >> 4;
  const double *pa = &S.a[buf][32 * (wave & 1) + i16][2 * g4], *pb = &S.b[buf][32 * (wave >> 1) + i16][2 * g4];
#pragma unroll
  for (int kk = 0; kk < KC; kk += 8) {
    f64x2 a[2], b[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      a[m] = *reinterpret_cast<const f64x2*>(pa + 16 * m * LP + kk);
      b[m] = *reinterpret_cast<const f64x2*>(pb + 16 * m * LP + kk);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc.d[m][n] = mfma4(a[m][e], b[n][e], acc.d[m][n]);
  }
}

// ... between the requests before it and what waits for them behind it (left to the compiler, the wait comes before the products).
__device__ __forceinline__ void multiply_between(Tile& acc, const Stage& S, int buf) {
  __builtin_amdgcn_sched_barrier(0);
  multiply(acc, S, buf);
  __builtin_amdgcn_sched_barrier(0);
}

// acc += A B^T over `stages` stages of KC; a barrier begins it (a product before may still be read) and ends it.
template <class A, class B>
__device__ __forceinline__ void tile_product(Tile& acc, A a, B b, int stages, Stage& S) {
  __syncthreads();
  if (stages <= 0) return;                   // workgroup-uniform
  f64x2 pa[2], pb[2];
  a.fetch(pa); b.fetch(pb);
  stash<A, B>(S, 0, pa, pb);
  __syncthreads();
  for (int s = 1; s < stages; s += 2) {      // stage s - 1 lies in the first buffer
    a.advance(1); b.advance(1);
    a.fetch(pa); b.fetch(pb);
    multiply_between(acc, S, 0);
    stash<A, B>(S, 1, pa, pb);
    __syncthreads();
    const int more = s + 1 < stages ? 1 : 0; // (behind the last stage that one again, unused)
    a.advance(more); b.advance(more);
    a.fetch(pa); b.fetch(pb);
    multiply_between(acc, S, 1);
    stash<A, B>(S, 0, pa, pb);
    __syncthreads();
  }
  if (stages & 1) {
    multiply(acc, S, 0);
    __syncthreads();
  }
}

// f(row, column, value) for the tile's elements of this thread.
template <class F>
__device__ __forceinline__ void each_element(const Tile& acc, F f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 32 * (wave & 1) + (lane >> 4), c0 = 32 * (wave >> 1) + (lane & 15);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) f(r0 + 16 * a + 4 * r, c0 + 16 * b, acc.d[a][b][r]);
}
// The tile with f(row, column) as this thread's elements.
template <class F>
__device__ __forceinline__ Tile load_tile(F f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = 32 * (wave & 1) + (lane >> 4), c0 = 32 * (wave >> 1) + (lane & 15);
  Tile t;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) t.d[a][b][r] = f(r0 + 16 * a + 4 * r, c0 + 16 * b);
  return t;
}

// Number of a cell of an upper triangle (row by row, `side` cells in the first) -> row and column.
__device__ __forceinline__ void upper_cell(int at, int side, int* row, int* col) {
  int r = 0;
  for (int left = side; at >= left; --left, ++r) at -= left;
  *row = r;
  *col = r + at;
}

// H = 2 X X^T, tiles on and above the diagonal, mirrored.  Squares of SQ x SQ tiles, a run of them for each of the 8 XCDs
// (workgroups go to the XCDs in turn): the tiles that run side by side on an XCD share rows of X in its L2.
constexpr int SQ = 2;
// 64 rows of it are within reach of a 32-bit offset.  Deeper, n = 128, d = 2^22 + 16: 259 ms with pointers checked element by element, 355
// stage after stage without overlap, 194 as it is (197 with offsets, d = 2^22); n = 1024: 268, 401, 212.
constexpr int kMostDepth = 1 << 22;
template <bool FAR>
__global__ void __launch_bounds__(256) hessian_kernel(const double* __restrict__ X, int n, int d, double* __restrict__ H, int squares, int run) {
  __shared__ Stage S;
  const int xcd = blockIdx.x % 8, at = blockIdx.x / 8, square = xcd * run + at / (SQ * SQ), side = (n + SQ * NB - 1) / (SQ * NB);
  if (square >= squares) return;             // workgroup-uniform
  int sr, sc;
  upper_cell(square, side, &sr, &sc);
  const int i0 = (sr * SQ + at % (SQ * SQ) / SQ) * NB, j0 = (sc * SQ + at % SQ) * NB;
  if (j0 < i0 || j0 >= n) return;            // below the diagonal or behind the matrix
  Tile acc = {};
  // (rows behind the last: the last, their sums are not written)
  auto rows = [&](int first) {
    const double* x = X + (size_t)first * d;
    if constexpr (FAR) return ByFarRows(x, d, n - 1 - first);
    else {
      ByRows o(x, d);
#pragma unroll
      for (int q = 0; q < 2; ++q) o.off[q] = ((uint32_t)min(ByRows::row(q), n - 1 - first) * (uint32_t)d + (uint32_t)ByRows::k(q)) * 8u;
      return o;
    }
  };
  const int stages = d / KC;
  tile_product(acc, rows(i0), rows(j0), stages, S);
  for (int64_t k0 = (int64_t)stages * KC; k0 < d; k0 += KC) {        // the rest of the depth, zeros behind it
    f64x2 pa[2], pb[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t k = k0 + ByRows::k(q);
      auto pair = [&](int row) {
        const double* x = X + (size_t)min(row, n - 1) * d + k;
        return f64x2{k < d ? x[0] : 0.0, k + 1 < d ? x[1] : 0.0};
      };
      pa[q] = pair(i0 + ByRows::row(q));
      pb[q] = pair(j0 + ByRows::row(q));
    }
    stash<ByRows, ByRows>(S, 0, pa, pb);
    __syncthreads();
    multiply(acc, S, 0);
    __syncthreads();
  }
  each_element(acc, [&](int r, int c, double v) {
    const int i = i0 + r, j = j0 + c;
    if (i <= j && j < n) {
      H[(size_t)i * n + j] = 2.0 * v;
      H[(size_t)j * n + i] = 2.0 * v;
    }
  });
}

// A row a workgroup up to the end of its diagonal block: nobody reads the blocks right of that (n = 4096: 46 us for every
// element of the square, 27 as it is).
__global__ void __launch_bounds__(256) init_reversed_kernel(const double* __restrict__ H, int n, int np, double lambda,
                                                           double* __restrict__ L) {
  const int a = blockIdx.x, end = (a | (NB - 1)) + 1;
  for (int b = threadIdx.x; b < end; b += 256) {
    double v = 0.0;
    if (b <= a) {
      if (a < n) v = H[(size_t)(n - 1 - a) * n + (n - 1 - b)] + (a == b ? lambda : 0.0);   // lower triangle of J A J
      else v = a == b ? 1.0 : 0.0;
    }
    L[(size_t)a * np + b] = v;
  }
}

// 1 / sqrt(x) to about a unit in the last place (x <= 0: NaN).  The hardware's estimate is good to 2^-24 or better; with
// e = 1 - x y^2 the true value is y (1 - e)^-1/2 = y (1 + e / 2 + 3 e^2 / 8 + ...), and what follows is below 2^-69.
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// d -= (s of lane LANE of the row of 16) * m, as one instruction: v_fmac_f64 takes that operand across lanes by itself.  The compiler does
// not look into the text for the two wait states between a write of `s` and its reading across lanes: the first reading after a write
// (FRESH) waits in its own text; that no later one follows a copy of `s` is looked after by a test, which reads the assembly.
template <int LANE, bool FRESH>
__device__ __forceinline__ void fnma_bcast(double& d, double s, double m) {
  if constexpr (FRESH)
    asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(m), "n"(LANE));
  else
    asm volatile("v_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(s), "v"(m), "n"(LANE));
}
template <int LANE>
__device__ __forceinline__ double bcast(double s) {                  // always the first
  double d;
  asm volatile("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(s), "n"(LANE));
  return d;
}
template <int... I, class F> __device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }

// Diagonal block kb: the inverse of its Cholesky factor in its place (nobody reads the factor's own block).  Four panels of 16 columns.
// A panel's own 16 x 16 block is the chain: wavefront 0 factorises and inverts it in registers, a lane per row of the factor and per
// column of the inverse (the four groups of 16 lanes do the same), 2 (15 - j) updates a step of one instruction each, which take the
// step's column of the factor across lanes themselves.  The next step's root hangs on the first of them; the others stand between
// the operations of that root, in the clocks these wait for one another.
//
// Everything else is products of blocks of 16 on the matrix cores, and all of it that the next chain does not need is done beside it by
// the other wavefronts: the blocks right of the next panel, and of row p of the inverse, X[p][j] = -X[p][p] W[j], the sums
// W[j] = L[p][j] X[j][j] + ... + L[p][p - 1] X[p - 1][j], which wavefront j + 1 keeps in registers: an accumulator's layout is that
// of a right operand.
//
// n = 4096, the launch of a block column with few tiles left: a lane per row of the whole panel, the column by two v_readlane a lane
// and the inverses afterwards row by row out of LDS 22.5 us; updates across lanes and the inverse joined by doubling at the end 17.0;
// as it is 12.0 (the diagonal entry itself, which nobody reads, no longer formed, a root by one step of third order instead of
// two of second, the updates in its gaps, 4 of 8 products and barriers after the last chain gone).
struct Diagonal {
  static constexpr int DP = NB + 2;
  double D[NB][DP];                          // the block; block (i, j) of the inverse in the place of block (j, i), which nobody reads by then
};
// The chain: r is row i of the block (what stands right of the diagonal means nothing), v column i of the identity, then of the inverse.
__device__ __forceinline__ void potrf_chain(double (&r)[16], double (&v)[16]) {
  double y = rsqrt_f64(bcast<0>(r[0]));
  unrolled(std::make_integer_sequence<int, 16>{}, [&](auto column) __attribute__((always_inline)) {
    constexpr int j = decltype(column)::value, updates = 2 * (15 - j), gap = (updates - 1 + 5) / 6;
    v[j] *= y;
    if constexpr (j < 15) {
      const double l = r[j] * y;
      // update 2 i of row or column j + 1 + i of r, 2 i + 1 of v
      const auto update = [&](auto from, auto count) __attribute__((always_inline)) {
        unrolled(std::make_integer_sequence<int, decltype(count)::value>{}, [&](auto at) __attribute__((always_inline)) {
          constexpr int u = decltype(from)::value + decltype(at)::value, k = j + 1 + u / 2;
          if constexpr (u < updates && u % 2 == 0) fnma_bcast<k, u == 0>(r[k], l, l);
          if constexpr (u < updates && u % 2 == 1) fnma_bcast<k, false>(v[k], l, v[j]);
        });
        __builtin_amdgcn_sched_barrier(0);
      };
#define SPQR_STEP(n, ...) __VA_ARGS__; update(std::integral_constant<int, 1 + (n)*gap>{}, std::integral_constant<int, gap>{})
      update(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
      SPQR_STEP(0, const double x = bcast<j + 1>(r[j + 1]));
      SPQR_STEP(1, const double y0 = __builtin_amdgcn_rsq(x));      // rsqrt_f64(x)
      SPQR_STEP(2, const double xy = x * y0);
      SPQR_STEP(3, const double e = fma(-xy, y0, 1.0));
      SPQR_STEP(4, const double h = fma(e, 0.375, 0.5); const double ye = y0 * e);
      SPQR_STEP(5, y = fma(ye, h, y0));
#undef SPQR_STEP
    }
  });
}
// `S.D` holds the block; every thread of the workgroup.
__device__ __forceinline__ void potrf_diag(Diagonal& S, double* __restrict__ L, int np, int kb) {
  double (&D)[NB][Diagonal::DP] = S.D;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15, g4 = lane >> 4;
  double* blk = L + (size_t)kb * NB * np + (size_t)kb * NB;
  const auto put = [&](int bi, int bj, auto value) __attribute__((always_inline)) {    // block (bi, bj) of the result, in an accumulator's layout
#pragma unroll
    for (int r = 0; r < 4; ++r) blk[(size_t)(16 * bi + g4 + 4 * r) * np + 16 * bj + i16] = value(r);
  };
  const auto trailing = [&](int p, int bi, int bj) __attribute__((always_inline)) {     // block (bi, bj) minus L[bi][p] L[bj][p]^T
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 16; q += 4) d = mfma4(D[16 * bi + i16][16 * p + q + g4], D[16 * bj + i16][16 * p + q + g4], d);
#pragma unroll
    for (int r = 0; r < 4; ++r) D[16 * bi + g4 + 4 * r][16 * bj + i16] -= d[r];
  };
  f64x4 W = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int p = 0; p < 4; ++p) {              // panel of columns 16 p ..
    const int c0 = 16 * p;
    if (wave == 0) {
      if (p > 0) trailing(p - 1, p, p);
      double r[16], v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) { r[k] = D[c0 + i16][c0 + k]; v[k] = k == i16 ? 1.0 : 0.0; }
      potrf_chain(r, v);
      if (g4 == 0) {
#pragma unroll
        for (int k = 0; k < 16; ++k) D[c0 + k][c0 + i16] = v[k];
      }
    } else {                                 // beside the chain
      if (p > 0) {
        int turn = 0;
        for (int bi = p + 1; bi < 4; ++bi)
          for (int bj = p; bj <= bi; ++bj)
            if (turn++ % 3 == wave - 1) trailing(p - 1, bi, bj);
        if (wave <= p) {
          const int j = wave - 1;
          W = f64x4{0.0, 0.0, 0.0, 0.0};
          for (int k = j; k < p; ++k)
#pragma unroll
            for (int q = 0; q < 16; q += 4) W = mfma4(D[c0 + i16][16 * k + q + g4], D[16 * j + q + g4][16 * k + i16], W);
        }
        if (wave == 3) put(p - 1, p - 1, [&](int r) { return D[c0 - 16 + g4 + 4 * r][c0 - 16 + i16]; });
      } else {                               // above the diagonal
        put(0, wave, [](int) { return 0.0; });
        put(wave == 3 ? 2 : 1, wave == 1 ? 2 : 3, [](int) { return 0.0; });
      }
    }
    __syncthreads();
    if (wave > p) {                          // the rows of block `wave` times the inverse, transposed
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 16; q += 4) d = mfma4(D[16 * wave + i16][c0 + q + g4], D[c0 + i16][c0 + q + g4], d);
#pragma unroll
      for (int r = 0; r < 4; ++r) D[16 * wave + g4 + 4 * r][c0 + i16] = d[r];
    } else if (wave > 0) {                   // block (p, wave - 1) of the inverse
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 16; q += 4) d = mfma4(D[c0 + i16][c0 + q + g4], W[q / 4], d);
      if (p < 3) {
#pragma unroll
        for (int r = 0; r < 4; ++r) D[16 * (wave - 1) + g4 + 4 * r][c0 + i16] = -d[r];
      }
      put(p, wave - 1, [&](int r) { return -d[r]; });
    } else if (p == 3) {
      put(3, 3, [&](int r) { return D[48 + g4 + 4 * r][48 + i16]; });
    }
    if (p < 3) __syncthreads();
  }
}

// The first diagonal block.
__global__ void __launch_bounds__(256) potrf_first_kernel(double* __restrict__ L, int np) {
  __shared__ Diagonal S;
  for (int idx = threadIdx.x; idx < NB * NB; idx += 256) S.D[idx >> 6][idx & 63] = L[(size_t)(idx >> 6) * np + (idx & 63)];
  __syncthreads();
  potrf_diag(S, L, np, 0);
}

// Panel below diagonal block kb: A[ib, kb] <- A[ib, kb] . inv(L_kk)^T
__global__ void __launch_bounds__(256) trsm_panel_kernel(double* __restrict__ L, int np, int kb) {
  __shared__ Stage S;
  const int ib = kb + 1 + blockIdx.x;
  double* blk = L + (size_t)ib * NB * np + (size_t)kb * NB;
  Tile acc = {};
  tile_product(acc, ByRows(blk, np), ByRows(L + (size_t)kb * NB * np + (size_t)kb * NB, np), NB / KC, S);   // every read of the block is done when it returns
  each_element(acc, [&](int r, int c, double v) { blk[(size_t)r * np + c] = v; });
}

// Trailing update: A[ib, jb] -= P_ib . P_jb^T for kb < jb <= ib, tile by tile of the lower triangle.  The first workgroup's is the
// next diagonal block, which it then factorises: a launch lasts as long as the longer of the two, and the chain of block
// columns is this launch and the panel's (n = 4096: 64 of 47 us, diagonal block, panel and update one after the other).
//
// A tile is 64 KiB of traffic however many panels it takes, and the workgroups beside the chain on its CU hold it up (12 us alone, 18 with
// one, 28 with three: a binary64 matrix instruction keeps the vector unit for 64 clocks).  So a column of tiles takes its panels kLag
// at a time, a launch before it becomes the panel itself and every kLag-th before that, and a launch has a kLag-th of the columns.
// What stands before the chain stays 64 deep: the diagonal block that comes after the next takes what it lacks a launch early, by the
// last workgroup.  The 63 launches of n = 4096 (warm): 1, 2, 3 and 4 panels at a time 1183, 1130, 1052 and 1146 us
// (one, two workgroups more of which fit a CU beside the chain than with the inverse in an array of its own: 1214).
// The whole factor, ms with 2, 3 and 4 at a time: 1024 inputs 0.398, 0.395 and 0.414, 4096 1.99, 1.96 and 2.01, 8192 9.39, 9.11 and 9.02, 11008 21.7,
// 20.9 and 20.4.
constexpr int kLag = 3;
// Tiles of the columns before column c of those of a launch; `rest` block rows are left.
__host__ __device__ constexpr int tiles_before(int c, int rest) { return c * rest - kLag * (c * (c - 1) / 2); }
static int update_tiles(int rest) { return tiles_before((rest + kLag - 1) / kLag, rest) + (rest > 1 ? 1 : 0); }
__global__ void __launch_bounds__(256) update_kernel(double* __restrict__ L, int np, int kb) {
  union Shared { Stage stage; Diagonal diagonal; };
  __shared__ Shared S;
  const int at = blockIdx.x, rest = np / NB - kb - 1;
  int ib = kb + 1, jb = kb + 1, from = kb;   // row and column; first panel
  if (at > 0 && at == (int)gridDim.x - 1) {
    ib = jb = kb + 2;
    from = max(kb - kLag + 2, 0);
  } else if (at > 0) {                       // tile number -> column and row of it
    const float h = (float)rest + 0.5f * kLag;
    int c = max((int)((h - sqrtf(fmaxf(h * h - 2.0f * kLag * (float)at, 0.0f))) * (1.0f / kLag)), 0);
    while (tiles_before(c, rest) > at) --c;
    while (tiles_before(c + 1, rest) <= at) ++c;
    jb = kb + 1 + kLag * __builtin_amdgcn_readfirstlane(c);
    ib = __builtin_amdgcn_readfirstlane(jb + at - tiles_before(c, rest));
    from = max(kb - kLag + 1, 0);
  }
  // the tile itself, on its way while the product is formed (64 deep, that is short: 4096 inputs 4.51 -> 4.42 ms)
  double* blk = L + (size_t)ib * NB * np + (size_t)jb * NB;
  const Tile before = load_tile([&](int r, int c) { return blk[(size_t)r * np + c]; });
  Tile acc = {};
  tile_product(acc, ByRows(L + (size_t)ib * NB * np + (size_t)from * NB, np), ByRows(L + (size_t)jb * NB * np + (size_t)from * NB, np),
               (kb + 1 - from) * (NB / KC), S.stage);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc.d[a][b] = before.d[a][b] - acc.d[a][b];
  if (at > 0) {                              // workgroup-uniform
    each_element(acc, [&](int r, int c, double v) { blk[(size_t)r * np + c] = v; });
    return;
  }
  each_element(acc, [&](int r, int c, double v) { S.diagonal.D[r][c] = v; });   // (the product is over: a barrier ends it)
  __syncthreads();
  potrf_diag(S.diagonal, L, np, kb + 1);
}

// The tiles of one pair of a level, `tiles` a side (a power of two), in such an order that the workgroups that share a CU, every 256th,
// have much the same to do in all: the depth falls along the columns in step 1 and grows along the rows in step 2, and every other
// 256 tiles go through them the other way (n = 4096, the last level: 319 and 235 us -> 188 and 205; 163 and 164 with
// tile_product as it is; the level before, two pairs of 256 tiles: 81 -> 51, counted through the pairs).  The whole factor without and
// with it: 2048 inputs the same, 3072 1.37 and 1.29 ms, 8192 9.87 and 9.11, 11008 22.0 and 20.9.
__device__ __forceinline__ bool other_way(int tiles) { return tiles <= 256 && ((blockIdx.x + tiles * (blockIdx.y + tiles * blockIdx.z)) / 256 & 1); }

// Level with diagonal blocks of `b` rows: pair p joins A = [2pb, 2pb + b) and B = [2pb + b, min(2pb + 2b, np)).
// Step 1: T = C . A^-1 into `T` (at C's place);  C = L[B rows, A columns].
__global__ void __launch_bounds__(256) trtri_step1_kernel(const double* __restrict__ L, int np, int b, double* __restrict__ T) {
  __shared__ Stage S;
  const int a0 = 2 * b * blockIdx.z, b0 = a0 + b, tiles = gridDim.x;
  const int x = other_way(tiles) ? tiles - 1 - (int)blockIdx.x : (int)blockIdx.x;
  const int i0 = b0 + blockIdx.y * NB, j0 = a0 + x * NB;             // tile: rows i0.. (in B), columns j0.. (in A)
  if (i0 >= np) return;                                              // B is shorter than b, or missing
  Tile acc = {};
  // A^-1 is lower triangular: rows k >= j0 only
  tile_product(acc, ByRows(L + (size_t)i0 * np + j0, np), ByColumns(L + (size_t)j0 * np + j0, np), (b0 - j0) / KC, S);
  each_element(acc, [&](int r, int c, double v) { T[(size_t)(i0 + r) * np + j0 + c] = v; });
}

// Step 2: -B^-1 . T over C.
__global__ void __launch_bounds__(256) trtri_step2_kernel(double* __restrict__ L, int np, int b, const double* __restrict__ T) {
  __shared__ Stage S;
  const int a0 = 2 * b * blockIdx.z, b0 = a0 + b, tiles = gridDim.x;
  const int rows = min(max(256 / tiles, 1), tiles), y = other_way(tiles) ? (int)blockIdx.y + rows - 1 - 2 * ((int)blockIdx.y % rows) : (int)blockIdx.y;
  const int i0 = b0 + y * NB, j0 = a0 + blockIdx.x * NB;             // tile: rows i0.., columns j0..
  if (i0 >= np) return;
  Tile acc = {};
  // B^-1, lower triangular: columns up to the tile's own block.  Its blocks left of the diagonal were written by the lower levels,
  // which are complete; this level writes blocks of C only.
  tile_product(acc, ByRows(L + (size_t)i0 * np + b0, np), ByColumns(T + (size_t)b0 * np + j0, np), (i0 + NB - b0) / KC, S);
  each_element(acc, [&](int r, int c, double v) { L[(size_t)(i0 + r) * np + j0 + c] = -v; });
}

__global__ void __launch_bounds__(256) unreverse_kernel(const double* __restrict__ L, int n, int np, double* __restrict__ U) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)n * n) return;
  const int i = (int)(idx / n), j = (int)(idx % n);
  U[idx] = j >= i ? L[(size_t)(n - 1 - i) * np + (n - 1 - j)] : 0.0;
}

}  // namespace spqr_fac

extern "C" {

int spqr_hessian(const double* X, int32_t n, int32_t d, double* H, void* stream) {
  using namespace spqr_fac;
  if (!X || !H) return SPQR_ERR_NULL;
  if (n < 1 || d < 1) return SPQR_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(X) % 8 != 0 || reinterpret_cast<uintptr_t>(H) % 8 != 0) return SPQR_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int side = (n + SQ * NB - 1) / (SQ * NB), squares = side * (side + 1) / 2, run = (squares + 7) / 8;
  hipLaunchKernelGGL(d <= kMostDepth ? hessian_kernel<false> : hessian_kernel<true>, dim3(8 * run * SQ * SQ), dim3(256), 0, st, X, n, d, H, squares, run);
  return hipGetLastError() == hipSuccess ? SPQR_OK : SPQR_ERR_HIP;
}

size_t spqr_inverse_cholesky_workspace_bytes(int32_t n) {
  if (n < 1) return 0;
  const size_t np = ((size_t)n + spqr_fac::NB - 1) / spqr_fac::NB * spqr_fac::NB;
  return 2 * np * np * sizeof(double);
}

int spqr_inverse_cholesky(const double* H, int32_t n, double lambda, double* Hic, void* workspace,
                          size_t workspace_bytes, void* stream) {
  using namespace spqr_fac;
  if (!H || !Hic || !workspace) return SPQR_ERR_NULL;
  if (n < 1) return SPQR_ERR_SHAPE;
  if (lambda != lambda) return SPQR_ERR_PARAM;
  if (workspace_bytes < spqr_inverse_cholesky_workspace_bytes(n)) return SPQR_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0 || reinterpret_cast<uintptr_t>(H) % 8 != 0 ||
      reinterpret_cast<uintptr_t>(Hic) % 8 != 0)
    return SPQR_ERR_ALIGN;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int np = (n + NB - 1) / NB * NB, nb = np / NB;
  double* L = static_cast<double*>(workspace);
  double* X = L + (size_t)np * np;
  hipLaunchKernelGGL(init_reversed_kernel, dim3(np), dim3(256), 0, st, H, n, np, lambda, L);
  hipLaunchKernelGGL(potrf_first_kernel, dim3(1), dim3(256), 0, st, L, np);
  for (int kb = 0; kb + 1 < nb; ++kb) {
    const int rest = nb - kb - 1;
    hipLaunchKernelGGL(trsm_panel_kernel, dim3(rest), dim3(256), 0, st, L, np, kb);
    hipLaunchKernelGGL(update_kernel, dim3(update_tiles(rest)), dim3(256), 0, st, L, np, kb);
  }
  for (int b = NB; b < np; b *= 2) {
    const int tiles = b / NB, pairs = (np + 2 * b - 1) / (2 * b);
    hipLaunchKernelGGL(trtri_step1_kernel, dim3(tiles, tiles, pairs), dim3(256), 0, st, L, np, b, X);
    hipLaunchKernelGGL(trtri_step2_kernel, dim3(tiles, tiles, pairs), dim3(256), 0, st, L, np, b, X);
  }
  hipLaunchKernelGGL(unreverse_kernel, dim3((unsigned)(((size_t)n * n + 255) / 256)), dim3(256), 0, st, L, n, np, Hic);
  return hipGetLastError() == hipSuccess ? SPQR_OK : SPQR_ERR_HIP;
}

}  // extern "C"
