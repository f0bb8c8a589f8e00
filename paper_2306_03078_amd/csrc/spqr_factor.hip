// Lines 2 and 3 of Alg. 1 (SpQRQuantize): H = 2 X X^T and H^ic = Cholesky((H + lambda I)^-1), binary64.
//
// The factor the sweep needs is the upper triangular U with U^T U = (H + lambda I)^-1.  With A = H + lambda I
// and J the index reversal, a lower Cholesky factor L of J A J gives A = R R^T with R = J L J upper triangular,
// so A^-1 = R^-T R^-1 and U = R^-1 = J L^-1 J: one Cholesky factorisation and one triangular inverse, both in the
// reversed index space, no product of two triangular matrices and no second factorisation.
//
//   init      L <- lower triangle of J A J, padded with an identity to a multiple of 64
//   per block column k (64 wide): potrf of the diagonal block and its inverse (one workgroup, in LDS);
//             the panel below times that inverse (transposed); the trailing lower triangle minus panel x panel^T
//   trtri     X = L^-1 by doubling: with L = [[A, 0], [C, B]], L^-1 = [[A^-1, 0], [-B^-1 C A^-1, B^-1]].  Level s joins
//             neighbouring diagonal blocks of 64 * 2^s: two launches of 64 x 64 tile products per level (T = C A^-1,
//             then -B^-1 T written over C), every tile of every pair in parallel.  The inverse ends up where L was
//             (strictly lower blocks) plus the diagonal blocks' inverses from the potrf step.
//   final     U[i][j] = X[n-1-i][n-1-j] for j >= i
//
// Every tile product runs on the matrix cores (v_mfma_f64_16x16x4_f64).  Their binary64 rate is the vector ALU's, but an
// operand of one 8-byte LDS read per lane feeds two instructions of 64 clocks, where register tiles of 4 x 4 FMAs need
// eight LDS reads for sixteen instructions of 4, bound by LDS.  n = d = 4096: Hessian 3.4 -> 2.5 ms (28 of 68 TFLOP/s),
// trailing updates 23 -> 20 us and panels 11.8 -> 7.0 us each, diagonal blocks 51 -> 20 us, Hessian and factor together 10.9 -> 6.8
// ms; what is left is the Hessian's operands one step ahead in registers, and the chain of diagonal blocks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/spqr_encode.h"

namespace spqr_fac {

constexpr int NB = 64;                       // block size of the factorisation
constexpr int KC = 16;                       // depth of one LDS stage of a tile product
constexpr int LP = NB + 8;                   // padded row of a staged operand: an operand's four rows meet no bank twice more than they must

typedef double f64x4 __attribute__((ext_vector_type(4)));

// D += A B for one 16 x 16 block: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16], D[r] is row l / 16 + 4 r, column l % 16.
__device__ __forceinline__ f64x4 mfma4(double a, double b, f64x4 d) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0); }

// A 64 x 64 tile of four wavefronts, 32 x 32 each; two LDS buffers of KC steps, the next one's values in registers
// while this one is multiplied.
struct Tile { f64x4 d[2][2]; };
struct Stage { double a[2][KC][LP], b[2][KC][LP]; };

// get_a / get_b (idx, k0): staged value idx (0 .. 1023) of the step at k0; place_b: where one of B goes.
template <class GetA, class GetB, class PlaceB>
__device__ __forceinline__ void tile_product(Tile& acc, int kb, int ke, GetA get_a, GetB get_b, PlaceB place_b, Stage& S) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, i16 = lane & 15, g4 = lane >> 4;
  const int r0 = 32 * (wave & 1) + i16, c0 = 32 * (wave >> 1) + i16;
  double pa[4], pb[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) { pa[q] = get_a(t + 256 * q, k0); pb[q] = get_b(t + 256 * q, k0); }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = t + 256 * q;
      S.a[buf][idx & 15][idx >> 4] = pa[q];
      place_b(S.b[buf], idx, pb[q]);
    }
  };
  if (kb >= ke) return;                      // workgroup-uniform
  __syncthreads();                           // a product before this one may still be read
  fetch(kb);
  stash(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = kb; k0 < ke; k0 += KC, buf ^= 1) {
    if (k0 + KC < ke) fetch(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      const double *ra = S.a[buf][kk + g4], *rb = S.b[buf][kk + g4];
      const double a0 = ra[r0], a1 = ra[r0 + 16], b0 = rb[c0], b1 = rb[c0 + 16];
      acc.d[0][0] = mfma4(a0, b0, acc.d[0][0]);
      acc.d[0][1] = mfma4(a0, b1, acc.d[0][1]);
      acc.d[1][0] = mfma4(a1, b0, acc.d[1][0]);
      acc.d[1][1] = mfma4(a1, b1, acc.d[1][1]);
    }
    if (k0 + KC < ke) stash(buf ^ 1);
    __syncthreads();
  }
}

// sum_{k < K} fa(i, k) * fb(j, k): both operands given by rows; consecutive threads fetch consecutive k of one row.
template <class FA, class FB>
__device__ __forceinline__ void tile_nt(Tile& acc, int K, FA fa, FB fb, Stage& S) {
  tile_product(acc, 0, K, [&](int idx, int k0) { return fa(idx >> 4, k0 + (idx & 15)); },
               [&](int idx, int k0) { return fb(idx >> 4, k0 + (idx & 15)); },
               [](double (*b)[LP], int idx, double v) { b[idx & 15][idx >> 4] = v; }, S);
}

// sum_{kb <= k < ke} fa(i, k) * fb(k, j): the second operand by rows (k, j), consecutive threads fetch consecutive j.
template <class FA, class FB>
__device__ __forceinline__ void tile_nn(Tile& acc, int kb, int ke, FA fa, FB fb, Stage& S) {
  tile_product(acc, kb, ke, [&](int idx, int k0) { return fa(idx >> 4, k0 + (idx & 15)); },
               [&](int idx, int k0) { return fb(k0 + (idx >> 6), idx & 63); },
               [](double (*b)[LP], int idx, double v) { b[idx >> 6][idx & 63] = v; }, S);
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

// H = 2 X X^T, tiles on and above the diagonal, mirrored.
__global__ void __launch_bounds__(256) hessian_kernel(const double* __restrict__ X, int n, int d, double* __restrict__ H) {
  __shared__ Stage S;
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj < bi) return;
  const int i0 = bi * NB, j0 = bj * NB;
  Tile acc = {};
  auto fa = [&](int i, int k) { return (i0 + i < n && k < d) ? X[(size_t)(i0 + i) * d + k] : 0.0; };
  auto fb = [&](int j, int k) { return (j0 + j < n && k < d) ? X[(size_t)(j0 + j) * d + k] : 0.0; };
  tile_nt(acc, d, fa, fb, S);
  each_element(acc, [&](int r, int c, double v) {
    const int i = i0 + r, j = j0 + c;
    if (i < n && j < n) {
      H[(size_t)i * n + j] = 2.0 * v;
      if (bi != bj) H[(size_t)j * n + i] = 2.0 * v;
    }
  });
}

__global__ void __launch_bounds__(256) init_reversed_kernel(const double* __restrict__ H, int n, int np, double lambda,
                                                           double* __restrict__ L) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)np * np) return;
  const int a = (int)(idx / np), b = (int)(idx % np);
  double v = 0.0;
  if (b <= a) {
    if (a < n) v = H[(size_t)(n - 1 - a) * n + (n - 1 - b)] + (a == b ? lambda : 0.0);   // lower triangle of J A J
    else v = a == b ? 1.0 : 0.0;
  }
  L[idx] = v;
}

// A lane's double as every lane sees it (v_readlane: the source lane is uniform).
__device__ __forceinline__ double readlane_f64(double v, int src) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / sqrt(x) and sqrt(x) by Newton steps on the hardware's estimate, to about a unit in the last place (x <= 0: NaN).
__device__ __forceinline__ double rsqrt_f64(double x, double* root) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double e = fma(-x * y, y, 1.0);    // 1 - x y^2
    y = fma(0.5 * y, e, y);
  }
  const double r = x * y;
  *root = fma(fma(-r, r, x), 0.5 * y, r);
  return y;
}

// Diagonal block kb: Cholesky factor in place, its inverse to Dinv[kb].  Four panels of 16 columns: a panel's 16 steps
// depend on each other, so one wavefront takes them (a lane per row, the row in registers, column j handed to the other
// rows by v_readlane); the columns right of the panel are updated by all four on the matrix cores.  The inverse by
// doubling: the four diagonal blocks of 16 at once, a wavefront each, then 16 -> 32 -> 64 as products of blocks.  (One
// wavefront for all 64 columns and the inverse took 51 us: 2016 updates and as many LDS reads in one chain, and a
// division and a square root per step.)
__global__ void __launch_bounds__(256) potrf_diag_kernel(double* __restrict__ L, int np, int kb, double* __restrict__ Dinv) {
  constexpr int DP = NB + 2;
  __shared__ double D[NB][DP], X[NB][DP], T[32][34], rd[NB];     // block, inverse, a product between, 1 / diagonal
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, g4 = lane >> 4;
  double* blk = L + (size_t)kb * NB * np + (size_t)kb * NB;
  for (int idx = tid; idx < NB * NB; idx += 256) {
    D[idx >> 6][idx & 63] = blk[(size_t)(idx >> 6) * np + (idx & 63)];
    X[idx >> 6][idx & 63] = 0.0;
  }
  __syncthreads();
  for (int p = 0; p < 4; ++p) {              // panel of columns c0 .. c0 + 15
    const int c0 = 16 * p;
    if (wave == 0) {
      double r[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) r[k] = D[lane][c0 + k];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        double root;
        const double y = rsqrt_f64(readlane_f64(r[j], c0 + j), &root);
        const double l = r[j] * y;           // L[lane][c0 + j] for lane > c0 + j
        r[j] = lane == c0 + j ? root : l;
        if (lane == 0) rd[c0 + j] = y;
#pragma unroll
        for (int k = j + 1; k < 16; ++k) r[k] = fma(-l, readlane_f64(l, c0 + k), r[k]);   // meaningful for c0 + k <= lane
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) D[lane][c0 + k] = c0 + k <= lane ? r[k] : 0.0;
    }
    __syncthreads();
    // blocks (bi, bj), p < bj <= bi: minus L[bi][p] L[bj][p]^T, dealt to the wavefronts in turn
    int pair = 0;
    for (int bi = p + 1; bi < 4; ++bi)
      for (int bj = p + 1; bj <= bi; ++bj) {
        if ((pair++ & 3) != wave) continue;  // wave-uniform
        f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 16; q += 4) d = mfma4(D[16 * bi + i16][c0 + q + g4], D[16 * bj + i16][c0 + q + g4], d);
#pragma unroll
        for (int r = 0; r < 4; ++r) D[16 * bi + g4 + 4 * r][16 * bj + i16] -= d[r];
      }
    __syncthreads();
  }
  for (int idx = tid; idx < NB * NB; idx += 256)
    blk[(size_t)(idx >> 6) * np + (idx & 63)] = (idx & 63) <= (idx >> 6) ? D[idx >> 6][idx & 63] : 0.0;
  // inverse of diagonal block `wave`, column i16 per lane (the four lane groups do the same)
  {
    const int o = 16 * wave;
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int k = 0; k + 1 < i; k += 2) { s0 = fma(D[o + i][o + k], v[k], s0); s1 = fma(D[o + i][o + k + 1], v[k + 1], s1); }
      if (i & 1) s0 = fma(D[o + i][o + i - 1], v[i - 1], s0);
      v[i] = i < i16 ? 0.0 : (i == i16 ? rd[o + i] : -(s0 + s1) * rd[o + i]);
    }
    if (g4 == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) X[o + i][o + i16] = v[i];
    }
  }
  __syncthreads();
  // [[A, 0], [C, B]]^-1 = [[A^-1, 0], [-B^-1 C A^-1, B^-1]], first for the pairs of blocks of 16, then of 32
#pragma unroll
  for (int h = 16; h <= 32; h *= 2) {
    const int per = h / 16;                  // blocks of 16 per side of C
    const int pairs = 32 / h;                // joins of this level; per * per blocks each, one per wavefront
    const int join = wave / (per * per), b = wave % (per * per), bi = 16 * (b / per), bj = 16 * (b % per);
    const int a0 = 2 * h * join, b0 = a0 + h;
    const bool mine = join < pairs;          // wave-uniform
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
    if (mine) {
      for (int q = 0; q < h; q += 4) d = mfma4(D[b0 + bi + i16][a0 + q + g4], X[a0 + q + g4][a0 + bj + i16], d);   // C A^-1
#pragma unroll
      for (int r = 0; r < 4; ++r) T[(h == 16 ? 16 * join : bi) + g4 + 4 * r][bj + i16] = d[r];
    }
    __syncthreads();
    if (mine) {
      d = f64x4{0.0, 0.0, 0.0, 0.0};
      for (int q = 0; q < h; q += 4) d = mfma4(X[b0 + bi + i16][b0 + q + g4], T[(h == 16 ? 16 * join : 0) + q + g4][bj + i16], d);
#pragma unroll
      for (int r = 0; r < 4; ++r) X[b0 + bi + g4 + 4 * r][a0 + bj + i16] = -d[r];
    }
    __syncthreads();
  }
  double* inv = Dinv + (size_t)kb * NB * NB;
  for (int idx = tid; idx < NB * NB; idx += 256) inv[idx] = X[idx >> 6][idx & 63];
}

// Panel below diagonal block kb: A[ib, kb] <- A[ib, kb] . inv(L_kk)^T
__global__ void __launch_bounds__(256) trsm_panel_kernel(double* __restrict__ L, int np, int kb, const double* __restrict__ Dinv) {
  __shared__ Stage S;
  const int ib = kb + 1 + blockIdx.x;
  double* blk = L + (size_t)ib * NB * np + (size_t)kb * NB;
  const double* inv = Dinv + (size_t)kb * NB * NB;
  Tile acc = {};
  auto fa = [&](int r, int k) { return blk[(size_t)r * np + k]; };
  auto fb = [&](int c, int k) { return inv[c * NB + k]; };
  tile_nt(acc, NB, fa, fb, S);          // every read of the block is done when tile_nt returns
  each_element(acc, [&](int r, int c, double v) { blk[(size_t)r * np + c] = v; });
}

// Trailing update: A[ib, jb] -= P_ib . P_jb^T for kb < jb <= ib.
__global__ void __launch_bounds__(256) syrk_kernel(double* __restrict__ L, int np, int kb) {
  __shared__ Stage S;
  const int ib = kb + 1 + blockIdx.y, jb = kb + 1 + blockIdx.x;
  if (jb > ib) return;
  const double* pi = L + (size_t)ib * NB * np + (size_t)kb * NB;
  const double* pj = L + (size_t)jb * NB * np + (size_t)kb * NB;
  Tile acc = {};
  auto fa = [&](int r, int k) { return pi[(size_t)r * np + k]; };
  auto fb = [&](int c, int k) { return pj[(size_t)c * np + k]; };
  tile_nt(acc, NB, fa, fb, S);
  double* blk = L + (size_t)ib * NB * np + (size_t)jb * NB;
  each_element(acc, [&](int r, int c, double v) { blk[(size_t)r * np + c] -= v; });
}

// Element (r, c), r >= c, of the inverse as far as it is built: the diagonal 64-blocks live in Dinv, the blocks
// below them where L was.
__device__ __forceinline__ double inverse_at(const double* __restrict__ L, const double* __restrict__ Dinv, int np,
                                             int r, int c) {
  const int rb = r >> 6, cb = c >> 6;
  if (rb == cb) return Dinv[(size_t)rb * NB * NB + (r & 63) * NB + (c & 63)];
  return rb > cb ? L[(size_t)r * np + c] : 0.0;
}

// Level with diagonal blocks of `b` rows: pair p joins A = [2pb, 2pb + b) and B = [2pb + b, min(2pb + 2b, np)).
// Step 1: T = C . A^-1 into `T` (at C's place);  C = L[B rows, A columns].
__global__ void __launch_bounds__(256) trtri_step1_kernel(const double* __restrict__ L, const double* __restrict__ Dinv,
                                                         int np, int b, double* __restrict__ T) {
  __shared__ Stage S;
  const int a0 = 2 * b * blockIdx.z, b0 = a0 + b;
  const int i0 = b0 + blockIdx.y * NB, j0 = blockIdx.x * NB;        // tile: rows i0.. (in B), columns a0 + j0.. (in A)
  if (i0 >= np) return;                                              // B is shorter than b, or missing
  Tile acc = {};
  auto fa = [&](int i, int k) { return L[(size_t)(i0 + i) * np + a0 + k]; };
  auto fb = [&](int k, int j) { return inverse_at(L, Dinv, np, a0 + k, a0 + j0 + j); };
  tile_nn(acc, j0, b, fa, fb, S);                               // A^-1 is lower triangular: rows k >= j0 only
  each_element(acc, [&](int r, int c, double v) { T[(size_t)(i0 + r) * np + a0 + j0 + c] = v; });
}

// Step 2: -B^-1 . T over C.
__global__ void __launch_bounds__(256) trtri_step2_kernel(double* __restrict__ L, const double* __restrict__ Dinv, int np,
                                                         int b, const double* __restrict__ T) {
  __shared__ Stage S;
  const int a0 = 2 * b * blockIdx.z, b0 = a0 + b;
  const int i0 = blockIdx.y * NB, j0 = blockIdx.x * NB;              // tile: rows b0 + i0.., columns a0 + j0..
  if (b0 + i0 >= np) return;
  Tile acc = {};
  // B^-1 (lower triangular, rows / columns relative to b0): its blocks left of the diagonal were written by the
  // lower levels, which are complete; this level writes blocks of C only
  auto fa = [&](int i, int k) { return inverse_at(L, Dinv, np, b0 + i0 + i, b0 + k); };
  auto fb = [&](int k, int j) { return T[(size_t)(b0 + k) * np + a0 + j0 + j]; };
  tile_nn(acc, 0, i0 + NB, fa, fb, S);
  each_element(acc, [&](int r, int c, double v) { L[(size_t)(b0 + i0 + r) * np + a0 + j0 + c] = -v; });
}

__global__ void __launch_bounds__(256) unreverse_kernel(const double* __restrict__ L, const double* __restrict__ Dinv, int n,
                                                       int np, double* __restrict__ U) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)n * n) return;
  const int i = (int)(idx / n), j = (int)(idx % n);
  U[idx] = j >= i ? inverse_at(L, Dinv, np, n - 1 - i, n - 1 - j) : 0.0;
}

}  // namespace spqr_fac

extern "C" {

int spqr_hessian(const double* X, int32_t n, int32_t d, double* H, void* stream) {
  using namespace spqr_fac;
  if (!X || !H) return SPQR_ERR_NULL;
  if (n < 1 || d < 1) return SPQR_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(X) % 8 != 0 || reinterpret_cast<uintptr_t>(H) % 8 != 0) return SPQR_ERR_ALIGN;
  const int nb = (n + NB - 1) / NB;
  hipLaunchKernelGGL(hessian_kernel, dim3(nb, nb), dim3(256), 0, static_cast<hipStream_t>(stream), X, n, d, H);
  return hipGetLastError() == hipSuccess ? SPQR_OK : SPQR_ERR_HIP;
}

size_t spqr_inverse_cholesky_workspace_bytes(int32_t n) {
  if (n < 1) return 0;
  const size_t np = ((size_t)n + spqr_fac::NB - 1) / spqr_fac::NB * spqr_fac::NB;
  return (2 * np * np + np * spqr_fac::NB) * sizeof(double);
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
  double* Dinv = X + (size_t)np * np;
  const unsigned cells = (unsigned)(((size_t)np * np + 255) / 256);
  hipLaunchKernelGGL(init_reversed_kernel, dim3(cells), dim3(256), 0, st, H, n, np, lambda, L);
  for (int kb = 0; kb < nb; ++kb) {
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(256), 0, st, L, np, kb, Dinv);
    const int rest = nb - kb - 1;
    if (rest > 0) {
      hipLaunchKernelGGL(trsm_panel_kernel, dim3(rest), dim3(256), 0, st, L, np, kb, Dinv);
      hipLaunchKernelGGL(syrk_kernel, dim3(rest, rest), dim3(256), 0, st, L, np, kb);
    }
  }
  for (int b = NB; b < np; b *= 2) {
    const int tiles = b / NB, pairs = (np + 2 * b - 1) / (2 * b);
    hipLaunchKernelGGL(trtri_step1_kernel, dim3(tiles, tiles, pairs), dim3(256), 0, st, L, Dinv, np, b, X);
    hipLaunchKernelGGL(trtri_step2_kernel, dim3(tiles, tiles, pairs), dim3(256), 0, st, L, Dinv, np, b, X);
  }
  hipLaunchKernelGGL(unreverse_kernel, dim3((unsigned)(((size_t)n * n + 255) / 256)), dim3(256), 0, st, L, Dinv, n, np, Hic);
  return hipGetLastError() == hipSuccess ? SPQR_OK : SPQR_ERR_HIP;
}

}  // extern "C"
