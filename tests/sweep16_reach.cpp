// Walks the loads and stores of the 16-row sweep on the CPU: the functions of spqr_sweep16.h that touch the caller's matrices, with
// buffer accesses that only note where they go.  A buffer checks a lane's offset against its size; what is documented not to be part of
// that check (the scalar offset) is added without one.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <utility>

#define __device__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n)
#define asm
#define volatile(...)

struct Dim { int x; };
static Dim threadIdx, blockIdx;
static int min(int a, int b) { return a < b ? a : b; }
static uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
static int max(int a, int b) { return a > b ? a : b; }

struct Range { const char* at; size_t bytes; };
static Range U_range, W_range;                 // never read: addresses only
static long reads, writes;
struct HostBuffer { const char* base; uint32_t bytes; };
static bool inside(const Range& r, const char* at) { return at >= r.at && at + 8 <= r.at + r.bytes; }
static const char* g_what = "";
static bool touch(const HostBuffer& b, int off, int row_off) {
  if ((uint64_t)(uint32_t)off + 8 > b.bytes) return false;               // zeros, or nothing written
  const char* at = b.base + (uint32_t)off + (uint32_t)row_off;
  if (inside(U_range, at) || inside(W_range, at)) return true;
  std::printf("%s: %lld bytes behind the end of a matrix\n", g_what,
              (long long)(at + 8 - (at >= W_range.at ? W_range.at + W_range.bytes : U_range.at + U_range.bytes)));
  std::exit(1);
}
typedef uint32_t HostWords __attribute__((ext_vector_type(2)));
#define __amdgpu_buffer_rsrc_t HostBuffer
static HostBuffer __builtin_amdgcn_make_buffer_rsrc(double* p, int, int bytes, int) { return {reinterpret_cast<const char*>(p), (uint32_t)bytes}; }
static HostWords host_load(const HostBuffer& b, int off, int row_off, int) { reads += touch(b, off, row_off); return HostWords{0, 0}; }
static void host_store(HostWords, const HostBuffer& b, int off, int row_off, int) { writes += touch(b, off, row_off); }
#define __builtin_amdgcn_raw_buffer_load_b64 host_load
#define __builtin_amdgcn_raw_buffer_store_b64 host_store
// what the functions that are not called need to be compiled
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_mov_dpp(v, ...) (v)
#define __builtin_amdgcn_fence(...)
#define __builtin_amdgcn_s_sleep(x)
#define __builtin_amdgcn_s_setprio(x)
#define __builtin_amdgcn_s_waitcnt(x)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sbfe(v, at, bits) (v)
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_fetch_add(p, ...) (*(p))
#define __any(x) (x)
#define __all(x) (x)
#define __ballot(x) ((uint64_t)(x))
#define __syncthreads()
#define __syncthreads_or(x) (x)

struct spqr_quantized_t { uint8_t *Q, *s_q, *z_q; uint16_t *s_s, *z_s, *s_z, *z_z; uint8_t* outlier_mask; uint16_t* outlier_val; int32_t* row_ptr; double* W_final; };
namespace spqr_enc {
struct SweepArgs { const double* U; double* Wt; const double* W; int m, n, beta2; double w_top, s_top, z_top, tau; spqr_quantized_t out; };
uint16_t f64_to_f16_bits(double);
double quantize(double, double, double, double);
void fit_from_range(double, double, double, double*, double*);
void second_level_of_range(double, double, double, double, double*, uint8_t*, uint16_t*, uint16_t*);
}
#include "../paper_2306_03078_amd/csrc/spqr_sweep16.h"

using namespace spqr_enc;

static double lds[2 * kSuper16 + 8][kRows16];

template <int B1> static void walk(int m, int n) {
  const double* U = reinterpret_cast<const double*>((uintptr_t)1 << 40);
  double* W = reinterpret_cast<double*>((uintptr_t)1 << 44);
  U_range = {reinterpret_cast<const char*>(U), (size_t)n * n * 8};
  W_range = {reinterpret_cast<const char*>(W), (size_t)m * n * 8};
  for (int row0 = 0; row0 < m; row0 += kRows16) {
    const int rows = min(kRows16, m - row0);
    for (int sb = 0; sb < n; sb += kSuper16) {
      const int next = sb + kSuper16, sbw = min(kSuper16, n - sb), from = next + kSuper16, runs = sb > 0 && from < n ? (n - from + 63) / 64 : 0;
      for (int lane = 0; lane < 64; ++lane) {
        g_what = "first corner";
        if (sb == 0)
          for (int wave = 0; wave < kWaves16; ++wave) { CornerRows<kSuper16 / kWaves16> c; fetch_corner(c, U, n, 0, wave, kWaves16, lane); }
        if (next >= n) continue;
        for (int half = 0; half < 2; ++half) {
          const int noff = (next + 64 * half + lane) * 8;
          Near N = {};
          g_what = "near factor";
          for (int j = 0; j < kSuper16; j += Near::PF) near_fetch(N.u, U, n, sb + j, noff);
          g_what = "near weights";
          near_weights(N, W, n, row0, rows, noff);
          g_what = "next corner";
          for (int b = 2; b < sbw / B1; ++b) { CornerRows<B1 / 2> c; fetch_corner(c, U, n, next, (b - 2) * B1 + half, 2, lane); }
          for (int j = kSuper16 - 2 * B1 + half; j < kSuper16; j += B1 < 8 ? 2 * B1 : 16) {
            CornerRows<B1 < 8 ? B1 : 8> c;
            fetch_corner(c, U, n, next, j, 2, lane);
          }
        }
        if (sb == 0) continue;
        g_what = "far, to the near columns";
        for (int r0 = 0; r0 < kRows16; r0 += 4) far_feedback<2, 4>(W, W, U, n, row0, rows, lane, sb - kSuper16, next, r0, lds);
        g_what = "far";
        for (int first = 0; first < runs; first += 4) {
          far_task<16>(min(4, runs - first), W, W, U, n, row0, rows, lane, sb - kSuper16, from + 64 * first, 0, lds);
          for (int r0 = 0; r0 < kRows16; r0 += 8) far_task<8>(min(4, runs - first), W, W, U, n, row0, rows, lane, sb - kSuper16, from + 64 * first, r0, lds);
        }
        for (int first = 0; first < runs; first += 2)
          for (int r0 = 0; r0 < kRows16; r0 += 8) far_task<8>(min(2, runs - first), W, W, U, n, row0, rows, lane, sb - kSuper16, from + 64 * first, r0, lds);
      }
    }
  }
}

// arguments: beta1 m n, any number of times
int main(int argc, char** argv) {
  for (int i = 1; i + 2 < argc; i += 3) {
    const int b1 = std::atoi(argv[i]), m = std::atoi(argv[i + 1]), n = std::atoi(argv[i + 2]);
    reads = writes = 0;
    std::printf("%d %d x %d ", b1, m, n);
    switch (b1) {
      case 4: walk<4>(m, n); break;
      case 8: walk<8>(m, n); break;
      case 16: walk<16>(m, n); break;
      default: walk<32>(m, n); break;
    }
    std::printf("%ld reads, %ld writes\n", reads, writes);
  }
  return 0;
}
