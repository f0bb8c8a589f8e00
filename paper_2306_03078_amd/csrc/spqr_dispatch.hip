// Which kernels a product call takes: host logic only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>

#include "../../include/spqr.h"
#include "spqr_kernels.h"

namespace spqr {

// Process-wide switches for tuning runs and tests (spqr_set_option); all zero in production.
static std::atomic<int> g_options[SPQR_OPT_COUNT_];
int option(int which) {
  return which >= 0 && which < SPQR_OPT_COUNT_ ? g_options[which].load(std::memory_order_relaxed) : 0;
}
bool set_option(int which, int value) {
  if (which < 0 || which >= SPQR_OPT_COUNT_) return false;
  g_options[which].store(value, std::memory_order_relaxed);
  return true;
}

// Smallest batch the matrix-core path is considered for (below it the vector kernel's 2- and 4-vector forms win
// or tie on every layer measured).
static constexpr int kMfmaMinBatch = 4;

// Y[b][m] = X[b][n] . W_hat^T.  Up to 4 activation vectors: the tuned vector kernel, all of them in one launch
// (4 vectors on a large layer: the matrix cores, see mfma_wanted).  More, where a matrix-core instance exists and
// it pays: slices of up to 16 on the matrix cores (weights stream once per slice), outliers in the same kernel, then the
// partial results are added.  Else slices of 4.
// ws.from_caller: scratch comes from the caller; nothing is allocated, freed or waited for, the choice of path
// never depends on the stream's state, and a workspace that is too small is hipErrorOutOfMemory.
hipError_t launch_gemm(const DevMatrix& A, const uint16_t* X, int b, void* Y, int y_dtype,
                       hipStream_t stream, const Workspace& ws) {
  const Geometry& g = A.g;
  const size_t ysz = y_dtype == SPQR_F32 ? 4 : 2;
  const bool force_generic = option(SPQR_OPT_FORCE_GENERIC) != 0;
  bool mfma_ok = !force_generic && mfma_has_instance(g);
  const bool alloc_nodes = mfma_ok && !ws.from_caller && b >= kMfmaMinBatch && stream_is_capturing(stream);
  // A prompt-sized batch: the product straight from the compressed weights, or (formats, sizes and outlier rates that path does
  // not take) one dense binary16 copy of the matrix in scratch and one matrix-core multiply for all vectors.  Both write Y 16
  // bytes at a time.
  const BatchRoute route = force_generic || reinterpret_cast<uintptr_t>(Y) % 16 != 0 ? kRouteSlices : batch_route(A, b, ws);
  if (route != kRouteSlices) {
    const hipError_t e = route == kRouteOnePass ? launch_prompt_scratch(&A, 1, X, b, &Y, y_dtype, stream, ws)
                                                : launch_prefill_scratch(A, X, b, Y, y_dtype, stream, ws);
    if (e != hipErrorNotSupported) return e;   // no library scratch of that size to be had: the slices below
  }
  int k = 0;
  while (k < b) {
    const uint16_t* xk = X + (size_t)k * g.n;
    void* yk = static_cast<uint8_t*>(Y) + (size_t)k * g.m * ysz;
    const int left = b - k;
    hipError_t e;
    int done = 1;
    // the matrix-core path takes up to 16 vectors per pass over the weights
    const int nb16 = left < 16 ? left : 16;
    if (mfma_ok && left >= kMfmaMinBatch && mfma_wanted(g, nb16, alloc_nodes)) {
      e = launch_mfma(A, xk, nb16, yk, y_dtype, stream, ws);
      if (e == hipErrorNotSupported) { mfma_ok = false; continue; }   // no scratch to be had: the vector path from now on
      if (e != hipSuccess) return e;
      k += nb16;
      continue;
    }
    const int nb = force_generic ? 0 : tuned_batch_width(g, left);
    if (nb >= 1) { e = launch_tuned(A, xk, nb, yk, y_dtype, stream); done = nb; }
    else e = launch_generic(A, xk, yk, y_dtype, stream);
    if (e != hipSuccess) return e;
    k += done;
  }
  return hipSuccess;
}

BatchRoute batch_route(const DevMatrix& A, int b, const Workspace& ws) {
  if (prompt_wanted(A, b) && prompt_fit(&A, 1, b, ws) >= 0) return kRouteOnePass;
  const bool copy = prefill_has_instance(A.g) && prefill_wanted(A, b) && (!ws.from_caller || ws.bytes >= prefill_workspace_bytes(A, b));
  return copy ? kRouteCopy : kRouteSlices;
}

// Whether launch_gemm_fused gives several matrices to the one-pass kernel together: where all of them are its own and that is
// faster than one after the other by its plans' model.  It hardly ever is not: the partial results of all of them have the room of
// one's (64 MB), so with very many rows and vectors groups of rows have to stay whole.  (Gate and up 17920 x 6656, 4-bit, 256
// vectors: 236 to 262 us together, 222 one by one; 22016 x 8192 289 and 361; the model 304 and 280, 398 and 424.)
static bool prompt_set_wanted(const DevMatrix* As, int count, int b) {
  if (count < 2) return false;
  int64_t nnz = 0;                           // (counted in 32 bits there)
  double apart = 0.0;
  for (int i = 0; i < count; ++i) {
    if (!prompt_wanted(As[i], b)) return false;
    nnz += As[i].nnz;
    apart += prompt_us(&As[i], 1, b);
  }
  return nnz < 0x7FFF0000ll && (option(SPQR_OPT_PROMPT_PLAN) >= 1 || prompt_us(As, count, b) <= apart);
}

// Whether launch_gemm_fused takes the fused matrix-core launches for a slice of nb vectors.
static bool fused_mfma_wanted(const DevMatrix* As, int count, int nb, bool alloc_nodes) {
  Geometry all = As[0].g;                    // the rule looks at the weights of all matrices together
  int64_t rows = 0;
  for (int i = 0; i < count; ++i) rows += As[i].g.m;
  all.m = (int)(rows < (1 << 30) ? rows : (1 << 30));
  return nb >= kMfmaMinBatch && mfma_wanted(all, nb, alloc_nodes);
}

// Y_i[b][m_i] = X[b][n] . W_hat_i^T for matrices that share X.  Batches the matrix-core path takes go through it
// fused (slices of 16); everything else is one launch_gemm per matrix.
hipError_t launch_gemm_fused(const DevMatrix* As, int count, const uint16_t* X, int b, void* const* Ys, int y_dtype,
                             hipStream_t stream, const Workspace& ws) {
  const Geometry& g = As[0].g;
  const size_t ysz = y_dtype == SPQR_F32 ? 4 : 2;
  const bool force_generic = option(SPQR_OPT_FORCE_GENERIC) != 0;
  bool mfma_ok = count > 1 && !force_generic && mfma_has_instance(g);
  // Not while the stream is being captured into a graph: a replay of a graph that held 12 fused batch calls among
  // 42 calls (a whole decoder block, six weight copies) once ended in a memory fault inside the fused kernel that
  // added the outliers (gone since: batch_group_fused_kernel adds them), while the same calls passed eagerly and
  // graphs of the per-matrix path replay correctly; the cause was never known, so captured calls take the per-matrix path.
  // That holds for the one-pass kernel's sets too: it is another kernel, but several matrices in a captured launch set are what
  // the calls of that graph had and the others had not.  (Results then differ from the eager call's in the order of sums.)
  const bool capturing = mfma_ok && b >= kMfmaMinBatch && stream_is_capturing(stream);
  if (capturing) mfma_ok = false;
  // a large batch: all matrices in the launches of the one-pass kernel where every one of them takes it, else one matrix at a
  // time (launch_gemm falls back to the slices where it has to)
  bool dense = !force_generic && prefill_has_instance(g);
  for (int i = 0; i < count && dense; ++i) dense = prefill_wanted(As[i], b);   // (prompt_wanted is a part of that)
  if (dense) {
    bool one_pass = mfma_ok && prompt_set_wanted(As, count, b);
    for (int i = 0; i < count && one_pass; ++i) one_pass = reinterpret_cast<uintptr_t>(Ys[i]) % 16 == 0;
    if (one_pass) {
      const hipError_t e = launch_prompt_scratch(As, count, X, b, Ys, y_dtype, stream, ws);
      if (e != hipErrorNotSupported) return e;
    }
    mfma_ok = false;
  }
  int k = 0;
  while (k < b) {
    const int left = b - k, nb16 = left < 16 ? left : 16;
    const uint16_t* xk = X + (size_t)k * g.n;
    void* yk[SPQR_MAX_FUSED];
    for (int i = 0; i < count; ++i) yk[i] = static_cast<uint8_t*>(Ys[i]) + (size_t)k * As[i].g.m * ysz;
    if (mfma_ok && fused_mfma_wanted(As, count, nb16, false)) {
      hipError_t e = launch_mfma_fused(As, count, xk, nb16, yk, y_dtype, stream, ws);
      if (e == hipErrorNotSupported) { mfma_ok = false; continue; }
      if (e != hipSuccess) return e;
      k += nb16;
      continue;
    }
    // the rest of the batch, matrix by matrix (each call applies its own rule)
    for (int i = 0; i < count; ++i) {
      hipError_t e = launch_gemm(As[i], xk, left, yk[i], y_dtype, stream, ws);
      if (e != hipSuccess) return e;
    }
    k = b;
  }
  return hipSuccess;
}

// Device scratch a product of these matrices with a batch of b needs at most when the caller brings it
// (0: the call takes kernels that need none).  One matrix: launch_gemm; several: launch_gemm_fused, which may
// fall back to one launch_gemm per matrix, so the bound covers both.
size_t workspace_bound(const DevMatrix* As, int count, int b, bool with_dense_copy) {
  if (option(SPQR_OPT_FORCE_GENERIC) != 0) return 0;
  size_t worst = 0;
  // a large batch: one matrix at a time, in one pass or through the dense copy (a smaller workspace sends the call to the
  // slices of 16, see prompt_line_bytes)
  if (with_dense_copy && prefill_has_instance(As[0].g))
    for (int i = 0; i < count; ++i) {
      if (!prefill_wanted(As[i], b)) continue;
      if (prompt_wanted(As[i], b)) worst = std::max({worst, prompt_workspace_bytes(&As[i], 1, b), prompt_line_bytes(As[i], b)});
      else worst = std::max(worst, prefill_workspace_bytes(As[i], b));
    }
  if (with_dense_copy && prompt_set_wanted(As, count, b)) {
    const size_t need = prompt_workspace_bytes(As, count, b);
    if (need > worst) worst = need;
  }
  if (!mfma_has_instance(As[0].g) || b < kMfmaMinBatch) return worst;
  // slices of 16, then the rest: the needs of min(b, 16) vectors and of the last slice bound all of them
  const int sizes[2] = {b < 16 ? b : 16, b % 16};
  for (int si = 0; si < 2; ++si) {
    const int nb = sizes[si];
    if (nb < kMfmaMinBatch) continue;
    const bool fused = count > 1 && fused_mfma_wanted(As, count, nb, false);
    bool any_single = false;
    for (int i = 0; i < count; ++i) any_single = any_single || mfma_wanted(As[i].g, nb, false);
    if (!fused && !any_single) continue;
    const size_t need = mfma_workspace_bound(As, count, nb, fused);
    if (need > worst) worst = need;
  }
  return worst;
}

hipError_t launch_gemv(const DevMatrix& A, const uint16_t* x, void* y, int y_dtype, hipStream_t stream) {
  Workspace none;
  return launch_gemm(A, x, 1, y, y_dtype, stream, none);
}

}  // namespace spqr
