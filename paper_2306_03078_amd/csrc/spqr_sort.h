// Index arithmetic of the outlier sort of spqr_prompt.hip, shared with the host (its test runs there).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spqr {

constexpr int kSortChunk = 4096;             // entries a workgroup counts or places at a time

struct GroupRange { int s, z; };             // entries s .. z - 1

// The entries of a group of `rows` rows.  Row pointers are trusted to be a valid prefix everywhere else; here they also size
// writes, so whatever they hold 0 <= s <= z <= nnz.  (The dense copy finds rows by bisection and stays in bounds with any
// row pointers, and these are calls that took it.)
__host__ __device__ inline GroupRange group_range(const int32_t* row_ptr, int group, int rows, int m, int nnz) {
  const int lo = row_ptr[group * rows], hi = row_ptr[group * rows + rows < m ? group * rows + rows : m];
  const int s = lo < 0 ? 0 : (lo > nnz ? nnz : lo);
  return {s, hi < s ? s : (hi > nnz ? nnz : hi)};
}
__host__ __device__ inline int sort_chunks(GroupRange r) { return (r.z - r.s + kSortChunk - 1) / kSortChunk; }
// Chunk k of group g counts into this slot; a chunk never spans two groups, and with a valid prefix no two chunks share one.
__host__ __device__ inline int64_t count_slot(GroupRange r, int group, int k) { return (int64_t)(r.s / kSortChunk) + group + k; }
inline int64_t count_slots(int64_t nnz, int groups) { return nnz / kSortChunk + groups + 1; }

}  // namespace spqr
