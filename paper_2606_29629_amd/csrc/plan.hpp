// Arithmetic of the launches that needs no GPU (no HIP in here: the host tests
// compile it by itself).
#pragma once

#include <stdint.h>

namespace tri {

constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }

// Bytes of a residual [M, ld] (bf16) that a tile of `rows` rows at (row0, col0)
// may read, counted from its first element: its valid rows, and in the last of
// them nothing past the row's end (for the last row, the tensor's).
constexpr int resid_range_bytes(int M, int ld, int row0, int col0, int rows) {
  const int valid = rows < M - row0 ? rows : M - row0;
  return (valid * ld - col0) * 2;
}

// A launch holds fewer than 2^32 threads per grid dimension: of the jobs
// first .. n - 1 with `threads` threads each, the end of those that fit in one
// launch together (at least one: a job that does not fit fails as it would alone).
constexpr int64_t kMaxGridThreads = ((int64_t)1 << 32) - 256;
constexpr int jobs_of_launch(const int64_t* threads, int first, int n) {
  int64_t sum = threads[first];
  int end = first + 1;
  while (end < n && sum + threads[end] <= kMaxGridThreads) sum += threads[end++];
  return end;
}

}  // namespace tri
