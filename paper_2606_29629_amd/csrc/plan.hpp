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

// Most rows with which a projection of N weight rows over K runs as a weight
// stream (gemm_stream.hip); beyond them it takes the skinny tiles, split in K.
// paired: SwiGLU and q/k/v, whose blocks hold 32 weight rows instead of 16.
//
// A stream's workgroup walks the whole K alone, so a narrow matrix with a long
// K has too few of them, and the more rows the longer each k-tile takes; the
// skinny tiles pay a second launch, but split K over all CUs.  Measured (skinny
// against stream, us): wide, 3584 x 18944 at 12 / 16 rows 31.1 / 31.2 against
// 30.6 / 33.0, 4096 x 16384 at 16 34.7 against 31.8; narrow, 1024 x 4096 at 5 / 16
// rows 8.4 / 8.7 against 6.7 / 7.7, 1024 x 8192 9.9 / 10.2 against 9.8 / 12.0, 1024 x
// 16384 12.5 / 12.8 against 16.8 / 21.2, 2048 x 8192 12.4 / 12.6 against 12.5 / 13.9;
// paired (a layer's stage), gate/up 1024 x 8192 11.8 / 12.4 against 15.0 / 17.7, 2048
// x 4096 11.8 / 11.9 against 10.6 / 12.3, q/k/v 1024 x 6144 13.9 / 14.0 against 14.7
// / 16.9, 768 x 4096 13.0 / 12.9 against 11.3 / 12.7.
constexpr int kStreamMaxRows = 16;
constexpr int stream_rows(int N, int K, bool paired) {
  const bool wide = N >= (paired ? 4096 : 3072);
  const int most = wide ? (1 << 18) / K : (paired ? 164000 : 215000) / K - 24;
  return most < 0 ? 0 : most < kStreamMaxRows ? most : kStreamMaxRows;
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
