// Arithmetic of the launches that needs no GPU (no HIP in here: the host tests
// compile it by itself).
#pragma once

namespace tri {

constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }

// Bytes of a residual [M, ld] (bf16) that a tile of `rows` rows at (row0, col0)
// may read, counted from its first element: its valid rows, and in the last of
// them nothing past the row's end (for the last row, the tensor's).
constexpr int resid_range_bytes(int M, int ld, int row0, int col0, int rows) {
  const int valid = rows < M - row0 ? rows : M - row0;
  return (valid * ld - col0) * 2;
}

}  // namespace tri
