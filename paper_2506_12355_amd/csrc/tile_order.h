// The order in which workgroups take causal query blocks that all run at once,
// two or three to a CU.
#pragma once

#include <hip/hip_runtime.h>

namespace qm {

// The tile of workgroup w (runs on XCD w % 8) of `total`.  The tiles' query blocks lie
// head by head, each head's nq longest first; tile t is block (t % 8) P + t / 8 with
// P = total / 8, the last total % 8 tiles are the last blocks.
//
// An XCD's workgroups reach its `row` CUs in rows: the first `row` of them one to a
// CU, the next `row` beside these, and so on.  A long block is to share a CU with a
// short one, so of the XCD's blocks (a range of P or P + 1) the longest take the first
// row, longest first, and the next the second, shortest first.  (Head by head instead,
// a CU could hold the longest blocks of two heads.  Heads of two blocks stay head by
// head, the second row from the end.)  us, B = 1, head by head -> so: d = 128 bf16
// N = 2048 H = 24 47.5 -> 36.6, H = 32 42.0 -> 41.4, N = 1024 H = 40 27.3 -> 22.1; d = 64
// N = 2048 H = 40 45.8 -> 31.6; FP8 N = 2048 H = 24 34.7 -> 25.6; at worst N = 320
// H = 160 14.8 -> 15.5, where a head's last block is half empty.
//
// heads: heads per XCD where they are whole, else 0.
__host__ __device__ constexpr int balanced_tile(int w, int total, int row, int nq, int heads) {
  const int x = w % 8, j = w / 8, p = total / 8, left = total % 8;
  const int n = p + (x < left);   // the XCD's blocks
  const int rest = n - row, second = rest < row ? rest : row;
  const bool in_second = j >= row && j < row + second;
  if (nq == 2 && heads) return (in_second ? n - 1 - (j - row) : j < row ? j : j - row) * 8 + x;
  // k: how many of the XCD's blocks are longer than this one (or as long and before it);
  // i: the block's place in its head, 0 the longest; r: the head, of those with this place
  const int k = in_second ? 2 * row + second - 1 - j : j;
  if (heads) {
    const int i = k / heads, r = k - i * heads;
    return (r * nq + i) * 8 + x;
  }
  // the first f blocks of the XCD's first head and all but e of its last belong to its
  // neighbours
  const int first = x * p + (x < left ? x : left);
  const int f = first % nq;
  heads = (f + n + nq - 1) / nq;
  const int e = f + n - (heads - 1) * nq;
  int i = k / heads, r = 0;
  for (;; ++i) {
    r = k - (i * heads - (i < f ? i : f) - (i > e ? i - e : 0));
    if (r < heads - (i < f) - (i >= e)) break;
  }
  const int id = first - f + (r + (i < f)) * nq + i;
  return id < 8 * p ? id % p * 8 + id / p : id;
}

}  // namespace qm
