// Index arithmetic of V+- stored as upper triangles, and of the rows that a streaming step holds.
// Shared by the kernels and their replay on the host.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define PPL_HD __host__ __device__
#else
#define PPL_HD
#endif

namespace ppl {

// ------------------------------------------------------------------ pair indices
// Row-major packed upper triangles of an n x n index space:
//   plus : pairs (a, b) with a <= b, index a*n - a(a+1)/2 + b
//   minus: pairs (a, b) with a <  b, index a*(n-1) - a(a+1)/2 + b - 1
PPL_HD inline int64_t pair_plus(int64_t a, int64_t b, int64_t n) { return a * n - a * (a + 1) / 2 + b; }
PPL_HD inline int64_t pair_minus(int64_t a, int64_t b, int64_t n) { return a * (n - 1) - a * (a + 1) / 2 + b - 1; }

// Resident V+- are stored as upper triangles: entry [r][q] is valid where
// q >= r or r / kTriBlock == q / kTriBlock (whole diagonal blocks), and the rest is never
// read. Every column tile of a contraction (64, 128 or 256 wide, from a multiple of its
// width) then lies in one diagonal block.
constexpr int kTriBlock = 256;

// Of the K chunks [kc0, kc1) of column tile n0, those from the returned one on are read along rows n
// of a triangular operand, the ones before it (k < n0) along its rows k.
PPL_HD inline int64_t tri_split(int64_t n0, int64_t kc0, int64_t kc1, int kc) {
  const int64_t c = n0 / kc;
  return c < kc0 ? kc0 : (c > kc1 ? kc1 : c);
}

// ------------------------------------------------------------------ streaming steps
// A step holds the rows [p0, p1) of U (V = U + U^T: entries at and right of the row's own pair, its
// diagonal halved) from global row step_row0(p0) on, zero in the rows before p0 and in kStepRows rows
// from p1 on, and in the columns of a row's kTriBlock block before its own pair.
constexpr int kStepRows = 16;
PPL_HD inline int64_t step_row0(int64_t p0) { return p0 / kStepRows * kStepRows; }

// first and last + 1 of the columns of global row k that are zeroed
PPL_HD inline int64_t step_zero_from(int64_t k, int64_t p0, int64_t p1) {
  return (k >= p0 && k < p1 ? k : step_row0(p0)) / kTriBlock * kTriBlock;
}
PPL_HD inline int64_t step_zero_to(int64_t k, int64_t p0, int64_t p1, int64_t ld) { return k >= p0 && k < p1 ? k : ld; }

// The stored row that column n of the result takes: columns outside the step take a zero row.
PPL_HD inline int64_t step_row(int64_t n, int64_t p0, int64_t p1) {
  const int64_t k0 = step_row0(p0);
  return n < k0 || n >= p1 ? p1 - k0 : n - k0;
}

// Slice s of `splits` of column tile [n0, n0 + bn): chunks [c0, cd) of kc rows of U, K-major (U^T, the
// step's rows k < n0 + bn), then, where the tile meets the step's own columns, chunks [t0, c1) along
// the rows n (U, from the tile's first column to chunk nk, the end of a row).
struct StepChunks {
  int64_t c0, cd, t0, c1;
};
PPL_HD inline StepChunks step_chunks(int64_t n0, int bn, int64_t p0, int64_t p1, int64_t nk, int kc, int s, int splits) {
  const int64_t ka = step_row0(p0) / kc, ke = (p1 + kc - 1) / kc, ne = (n0 + bn) / kc;
  const int64_t nn = (ke < ne ? ke : ne) - ka;
  const int64_t ta = n0 / kc > ka ? n0 / kc : ka, total = nn + (n0 < p1 ? nk - ta : 0);
  const int64_t lo = total * s / splits, hi = total * (s + 1) / splits;
  return StepChunks{ka + (lo < nn ? lo : nn), ka + (hi < nn ? hi : nn), ta + (lo > nn ? lo - nn : 0),
                    ta + (hi > nn ? hi - nn : 0)};
}

}  // namespace ppl
