// Replay, on the CPU, of V+- as upper triangles and as the rows of streaming steps: the packing kernel
// (pack_vpm_tri_kernel with its LDS transposes, step_zero_kernel) and the reads of the contractions
// (tile_body_direct3 and the BF16 tiles over MapGrid, EpiStep over MapStep) through the index
// functions that the kernels call (pack_cubes.h, triangle.h). Every buffer starts poisoned.
//   - every entry that a contraction reads is written, exactly once (the diagonal of a triangle twice, as
//     its own mirror entry), with the value of its definition; nothing else is written;
//   - every K index of every result column is taken exactly once, from an address inside the rows;
//   - the steps of a partition add up to the full product, for any number of slices and sums.
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

#include "pack_cubes.h"
#include "triangle.h"

using namespace ppl;

static int failures = 0, checks = 0;
#define CHECK(cond)                                                                       \
  do {                                                                                    \
    ++checks;                                                                             \
    if (!(cond)) {                                                                        \
      fprintf(stderr, "CHECK failed at %s:%d: %s [%s]\n", __FILE__, __LINE__, #cond, where); \
      ++failures;                                                                         \
    }                                                                                     \
  } while (0)
static char where[256] = "";

static const double kPoison = std::numeric_limits<double>::quiet_NaN();
static int64_t pad64(int64_t n) { return (n + 63) / 64 * 64; }

// (pq|rs) as a small even integer with the symmetries of the integrals
static double integral(int64_t p, int64_t q, int64_t r, int64_t s) {
  if (p > q) std::swap(p, q);
  if (r > s) std::swap(r, s);
  uint64_t x = (uint64_t)(p * 1000 + q), y = (uint64_t)(r * 1000 + s);
  if (x > y) std::swap(x, y);
  uint64_t h = x * 0x9E3779B97F4A7C15ull ^ (y + 0x7F4A7C15ull) * 0xC2B2AE3D27D4EB4Full;
  h ^= h >> 29;
  h *= 0xBF58476D1CE4E5B9ull;
  return 2.0 * (double)((h >> 40) % 63) - 62.0;
}

struct Problem {
  int v;
  int64_t Pp, Pm, ldp, ldm;
  std::vector<int> first, second;             // packed pair -> (x <= y)
  std::vector<double> Vp, Vm;                 // the full matrices, Pp x Pp and Pm x Pm
  std::vector<int64_t> off;
  explicit Problem(int v_) : v(v_) {
    Pp = (int64_t)v * (v + 1) / 2;
    Pm = (int64_t)v * (v - 1) / 2;
    ldp = pad64(Pp);
    ldm = pad64(std::max<int64_t>(Pm, 1));
    for (int x = 0; x < v; ++x)
      for (int y = x; y < v; ++y) {
        first.push_back(x);
        second.push_back(y);
      }
    Vp.assign((size_t)(Pp * Pp), 0.0);
    Vm.assign((size_t)(Pm * Pm), 0.0);
    for (int64_t r = 0; r < Pp; ++r)
      for (int64_t q = 0; q < Pp; ++q) {
        const int a = first[r], b = second[r], c = first[q], d = second[q];
        const double x = integral(a, c, b, d), y = integral(a, d, b, c);
        Vp[r * Pp + q] = 0.5 * (x + y);
        if (a < b && c < d) Vm[pair_minus(a, b, v) * Pm + pair_minus(c, d, v)] = 0.5 * (x - y);
      }
    off.assign(v + 1, 0);
    for (int a = 0; a < v; ++a) off[a + 1] = off[a] + cubes_of(v, a);
  }
};

// A stored matrix: entries, and how often each was written
struct Rows {
  int64_t n, ld;
  std::vector<double> x;
  std::vector<int> hits;
  Rows(int64_t n_, int64_t ld_) : n(n_), ld(ld_), x((size_t)(n_ * ld_), kPoison), hits((size_t)(n_ * ld_), 0) {}
  bool put(int64_t r, int64_t q, double y) {
    if (r < 0 || r >= n || q < 0 || q >= ld) return false;
    x[r * ld + q] = y;
    hits[r * ld + q]++;
    return true;
  }
};

// the packing of the step [a0, a1) into vp, vm (stored rows from row0p / row0m on)
static void pack(const Problem& P, int a0, int a1, bool step, Rows& vp, Rows& vm, int64_t row0p, int64_t row0m) {
  const int v = P.v, C = kCube, LD = kCube + 1, LB = kCube * LD + 1;
  const int64_t pr0 = pair_plus(a0, a0, v), W = v - a0, ldt = W * (W + 1) / 2;
  const int64_t M = (a1 >= v ? P.Pp : pair_plus(a1, a1, v)) - pr0;
  const int64_t g0 = P.off[a0], n = P.off[a1] - g0;
  bool ok = true;
  std::vector<int> seen((size_t)n, 0);
  for (int64_t bid = 0; bid < n; ++bid) {
    const int64_t g = g0 + cube_of_slot(bid, n);
    if (g < g0 || g >= g0 + n) { ok = false; continue; }
    seen[(size_t)(g - g0)]++;
    const int a = cube_virtual(P.off.data(), a0, a1, g);
    int bi = -1, ci = -1, di = -1;
    const int nt = cube_blocks(v, a);
    cube_decode_rows(g - P.off[a], nt, bi, ci, di);
    if (a < a0 || a >= a1 || bi < 0 || bi >= nt || ci < 0 || ci > di || di >= nt) { ok = false; continue; }
    const int b0 = a + C * bi, c0 = a + C * ci, d0 = a + C * di;
    auto at = [&](int r, int x, int y) {
      const int lo = std::min(x, y), hi = std::max(x, y);
      if (!(r < v && hi < v)) return 0.0;
      const int64_t m = pair_plus(a, r, v) - pr0, col = pair_plus(lo, hi, v) - pr0;
      // (columns left of the row's virtual are not computed by the build)
      if (m < 0 || m >= M || col < 0 || col >= ldt || lo < a) { ok = false; return kPoison; }
      return integral(a, r, lo, hi);
    };
    double s[kCube * (kCube * (kCube + 1) + 1)];
    static double gcd[256][kCube], gdc[256][kCube];
    auto each = [&](auto fn) {
      for (int t = 0; t < 256; ++t) fn(t, t & 15, t >> 4);
    };
    const bool swapped = bi > di;
    each([&](int t, int f, int m) {
      for (int k = 0; k < C; ++k) gdc[t][k] = bi <= ci ? at(d0 + m, b0 + k, c0 + f) : at(d0 + k, c0 + m, b0 + f);
    });
    if (swapped) {
      each([&](int t, int f, int m) {
        for (int k = 0; k < C; ++k) s[f * LB + k * LD + m] = at(c0 + m, d0 + k, b0 + f);
      });
      each([&](int t, int f, int m) {
        for (int k = 0; k < C; ++k) gcd[t][k] = s[k * LB + f * LD + m];
      });
    } else {
      each([&](int t, int f, int m) {
        for (int k = 0; k < C; ++k) gcd[t][k] = at(c0 + m, b0 + k, d0 + f);
      });
    }
    each([&](int t, int f, int m) {
      for (int k = 0; k < C; ++k) {
        if (bi <= ci) s[k * LB + m * LD + f] = gdc[t][k];
        else s[f * LB + k * LD + m] = gdc[t][k];
      }
    });
    each([&](int t, int f, int m) {
      for (int k = 0; k < C; ++k) gdc[t][k] = s[k * LB + f * LD + m];
    });
    each([&](int t, int f, int m) {
      const int c = c0 + m, d = d0 + f;
      if (!(d < v && c <= d)) return;
      const int kmax = cube_rows(v, a, b0, c, d);
      const int64_t rp = pair_plus(a, b0, v), cp = pair_plus(c, d, v);
      const int64_t rm = pair_minus(a, b0, v), cm = pair_minus(c, d, v);
      const bool near = !step && cube_near(v, a, b0, c0, d0);
      for (int k = 0; k < kmax && k < C; ++k) {
        const double x = gcd[t][k], y = gdc[t][k];
        const bool minus = c < d && (k > 0 || b0 > a);
        const double w = step && cp == rp + k ? 0.25 : 0.5;
        ok &= vp.put(rp + k - row0p, cp, w * (x + y));
        if (minus) ok &= vm.put(rm + k - row0m, cm, w * (x - y));
        if (near) {
          if ((rp + k) / kTriBlock == cp / kTriBlock) ok &= vp.put(cp, rp + k, 0.5 * (x + y));
          if (minus && (rm + k) / kTriBlock == cm / kTriBlock) ok &= vm.put(cm, rm + k, 0.5 * (x - y));
        }
      }
    });
    if (ci == 0 && di == 0)
      for (int b = b0; b < std::min(v, b0 + C); ++b) {
        for (int64_t q = P.Pp; q < P.ldp; ++q) ok &= vp.put(pair_plus(a, b, v) - row0p, q, 0.0);
        if (a < b)
          for (int64_t q = P.Pm; q < P.ldm; ++q) ok &= vm.put(pair_minus(a, b, v) - row0m, q, 0.0);
      }
  }
  for (int x : seen) ok = ok && x == 1;
  CHECK(ok);
}

// what a resident triangle must hold: V at and right of the diagonal and in diagonal blocks, zero padding
static void check_triangle(const Rows& R, const std::vector<double>& V, int64_t N) {
  bool exact = true;
  for (int64_t r = 0; r < N; ++r)
    for (int64_t q = 0; q < R.ld; ++q) {
      const bool pad = q >= N, valid = pad || q >= r || q / kTriBlock == r / kTriBlock;
      const double x = R.x[r * R.ld + q];
      exact = exact && R.hits[r * R.ld + q] == (!valid ? 0 : r == q ? 2 : 1);
      exact = exact && (!valid || x == (pad ? 0.0 : V[r * N + q]));
    }
  CHECK(exact);
}

// the reads of a contraction over a resident triangle, on tiles of bn columns and chunks of kc
static void check_triangle_reads(const Rows& R, const std::vector<double>& V, int64_t N, int bn, int kc, int splits) {
  const int64_t nk = R.ld / kc;
  splits = (int)std::min<int64_t>(splits, nk);
  const int64_t kps = (nk + splits - 1) / splits;
  splits = (int)((nk + kps - 1) / kps);
  bool inside = true, exact = true;
  for (int64_t n0 = 0; n0 < N; n0 += bn) {
    std::vector<int> taken((size_t)(bn * R.ld), 0);
    for (int s = 0; s < splits; ++s) {
      const int64_t kc0 = s * kps, kc1 = std::min(nk, kc0 + kps), cd = tri_split(n0, kc0, kc1, kc);
      if (cd < kc0 || cd > kc1) { inside = false; continue; }
      for (int64_t k = kc0 * kc; k < kc1 * kc; ++k)
        for (int64_t n = n0; n < n0 + bn; ++n) {
          const int64_t row = k < cd * kc ? k : std::min(n, N - 1), col = k < cd * kc ? n : k;
          const int64_t at = row * R.ld + col;       // (a tile's last columns may run into the next row)
          if (at < 0 || at >= N * R.ld) { inside = false; continue; }
          if (n >= N) continue;
          taken[(n - n0) * R.ld + k]++;
          exact = exact && R.x[at] == (k < N ? V[n * N + k] : 0.0);
        }
    }
    for (int64_t n = n0; n < std::min(N, n0 + bn); ++n)
      for (int64_t k = 0; k < R.ld; ++k) exact = exact && taken[(n - n0) * R.ld + k] == 1;
  }
  CHECK(inside && exact);
}

// One row of S against the rows of a step, as the step kernel accumulates it: `sums` sums, slice s
// into sum s mod sums. rows: stored rows that the plan holds.
static void step_product(const std::vector<double>& S, const Rows& U, int64_t rows, int64_t N, int64_t p0, int64_t p1,
                         bool first, int bn, int splits, int sums, std::vector<std::vector<double>>& C) {
  const int kc = kStepRows;
  const int64_t k0 = step_row0(p0), nk = U.ld / kc;
  bool inside = true;
  for (int s0 = 0; s0 < splits; s0 += sums)
    for (int j = 0; j < std::min(sums, splits - s0); ++j)
      for (int64_t n0 = p0 / bn * bn; n0 < N; n0 += bn) {
        const StepChunks c = step_chunks(n0, bn, p0, p1, nk, kc, s0 + j, splits);
        inside = inside && c.c0 * kc >= k0 && c.cd * kc - k0 <= rows && c.t0 >= 0 && c.c1 <= nk;
        for (int64_t n = n0; n < n0 + bn; ++n) {
          double acc = 0.0;
          for (int64_t k = c.c0 * kc; k < c.cd * kc; ++k) {
            const int64_t at = (k - k0) * U.ld + n;
            // (the last tile's surplus columns: the following row, at the very end at most bn elements behind)
            inside = inside && at >= 0 && at < rows * U.ld + (n >= N ? bn : 0);
            if (n < N) acc += S[k] * U.x[at];
          }
          for (int64_t k = c.t0 * kc; k < c.c1 * kc; ++k) {
            const int64_t at = step_row(std::min(n, N - 1), p0, p1) * U.ld + k;
            inside = inside && at >= 0 && at < rows * U.ld;
            if (n < N) acc += S[k] * U.x[at];
          }
          if (n >= N) continue;
          if (first && s0 == 0) C[j][n] = acc;
          else C[j][n] += acc;
        }
      }
  CHECK(inside);
}

static void check_steps(const Problem& P, const std::vector<int>& cuts) {
  const int v = P.v;
  int64_t most = 0;
  for (size_t i = 0; i + 1 < cuts.size(); ++i) {
    const int a1 = cuts[i + 1];
    most = std::max(most, (a1 >= v ? P.Pp : pair_plus(a1, a1, v)) - pair_plus(cuts[i], cuts[i], v));
  }
  const int64_t rows = most + 2 * kStepRows - 1;
  // the row of S: zero in its padding
  auto row = [&](int64_t N, int64_t ld) {
    std::vector<double> S((size_t)ld, 0.0);
    for (int64_t k = 0; k < N; ++k) S[k] = (double)((k * 37 + 11) % 41) - 20.0;
    return S;
  };
  const std::vector<double> Sp = row(P.Pp, P.ldp), Sm = row(P.Pm, P.ldm);
  std::vector<double> refp(P.Pp, 0.0), refm(P.Pm, 0.0);
  for (int64_t n = 0; n < P.Pp; ++n)
    for (int64_t k = 0; k < P.Pp; ++k) refp[n] += Sp[k] * P.Vp[n * P.Pp + k];
  for (int64_t n = 0; n < P.Pm; ++n)
    for (int64_t k = 0; k < P.Pm; ++k) refm[n] += Sm[k] * P.Vm[n * P.Pm + k];
  struct Step {
    Rows up, um;
    int64_t p0, p1, q0, q1;
  };
  std::vector<Step> steps;
  for (size_t i = 0; i + 1 < cuts.size(); ++i) {
    const int a0 = cuts[i], a1 = cuts[i + 1];
    const int64_t p0 = pair_plus(a0, a0, v), p1 = a1 >= v ? P.Pp : pair_plus(a1, a1, v);
    const int64_t q0 = a0 + 1 < v ? pair_minus(a0, a0 + 1, v) : P.Pm, q1 = a1 + 1 < v ? pair_minus(a1, a1 + 1, v) : P.Pm;
    Step s{Rows(rows, P.ldp), Rows(rows, P.ldm), p0, p1, q0, q1};
    pack(P, a0, a1, true, s.up, s.um, step_row0(p0), step_row0(q0));
    auto zero = [&](Rows& U, int64_t r0, int64_t r1) {
      bool ok = true;
      for (int64_t x = 0; x < r1 - step_row0(r0) + kStepRows; ++x) {
        const int64_t k = step_row0(r0) + x;
        for (int64_t c = step_zero_from(k, r0, r1); c < step_zero_to(k, r0, r1, U.ld); ++c) ok &= U.put(x, c, 0.0);
      }
      for (int h : U.hits) ok = ok && h <= 1;
      CHECK(ok);
    };
    zero(s.up, p0, p1);
    if (q1 > q0) zero(s.um, q0, q1);
    steps.push_back(s);
  }
  for (int bn : {64, 128, 256})
    for (int splits : {1, 3, 8})
      for (int sums : {1, 2, 8}) {
        std::vector<std::vector<double>> Cp(sums, std::vector<double>(P.Pp, 0.0)), Cm(sums, std::vector<double>(P.Pm, 0.0));
        bool first = true;
        for (const Step& s : steps) {
          step_product(Sp, s.up, rows, P.Pp, s.p0, s.p1, first, bn, splits, sums, Cp);
          if (s.q1 > s.q0) step_product(Sm, s.um, rows, P.Pm, s.q0, s.q1, first, bn, splits, sums, Cm);
          first = false;
        }
        bool exact = true;             // (integers and halves: every sum is exact)
        auto sum = [&](const std::vector<std::vector<double>>& C, int64_t n) {
          double x = 0.0;
          for (int j = 0; j < std::min(sums, splits); ++j) x += C[j][n];
          return x;
        };
        for (int64_t n = 0; n < P.Pp; ++n) exact = exact && sum(Cp, n) == refp[n];
        for (int64_t n = 0; n < P.Pm; ++n) exact = exact && sum(Cm, n) == refm[n];
        CHECK(exact);
      }
}

int main() {
  // (P+, P-) from one pair over chunk, tile and block edges: 256-blocks start to matter at v = 23
  for (int v : {1, 2, 3, 10, 16, 17, 23, 32, 33, 45}) {
    const Problem P(v);
    for (int nsteps : {1, 3})
      for (int reverse = 0; reverse < 2; ++reverse) {
        snprintf(where, sizeof(where), "triangle v=%d steps=%d reverse=%d", v, nsteps, reverse);
        Rows vp(P.Pp, P.ldp), vm(std::max<int64_t>(P.Pm, 1), P.ldm);
        for (int i = 0; i < nsteps; ++i) {
          const int k = reverse ? nsteps - 1 - i : i, a0 = v * k / nsteps, a1 = v * (k + 1) / nsteps;
          if (a0 < a1) pack(P, a0, a1, false, vp, vm, 0, 0);
        }
        check_triangle(vp, P.Vp, P.Pp);
        check_triangle(vm, P.Vm, P.Pm);
        if (nsteps > 1) continue;
        for (int bn : {64, 128, 256})
          for (int kc : {16, 32, 64})
            for (int splits : {1, 3, 8}) {
              check_triangle_reads(vp, P.Vp, P.Pp, bn, kc, splits);
              if (P.Pm > 0) check_triangle_reads(vm, P.Vm, P.Pm, bn, kc, splits);
            }
      }
    if (v < 2) continue;
    for (int kind = 0; kind < 3; ++kind) {
      std::vector<int> cuts{0};      // one virtual at a time, a few, all at once
      while (cuts.back() < v) cuts.push_back(std::min(v, cuts.back() + (kind == 0 ? 1 : kind == 1 ? 4 + cuts.back() / 3 : v)));
      if (kind == 0 && v > 23) continue;
      snprintf(where, sizeof(where), "steps v=%d kind=%d", v, kind);
      check_steps(P, cuts);
    }
  }
  printf("triangle checks: %d of %d failed\n", failures, checks);
  return failures ? 1 : 0;
}
