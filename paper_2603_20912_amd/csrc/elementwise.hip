// Memory-bound kernels around the MFMA GEMMs: staging of the Cholesky blocks,
// packing into the symmetric/antisymmetric pair layout, unpacking of results,
// the packed Jacobi update with its FP64 residual/energy reductions.
//
// Pair layout (i<=j / a<=b, "+"; i<j / a<b, "-"), for pair-symmetric t
// (t_ij^ab = t_ji^ba, eq. (2)):
//   s_ij^ab = (t_ij^ab + t_ij^ba)/2 is symmetric in (a,b) and in (i,j),
//   a_ij^ab = (t_ij^ab - t_ij^ba)/2 is antisymmetric in both,
// and the ladder term of eq. (vfunction-chol) splits into
//   R+ = V+ S',  S'[(ij)][(cd)] = (2 - delta_cd) s_ij^cd,
//   R- = V- A',  A'[(ij)][(cd)] = 2 a_ij^cd,
// with V+-[(ab)][(cd)] = ((ac|bd) +- (ad|bc))/2, and R = R+ + R- on the
// (i<=j, a<=b) half, the rest following from the two (anti)symmetries.
// The Fock denominator D_ij^ab = e_i + e_j - e_a - e_b is symmetric in (a,b) and
// (i,j), so the update t <- (V + R)/D acts on each part separately.
#include <algorithm>

#include "ppl_internal.h"
#include "pack_cubes.h"

namespace ppl {

static inline unsigned grid_for(int64_t n, int threads, int64_t cap = 65536) {
  int64_t g = (n + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

#define PPL_LAUNCH_CHECK() PPL_HIP_TRY(hipGetLastError())

// ------------------------------------------------------------------ fill / tables
__global__ void zero_kernel(uint4* p, int64_t n16) {
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16; i += st)
    p[i] = uint4{0, 0, 0, 0};
}

int zero_bytes(hipStream_t s, void* p, uint64_t bytes) {
  if (bytes == 0) return PPL_OK;
  if (bytes % 16 != 0 || ((uintptr_t)p) % 16 != 0)
    return fail(PPL_E_ARG, "zero_bytes: unaligned range");
  const int64_t n16 = (int64_t)(bytes / 16);
  hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n16, 256, 8192)), dim3(256), 0, s, (uint4*)p, n16);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

__global__ void tables_kernel(int n, int* plus, int* minus) {
  const int64_t total = (int64_t)n * n;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < total; x += st) {
    const int a = (int)(x / n), b = (int)(x % n);
    if (a <= b) plus[pair_plus(a, b, n)] = (a << 16) | b;
    if (a < b) minus[pair_minus(a, b, n)] = (a << 16) | b;
  }
}

int fill_tables(hipStream_t s, int o, int v, int* tab_vp, int* tab_vm, int* tab_op, int* tab_om) {
  hipLaunchKernelGGL(tables_kernel, dim3(grid_for((int64_t)v * v, 256)), dim3(256), 0, s, v, tab_vp, tab_vm);
  PPL_LAUNCH_CHECK();
  hipLaunchKernelGGL(tables_kernel, dim3(grid_for((int64_t)o * o, 256)), dim3(256), 0, s, o, tab_op, tab_om);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// ------------------------------------------------------------------ precision helpers
template <int PREC> struct Store;
template <> struct Store<PPL_FP64> {
  __device__ static void put(void* hi, void*, int64_t i, double x) { ((double*)hi)[i] = x; }
};
template <> struct Store<PPL_FP32> {
  __device__ static void put(void* hi, void*, int64_t i, double x) { ((float*)hi)[i] = (float)x; }
};
template <> struct Store<PPL_BF16X3> {
  // x -> FP32 (round to nearest), hi = bf16(x32), lo = bf16(x32 - hi); both round to nearest even.
  // (The compiler may round x to hi in one step: where x32 lies halfway between two bf16 numbers and x
  // does not, hi is then the one nearer to x. x32 = hi + lo to the same 17 bits either way. A kernel
  // that must go through x32 passes via_f32(x).)
  __device__ static void put(void* hi, void* lo, int64_t i, double x) {
    const float xf = (float)x;
    const __bf16 h = (__bf16)xf;
    const __bf16 l = (__bf16)(xf - (float)h);
    ((__bf16*)hi)[i] = h;
    ((__bf16*)lo)[i] = l;
  }
};
template <> struct Store<PPL_BF16X6> {
  // x -> FP32 (round to nearest), hi = bf16(x32), mid = bf16(x32 - hi), lo = bf16(x32 - hi - mid),
  // each rounded to nearest even (both differences are exact in FP32). The three planes lie
  // equally far apart: hi at h, mid at m, lo at m + (m - h).
  __device__ static void put(void* hi, void* mid, int64_t i, double x) {
    const float xf = (float)x;
    const __bf16 h = (__bf16)xf;
    const float r1 = xf - (float)h;
    const __bf16 m = (__bf16)r1;
    const __bf16 l = (__bf16)(r1 - (float)m);
    __bf16* ph = (__bf16*)hi;
    __bf16* pm = (__bf16*)mid;
    ph[i] = h;
    pm[i] = m;
    (pm + (pm - ph))[i] = l;
  }
};

// x, rounded to FP32 first for a bf16 operand
template <int PREC>
__device__ inline double via_f32(double x) {
  if constexpr (PREC == PPL_BF16X3 || PREC == PPL_BF16X6) {
    float y = (float)x;
    asm("" : "+v"(y));
    return y;
  }
  return x;
}

// ------------------------------------------------------------------ staging (transposing copy)
// X[r1*R2 + r2][P] = L[P][r1_off + r1][r2_off + r2] for P < naux, 0 for naux <= P < ldx.
template <int PREC>
__global__ void __launch_bounds__(256)
stage_kernel(const double* __restrict__ L, int n, int naux, int r1_off, int r2_off, int R2,
             int64_t rows, int64_t ldx, void* xh, void* xl) {
  __shared__ double sh[32][65];
  const int64_t r0 = (int64_t)blockIdx.x * 64;
  const int P0 = blockIdx.y * 32;
  const int tid = threadIdx.x;
  {  // load: 64 consecutive rows for each of 32 vectors P
    const int rr = tid & 63;
    const int64_t r = r0 + rr;
    int64_t src = -1;
    if (r < rows) {
      const int64_t r1 = r / R2, r2 = r - r1 * R2;
      src = (r1_off + r1) * (int64_t)n + r2_off + r2;
    }
    for (int pp = tid >> 6; pp < 32; pp += 4) {
      const int P = P0 + pp;
      double x = 0.0;
      if (src >= 0 && P < naux) x = L[(int64_t)P * n * n + src];
      sh[pp][rr] = x;
    }
  }
  __syncthreads();
  {  // store: 32 consecutive P for each row
    const int pp = tid & 31;
    for (int rr = tid >> 5; rr < 64; rr += 8) {
      const int64_t r = r0 + rr;
      const int P = P0 + pp;
      if (r < rows && P < ldx) Store<PREC>::put(xh, xl, r * ldx + P, sh[pp][rr]);
    }
  }
}

template <int PREC>
static int stage_launch(hipStream_t s, const double* L, int n, int naux, int r1_off, int r2_off,
                        int R1, int R2, int64_t ldx, void* xh, void* xl) {
  const int64_t rows = (int64_t)R1 * R2;
  dim3 grid((unsigned)((rows + 63) / 64), (unsigned)((ldx + 31) / 32));
  hipLaunchKernelGGL(stage_kernel<PREC>, grid, dim3(256), 0, s, L, n, naux, r1_off, r2_off, R2, rows,
                     ldx, xh, xl);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int stage_vv(hipStream_t s, int prec, const double* L, int o, int v, int naux, int64_t ldx, void* xt,
             void* xt_lo) {
  const int n = o + v;
  if (prec == PPL_FP64) return stage_launch<PPL_FP64>(s, L, n, naux, o, o, v, v, ldx, xt, xt_lo);
  if (prec == PPL_FP32) return stage_launch<PPL_FP32>(s, L, n, naux, o, o, v, v, ldx, xt, xt_lo);
  if (prec == PPL_BF16X3) return stage_launch<PPL_BF16X3>(s, L, n, naux, o, o, v, v, ldx, xt, xt_lo);
  if (prec == PPL_BF16X6) return stage_launch<PPL_BF16X6>(s, L, n, naux, o, o, v, v, ldx, xt, xt_lo);
  return fail(PPL_E_ARG, "stage_vv: unknown precision %d", prec);
}

int stage_ov(hipStream_t s, const double* L, int o, int v, int naux, int64_t ldx, double* xov) {
  return stage_launch<PPL_FP64>(s, L, o + v, naux, 0, o, o, v, ldx, xov, nullptr);
}

// ------------------------------------------------------------------ G -> V+ / V- rows
// One block per pair (a,b) of the batch; 32 x 32 tiles (cB <= dB) of G_ab and
// of its transpose are staged through LDS so that both reads and the packed
// row writes are contiguous.
template <class Tg, int PREC>
__global__ void __launch_bounds__(256)
pack_vpm_kernel(int v, int64_t pair0, const Tg* __restrict__ G, const int* __restrict__ tab_vp,
                void* vp, void* vp_lo, int64_t ldp, int64_t vp_row0, void* vm, void* vm_lo,
                int64_t ldm, int64_t vm_row0, int64_t Pp, int64_t Pm) {
  __shared__ double t1[32][33], t2[32][33];
  const int64_t pr = pair0 + blockIdx.x;           // global V+ row of this block
  const int ab = tab_vp[pr];
  const int a = pair_first(ab), b = pair_second(ab);
  const Tg* g = G + (int64_t)blockIdx.x * v * v;
  const int64_t rowp = pr - vp_row0;
  const bool has_minus = a < b;
  const int64_t rowm = has_minus ? pair_minus(a, b, v) - vm_row0 : 0;
  const int tid = threadIdx.x;
  const int nt = (v + 31) / 32;
  for (int cb = 0; cb < nt; ++cb) {
    for (int db = cb; db < nt; ++db) {
      // t1[c][d] = G[cB+c][dB+d], t2[c][d] = G[dB+d][cB+c]
      for (int e = tid; e < 1024; e += 256) {
        const int r = e >> 5, q = e & 31;
        const int c1 = cb * 32 + r, d1 = db * 32 + q;
        t1[r][q] = (c1 < v && d1 < v) ? (double)g[(int64_t)c1 * v + d1] : 0.0;
        const int c2 = db * 32 + r, d2 = cb * 32 + q;   // row d, col c
        t2[q][r] = (c2 < v && d2 < v) ? (double)g[(int64_t)c2 * v + d2] : 0.0;
      }
      __syncthreads();
      for (int e = tid; e < 1024; e += 256) {
        const int r = e >> 5, q = e & 31;
        const int c = cb * 32 + r, d = db * 32 + q;
        if (c < v && d < v && c <= d) {
          const double gcd = t1[r][q], gdc = t2[r][q];
          Store<PREC>::put(vp, vp_lo, rowp * ldp + pair_plus(c, d, v), 0.5 * (gcd + gdc));
          if (has_minus && c < d)
            Store<PREC>::put(vm, vm_lo, rowm * ldm + pair_minus(c, d, v), 0.5 * (gcd - gdc));
        }
      }
      __syncthreads();
    }
  }
  // zero padding columns
  for (int64_t k = Pp + tid; k < ldp; k += 256) Store<PREC>::put(vp, vp_lo, rowp * ldp + k, 0.0);
  if (has_minus)
    for (int64_t k = Pm + tid; k < ldm; k += 256) Store<PREC>::put(vm, vm_lo, rowm * ldm + k, 0.0);
}

int pack_vpm(hipStream_t s, int prec, int v, int a0, int a1, const void* G, void* vp, void* vp_lo,
             int64_t ldp, int64_t vp_row0, void* vm, void* vm_lo, int64_t ldm, int64_t vm_row0,
             const int* tab_vp, const int* tab_vm) {
  (void)tab_vm;
  const int64_t p0 = pair_plus(a0, a0, v);
  const int64_t p1 = (a1 >= v) ? npairs_plus(v) : pair_plus(a1, a1, v);
  const int64_t npairs = p1 - p0;
  if (npairs <= 0) return PPL_OK;
  const int64_t Pp = npairs_plus(v), Pm = npairs_minus(v);
  dim3 grid((unsigned)npairs);
  if (prec == PPL_FP64)
    hipLaunchKernelGGL((pack_vpm_kernel<double, PPL_FP64>), grid, dim3(256), 0, s, v, p0,
                       (const double*)G, tab_vp, vp, vp_lo, ldp, vp_row0, vm, vm_lo, ldm, vm_row0, Pp, Pm);
  else if (prec == PPL_FP32)
    hipLaunchKernelGGL((pack_vpm_kernel<float, PPL_FP32>), grid, dim3(256), 0, s, v, p0,
                       (const float*)G, tab_vp, vp, vp_lo, ldp, vp_row0, vm, vm_lo, ldm, vm_row0, Pp, Pm);
  else if (prec == PPL_BF16X3)
    hipLaunchKernelGGL((pack_vpm_kernel<float, PPL_BF16X3>), grid, dim3(256), 0, s, v, p0,
                       (const float*)G, tab_vp, vp, vp_lo, ldp, vp_row0, vm, vm_lo, ldm, vm_row0, Pp, Pm);
  else if (prec == PPL_BF16X6)
    hipLaunchKernelGGL((pack_vpm_kernel<float, PPL_BF16X6>), grid, dim3(256), 0, s, v, p0,
                       (const float*)G, tab_vp, vp, vp_lo, ldp, vp_row0, vm, vm_lo, ldm, vm_row0, Pp, Pm);
  else
    return fail(PPL_E_ARG, "pack_vpm: unknown precision %d", prec);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

constexpr int kPackThreads = 256;
static_assert(kCube == 16, "the cube packing splits an element index into 4-bit fields");

// Rows of V+- of an upper-triangle build step from the natural build output T: T[(pair(a, r) - pr0) *
// ldt + pair(x, y) - pr0] = (ar|xy) for the step's virtuals a in [a0, a1), r >= a and
// a <= x <= y (pr0 = pair(a0, a0)); T is symmetric in (x, y) since the Cholesky vectors are. For
// row (ab) and column (cd) >= (ab) in packed order
//   V+[ab][cd] = ((ac|bd) + (ad|bc)) / 2,   V-[ab][cd] = ((ac|bd) - (ad|bc)) / 2  (a < b, c < d).
// Of the entries below the diagonal those inside a diagonal block (kTriBlock) are written; a
// streaming step (STEP, EpiStep) has none, halves its diagonal and stores its rows from global rows
// row0p / row0m on. One workgroup per cube of 16 x 16 x 16
// indices (b, c, d), thread (c, d), b unrolled, so that the rows are written along d. (ac|bd) is
// read in that shape where b <= d (contiguous along d); (ad|bc) is contiguous along c (b <= c) or
// b and goes through one LDS array s[b][d][c], and where b > d so does (ac|bd), contiguous along
// b, in a round of its own. The cubes with ci == di == 0 also zero the rows' padding.
// Bound by the writes of its 16 x 16 row segments: the lines that segments share are merged in
// L2 only while few are open, so spare LDS holds it to a few workgroups per CU (TriLds). By workgroups
// per CU, the most being what fits (ms per build):
//   FP64, v = 200 in one step (3.2 GB written, 1.6 read)   two 1.74   three 1.94   four 2.01
//   FP64, v = 300 in eight steps                           two 9.3    three 10.2   four 10.5
//   FP32, v = 151                                          two 0.374  four 0.356   eight 0.420
//   BF16x6, v = 137                                        two 0.388  three 0.379 four 0.411   eight 0.471
//   BF16x3, v = 137                                        two 0.319  three 0.285 four 0.299   eight 0.361
// Writing every mirror entry here, along b, took 3.35 ms (FP64), 0.58 ms (FP32) and 0.845 ms (BF16x6).
template <class Tg, int PREC>
struct TriLds {
  static constexpr int LD = kCube + 1, LB = kCube * LD + 1;   // odd strides: at most a few lanes meet on a bank
  static constexpr unsigned bytes = kCube * LB * sizeof(Tg);
  // workgroups per CU (160 KB of LDS, dealt in units of 1280 bytes) and the least that holds it to them
  static constexpr unsigned groups = PREC == PPL_FP64 ? 2 : PREC == PPL_FP32 ? 4 : 3;
  static constexpr unsigned cu = 160 * 1024, unit = 1280, all = (cu / (groups + 1) / unit + 1) * unit;
  static constexpr unsigned spare = all - bytes;
  static_assert(all >= bytes && groups * all <= cu && (groups + 1) * all > cu, "workgroups per CU");
};

template <class Tg, int PREC, bool STEP>
__global__ void __launch_bounds__(kPackThreads)
pack_vpm_tri_kernel(int v, int a0, int a1, const Tg* __restrict__ T, int64_t ldt, const int64_t* __restrict__ off,
                    int64_t g0, int64_t ncubes, void* vp, void* vp_lo, int64_t ldp, void* vm, void* vm_lo,
                    int64_t ldm, int64_t Pp, int64_t Pm, int64_t row0p, int64_t row0m) {
  constexpr int C = kCube, LD = TriLds<Tg, PREC>::LD, LB = TriLds<Tg, PREC>::LB;
  __shared__ Tg s[C * LB];
  const int64_t g = g0 + cube_of_slot(blockIdx.x, ncubes);
  const int a = cube_virtual(off, a0, a1, g);
  const int nt = cube_blocks(v, a);
  int bi, ci, di;
  cube_decode_rows(g - off[a], nt, bi, ci, di);
  const int b0 = a + C * bi, c0 = a + C * ci, d0 = a + C * di;
  const int64_t pr0 = pair_plus(a0, a0, v);
  const int f = threadIdx.x & 15, m = threadIdx.x >> 4;
  // (a r | x y), zero outside v
  auto at = [&](int r, int x, int y) __attribute__((always_inline)) {
    const int lo = x < y ? x : y, hi = x < y ? y : x;
    return (r < v && hi < v) ? T[(pair_plus(a, r, v) - pr0) * ldt + (pair_plus(lo, hi, v) - pr0)] : Tg(0);
  };
  const bool swapped = bi > di;               // b > d: (ac|bd) is contiguous along b
  Tg gcd[C], gdc[C];
  if (bi <= ci) {
#pragma unroll
    for (int k = 0; k < C; ++k) gdc[k] = at(d0 + m, b0 + k, c0 + f);   // s[k][m][f]
  } else {
#pragma unroll
    for (int k = 0; k < C; ++k) gdc[k] = at(d0 + k, c0 + m, b0 + f);   // s[f][k][m]
  }
  if (swapped) {
#pragma unroll
    for (int k = 0; k < C; ++k) gcd[k] = at(c0 + m, d0 + k, b0 + f);   // s[f][k][m]
#pragma unroll
    for (int k = 0; k < C; ++k) s[f * LB + k * LD + m] = gcd[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C; ++k) gcd[k] = s[k * LB + f * LD + m];
    __syncthreads();
  } else {
#pragma unroll
    for (int k = 0; k < C; ++k) gcd[k] = at(c0 + m, b0 + k, d0 + f);
  }
  if (bi <= ci) {
#pragma unroll
    for (int k = 0; k < C; ++k) s[k * LB + m * LD + f] = gdc[k];
  } else {
#pragma unroll
    for (int k = 0; k < C; ++k) s[f * LB + k * LD + m] = gdc[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < C; ++k) gdc[k] = s[k * LB + f * LD + m];
  const int c = c0 + m, d = d0 + f;
  if (d < v && c <= d) {
    const int kmax = cube_rows(v, a, b0, c, d);
    const int64_t rp = pair_plus(a, b0, v), cp = pair_plus(c, d, v);
    const int64_t rm = pair_minus(a, b0, v), cm = pair_minus(c, d, v);
    const bool near = !STEP && cube_near(v, a, b0, c0, d0);   // (the same for every thread)
#pragma unroll
    for (int k = 0; k < C; ++k) {
      if (k < kmax) {
        const double x = (double)gcd[k], y = (double)gdc[k];
        const bool minus = c < d && (k > 0 || b0 > a);
        const double w = STEP && cp == rp + k ? 0.25 : 0.5;   // (V+ and V- meet their diagonals together)
        Store<PREC>::put(vp, vp_lo, (rp + k - row0p) * ldp + cp, w * (x + y));
        if (minus) Store<PREC>::put(vm, vm_lo, (rm + k - row0m) * ldm + cm, w * (x - y));
        if (near) {
          if ((rp + k) / kTriBlock == cp / kTriBlock) Store<PREC>::put(vp, vp_lo, cp * ldp + rp + k, 0.5 * (x + y));
          if (minus && (rm + k) / kTriBlock == cm / kTriBlock)
            Store<PREC>::put(vm, vm_lo, cm * ldm + rm + k, 0.5 * (x - y));
        }
      }
    }
  }
  if (ci == 0 && di == 0) {
    const int64_t padp = ldp - Pp, padm = ldm - Pm;
    for (int e = threadIdx.x; e < C * padp; e += kPackThreads) {
      const int b = b0 + (int)(e / padp);
      if (b < v) Store<PREC>::put(vp, vp_lo, (pair_plus(a, b, v) - row0p) * ldp + Pp + e % padp, 0.0);
    }
    for (int e = threadIdx.x; e < C * padm; e += kPackThreads) {
      const int b = b0 + (int)(e / padm);
      if (b < v && a < b) Store<PREC>::put(vm, vm_lo, (pair_minus(a, b, v) - row0m) * ldm + Pm + e % padm, 0.0);
    }
  }
}

template <class Tg, int PREC, bool STEP = false>
static int launch_vpm_tri(hipStream_t s, int v, int a0, int a1, const void* T, int64_t ldt, const int64_t* off,
                          void* vp, void* vp_lo, int64_t ldp, void* vm, void* vm_lo, int64_t ldm, int64_t row0p = 0,
                          int64_t row0m = 0) {
  int64_t g0 = 0, n = 0;
  for (int a = 0; a < a1; ++a) (a < a0 ? g0 : n) += cubes_of(v, a);
  if (n <= 0) return PPL_OK;
  if (n > 0x7fffffffLL) return fail(PPL_E_ARG, "pack_vpm_tri: %lld cubes", (long long)n);
  hipLaunchKernelGGL((pack_vpm_tri_kernel<Tg, PREC, STEP>), dim3((unsigned)n), dim3(kPackThreads),
                     (TriLds<Tg, PREC>::spare), s, v, a0, a1, (const Tg*)T, ldt, off, g0, n, vp, vp_lo, ldp, vm, vm_lo,
                     ldm, npairs_plus(v), npairs_minus(v), row0p, row0m);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int pack_vpm_tri(hipStream_t s, int prec, int v, int a0, int a1, const void* T, int64_t ldt, const int64_t* off,
                 void* vp, void* vp_lo, int64_t ldp, void* vm, void* vm_lo, int64_t ldm) {
  switch (prec) {
    case PPL_FP64:
      return launch_vpm_tri<double, PPL_FP64>(s, v, a0, a1, T, ldt, off, vp, nullptr, ldp, vm, nullptr, ldm);
    case PPL_FP32:
      return launch_vpm_tri<float, PPL_FP32>(s, v, a0, a1, T, ldt, off, vp, nullptr, ldp, vm, nullptr, ldm);
    case PPL_BF16X3:
      return launch_vpm_tri<float, PPL_BF16X3>(s, v, a0, a1, T, ldt, off, vp, vp_lo, ldp, vm, vm_lo, ldm);
    case PPL_BF16X6:
      return launch_vpm_tri<float, PPL_BF16X6>(s, v, a0, a1, T, ldt, off, vp, vp_lo, ldp, vm, vm_lo, ldm);
  }
  return fail(PPL_E_ARG, "pack_vpm_tri: unknown precision %d", prec);
}

// The zeros of a step's rows (triangle.h)
__global__ void __launch_bounds__(256)
step_zero_kernel(double* U, int64_t ld, int64_t p0, int64_t p1) {
  const int64_t k = step_row0(p0) + blockIdx.x, c1 = step_zero_to(k, p0, p1, ld);
  for (int64_t c = step_zero_from(k, p0, p1) + threadIdx.x; c < c1; c += 256) U[(int64_t)blockIdx.x * ld + c] = 0.0;
}

int pack_vpm_step(hipStream_t s, int v, const Batch& b, const double* T, int64_t ldt, const int64_t* off, double* vp,
                  int64_t ldp, double* vm, int64_t ldm) {
  const int64_t kp = step_row0(b.p0), km = step_row0(b.q0);
  PPL_TRY((launch_vpm_tri<double, PPL_FP64, true>(s, v, b.a0, b.a1, T, ldt, off, vp, nullptr, ldp, vm, nullptr, ldm, kp,
                                                  km)));
  hipLaunchKernelGGL(step_zero_kernel, dim3((unsigned)(b.p1 - kp + kStepRows)), dim3(256), 0, s, vp, ldp, b.p0, b.p1);
  if (b.q1 > b.q0)
    hipLaunchKernelGGL(step_zero_kernel, dim3((unsigned)(b.q1 - km + kStepRows)), dim3(256), 0, s, vm, ldm, b.q0, b.q1);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// Y[p][q] = w X[q][p] for q < nq, p < np, and Y[p][q] = 0 for nq <= q < ldy (rows of X
// hold ldx, rows of Y ldy doubles). scaled: w = (2 - d_kl) / (2 - d_ab) with (k, l) =
// tab_q[q] and (a, b) = tab_p[p] (S' rows to the transposed symmetric operand of the
// hole-hole ladder); otherwise w = 1.
__global__ void __launch_bounds__(256)
transpose_pm_kernel(const double* __restrict__ X, int64_t ldx, double* __restrict__ Y, int64_t ldy, int64_t nq,
                    int64_t np, const int* __restrict__ tab_q, const int* __restrict__ tab_p, int scaled,
                    int64_t qwrite, int64_t tiles_q) {
  __shared__ double sh[64][65];
  const int64_t tp = blockIdx.x / tiles_q, tq = blockIdx.x % tiles_q;
  const int64_t p0 = tp * 64, q0 = tq * 64;
  const int tid = threadIdx.x;
  for (int e = tid; e < 64 * 64; e += 256) {
    const int ql = e >> 6, pl = e & 63;                   // read X row q0 + ql, column p0 + pl
    const int64_t q = q0 + ql, p = p0 + pl;
    double x = 0.0;
    if (q < nq && p < np) {
      x = X[q * ldx + p];
      if (scaled) {
        const int kl = tab_q[q], ab = tab_p[p];
        const double wq = pair_first(kl) == pair_second(kl) ? 1.0 : 2.0;
        const double wp = pair_first(ab) == pair_second(ab) ? 1.0 : 2.0;
        x *= wq / wp;
      }
    }
    sh[ql][pl] = x;
  }
  __syncthreads();
  for (int e = tid; e < 64 * 64; e += 256) {
    const int pl = e >> 6, ql = e & 63;                   // write Y row p0 + pl, column q0 + ql
    const int64_t p = p0 + pl, q = q0 + ql;
    if (p < np && q < qwrite) Y[p * ldy + q] = sh[ql][pl];
  }
}

int transpose_pm(hipStream_t s, const double* X, int64_t ldx, double* Y, int64_t ldy, int64_t nq, int64_t np,
                 const int* tab_q, const int* tab_p, int scaled, int pad) {
  if (np <= 0 || ldy <= 0) return PPL_OK;
  const int64_t qwrite = pad ? ldy : nq;          // columns written per row of Y
  const int64_t tq = (qwrite + 63) / 64, tp = (np + 63) / 64;
  if (tq * tp > 0x7fffffffLL) return fail(PPL_E_ARG, "transpose of %lld x %lld too large", (long long)np,
                                          (long long)ldy);
  hipLaunchKernelGGL(transpose_pm_kernel, dim3((unsigned)(tq * tp)), dim3(256), 0, s, X, ldx, Y, ldy, nq, np, tab_q,
                     tab_p, scaled, qwrite, tq);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// C[q][p] += T[p][q] for q < nq, p < np (C rows of ldc, T rows of ldt), 64 x 64 LDS tiles.
template <class Tc>
__global__ void __launch_bounds__(256)
add_transposed_kernel(Tc* __restrict__ C, int64_t ldc, const double* __restrict__ T, int64_t ldt, int64_t nq,
                      int64_t np, int64_t tiles_p) {
  __shared__ double sh[64][65];
  const int64_t tq = blockIdx.x / tiles_p, tp = blockIdx.x % tiles_p;
  const int64_t q0 = tq * 64, p0 = tp * 64;
  const int tid = threadIdx.x;
  for (int e = tid; e < 64 * 64; e += 256) {
    const int pl = e >> 6, ql = e & 63;                   // read T row p0 + pl, column q0 + ql
    const int64_t pp = p0 + pl, q = q0 + ql;
    sh[pl][ql] = (pp < np && q < nq) ? T[pp * ldt + q] : 0.0;
  }
  __syncthreads();
  for (int e = tid; e < 64 * 64; e += 256) {
    const int ql = e >> 6, pl = e & 63;                   // update C row q0 + ql, column p0 + pl
    const int64_t q = q0 + ql, pp = p0 + pl;
    if (q < nq && pp < np) C[q * ldc + pp] = (Tc)((double)C[q * ldc + pp] + sh[pl][ql]);
  }
}

int add_transposed(hipStream_t s, int c_prec, void* C, int64_t ldc, const double* T, int64_t ldt, int64_t nq,
                   int64_t np) {
  if (nq <= 0 || np <= 0) return PPL_OK;
  const int64_t tq = (nq + 63) / 64, tp = (np + 63) / 64;
  if (tq * tp > 0x7fffffffLL) return fail(PPL_E_ARG, "transposed add of %lld x %lld too large", (long long)nq,
                                          (long long)np);
  if (c_prec == PPL_FP64)
    hipLaunchKernelGGL(add_transposed_kernel<double>, dim3((unsigned)(tq * tp)), dim3(256), 0, s, (double*)C, ldc, T,
                       ldt, nq, np, tp);
  else
    hipLaunchKernelGGL(add_transposed_kernel<float>, dim3((unsigned)(tq * tp)), dim3(256), 0, s, (float*)C, ldc, T,
                       ldt, nq, np, tp);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// ------------------------------------------------------------------ generic (i,j,a,b) -> +/- packing
// Work items are one occupied pair (i <= j) and one 32 x 32 block pair (A <= B) of virtual
// indices: block (A, B) of X_ij is read along rows, block (B, A) too and transposed through LDS,
// and both packed rows are written along b, so X is read once and every access is
// coalesced for sb = 1 (48 + 39 us as two kernels with strided partners at (20, 200), 24 us). The
// item of the last block also zeroes the rows' padding. With t1 ([i][a], row length v1) the
// packed tensor is X_ij^ab + t1_i^a t1_j^b.
struct PackArgs {
  int64_t si, sj, sa, sb;
  double s_off, s_diag, am;
  void *plus, *plus_lo, *minus, *minus_lo;
  int64_t ldp, ldm, v1;
};

template <int PREC>
__global__ void __launch_bounds__(256)
pack_tiled_kernel(int o, int v, const double* __restrict__ X, PackArgs g, const int* __restrict__ tab_op,
                  const double* __restrict__ t1) {
  __shared__ double tr[32][33];
  const int nb = (v + 31) / 32;
  const int64_t per = (int64_t)nb * (nb + 1) / 2, items = npairs_plus(o) * per;
  const int64_t Pp = npairs_plus(v), Pm = npairs_minus(v);
  const int f = threadIdx.x & 31, m = threadIdx.x >> 5;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t pr = it / per;
    int k = (int)(it % per), A = 0;
    while (k >= nb - A) k -= nb - A++;          // block pair (A, B = A + k)
    const int B = A + k, ij = tab_op[pr], i = pair_first(ij), j = pair_second(ij);
    const bool offd = i < j;
    const double* x = X + i * g.si + j * g.sj;
    double ab[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m + 8 * e, a = A * 32 + r, b = B * 32 + f;
      ab[e] = (a < v && b < v) ? x[a * g.sa + b * g.sb] : 0.0;
      if (t1 && a < v && b < v) ab[e] += t1[i * g.v1 + a] * t1[j * g.v1 + b];
    }
    if (A != B) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = m + 8 * e, b = B * 32 + r, a = A * 32 + f;
        double y = (a < v && b < v) ? x[b * g.sa + a * g.sb] : 0.0;
        if (t1 && a < v && b < v) y += t1[i * g.v1 + b] * t1[j * g.v1 + a];
        tr[f][r] = y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) tr[f][m + 8 * e] = ab[e];
    }
    __syncthreads();
    const int64_t qr = offd ? pair_minus(i, j, o) : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m + 8 * e, a = A * 32 + r, b = B * 32 + f;
      if (b < v && a <= b) {
        const double y = tr[r][f];
        Store<PREC>::put(g.plus, g.plus_lo, pr * g.ldp + pair_plus(a, b, v), (a == b ? g.s_diag : g.s_off) * (ab[e] + y));
        if (offd && a < b)
          Store<PREC>::put(g.minus, g.minus_lo, qr * g.ldm + pair_minus(a, b, v), g.am * (ab[e] - y));
      }
    }
    if (A == nb - 1) {                          // (A = B: the last block of the pair)
      for (int64_t q = Pp + threadIdx.x; q < g.ldp; q += 256) Store<PREC>::put(g.plus, g.plus_lo, pr * g.ldp + q, 0.0);
      if (offd)
        for (int64_t q = Pm + threadIdx.x; q < g.ldm; q += 256)
          Store<PREC>::put(g.minus, g.minus_lo, qr * g.ldm + q, 0.0);
    }
    __syncthreads();
  }
}

int pack_pm(hipStream_t s, int prec, int o, int v, const double* X, int64_t si, int64_t sj, int64_t sa, int64_t sb,
            double sp_off, double sp_diag, double am, void* plus, void* plus_lo, int64_t ldp, void* minus,
            void* minus_lo, int64_t ldm, const int* tab_op, const double* t1) {
  const int64_t nb = (v + 31) / 32, items = npairs_plus(o) * (nb * (nb + 1) / 2);
  const dim3 grid((unsigned)std::min<int64_t>(items, 16384));
  const PackArgs g{si, sj, sa, sb, sp_off, sp_diag, am, plus, plus_lo, minus, minus_lo, ldp, ldm, (int64_t)v};
  if (prec == PPL_FP64)
    hipLaunchKernelGGL(pack_tiled_kernel<PPL_FP64>, grid, dim3(256), 0, s, o, v, X, g, tab_op, t1);
  else if (prec == PPL_FP32)
    hipLaunchKernelGGL(pack_tiled_kernel<PPL_FP32>, grid, dim3(256), 0, s, o, v, X, g, tab_op, t1);
  else if (prec == PPL_BF16X3)
    hipLaunchKernelGGL(pack_tiled_kernel<PPL_BF16X3>, grid, dim3(256), 0, s, o, v, X, g, tab_op, t1);
  else if (prec == PPL_BF16X6)
    hipLaunchKernelGGL(pack_tiled_kernel<PPL_BF16X6>, grid, dim3(256), 0, s, o, v, X, g, tab_op, t1);
  else
    return fail(PPL_E_ARG, "pack_pm: unknown precision %d", prec);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int stage_oo(hipStream_t s, const double* L, int o, int v, int naux, int64_t ldx, double* xoo) {
  return stage_launch<PPL_FP64>(s, L, o + v, naux, 0, 0, o, o, ldx, xoo, nullptr);
}

// ------------------------------------------------------------------ FP64 rows -> operand precision
template <int PREC>
__global__ void convert_kernel(const double* __restrict__ src, int64_t n, void* dh, void* dl) {
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += st)
    Store<PREC>::put(dh, dl, x, src[x]);
}

int convert_rows(hipStream_t s, int prec, const double* src, int64_t rows, int64_t cols, int64_t ld,
                 void* dst, void* dst_lo) {
  (void)cols;
  const int64_t n = rows * ld;
  if (n <= 0) return PPL_OK;
  if (prec == PPL_FP32)
    hipLaunchKernelGGL(convert_kernel<PPL_FP32>, dim3(grid_for(n, 256)), dim3(256), 0, s, src, n, dst, dst_lo);
  else if (prec == PPL_BF16X3)
    hipLaunchKernelGGL(convert_kernel<PPL_BF16X3>, dim3(grid_for(n, 256)), dim3(256), 0, s, src, n, dst, dst_lo);
  else if (prec == PPL_BF16X6)
    hipLaunchKernelGGL(convert_kernel<PPL_BF16X6>, dim3(grid_for(n, 256)), dim3(256), 0, s, src, n, dst, dst_lo);
  else if (prec == PPL_FP64)
    hipLaunchKernelGGL(convert_kernel<PPL_FP64>, dim3(grid_for(n, 256)), dim3(256), 0, s, src, n, dst, dst_lo);
  else
    return fail(PPL_E_ARG, "convert_rows: unknown precision %d", prec);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// Four consecutive elements of an operand row (i a multiple of 4, rows 16-byte aligned)
template <int PREC>
__device__ inline void put4(void* hi, void* lo, int64_t i, const double (&x)[4]) {
  if constexpr (PREC == PPL_FP32) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<f32x4*>((float*)hi + i) = f32x4{(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
  } else {
    typedef __bf16 b16x4 __attribute__((ext_vector_type(4)));
    b16x4 pl[3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {     // as Store<PREC>::put
      const float xf = (float)x[k];
      pl[0][k] = (__bf16)xf;
      const float r1 = xf - (float)pl[0][k];
      pl[1][k] = (__bf16)r1;
      if (PREC == PPL_BF16X6) pl[2][k] = (__bf16)(r1 - (float)pl[1][k]);
    }
    __bf16 *ph = (__bf16*)hi, *pm = (__bf16*)lo;
    *reinterpret_cast<b16x4*>(ph + i) = pl[0];
    *reinterpret_cast<b16x4*>(pm + i) = pl[1];
    if (PREC == PPL_BF16X6) *reinterpret_cast<b16x4*>(pm + (pm - ph) + i) = pl[2];
  }
}

// An n x n FP64 matrix stored as its upper triangle (kTriBlock; rows of ld, a multiple of 64) to the
// same in an operand precision: one workgroup per row and share of its stored columns (a share
// per 4096 columns of a whole row), four entries per thread and step. Bound by memory: (20, 200) to
// BF16x3 516 us per sign for 2.4 GB (643 with the mirror half).
template <int PREC>
__global__ void __launch_bounds__(256)
convert_tri_kernel(const double* __restrict__ src, int64_t ld, void* dh, void* dl) {
  const int64_t r = blockIdx.x, b = r / kTriBlock * kTriBlock;
  const int64_t seg = ((ld - b) / 4 + gridDim.y - 1) / gridDim.y * 4;
  const int64_t q0 = b + blockIdx.y * seg, q1 = q0 + seg < ld ? q0 + seg : ld;
  for (int64_t q = q0 + threadIdx.x * 4; q < q1; q += 1024) {
    double x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = src[r * ld + q + k];
    put4<PREC>(dh, dl, r * ld + q, x);
  }
}

int convert_tri(hipStream_t s, int prec, const double* src, int64_t n, int64_t ld, void* dst, void* dst_lo) {
  if (n <= 0) return PPL_OK;
  if (ld % 64 != 0 || ld < n || n > 0x7fffffffLL)
    return fail(PPL_E_ARG, "convert_tri: %lld rows of %lld elements", (long long)n, (long long)ld);
  const dim3 grid((unsigned)n, (unsigned)std::max<int64_t>(1, ld / 4096));
  if (prec == PPL_FP32)
    hipLaunchKernelGGL(convert_tri_kernel<PPL_FP32>, grid, dim3(256), 0, s, src, ld, dst, dst_lo);
  else if (prec == PPL_BF16X3)
    hipLaunchKernelGGL(convert_tri_kernel<PPL_BF16X3>, grid, dim3(256), 0, s, src, ld, dst, dst_lo);
  else if (prec == PPL_BF16X6)
    hipLaunchKernelGGL(convert_tri_kernel<PPL_BF16X6>, grid, dim3(256), 0, s, src, ld, dst, dst_lo);
  else
    return fail(PPL_E_ARG, "convert_tri: unknown precision %d", prec);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// ------------------------------------------------------------------ unpack R and t
// Both unpackings over tiles: a work item is one occupied pair (i0 <= j0) and one 32 x 32
// block pair (A <= B) of virtual indices. The packed values of (a, b), a <= b, are read
// along their rows once and give the four entries (i0 j0 a b), (i0 j0 b a), (j0 i0 a b) and
// (j0 i0 b a); the (b a) entries are written from an LDS transpose, so that reads and
// writes both run along contiguous rows. MODE 0 unpacks R (R = alpha r + beta R), MODE 1
// the amplitudes (s = S' / (2 - delta_ab), a = A' / 2). R may come as K slices, summed here in
// slice order instead of in a pass of its own (100 us at (20, 200) with four and six slices,
// 47 + 72 us as unpacking and two passes).
template <class Tr>
struct SliceSum {
  const Tr* p;
  int n;
  int64_t stride;
  __device__ Tr operator[](int64_t i) const {
    Tr y[kMaxSplits];          // every slice's load in flight before the first sum
#pragma unroll
    for (int k = 0; k < kMaxSplits; ++k) y[k] = k < n ? p[i + k * stride] : Tr(0);
    Tr x = y[0];
#pragma unroll
    for (int k = 1; k < kMaxSplits; ++k)
      if (k < n) x += y[k];
    return x;
  }
};

template <class Tr, int MODE>
__global__ void __launch_bounds__(256)
unpack_tiled_kernel(int o, int v, SliceSum<Tr> xp, int64_t ldp, SliceSum<Tr> xm, int64_t ldm, double* out,
                    double alpha, double beta) {
  __shared__ double sp_[32][33], sm_[32][33];
  const int nb = (v + 31) / 32;
  const int64_t per = (int64_t)nb * (nb + 1) / 2;
  const int64_t items = npairs_plus(o) * per;
  const int tid = threadIdx.x;
  auto put = [&](int64_t x, double val) __attribute__((always_inline)) {
    out[x] = (MODE == 1 || beta == 0.0) ? alpha * val : alpha * val + beta * out[x];
  };
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t pr = it / per;
    int k = (int)(it % per), A = 0;
    while (k >= nb - A) k -= nb - A++;          // block pair (A, B = A + k)
    const int B = A + k;
    int i0 = 0;                                 // occupied pair pr = (i0, j0), i0 <= j0
    while (pair_plus(i0 + 1, i0 + 1, o) <= pr) ++i0;
    const int j0 = i0 + (int)(pr - pair_plus(i0, i0, o));
    const bool offd = i0 < j0;
    const int64_t qr = offd ? pair_minus(i0, j0, o) : 0;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const int e = tid + 256 * e4, r = e >> 5, c = e & 31;
      const int a = A * 32 + r, b = B * 32 + c;
      const bool ok = a < v && b < v && a <= b;
      double pv = ok ? (double)xp[pr * ldp + pair_plus(a, b, v)] : 0.0;
      double mv = (ok && offd && a < b) ? (double)xm[qr * ldm + pair_minus(a, b, v)] : 0.0;
      if (MODE == 1) {
        if (a != b) pv *= 0.5;
        mv *= 0.5;
      }
      sp_[r][c] = pv;
      sm_[r][c] = mv;
    }
    __syncthreads();
    const int64_t row_ij = ((int64_t)i0 * o + j0) * v, row_ji = ((int64_t)j0 * o + i0) * v;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {            // entries (a, b), a <= b
      const int e = tid + 256 * e4, r = e >> 5, c = e & 31;
      const int a = A * 32 + r, b = B * 32 + c;
      if (a < v && b < v && a <= b) {
        const double pv = sp_[r][c], mv = sm_[r][c];
        put((row_ij + a) * v + b, pv + mv);
        if (offd) put((row_ji + a) * v + b, pv - mv);
      }
    }
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {            // entries (b, a), a < b, from the transpose
      const int e = tid + 256 * e4, rb = e >> 5, ca = e & 31;
      const int b = B * 32 + rb, a = A * 32 + ca;
      if (b < v && a < b) {
        const double pv = sp_[ca][rb], mv = sm_[ca][rb];
        put((row_ij + b) * v + a, pv - mv);
        if (offd) put((row_ji + b) * v + a, pv + mv);
      }
    }
    __syncthreads();
  }
}

static int64_t unpack_grid(int o, int v) {
  const int64_t nb = (v + 31) / 32, items = npairs_plus(o) * (nb * (nb + 1) / 2);
  return items < 8192 ? items : 8192;
}

template <class Tr>
static SliceSum<Tr> slice_sum(const Slices& x) {
  return SliceSum<Tr>{(const Tr*)x.p, x.n, x.stride};
}

int unpack_r(hipStream_t s, int acc_prec, int o, int v, const Slices& rp, int64_t ldp, const Slices& rm, int64_t ldm,
             double* R, double alpha, double beta) {
  if (o <= 0 || v <= 0) return PPL_OK;
  const unsigned g = (unsigned)unpack_grid(o, v);
  if (acc_prec == PPL_FP64)
    hipLaunchKernelGGL((unpack_tiled_kernel<double, 0>), dim3(g), dim3(256), 0, s, o, v, slice_sum<double>(rp), ldp,
                       slice_sum<double>(rm), ldm, R, alpha, beta);
  else
    hipLaunchKernelGGL((unpack_tiled_kernel<float, 0>), dim3(g), dim3(256), 0, s, o, v, slice_sum<float>(rp), ldp,
                       slice_sum<float>(rm), ldm, R, alpha, beta);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int unpack_t(hipStream_t s, int o, int v, const double* sp, int64_t ldp, const double* am,
             int64_t ldm, double* t2) {
  if (o <= 0 || v <= 0) return PPL_OK;
  hipLaunchKernelGGL((unpack_tiled_kernel<double, 1>), dim3((unsigned)unpack_grid(o, v)), dim3(256), 0, s, o, v,
                     SliceSum<double>{sp, 1, 0}, ldp, SliceSum<double>{am, 1, 0}, ldm, t2, 1.0, 0.0);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// ------------------------------------------------------------------ reductions
// Fixed grid (kReduceBlocks x kReduceThreads), grid-stride loops and a fixed
// tree order: the sums are bitwise reproducible for a given problem size.
// Sum over the workgroup in thread 0: halves of 256 and 128 threads through LDS, the rest of
// the same tree by lane shifts.
__device__ inline double block_sum(double x, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = x;
  __syncthreads();
  if (tid < 128) sh[tid] += sh[tid + 128];
  __syncthreads();
  if (tid < 64) {
    x = sh[tid] + sh[tid + 64];
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) x += __shfl_down(x, w, 64);
  }
  return x;
}
static_assert(kReduceThreads == 256, "block_sum adds four waves");

// one sum per value of this workgroup: partials[k][workgroup]
template <int NV>
__device__ inline void block_reduce_store(double (&vals)[NV], double* partials) {
  __shared__ double sh[NV][kReduceThreads];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double x = block_sum(vals[k], sh[k]);
    if (threadIdx.x == 0) partials[k * kReduceBlocks + blockIdx.x] = x;
  }
}

// out[k] = sum of partials[k][.], one workgroup per value k; values from n0 on come from a second
// partial buffer. out may be mapped host memory.
__global__ void __launch_bounds__(kReduceThreads)
final_reduce_kernel(const double* __restrict__ partials, int n0, const double* __restrict__ partials1, double* out) {
  __shared__ double sh[kReduceThreads];
  const int k = blockIdx.x;
  const double* p = k < n0 ? partials + k * kReduceBlocks : partials1 + (k - n0) * kReduceBlocks;
  double acc = 0.0;
#pragma unroll
  for (int b = 0; b < kReduceBlocks; b += kReduceThreads) acc += p[b + threadIdx.x];
  const double x = block_sum(acc, sh);
  if (threadIdx.x == 0) out[k] = x;
}

static int final_reduce(hipStream_t s, const double* partials, int n0, const double* partials1, int n1, double* out) {
  hipLaunchKernelGGL(final_reduce_kernel, dim3((unsigned)(n0 + n1)), dim3(kReduceThreads), 0, s, partials, n0,
                     partials1, out);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

struct PairGeom {
  int o, v;
  int64_t Np, Nm, Pp, Pm, ldp, ldm;
  const int *tab_op, *tab_om, *tab_vp, *tab_vm;
};

// q = x / d, p = x - q d for x >= 0, d > 0; in 32 bits when the caller knows x < 2^31
// (the quotient is the same, the instruction sequence much shorter)
__device__ inline void row_col(int64_t x, int64_t d, bool narrow, int64_t& q, int64_t& p) {
  if (narrow) {
    const uint32_t q32 = (uint32_t)x / (uint32_t)d;
    q = q32;
  } else {
    q = x / d;
  }
  p = x - q * d;
}

// Denominator of a packed element
__device__ inline double denom(const double* e_occ, const double* e_vir, int ij, int ab) {
  return e_occ[pair_first(ij)] + e_occ[pair_second(ij)] - e_vir[pair_first(ab)] - e_vir[pair_second(ab)];
}

// mode 0: MP2 start   S' = (2-d_ab) VS / D, A' = 2 VA / D, energy of the result
// mode 1: Jacobi update from R+- (type Tr, K slices summed here); residual^2, energy, non-finite count
// mode 2: energy of the current S'/A' only
// ND >= 0 (mode 1): a DIIS sweep. Also writes the new amplitudes and the error e (new - old), both
// in the packed S'/A' scaling, to one slot each (plus part, then minus part at offset Np * ldp;
// padding columns of the slots are not written), and forms the inner products of e with up to ND
// earlier errors over the full o x o x v x v tensors: a "+" entry of S' scaling carries weight
// (2 - d_ij) / (2 - d_ab) (its full-tensor multiplicity over the square of its packing factor), a
// "-" entry of A' scaling weight 1 (four entries, each half of A'). <e, e> is the residual^2.
// PREC != PPL_FP64 (mode 1): also the new amplitudes as the operands of the next sweep's GEMMs.
struct SweepArgs {
  const double *e_occ, *e_vir, *vs, *va;
  double *sp, *am, *partials;
  void *op, *op_lo, *om, *om_lo;       // operand rows S', A'
  double *tslot, *eslot;
  const double* E;                     // error slots
  int64_t slot_n;
  DiisSet set;                         // the earlier errors
  double* dots;                        // partials of their inner products
};

template <int MODE, class Tr, int PREC = PPL_FP64, int ND = -1>
__global__ void __launch_bounds__(kReduceThreads)
sweep_kernel(PairGeom g, SweepArgs w, SliceSum<Tr> rp, SliceSum<Tr> rm) {
  constexpr bool SAVE = ND >= 0;
  constexpr int NS = ND > 0 ? ND : 1;
  double r2 = 0.0, en = 0.0, bad = 0.0, dot[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) dot[i] = 0.0;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  const int64_t tid0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  // "+" part: weights (2 - d_ij)(2 - d_ab) turn packed sums into full-tensor sums
  const int64_t totp = g.Np * g.ldp, totm = g.Nm * g.ldm;
  const bool narrow = totp < 0x7fffffffLL && totm < 0x7fffffffLL;
  for (int64_t x = tid0; x < totp; x += st) {
    int64_t q, p;
    row_col(x, g.ldp, narrow, q, p);
    if (p >= g.Pp) continue;
    const int ij = g.tab_op[q], ab = g.tab_vp[p];
    const bool dij = pair_first(ij) == pair_second(ij), dab = pair_first(ab) == pair_second(ab);
    const double wf = (dij ? 1.0 : 2.0) * (dab ? 1.0 : 2.0);
    const double wab = dab ? 1.0 : 2.0;             // S' = wab * s
    const double vsx = w.vs[x];
    double snew;
    if (MODE == 0) {
      snew = vsx / denom(w.e_occ, w.e_vir, ij, ab);
      w.sp[x] = wab * snew;
    } else if (MODE == 1) {
      snew = (vsx + (double)rp[x]) / denom(w.e_occ, w.e_vir, ij, ab);
      const double sold = w.sp[x] / wab;
      const double ds = snew - sold;
      r2 += wf * ds * ds;
      w.sp[x] = wab * snew;
      if constexpr (PREC != PPL_FP64) Store<PREC>::put(w.op, w.op_lo, x, wab * snew);
      if constexpr (SAVE) {
        w.tslot[x] = wab * snew;
        w.eslot[x] = wab * ds;
        const double a = (dij ? 1.0 : 2.0) / wab * (wab * ds);
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (i < w.set.n) dot[i] += a * w.E[w.set.id[i] * w.slot_n + x];
      }
    } else {
      snew = w.sp[x] / wab;
    }
    if (!isfinite(snew)) bad += 1.0;
    en += wf * vsx * snew;
  }
  // "-" part: every packed (i<j, a<b) entry stands for 4 full-tensor entries
  for (int64_t x = tid0; x < totm; x += st) {
    int64_t q, p;
    row_col(x, g.ldm, narrow, q, p);
    if (p >= g.Pm) continue;
    const int ij = g.tab_om[q], ab = g.tab_vm[p];
    const double vax = w.va[x];
    double anew;
    if (MODE == 0) {
      anew = vax / denom(w.e_occ, w.e_vir, ij, ab);
      w.am[x] = 2.0 * anew;
    } else if (MODE == 1) {
      anew = (vax + (double)rm[x]) / denom(w.e_occ, w.e_vir, ij, ab);
      const double da = anew - 0.5 * w.am[x];
      r2 += 4.0 * da * da;
      w.am[x] = 2.0 * anew;
      if constexpr (PREC != PPL_FP64) Store<PREC>::put(w.om, w.om_lo, x, 2.0 * anew);
      if constexpr (SAVE) {
        w.tslot[totp + x] = 2.0 * anew;
        w.eslot[totp + x] = 2.0 * da;
        const double a = 2.0 * da;
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (i < w.set.n) dot[i] += a * w.E[w.set.id[i] * w.slot_n + totp + x];
      }
    } else {
      anew = 0.5 * w.am[x];
    }
    if (!isfinite(anew)) bad += 1.0;
    en += 12.0 * vax * anew;                        // E = sum V^S s + 3 sum V^A a (full tensor)
  }
  double vals[3] = {r2, en, bad};
  block_reduce_store<3>(vals, w.partials);
  if constexpr (ND > 0) block_reduce_store<NS>(dot, w.dots);
}

static PairGeom geom(int o, int v, int64_t ldp, int64_t ldm, const int* tab_op, const int* tab_om,
                     const int* tab_vp, const int* tab_vm) {
  return PairGeom{o, v, npairs_plus(o), npairs_minus(o), npairs_plus(v), npairs_minus(v), ldp, ldm,
                  tab_op, tab_om, tab_vp, tab_vm};
}

template <int MODE, class Tr, int PREC = PPL_FP64, int ND = -1>
static int sweep_launch(hipStream_t s, const PairGeom& g, const SweepArgs& w, const Slices& rp, const Slices& rm) {
  hipLaunchKernelGGL((sweep_kernel<MODE, Tr, PREC, ND>), dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, g, w,
                     slice_sum<Tr>(rp), slice_sum<Tr>(rm));
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int mp2_start(hipStream_t s, int o, int v, const double* e_occ, const double* e_vir, const double* vs,
              const double* va, int64_t ldp, int64_t ldm, double* sp, double* am, const int* tab_op,
              const int* tab_om, const int* tab_vp, const int* tab_vm, double* partials,
              double* red_out) {
  const PairGeom g = geom(o, v, ldp, ldm, tab_op, tab_om, tab_vp, tab_vm);
  SweepArgs w{e_occ, e_vir, vs, va, sp, am, partials};
  PPL_TRY((sweep_launch<0, double>(s, g, w, Slices{}, Slices{})));
  return final_reduce(s, partials, 3, nullptr, 0, red_out);
}

int update_sweep(hipStream_t s, int acc_prec, int o, int v, const double* e_occ, const double* e_vir,
                 const double* vs, const double* va, const Slices& rp, const Slices& rm, int64_t ldp, int64_t ldm,
                 double* sp, double* am, const int* tab_op, const int* tab_om, const int* tab_vp, const int* tab_vm,
                 double* partials, double* red_out, const OperandRows& op, const DiisSlot& d) {
  const PairGeom g = geom(o, v, ldp, ldm, tab_op, tab_om, tab_vp, tab_vm);
  const SweepArgs w{e_occ, e_vir, vs,       va,       sp,       am,       partials, op.sp,   op.sp_lo, op.am,
                    op.am_lo, d.t,   d.e,   d.E,      d.slot_n, d.others, d.partials};
  if (!d.t) {
    if (acc_prec == PPL_FP64) PPL_TRY((sweep_launch<1, double>(s, g, w, rp, rm)));
    else if (op.prec == PPL_FP32) PPL_TRY((sweep_launch<1, float, PPL_FP32>(s, g, w, rp, rm)));
    else if (op.prec == PPL_BF16X3) PPL_TRY((sweep_launch<1, float, PPL_BF16X3>(s, g, w, rp, rm)));
    else if (op.prec == PPL_BF16X6) PPL_TRY((sweep_launch<1, float, PPL_BF16X6>(s, g, w, rp, rm)));
    else PPL_TRY((sweep_launch<1, float>(s, g, w, rp, rm)));
    return final_reduce(s, partials, 3, nullptr, 0, red_out);
  }
  const int n = d.others.n;
  if (n < 0 || n >= kDiisMax) return fail(PPL_E_ARG, "DIIS set of %d vectors", n);
  // the smallest count of inner products that covers the subspace (their sums live in registers)
  if (acc_prec == PPL_FP64) {
    if (n == 0) PPL_TRY((sweep_launch<1, double, PPL_FP64, 0>(s, g, w, rp, rm)));
    else if (n <= 3) PPL_TRY((sweep_launch<1, double, PPL_FP64, 3>(s, g, w, rp, rm)));
    else if (n <= 7) PPL_TRY((sweep_launch<1, double, PPL_FP64, 7>(s, g, w, rp, rm)));
    else PPL_TRY((sweep_launch<1, double, PPL_FP64, 15>(s, g, w, rp, rm)));
  } else {
    if (n == 0) PPL_TRY((sweep_launch<1, float, PPL_FP64, 0>(s, g, w, rp, rm)));
    else if (n <= 3) PPL_TRY((sweep_launch<1, float, PPL_FP64, 3>(s, g, w, rp, rm)));
    else if (n <= 7) PPL_TRY((sweep_launch<1, float, PPL_FP64, 7>(s, g, w, rp, rm)));
    else PPL_TRY((sweep_launch<1, float, PPL_FP64, 15>(s, g, w, rp, rm)));
  }
  return final_reduce(s, partials, 3, d.partials, n, red_out);
}

// ------------------------------------------------------------------ DIIS subspace
// S'/A' = sum_i c_i T_i over the slots of the set; padding columns set to zero. PREC != PPL_FP64:
// also as the operands of the next sweep's GEMMs.
template <int PREC>
__global__ void __launch_bounds__(256)
diis_combine_kernel(PairGeom g, const double* __restrict__ T, int64_t slot_n, DiisSet set, double* sp, double* am,
                    OperandRows op) {
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  const int64_t tid0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t totp = g.Np * g.ldp, totm = g.Nm * g.ldm;
  const bool narrow = totp < 0x7fffffffLL && totm < 0x7fffffffLL;
  for (int64_t x = tid0; x < totp; x += st) {
    int64_t q, p;
    row_col(x, g.ldp, narrow, q, p);
    double y = 0.0;
    if (p < g.Pp)
      for (int i = 0; i < set.n; ++i) y += set.c[i] * T[set.id[i] * slot_n + x];
    sp[x] = y;
    if constexpr (PREC != PPL_FP64) Store<PREC>::put(op.sp, op.sp_lo, x, y);
  }
  for (int64_t x = tid0; x < totm; x += st) {
    int64_t q, p;
    row_col(x, g.ldm, narrow, q, p);
    double y = 0.0;
    if (p < g.Pm)
      for (int i = 0; i < set.n; ++i) y += set.c[i] * T[set.id[i] * slot_n + totp + x];
    am[x] = y;
    if constexpr (PREC != PPL_FP64) Store<PREC>::put(op.am, op.am_lo, x, y);
  }
}

int diis_combine(hipStream_t s, int o, int v, int64_t ldp, int64_t ldm, const double* T, int64_t slot_n,
                 const DiisSet& set, double* sp, double* am, const OperandRows& op) {
  if (set.n < 1 || set.n > kDiisMax) return fail(PPL_E_ARG, "DIIS set of %d vectors", set.n);
  PairGeom g = geom(o, v, ldp, ldm, nullptr, nullptr, nullptr, nullptr);
  const dim3 grid(grid_for(std::max(g.Np * ldp, g.Nm * ldm), 256));
  if (op.prec == PPL_FP32)
    hipLaunchKernelGGL(diis_combine_kernel<PPL_FP32>, grid, dim3(256), 0, s, g, T, slot_n, set, sp, am, op);
  else if (op.prec == PPL_BF16X3)
    hipLaunchKernelGGL(diis_combine_kernel<PPL_BF16X3>, grid, dim3(256), 0, s, g, T, slot_n, set, sp, am, op);
  else if (op.prec == PPL_BF16X6)
    hipLaunchKernelGGL(diis_combine_kernel<PPL_BF16X6>, grid, dim3(256), 0, s, g, T, slot_n, set, sp, am, op);
  else
    hipLaunchKernelGGL(diis_combine_kernel<PPL_FP64>, grid, dim3(256), 0, s, g, T, slot_n, set, sp, am, op);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int energy_only(hipStream_t s, int o, int v, const double* vs, const double* va, const double* sp,
                const double* am, int64_t ldp, int64_t ldm, const int* tab_op, const int* tab_om,
                const int* tab_vp, const int* tab_vm, double* partials, double* red_out) {
  PairGeom g = geom(o, v, ldp, ldm, tab_op, tab_om, tab_vp, tab_vm);
  SweepArgs w{nullptr, nullptr, vs, va, (double*)sp, (double*)am, partials};
  PPL_TRY((sweep_launch<2, double>(s, g, w, Slices{}, Slices{})));
  return final_reduce(s, partials, 3, nullptr, 0, red_out);
}

// Sums of (L^P_ac - L^P_ca)^2 and (L^P_ac)^2 + (L^P_ca)^2 over the virtual block, a < c
// (red_out[0], red_out[1]): the relative asymmetry of the Cholesky vectors. Work items are
// 32 x 32 block pairs (P, A <= C): block (A, C) and block (C, A) are both read along rows
// and the second is transposed through LDS, so that every read is coalesced.
__global__ void __launch_bounds__(kReduceThreads)
asym_kernel(const double* __restrict__ L, int n, int o, int v, int naux, double* partials) {
  static_assert(kReduceThreads == 256, "four elements of a 32 x 32 block per thread");
  __shared__ double tr[32][33];
  double d2 = 0.0, l2 = 0.0;
  const int nb = (v + 31) / 32;
  const int64_t per_p = (int64_t)nb * (nb + 1) / 2;
  const int64_t items = (int64_t)naux * per_p;
  const int tid = threadIdx.x;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t P = it / per_p;
    int k = (int)(it % per_p), A = 0;
    while (k >= nb - A) k -= nb - A++;           // block pair (A, C = A + k)
    const int C = A + k;
    const double* Lp = L + P * n * n;
    // blocks (C, A) and (A, C) by rows, all loads in flight; the first is stored transposed
    double ca[4], ac[4];
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const int e = tid + 256 * e4, r = e >> 5, q = e & 31;
      ca[e4] = (C * 32 + r < v && A * 32 + q < v) ? Lp[(int64_t)(o + C * 32 + r) * n + o + A * 32 + q] : 0.0;
      ac[e4] = (A * 32 + r < v && C * 32 + q < v) ? Lp[(int64_t)(o + A * 32 + r) * n + o + C * 32 + q] : 0.0;
    }
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const int e = tid + 256 * e4, r = e >> 5, q = e & 31;
      tr[q][r] = ca[e4];
    }
    __syncthreads();
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const int e = tid + 256 * e4, r = e >> 5, q = e & 31;
      const int a = A * 32 + r, c = C * 32 + q;
      if (a < c && c < v) {
        const double lac = ac[e4], lca = tr[r][q];
        d2 += (lac - lca) * (lac - lca);
        l2 += lac * lac + lca * lca;
      }
    }
    __syncthreads();
  }
  double vals[3] = {d2, l2, 0.0};
  block_reduce_store<3>(vals, partials);
}

int asymmetry_vv(hipStream_t s, const double* L, int o, int v, int naux, double* partials, double* red_out) {
  hipLaunchKernelGGL(asym_kernel, dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, L, o + v, o, v, naux, partials);
  PPL_LAUNCH_CHECK();
  return final_reduce(s, partials, 3, nullptr, 0, red_out);
}

__global__ void __launch_bounds__(kReduceThreads)
nonfinite_kernel(const double* __restrict__ x, int64_t n, double* partials) {
  double bad = 0.0;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += st)
    if (!isfinite(x[i])) bad += 1.0;
  double vals[3] = {0.0, 0.0, bad};
  block_reduce_store<3>(vals, partials);
}

int count_nonfinite(hipStream_t s, const double* x, int64_t n, double* partials, double* red_out) {
  hipLaunchKernelGGL(nonfinite_kernel, dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, x, n, partials);
  PPL_LAUNCH_CHECK();
  return final_reduce(s, partials, 3, nullptr, 0, red_out);
}


// ------------------------------------------------------------------ ring terms
// Operands of the ring terms as (o v) x (o v) matrices over the pairs (i,a) and (k,c),
// rows of ld elements (columns from o v on zero), stored in the operand precision PREC
// (FP64, FP32, or bf16 planes: the second pointer of each is its lo / mid plane):
//   Xa[(i,a)][(k,c)] = 2 t_ik^ac - t_ik^ca,  An[(i,a)][(k,c)] = -t_ik^ac,  B[(i,a)][(k,c)] = t_ik^ca.
// These passes move 32 x 32 blocks through LDS, so that both index orders are read and written
// along rows; bound by memory. (18, 190), FP64: packing 89 us for 0.37 GB, 154 element by element
// with strided partners; ring_exchange 42 for 0.19 GB, 111; ring_unpack 83 for 0.37 GB, 249.
template <int PREC>
__global__ void __launch_bounds__(256)
ring_pack_kernel(int o, int v, const double* __restrict__ t, int64_t ld, void* Xa, void* Xa_lo, void* An,
                 void* An_lo, void* B, void* B_lo) {
  __shared__ double sp[32][33], sq[32][33];
  const int nb = (v + 31) / 32;
  const int64_t per = (int64_t)nb * (nb + 1) / 2, items = (int64_t)o * o * per, ov = (int64_t)o * v;
  const int f = threadIdx.x & 31, m = threadIdx.x >> 5;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t ik = it / per, i = ik / o, k = ik - i * o;
    int q = (int)(it % per), ba = 0;
    while (q >= nb - ba) q -= nb - ba++;        // block pair (ba, bc = ba + q)
    const int a0 = ba * 32, c0 = (ba + q) * 32;
    const double* x = t + ik * v * v;
    double ac[4], ca[4];                        // x[a][c] at (a0 + r, c0 + f), x[c][a] at (c0 + r, a0 + f)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m + 8 * e;
      ac[e] = (a0 + r < v && c0 + f < v) ? x[(int64_t)(a0 + r) * v + c0 + f] : 0.0;
      ca[e] = (c0 + r < v && a0 + f < v) ? x[(int64_t)(c0 + r) * v + a0 + f] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sp[m + 8 * e][f] = ac[e];
      sq[m + 8 * e][f] = ca[e];
    }
    __syncthreads();
    auto put = [&](int row, int col, double u, double w) __attribute__((always_inline)) {
      if (row >= v || col >= v) return;
      const int64_t y = (i * v + row) * ld + k * v + col;
      Store<PREC>::put(Xa, Xa_lo, y, via_f32<PREC>(2.0 * u - w));
      Store<PREC>::put(An, An_lo, y, via_f32<PREC>(-u));
      Store<PREC>::put(B, B_lo, y, via_f32<PREC>(w));
    };
#pragma unroll
    for (int e = 0; e < 4; ++e) put(a0 + m + 8 * e, c0 + f, ac[e], sq[f][m + 8 * e]);
    if (q > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) put(c0 + m + 8 * e, a0 + f, ca[e], sp[f][m + 8 * e]);
    }
    if (k == o - 1 && ba + q == nb - 1) {       // the padding of rows (i, a)
      const int64_t pad = ld - ov;
      for (int64_t z = threadIdx.x; z < 32 * pad; z += 256) {
        const int a = a0 + (int)(z / pad);
        if (a >= v) break;
        const int64_t y = (i * v + a) * ld + ov + z % pad;
        Store<PREC>::put(Xa, Xa_lo, y, 0.0);
        Store<PREC>::put(An, An_lo, y, 0.0);
        Store<PREC>::put(B, B_lo, y, 0.0);
      }
    }
    __syncthreads();
  }
}

static dim3 ring_grid(int64_t items) { return dim3((unsigned)std::min<int64_t>(items, 16384)); }

int ring_pack(hipStream_t s, int o, int v, const double* t, int64_t ld, double* Xa, double* An, double* B) {
  return ring_pack_lp(s, PPL_FP64, o, v, t, ld, Xa, nullptr, An, nullptr, B, nullptr);
}

int ring_pack_lp(hipStream_t s, int prec, int o, int v, const double* t, int64_t ld, void* Xa, void* Xa_lo,
                 void* An, void* An_lo, void* B, void* B_lo) {
  if (o <= 0 || v <= 0) return PPL_OK;
  const int64_t nb = (v + 31) / 32;
  const dim3 grid = ring_grid((int64_t)o * o * (nb * (nb + 1) / 2));
  if (prec == PPL_FP64)
    hipLaunchKernelGGL(ring_pack_kernel<PPL_FP64>, grid, dim3(256), 0, s, o, v, t, ld, Xa, Xa_lo, An, An_lo, B, B_lo);
  else if (prec == PPL_FP32)
    hipLaunchKernelGGL(ring_pack_kernel<PPL_FP32>, grid, dim3(256), 0, s, o, v, t, ld, Xa, Xa_lo, An, An_lo, B, B_lo);
  else if (prec == PPL_BF16X3)
    hipLaunchKernelGGL(ring_pack_kernel<PPL_BF16X3>, grid, dim3(256), 0, s, o, v, t, ld, Xa, Xa_lo, An, An_lo, B,
                       B_lo);
  else if (prec == PPL_BF16X6)
    hipLaunchKernelGGL(ring_pack_kernel<PPL_BF16X6>, grid, dim3(256), 0, s, o, v, t, ld, Xa, Xa_lo, An, An_lo, B,
                       B_lo);
  else
    return fail(PPL_E_ARG, "ring_pack: unknown precision %d", prec);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// K[(k,c)][(j,b)] = (kj|bc) = G[(k,j)][(b,c)] (G rows of ldg elements); columns from o v on zero, in
// K and in J
__global__ void __launch_bounds__(256)
ring_exchange_kernel(int o, int v, const double* __restrict__ G, int64_t ldg, double* K, double* J, int64_t ld) {
  __shared__ double sh[32][33];
  const int nb = (v + 31) / 32;
  const int64_t items = (int64_t)o * o * nb * nb, ov = (int64_t)o * v;
  const int f = threadIdx.x & 31, m = threadIdx.x >> 5;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int64_t kj = it / (nb * nb), k = kj / o, j = kj - k * o;
    const int b0 = (int)(it / nb % nb) * 32, c0 = (int)(it % nb) * 32;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int b = b0 + m + 8 * e, c = c0 + f;
      sh[m + 8 * e][f] = (b < v && c < v) ? G[kj * ldg + (int64_t)b * v + c] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = c0 + m + 8 * e, b = b0 + f;
      if (b < v && c < v) K[(k * v + c) * ld + j * v + b] = sh[f][m + 8 * e];
    }
    if (j == o - 1 && b0 + 32 >= v) {
      const int64_t pad = ld - ov;
      for (int64_t z = threadIdx.x; z < 32 * pad; z += 256) {
        const int c = c0 + (int)(z / pad);
        if (c >= v) break;
        const int64_t y = (k * v + c) * ld + ov + z % pad;
        K[y] = 0.0;
        J[y] = 0.0;
      }
    }
    __syncthreads();
  }
}

int ring_exchange(hipStream_t s, int o, int v, const double* G, int64_t ldg, double* K, double* J, int64_t ld) {
  if (o <= 0 || v <= 0) return PPL_OK;
  const int64_t nb = (v + 31) / 32;
  hipLaunchKernelGGL(ring_exchange_kernel, ring_grid((int64_t)o * o * nb * nb), dim3(256), 0, s, o, v, G, ldg, K, J, ld);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// R_ij^ab = beta R_ij^ab + alpha (Y_ij^ab + Y_ji^ba) with Y_ij^ab = C1[(i,a)][(j,b)] - C2[(i,b)][(j,a)]
// (C1, C2 in the accumulator type Tc of the ring GEMMs). A block (a, b) of a pair i <= j writes
// R_ij^ab and R_ji^ba, which are the same sum.
template <class Tc>
__global__ void __launch_bounds__(256)
ring_unpack_kernel(int o, int v, const Tc* __restrict__ C1, const Tc* __restrict__ C2, int64_t ld, double* R,
                   double alpha, double beta) {
  __shared__ double s1[32][33], s2[32][33];
  const int nb = (v + 31) / 32;
  const int64_t items = npairs_plus(o) * nb * nb;
  const int f = threadIdx.x & 31, m = threadIdx.x >> 5;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    int64_t j = it / (nb * nb), i = 0;
    while (j >= o - i) j -= o - i++;            // pair (i, i + j)
    j += i;
    const int a0 = (int)(it / nb % nb) * 32, b0 = (int)(it % nb) * 32;
    double d1[4], d2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m + 8 * e;
      const bool in = a0 + r < v && b0 + f < v, tr = b0 + r < v && a0 + f < v;
      d1[e] = in ? (double)C1[(i * v + a0 + r) * ld + j * v + b0 + f] : 0.0;
      d2[e] = in ? (double)C2[(j * v + a0 + r) * ld + i * v + b0 + f] : 0.0;
      s1[r][f] = tr ? (double)C1[(j * v + b0 + r) * ld + i * v + a0 + f] : 0.0;
      s2[r][f] = tr ? (double)C2[(i * v + b0 + r) * ld + j * v + a0 + f] : 0.0;
    }
    __syncthreads();
    double y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m + 8 * e;
      y[e] = alpha * ((d1[e] - s2[f][r]) + (s1[f][r] - d2[e]));
      if (a0 + r < v && b0 + f < v) {
        double* p = R + (((int64_t)i * o + j) * v + a0 + r) * v + b0 + f;
        *p = beta == 0.0 ? y[e] : beta * *p + y[e];
      }
    }
    __syncthreads();
    if (i < j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s1[m + 8 * e][f] = y[e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = m + 8 * e;
        if (b0 + r < v && a0 + f < v) {
          double* p = R + (((int64_t)j * o + i) * v + b0 + r) * v + a0 + f;
          *p = beta == 0.0 ? s1[f][r] : beta * *p + s1[f][r];
        }
      }
      __syncthreads();
    }
  }
}

int ring_unpack(hipStream_t s, int o, int v, const double* C1, const double* C2, int64_t ld, double* R, double alpha,
                double beta) {
  if (o <= 0 || v <= 0) return PPL_OK;
  const int64_t nb = (v + 31) / 32;
  hipLaunchKernelGGL(ring_unpack_kernel<double>, ring_grid(npairs_plus(o) * nb * nb), dim3(256), 0, s, o, v, C1, C2,
                     ld, R, alpha, beta);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

int ring_unpack_f32(hipStream_t s, int o, int v, const float* C1, const float* C2, int64_t ld, double* R, double alpha,
                    double beta) {
  if (o <= 0 || v <= 0) return PPL_OK;
  const int64_t nb = (v + 31) / 32;
  hipLaunchKernelGGL(ring_unpack_kernel<float>, ring_grid(npairs_plus(o) * nb * nb), dim3(256), 0, s, o, v, C1, C2,
                     ld, R, alpha, beta);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

// R+- += the pair parts of a pair-symmetric full tensor (the inverse of unpack_r)
template <class Tc>
__global__ void __launch_bounds__(256)
add_pm_kernel(int o, int v, const double* __restrict__ R, Tc* rp, int64_t ldp, Tc* rm, int64_t ldm, int64_t Np,
              int64_t Pp, int64_t Nm, int64_t Pm, const int* __restrict__ tab_op, const int* __restrict__ tab_om,
              const int* __restrict__ tab_vp, const int* __restrict__ tab_vm) {
  const int64_t np = Np * Pp, total = np + Nm * Pm;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < total; x += st) {
    const bool plus = x < np;
    const int64_t y = plus ? x : x - np;
    const int64_t P = plus ? Pp : Pm;
    const int64_t q = y / P, c = y - q * P;
    const int ij = plus ? tab_op[q] : tab_om[q];
    const int ab = plus ? tab_vp[c] : tab_vm[c];
    const int64_t i = pair_first(ij), j = pair_second(ij), a = pair_first(ab), b = pair_second(ab);
    const double r1 = R[((i * o + j) * v + a) * v + b], r2 = R[((i * o + j) * v + b) * v + a];
    if (plus) {
      Tc* d = rp + q * ldp + c;
      *d = (Tc)((double)*d + 0.5 * (r1 + r2));
    } else {
      Tc* d = rm + q * ldm + c;
      *d = (Tc)((double)*d + 0.5 * (r1 - r2));
    }
  }
}

int add_pm(hipStream_t s, int c_prec, int o, int v, const double* R, void* rp, int64_t ldp, void* rm, int64_t ldm,
           const int* tab_op, const int* tab_om, const int* tab_vp, const int* tab_vm) {
  const int64_t Np = npairs_plus(o), Nm = npairs_minus(o), Pp = npairs_plus(v), Pm = npairs_minus(v);
  const int64_t n = Np * Pp + Nm * Pm;
  if (n <= 0) return PPL_OK;
  if (c_prec == PPL_FP64)
    hipLaunchKernelGGL(add_pm_kernel<double>, dim3(grid_for(n, 256)), dim3(256), 0, s, o, v, R, (double*)rp, ldp,
                       (double*)rm, ldm, Np, Pp, Nm, Pm, tab_op, tab_om, tab_vp, tab_vm);
  else
    hipLaunchKernelGGL(add_pm_kernel<float>, dim3(grid_for(n, 256)), dim3(256), 0, s, o, v, R, (float*)rp, ldp,
                       (float*)rm, ldm, Np, Pp, Nm, Pm, tab_op, tab_om, tab_vp, tab_vm);
  PPL_LAUNCH_CHECK();
  return PPL_OK;
}

}  // namespace ppl
