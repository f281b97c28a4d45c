// Learned start of the amplitude iteration: a 4 -> 128 -> 128 -> 1 SiLU network
// that maps per-element features of the first-order amplitudes,
//     x = (t_MP2 / sigma, D_ij^ab, e_i + e_j, e_a + e_b),
// to a correction f(x), giving the guess t = t_MP2 + sigma * f(x).
// Every feature is invariant under (i,j,a,b) -> (j,i,b,a), so the guess keeps
// the amplitudes' pair symmetry (eq. (2)).
//
// Training (FP32): one fused kernel per minibatch computes the forward pass,
// the mean-squared-error loss and the full backward pass for blocks of rows on
// the FP32 matrix cores, and writes per-workgroup gradient partials; a second
// kernel sums them in a fixed order (bitwise reproducible) and applies Adam.
// Inference: the 128 x 128 hidden layer runs on the BF16 matrix cores
// (16x16x32, FP32 accumulation); the small layers stay in FP32.
//
// Flat parameter order: W1 [128][4], b1 [128], W2 [128][128], b2 [128], W3 [128], b3 [1].
#include <algorithm>

#include "ppl_internal.h"

namespace ppl {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int kH = 128;
constexpr int kOffW1 = 0, kOffB1 = kH * 4, kOffW2 = kOffB1 + kH, kOffB2 = kOffW2 + kH * kH,
              kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH, kNParams = kOffB3 + 1;
constexpr int kTrainRows = 32;     // rows per block of a training workgroup
// training workgroups at most, one per CU; each further block of rows costs a workgroup less
// than another partial gradient (69 KB written and read) would
constexpr int kTrainGroups = 256;

int mlp_param_count() { return kNParams; }
int64_t mlp_train_partials(int64_t max_batch) {
  return std::min<int64_t>((max_batch + kTrainRows - 1) / kTrainRows, kTrainGroups);
}

// z / (1 + exp(-z)) with one reciprocal and one residual step for the quotient. Compared over every
// float on gfx950 with that expression as written: the same bits, except for -89 < z < -87.3, where
// it gives -0 for values of at most 1.1e-36, and z = +inf, where it gives NaN for +inf (silu_any has
// +inf). The exponential is held below 2^128, so that 1 + exp(-z) is finite; its reciprocal is flushed
// to zero above 2^126, which makes the result -0 for every finite z beyond.
__device__ inline float silu_f(float z) {
  const float d = 1.0f + __builtin_amdgcn_exp2f(fminf(-1.44269504088896340736f * z, 127.99f));
  const float r = __builtin_amdgcn_rcpf(d);
  const float y = z * r;
  return fmaf(fmaf(-d, y, z), r, y);
}
__device__ inline float silu_any(float z) { return z == __builtin_huge_valf() ? z : silu_f(z); }

// Sum over the 16 lanes of a row (l / 16 equal), the same in each: x + x(l^1), then l^2, then the
// other half of eight and of sixteen, whose lanes already hold equal sums.
__device__ inline float row_sum16(float x) {
  auto add = [&](int y) { x += __builtin_bit_cast(float, y); };
  auto bits = [&]() { return __builtin_bit_cast(int, x); };
  add(__builtin_amdgcn_update_dpp(0, bits(), 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  add(__builtin_amdgcn_update_dpp(0, bits(), 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  add(__builtin_amdgcn_update_dpp(0, bits(), 0x141, 0xF, 0xF, true));   // row_half_mirror
  add(__builtin_amdgcn_update_dpp(0, bits(), 0x140, 0xF, 0xF, true));   // row_mirror
  return x;
}

// ------------------------------------------------------------------ training
// grid = min(ceil(n / kTrainRows), kTrainGroups) workgroups of eight waves; a workgroup takes
// every gridDim.x-th block of kTrainRows rows, keeps the 128 x 128 weights in LDS and its
// gradient sums in registers, and writes one partial gradient. The three 128 x 128 products
// (Z2 = H1 W2^T, dH1 = dZ2 W2, dW2 = dZ2^T H1) run on the FP32 matrix cores (16x16x4: lane l
// holds A[l%16][l/16], B[l/16][l%16], D[4 (l/16) + r][l%16]). Wave w owns the columns
// [16 w, 16 w + 16) of H1, Z2 and dH1 and the same rows of dW2; 16-element groups of the summed
// index are read as k = 16 g + 4 (l/16) + e in step e, the same for both operands.
// Bound by the latencies of its phases (loads, three dependent products, six barriers):
// the products are 0.8 GFLOP at 8192 rows, 5 us of the matrix cores; 22 us (98 on the vector
// unit, with the weights and the gradient partials of every 32 rows moved per workgroup).
constexpr int kTrainThreads = 512;
constexpr int kTrainLd = kH + 4;   // 16-byte rows; 16 rows start in 16 different bank groups

__global__ void __launch_bounds__(kTrainThreads)
mlp_train_kernel(const float* __restrict__ prm, const float* __restrict__ X, const float* __restrict__ Y,
                 int64_t n, float inv_n, float* __restrict__ gpart, float* __restrict__ lpart) {
  constexpr int LD = kTrainLd, R = kTrainRows, NW = kTrainThreads / 64;
  static_assert(R == 32 && NW * 16 == kH, "two 16-row blocks, one 16-column block per wave");
  __shared__ __attribute__((aligned(16))) float sW2[kH * LD], sH1[R * LD], sZ2[R * LD];
  __shared__ __attribute__((aligned(16))) float sX[R][4];
  __shared__ float sY[R], sdy[R], sy[NW][R], sl[R], sb[R];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c16 = lane & 15, q = lane >> 4;
  const int col = 16 * wave + c16;
  for (int e = tid; e < kH * kH / 4; e += kTrainThreads) {
    const int h = e / (kH / 4), k = e % (kH / 4) * 4;
    *reinterpret_cast<f4*>(&sW2[h * LD + k]) = *reinterpret_cast<const f4*>(&prm[kOffW2 + h * kH + k]);
  }
  const f4 w1 = *reinterpret_cast<const f4*>(&prm[kOffW1 + col * 4]);
  const float b1 = prm[kOffB1 + col], b2 = prm[kOffB2 + col], w3 = prm[kOffW3 + col], b3 = prm[kOffB3];
  f4 gW2[kH / 16], gW1 = f4{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < kH / 16; ++j) gW2[j] = f4{0, 0, 0, 0};
  float gb1 = 0.0f, gb2 = 0.0f, gW3 = 0.0f, gb3 = 0.0f, lsum = 0.0f;
  const int64_t nblk = (n + R - 1) / R;
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t r0 = blk * R;
    __syncthreads();
    if (tid < R * 4) {
      const int r = tid / 4, c = tid % 4;
      sX[r][c] = (r0 + r < n) ? X[(r0 + r) * 4 + c] : 0.0f;
    }
    if (tid < R) sY[tid] = (r0 + tid < n) ? Y[r0 + tid] : 0.0f;
    __syncthreads();
    // layer 1: the wave's 16 columns, rows 16 mb + 4 q + r of this lane
    float d1[2][4];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * mb + 4 * q + r;
        const f4 x = *reinterpret_cast<const f4*>(sX[row]);
        float z = b1;
#pragma unroll
        for (int c = 0; c < 4; ++c) z += w1[c] * x[c];
        const float sg = 1.0f / (1.0f + __expf(-z));
        sH1[row * LD + col] = z * sg;
        d1[mb][r] = sg * (1.0f + z * (1.0f - sg));
      }
    __syncthreads();
    // layer 2 and the output
    f4 acc[2] = {f4{0, 0, 0, 0}, f4{0, 0, 0, 0}};
#pragma unroll
    for (int g = 0; g < kH / 16; ++g) {
      const f4 bw = *reinterpret_cast<const f4*>(&sW2[col * LD + 16 * g + 4 * q]);
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const f4 a = *reinterpret_cast<const f4*>(&sH1[(16 * mb + c16) * LD + 16 * g + 4 * q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], bw[e], acc[mb], 0, 0, 0);
      }
    }
    float h2[2][4], d2[2][4];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = acc[mb][r] + b2;
        const float sg = 1.0f / (1.0f + __expf(-z));
        h2[mb][r] = z * sg;
        d2[mb][r] = sg * (1.0f + z * (1.0f - sg));
        const float y = row_sum16(w3 * h2[mb][r]);
        if (c16 == 0) sy[wave][16 * mb + 4 * q + r] = y;
      }
    __syncthreads();
    if (tid < R) {
      float y = b3;
#pragma unroll
      for (int w = 0; w < NW; ++w) y += sy[w][tid];
      const float diff = (r0 + tid < n) ? (y - sY[tid]) : 0.0f;
      const float dy = 2.0f * diff * inv_n;
      sdy[tid] = dy;
      gb3 += dy;
      lsum += diff * diff;
    }
    __syncthreads();
    // dZ2, dW3, db2
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * mb + 4 * q + r;
        const float dy = sdy[row];
        gW3 += dy * h2[mb][r];
        const float dz = dy * w3 * d2[mb][r];
        gb2 += dz;
        sZ2[row * LD + col] = dz;
      }
    __syncthreads();
    // dW2[h][k] += sum_r dZ2[r][h] H1[r][k], h in the wave's 16 rows
#pragma unroll
    for (int g = 0; g < R / 16; ++g) {
      float a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = sZ2[(16 * g + 4 * q + e) * LD + col];
#pragma unroll
      for (int j = 0; j < kH / 16; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          gW2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], sH1[(16 * g + 4 * q + e) * LD + 16 * j + c16], gW2[j],
                                                        0, 0, 0);
    }
    // dH1[r][k] = sum_h dZ2[r][h] W2[h][k], then dZ1, dW1, db1
    acc[0] = acc[1] = f4{0, 0, 0, 0};
#pragma unroll
    for (int g = 0; g < kH / 16; ++g) {
      float bw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) bw[e] = sW2[(16 * g + 4 * q + e) * LD + col];
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const f4 a = *reinterpret_cast<const f4*>(&sZ2[(16 * mb + c16) * LD + 16 * g + 4 * q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], bw[e], acc[mb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dz = acc[mb][r] * d1[mb][r];
        const f4 x = *reinterpret_cast<const f4*>(sX[16 * mb + 4 * q + r]);
        gb1 += dz;
#pragma unroll
        for (int c = 0; c < 4; ++c) gW1[c] += dz * x[c];
      }
  }
  // the partial gradient: the four lane groups of a column hold disjoint rows
  float* gp = gpart + (int64_t)blockIdx.x * kNParams;
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
    gb1 += __shfl_xor(gb1, off, 64);
    gb2 += __shfl_xor(gb2, off, 64);
    gW3 += __shfl_xor(gW3, off, 64);
#pragma unroll
    for (int c = 0; c < 4; ++c) gW1[c] += __shfl_xor(gW1[c], off, 64);
  }
  if (q == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) gp[kOffW1 + col * 4 + c] = gW1[c];
    gp[kOffB1 + col] = gb1;
    gp[kOffB2 + col] = gb2;
    gp[kOffW3 + col] = gW3;
  }
#pragma unroll
  for (int j = 0; j < kH / 16; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) gp[kOffW2 + (16 * wave + 4 * q + r) * kH + 16 * j + c16] = gW2[j][r];
  if (tid < R) {
    sl[tid] = lsum;
    sb[tid] = gb3;
  }
  __syncthreads();
  if (tid == 0) {
    float l = 0.0f, b = 0.0f;
    for (int r = 0; r < R; ++r) {
      l += sl[r];
      b += sb[r];
    }
    lpart[blockIdx.x] = l;
    gp[kOffB3] = b;
  }
}

// grad[p] = sum_w gpart[w][p], loss = inv_n sum_w lpart[w], and with ADAM the update of the
// parameters. One workgroup per 64 parameters; wave w sums the partials of its share in order,
// and the shares are added in order: the same bits in every run. All of a wave's loads are in
// flight together (at most kTrainGroups / 16 of them): one read latency where the sum over the
// partials by one thread per parameter waited for each (6.3 us with the Adam update, against 70 + 5
// us, at 256 partials).
template <bool ADAM>
__global__ void __launch_bounds__(1024)
mlp_reduce_kernel(const float* __restrict__ gpart, const float* __restrict__ lpart, int nwg, float inv_n,
                  float* __restrict__ grad, float* __restrict__ loss, float* __restrict__ prm, float* __restrict__ m,
                  float* __restrict__ v, float lr, float b1, float b2, float bc1, float bc2, float eps) {
  constexpr int NW = 16, C = kTrainGroups / NW;
  __shared__ float sh[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  const int per = (nwg + NW - 1) / NW, w0 = wave * per;   // per <= C
  float x[C];
#pragma unroll
  for (int k = 0; k < C; ++k)
    x[k] = (p < kNParams && k < per && w0 + k < nwg) ? gpart[(int64_t)(w0 + k) * kNParams + p] : 0.0f;
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < C; ++k) s += x[k];
  sh[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && p < kNParams) {
    float g = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) g += sh[w][lane];
    grad[p] = g;
    if constexpr (ADAM) {
      const float mm = b1 * m[p] + (1.0f - b1) * g;
      const float vv = b2 * v[p] + (1.0f - b2) * g * g;
      m[p] = mm;
      v[p] = vv;
      prm[p] -= lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
    }
  }
  if (blockIdx.x == 0 && wave == 1) {        // the loss: lane l sums every 64th partial
    float l = 0.0f;
    for (int w = lane; w < nwg; w += 64) l += lpart[w];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) *loss = l * inv_n;
  }
}

static int train_groups(int64_t n) {
  const int64_t nblk = (n + kTrainRows - 1) / kTrainRows;
  return (int)(nblk < kTrainGroups ? nblk : kTrainGroups);
}

static int train_backward(hipStream_t s, const float* prm, const float* X, const float* Y, int64_t n, float* gpart,
                          float* lpart) {
  hipLaunchKernelGGL(mlp_train_kernel, dim3((unsigned)train_groups(n)), dim3(kTrainThreads), 0, s, prm, X, Y, n,
                     1.0f / (float)n, gpart, lpart);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

int mlp_grad_launch(hipStream_t s, const float* prm, const float* X, const float* Y, int64_t n, float* gpart,
                    float* lpart, float* grad, float* loss) {
  PPL_TRY(train_backward(s, prm, X, Y, n, gpart, lpart));
  hipLaunchKernelGGL(mlp_reduce_kernel<false>, dim3((kNParams + 63) / 64), dim3(1024), 0, s, gpart, lpart,
                     train_groups(n), 1.0f / (float)n, grad, loss, nullptr, nullptr, nullptr, 0.0f, 0.0f, 0.0f, 1.0f,
                     1.0f, 0.0f);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

int mlp_step_launch(hipStream_t s, float* prm, const float* X, const float* Y, int64_t n, float* gpart, float* lpart,
                    float* grad, float* loss, float* m, float* v, float lr, int step, float beta1, float beta2,
                    float eps) {
  PPL_TRY(train_backward(s, prm, X, Y, n, gpart, lpart));
  const float bc1 = 1.0f - powf(beta1, (float)step), bc2 = 1.0f - powf(beta2, (float)step);
  hipLaunchKernelGGL(mlp_reduce_kernel<true>, dim3((kNParams + 63) / 64), dim3(1024), 0, s, gpart, lpart,
                     train_groups(n), 1.0f / (float)n, grad, loss, prm, m, v, lr, beta1, beta2, bc1, bc2, eps);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

// ------------------------------------------------------------------ features, samples, sigma
__device__ inline void element_ijab(int64_t x, int o, int v, int& i, int& j, int& a, int& b) {
  b = (int)(x % v);
  const int64_t y = x / v;
  a = (int)(y % v);
  const int64_t z = y / v;
  j = (int)(z % o);
  i = (int)(z / o);
}

__global__ void mlp_samples_kernel(int o, int v, const double* __restrict__ tm, const double* __restrict__ ts,
                                   const double* __restrict__ e_occ, const double* __restrict__ e_vir,
                                   double sigma, const int64_t* __restrict__ idx, int64_t n, float* X,
                                   float* Y) {
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += st) {
    const int64_t x = idx[k];
    int i, j, a, b;
    element_ijab(x, o, v, i, j, a, b);
    const double eij = e_occ[i] + e_occ[j], eab = e_vir[a] + e_vir[b];
    X[k * 4 + 0] = (float)(tm[x] / sigma);
    X[k * 4 + 1] = (float)(e_occ[i] + e_occ[j] - e_vir[a] - e_vir[b]);
    X[k * 4 + 2] = (float)eij;
    X[k * 4 + 3] = (float)eab;
    if (Y) Y[k] = (float)((ts[x] - tm[x]) / sigma);
  }
}

int mlp_samples_launch(hipStream_t s, int o, int v, const double* tm, const double* ts, const double* e_occ,
                       const double* e_vir, double sigma, const int64_t* idx, int64_t n, float* X, float* Y) {
  int64_t g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(mlp_samples_kernel, dim3((unsigned)g), dim3(256), 0, s, o, v, tm, ts, e_occ, e_vir,
                     sigma, idx, n, X, Y);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

// ------------------------------------------------------------------ inference (BF16 MFMA hidden layer)
// The network's output (without its bias) at x where some hidden unit is NaN or +inf, so that the
// output is NaN or infinite in any order of its sums: element by element, the first layer anew
// for each unit of the second.
__device__ inline float far_output(const float* __restrict__ prm, f4 x) {
  auto h1 = [&](int k) __attribute__((always_inline)) {
    const float* w = &prm[kOffW1 + 4 * k];
    const float z = fmaf(w[3], x[3], fmaf(w[2], x[2], fmaf(w[1], x[1], fmaf(w[0], x[0], prm[kOffB1 + k]))));
    return (float)(__bf16)silu_any(z);
  };
#pragma unroll 1
  for (int k = 0; k < kH; ++k)
    if (const float h = h1(k); h != h) return h;
  float y = 0.0f;
#pragma unroll 1
  for (int j = 0; j < kH; ++j) {
    float z = 0.0f;
#pragma unroll 1
    for (int k = 0; k < kH; ++k) z = fmaf((float)(__bf16)prm[kOffW2 + j * kH + k], h1(k), z);
    y = fmaf(prm[kOffW3 + j], silu_any(z + prm[kOffB2 + j]), y);
  }
  return y;
}

// A work item is one 16 x 16 tile (a, b) of an occupied pair: (i < j) all tiles, (i = j) the
// tiles A <= B and in them a <= b. Each element gives the guess at (i,j,a,b) and at its pair
// partner (j,i,b,a), so no entry is written twice; the partners are written along their rows
// from an LDS transpose. A wave takes items in turn and 16 elements (fixed a) at a time: lane
// l holds element b = l % 16 and computes the hidden units k = 32 kk + 8 (l / 16) + 0..7 of it,
// which is the A operand of the 16x16x32 MFMA, so the first layer never leaves the registers;
// so does not the second layer's weight matrix, 128 registers of bf16 per lane, loaded once.
// Bound by the vector unit, 256 SiLUs per element: 1.0 ms at (20, 200), 8.0e6 evaluations; 3.4
// with the weights staged in LDS for every 64 elements, scattered partners and the compiler's
// quotient (1.56 with that quotient). Results are bit-identical to that form.
constexpr int kInferThreads = 256;

__global__ void __launch_bounds__(kInferThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
mlp_infer_kernel(const float* __restrict__ prm, int o, int v, const double* __restrict__ tm,
                 const double* __restrict__ e_occ, const double* __restrict__ e_vir, double sigma,
                 const int* __restrict__ tab_om, int64_t n_first, int64_t n_items, int shift,
                 double* __restrict__ tout) {
  __shared__ __attribute__((aligned(16))) float sW1[kH][4], sb1[kH];
  __shared__ float sb2[kH], sW3[kH];
  __shared__ double sT[kInferThreads / 64][16][17];
  const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int e = tid; e < kH * 4; e += kInferThreads) sW1[e / 4][e % 4] = prm[kOffW1 + e];
  if (tid < kH) {
    sb1[tid] = prm[kOffB1 + tid];
    sb2[tid] = prm[kOffB2 + tid];
    sW3[tid] = prm[kOffW3 + tid];
  }
  const float b3 = prm[kOffB3];
  // B[k][n] = W2[n][k]: lane l holds n = 16 jb + l % 16, k = 32 kk + 8 (l / 16) + 0..7 (through LDS: read
  // by every wave from L2, 2048 waves took 10 us)
  constexpr int LD2 = kH + 8;
  __shared__ __attribute__((aligned(16))) __bf16 sW2[kH * LD2];
  for (int e = tid; e < kH * kH / 4; e += kInferThreads) {
    const f4 x = *reinterpret_cast<const f4*>(&prm[kOffW2 + 4 * e]);
#pragma unroll
    for (int k = 0; k < 4; ++k) sW2[e / (kH / 4) * LD2 + e % (kH / 4) * 4 + k] = (__bf16)x[k];
  }
  __syncthreads();
  bf8 w2[kH / 16][kH / 32];
#pragma unroll
  for (int jb = 0; jb < kH / 16; ++jb)
#pragma unroll
    for (int kk = 0; kk < kH / 32; ++kk)
      w2[jb][kk] = *reinterpret_cast<const bf8*>(&sW2[(16 * jb + c16) * LD2 + 32 * kk + 8 * q]);
  const int nb = (v + 15) / 16, per = nb * (nb + 1) / 2;
  const int64_t vv = (int64_t)v * v, nbb = (int64_t)nb * nb, nw = (int64_t)gridDim.x * (kInferThreads / 64);
  for (int64_t part = (int64_t)blockIdx.x * (kInferThreads / 64) + wave; part < n_items << shift; part += nw) {
    const int64_t it = part >> shift;
    int i, j, A, B;
    if (it < n_first) {
      const int ij = tab_om[it / nbb], rem = (int)(it % nbb);
      i = pair_first(ij);
      j = pair_second(ij);
      A = rem / nb;
      B = rem % nb;
    } else {
      i = j = (int)((it - n_first) / per);
      int r = (int)((it - n_first) % per);
      A = 0;
      while (r >= nb - A) r -= nb - A++;
      B = A + r;
    }
    const bool diag = i == j;
    const int b = 16 * B + c16;
    const double eo = e_occ[i] + e_occ[j], evb = b < v ? e_vir[b] : 0.0;
    const int64_t row_ij = ((int64_t)i * o + j) * vv, row_ji = ((int64_t)j * o + i) * vv;
    const int a0 = (int)(part & ((1 << shift) - 1)) * (16 >> shift), a1 = a0 + (16 >> shift);
    const int na = v - 16 * A < a1 ? v - 16 * A : a1;        // this part's rows a0 .. na - 1 of the tile
    if (a0 >= na) continue;
    bool nan = false;
    double t = b < v ? tm[row_ij + (int64_t)(16 * A + a0) * v + b] : 0.0;
    for (int al = a0; al < na; ++al) {
      const int a = 16 * A + al;
      const double tn = (al + 1 < na && b < v) ? tm[row_ij + (int64_t)(a + 1) * v + b] : 0.0;
      const double eva = e_vir[a];
      asm volatile("" ::: "memory");   // the first layer's weights stay in LDS, not in 160 registers
      const float x0 = (float)(t / sigma), x1 = (float)(eo - eva - evb), x2 = (float)eo, x3 = (float)(eva + evb);
      f4 acc[kH / 16];
#pragma unroll
      for (int jb = 0; jb < kH / 16; ++jb) acc[jb] = f4{0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < kH / 32; ++kk) {
        bf8 h1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int h = 32 * kk + 8 * q + e;
          const f4 w = *reinterpret_cast<const f4*>(sW1[h]);
          const float z = fmaf(w[3], x3, fmaf(w[2], x2, fmaf(w[1], x1, fmaf(w[0], x0, sb1[h]))));
          h1[e] = (__bf16)silu_f(z);
        }
#pragma unroll
        for (int jb = 0; jb < kH / 16; ++jb)
          acc[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, w2[jb][kk], acc[jb], 0, 0, 0);
      }
      // lane holds elements 4 (l / 16) + r of the 16, hidden units 16 jb + l % 16
      float part[4] = {0, 0, 0, 0};
#pragma unroll
      for (int jb = 0; jb < kH / 16; ++jb) {
        const float bb = sb2[16 * jb + c16], w = sW3[16 * jb + c16];
#pragma unroll
        for (int r = 0; r < 4; ++r) part[r] = fmaf(w, silu_f(acc[jb][r] + bb), part[r]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) part[r] = row_sum16(part[r]);
      if ((c16 >> 2) == q) {       // this lane's own element is among its group's four
        const int r = c16 & 3;
        const float y = r == 0 ? part[0] : (r == 1 ? part[1] : (r == 2 ? part[2] : part[3]));
        const double guess = fma(sigma, (double)(y + b3), t);
        nan |= guess != guess;
        sT[wave][c16][al] = guess;
        if (b < v && (!diag || a <= b)) tout[row_ij + (int64_t)a * v + b] = guess;
      }
      t = tn;
    }
    if (nan)                         // NaN where a hidden unit may be at +inf: which of the two it is
      for (int al = a0; al < na; ++al) {
        const int a = 16 * A + al;
        const double tx = b < v ? tm[row_ij + (int64_t)a * v + b] : 0.0, eva = e_vir[a];
        if (sT[wave][c16][al] == sT[wave][c16][al] || tx != tx) continue;
        const float y = far_output(prm, f4{(float)(tx / sigma), (float)(eo - eva - evb), (float)eo, (float)(eva + evb)});
        const double guess = fma(sigma, (double)(y + b3), tx);
        sT[wave][c16][al] = guess;
        if (b < v && (!diag || a <= b)) tout[row_ij + (int64_t)a * v + b] = guess;
      }
    // partners (j,i,b,a), along a (the wave's own LDS writes: in order, no barrier needed)
    __builtin_amdgcn_wave_barrier();
    const int a = 16 * A + c16;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int bl = 4 * k + q, bb = 16 * B + bl;
      if (c16 >= a0 && c16 < na && bb < v && (!diag || a < bb)) tout[row_ji + (int64_t)bb * v + a] = sT[wave][bl][c16];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

int mlp_infer_launch(hipStream_t s, const float* prm, int o, int v, const double* tm, const double* e_occ,
                     const double* e_vir, double sigma, const int* tab_om, double* tout) {
  const int64_t nb = (v + 15) / 16;
  const int64_t n_first = npairs_minus(o) * nb * nb, n_items = n_first + (int64_t)o * (nb * (nb + 1) / 2);
  // Two waves per SIMD (the weights take half of the registers), items dealt to them in turn, in parts of
  // fewer rows where there are less than kInferItems per wave: whole tiles of 16 rows leave most waves
  // without work at (3, 17) (46 us; 8.5 so, 15.1 by 64 elements per workgroup) and their last round
  // uneven at (10, 100) (91 us; 74 with two items per wave, 84 and 81 with one and four).
  constexpr int64_t kWaves = 512 * (kInferThreads / 64), kInferItems = 2;
  int shift = 0;
  while (shift < 4 && n_items << shift < kInferItems * kWaves) ++shift;
  const int64_t groups = ((n_items << shift) + kInferThreads / 64 - 1) / (kInferThreads / 64);
  hipLaunchKernelGGL(mlp_infer_kernel, dim3((unsigned)std::min<int64_t>(groups, 512)), dim3(kInferThreads), 0, s, prm,
                     o, v, tm, e_occ, e_vir, sigma, tab_om, n_first, n_items, shift, tout);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

// sum of squares of a tensor (red_out[0]) with the fixed-order reduction of the sweep kernels
__global__ void __launch_bounds__(kReduceThreads)
sumsq_kernel(const double* __restrict__ x, int64_t n, double* partials) {
  __shared__ double sh[kReduceThreads];
  double s = 0.0;
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += st) s += x[i] * x[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partials[blockIdx.x * 4 + 0] = sh[0];
    partials[blockIdx.x * 4 + 1] = 0.0;
    partials[blockIdx.x * 4 + 2] = 0.0;
    partials[blockIdx.x * 4 + 3] = 0.0;
  }
}

__global__ void final_reduce_kernel2(const double* __restrict__ partials, int nblocks, double* out) {
  __shared__ double sh[kReduceThreads];
  double acc = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += kReduceThreads) acc += partials[b * 4];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

int sumsq_launch(hipStream_t s, const double* x, int64_t n, double* partials, double* red_out) {
  hipLaunchKernelGGL(sumsq_kernel, dim3(kReduceBlocks), dim3(kReduceThreads), 0, s, x, n, partials);
  PPL_HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(final_reduce_kernel2, dim3(1), dim3(kReduceThreads), 0, s, partials, kReduceBlocks,
                     red_out);
  PPL_HIP_TRY(hipGetLastError());
  return PPL_OK;
}

}  // namespace ppl
