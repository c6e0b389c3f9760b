// Learned per-row Jacobi weights: omega_i = sigmoid(y_i) * 2|a_ii| /
// (|a_ii| + sum_{j != i} |a_ij|), y = MLP(features of row i), 9 -> 32 -> 32 -> 1
// with ReLU.  Operands are bfloat16 (round to nearest even), products and sums
// in FP32, biases FP32; hidden activations are rounded to bfloat16 before the
// next layer.  The bound makes 2 D Omega^-1 - A strictly diagonally dominant
// with a positive diagonal, so the smoother converges for SPD A.
//
// Training loss on a level (S samples with no coarse-space component,
// e = v - P P^T v):  L = (1/S) sum_s ||(I - W A) e||_A^2 / ||e||_A^2.
// Weight layout (1409 FP32 masters): W1[32][9], b1[32], W2[32][32], b2[32],
// W3[32], b3.
#include <algorithm>
#include <cmath>

#include "kernels_common.hpp"

namespace amg {

namespace {
constexpr int kIn = 9, kH = 32;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kH, kNP = oB3 + 1;   // 1409

__device__ __forceinline__ float bf16r(float x) {
  uint32_t u = __float_as_uint(x);
  u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
  return __uint_as_float(u);
}

// log|a_ii| summed over the level (for the level mean)
struct OpLogDiagSum {
  static constexpr int NV = 1;
  const double* diag;
  double* out;
  __device__ bool active() const { return true; }
  __device__ void idle() const {}
  __device__ void elem(int i, double* acc) const { acc[0] += log(fabs(diag[i])); }
  __device__ void finalize(const double* s) const { *out = s[0]; }
};

__global__ void __launch_bounds__(256) k_features(int n, int level, const int* __restrict__ rp,
                                                  const int* __restrict__ ci, const double* __restrict__ val,
                                                  const double* __restrict__ logsum, float* __restrict__ F,
                                                  double* __restrict__ beta) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double mean = *logsum / n;
  double d = 0.0;
  for (int k = rp[i]; k < rp[i + 1]; ++k)
    if (ci[k] == i) d = val[k];
  const double ad = fabs(d);
  double top[6] = {0, 0, 0, 0, 0, 0};
  double rs = 0.0, offabs = 0.0;
  for (int k = rp[i]; k < rp[i + 1]; ++k) {
    rs += val[k];
    if (ci[k] == i) continue;
    const double a = fabs(val[k]);
    offabs += a;
    double t = a / ad;
    for (int q = 0; q < 6; ++q) {   // keep the six largest, descending
      if (t > top[q]) { const double u = top[q]; top[q] = t; t = u; }
    }
  }
  float* f = F + (size_t)i * kIn;
  f[0] = bf16r((float)(log(ad) - mean));
  for (int q = 0; q < 6; ++q) f[1 + q] = bf16r((float)top[q]);
  f[7] = bf16r((float)(rs / d));
  f[8] = bf16r((float)level);
  if (beta) beta[i] = 2.0 * ad / (ad + offabs);
}

// The network's weights as the kernels use them: the matrices rounded to
// bfloat16, the biases as they are.
__global__ void k_round_weights(const float* __restrict__ wm, float* __restrict__ wr) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= kNP) return;
  const bool bias = (q >= oB1 && q < oW2) || (q >= oB2 && q < oW3) || q == oB3;
  wr[q] = bias ? wm[q] : bf16r(wm[q]);
}

// forward pass of one row (w: rounded weights, in LDS: with scalar loads, as
// the backward kernel takes them, the omega kernel measured 26 us on 64^3
// rows against 19)
struct Fwd {
  float h1[kH], h2[kH], y;
};

__device__ __forceinline__ void mlp_forward(const float* __restrict__ w, const float (&x)[kIn], Fwd& o) {
#pragma unroll
  for (int j = 0; j < kH; ++j) {
    float s = w[oB1 + j];
#pragma unroll
    for (int q = 0; q < kIn; ++q) s = fmaf(w[oW1 + j * kIn + q], x[q], s);
    o.h1[j] = bf16r(fmaxf(s, 0.f));
  }
#pragma unroll
  for (int j = 0; j < kH; ++j) {
    float s = w[oB2 + j];
#pragma unroll
    for (int q = 0; q < kH; ++q) s = fmaf(w[oW2 + j * kH + q], o.h1[q], s);
    o.h2[j] = bf16r(fmaxf(s, 0.f));
  }
  float y = w[oB3];
#pragma unroll
  for (int q = 0; q < kH; ++q) y = fmaf(w[oW3 + q], o.h2[q], y);
  o.y = y;
}

// omega_i and omega_i / a_ii for a level
__global__ void __launch_bounds__(256) k_mlp_omega(int n, const float* __restrict__ F, const double* __restrict__ beta,
                                                   const double* __restrict__ diag, const float* __restrict__ wr,
                                                   double* __restrict__ omega, double* __restrict__ wdinv,
                                                   float* __restrict__ wdinv32, double* __restrict__ sig_out) {
  __shared__ float s_w[kNP];
  for (int q = threadIdx.x; q < kNP; q += blockDim.x) s_w[q] = wr[q];
  __syncthreads();
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float x[kIn];
#pragma unroll
  for (int q = 0; q < kIn; ++q) x[q] = F[(size_t)i * kIn + q];
  Fwd o;
  mlp_forward(s_w, x, o);
  const double sg = 1.0 / (1.0 + exp(-(double)o.y));
  const double om = sg * beta[i];
  if (omega) omega[i] = om;
  if (sig_out) sig_out[i] = sg;
  if (wdinv) {
    const double wd = om / diag[i];
    wdinv[i] = wd;
    if (wdinv32) wdinv32[i] = (float)wd;
  }
}

// ---------------------------------------------------------------- loss pipeline
// v_s[i] = unit_uniform(i, seed + s) (or the caller's extra samples), then
// restricted per aggregate: c[I][s] = sum_{i in G_I} pval_i v_s[i]
__global__ void k_err_raw(int n, int S, int S_rand, uint32_t seed, const double* __restrict__ extra, double* __restrict__ V) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)n * S) return;
  const int i = (int)(t / S), s = (int)(t - (long)i * S);
  V[t] = s < S_rand ? unit_uniform((uint32_t)i, seed + (uint32_t)s) : extra[(size_t)i * (S - S_rand) + (s - S_rand)];
}

__global__ void k_err_restrict(int nc, int S, const int* __restrict__ agg_ptr, const int* __restrict__ agg_rows,
                               const double* __restrict__ pval, const double* __restrict__ V, double* __restrict__ C) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)nc * S) return;
  const int I = (int)(t / S), s = (int)(t - (long)I * S);
  double acc = 0.0;
  for (int k = agg_ptr[I]; k < agg_ptr[I + 1]; ++k) {
    const int i = agg_rows[k];
    acc += pval[i] * V[(size_t)i * S + s];
  }
  C[t] = acc;
}

// e_s -= P (P^T e_s) for the first S_proj samples (the others stay as given)
__global__ void k_err_project(int n, int S, int S_proj, const int* __restrict__ agg, const double* __restrict__ pval,
                              const double* __restrict__ C, double* __restrict__ E) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)n * S) return;
  const int i = (int)(t / S), s = (int)(t - (long)i * S);
  if (s < S_proj) E[t] -= pval[i] * C[(size_t)agg[i] * S + s];
}

// One product of the loss: Y = A X for a [n][S] block with the column dots
// d_s = sum_i X[i][s] Y[i][s], and what follows row by row in the same pass:
//   kFirst:  X = e, Y = A e kept, and the smoothed error E2 = e - (omega/a) A e
//   else:    X = E2; Y enters its dots and, with dy given, the derivative
//            dL/dy_i = (-2/S) sum_s Y[i][s] AE[i][s] / (ee_s a_ii) * beta_i sigma_i (1 - sigma_i)
//            and is not stored.
// A block takes 256/S whole rows at a time, so a thread keeps its column; the
// block's partial dots are summed over its rows in order.  64^3 rows, S = 8:
// the products, dots, smoothing and derivative as passes of their own took
// 51 + 45 + 10 + 14 us; the two passes here take 29 us each.
constexpr int kProdBlocks = 2048;
template <bool kFirst>
__global__ void __launch_bounds__(256) k_err_product(int n, int S, const int* __restrict__ rp,
                                                     const int* __restrict__ ci, const double* __restrict__ val,
                                                     const double* __restrict__ X, const double* __restrict__ omega,
                                                     const double* __restrict__ diag, double* __restrict__ AE,
                                                     double* __restrict__ E2, const double* __restrict__ ee,
                                                     const double* __restrict__ beta, const double* __restrict__ sig,
                                                     float* __restrict__ dy, double* __restrict__ part) {
  __shared__ double red[256];
  const int rpb = 256 / S;   // rows per pass of the block
  const int r = threadIdx.x / S, s = threadIdx.x - r * S;
  const bool on = r < rpb;
  const double inv = !kFirst && on ? ee[s] : 1.0;
  double dot = 0.0;
  for (int i0 = blockIdx.x * rpb; i0 < n; i0 += gridDim.x * rpb) {
    const int i = i0 + r;
    double term = 0.0;
    if (on && i < n) {
      const size_t t = (size_t)i * S + s;
      double acc = 0.0;
      for (int k = rp[i]; k < rp[i + 1]; ++k) acc += val[k] * X[(size_t)ci[k] * S + s];
      const double xi = X[t];
      dot += xi * acc;
      if constexpr (kFirst) {
        AE[t] = acc;
        E2[t] = xi - omega[i] / diag[i] * acc;
      } else if (dy) {
        term = acc * AE[t] / inv;
      }
    }
    if constexpr (!kFirst) {
      if (dy) {   // uniform over the grid
        red[threadIdx.x] = term;
        __syncthreads();
        if (on && s == 0 && i < n) {
          double a = 0.0;
          for (int q = 0; q < S; ++q) a += red[threadIdx.x + q];
          const double dom = -2.0 / S * a / diag[i];
          dy[i] = (float)(dom * beta[i] * sig[i] * (1.0 - sig[i]));
        }
        __syncthreads();
      }
    }
  }
  red[threadIdx.x] = dot;
  __syncthreads();
  if (threadIdx.x < S) {
    double a = 0.0;
    for (int q = 0; q < rpb; ++q) a += red[q * S + threadIdx.x];
    part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = a;
  }
}

// totals of the column dots, one block per column (fixed order)
__global__ void __launch_bounds__(256) k_coldot_final(int nb, const double* __restrict__ part,
                                                      double* __restrict__ out) {
  __shared__ double red[256 / kWave];
  double v[1] = {0.0};
  const double* p = part + (size_t)blockIdx.x * nb;
  for (int b = threadIdx.x; b < nb; b += 256) v[0] += p[b];
  block_sum<1>(v, red);
  if (threadIdx.x == 0) out[blockIdx.x] = v[0];
}

// Backward pass.  A wave takes tiles of 64 rows, a lane one row for the two
// layers' forward pass and dz1 = W2^T dz2 (FP32, scalar weights); the row
// vectors then go to the wave's own LDS, and the two weight matrices'
// gradients, sums over the tile's rows of outer products,
//   dW2 += dz2^T h1 (32 x 32),  dW1 += dz1^T x (32 x 9),
// are FP32 matrix-core steps with the rows as inner dimension
// (v_mfma_f32_32x32x2f32: lane l gives A[l % 32][l / 32] and B[l / 32][l % 32],
// two rows per step, and holds D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32] in
// element i); the bias and W3 gradients are summed by the lanes that read the
// same operands.  The vectors in LDS are padded to 33 floats a row, so that
// lanes writing their rows spread over the banks.  One partial gradient per
// block (its waves added in order).  The arithmetic is small (4.5 kFLOP a row);
// what bound the first version (one lane per gradient entry, walking the 64
// rows with two LDS reads per product, one wave per block) was the chain of
// LDS reads: 1889 us for 64^3 rows, 81 us now (2.2 GFLOP; two waves per SIMD
// wait on their scalar loads).
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kTile = 64;
constexpr int kBwdWaves = 2;     // waves per block
constexpr int kBwdBlocks = 1024;
constexpr int kPad = kH + 1;
constexpr int kXPad = kIn + 2;   // an odd stride
// A tile's vectors go through LDS in two turns: first dz2 (u) and h1 (v),
// then dz1 (u); h2, whose values are bfloat16, is kept in 16 bits.
struct BwdTile {
  float u[kTile * kPad], v[kTile * kPad];
  float x[kTile * kXPad];
  float dy[kTile];
  uint16_t h2[kTile * (kH + 2)];
};

__global__ void __launch_bounds__(kBwdWaves * kWave) k_mlp_backward(int n, const float* __restrict__ F,
                                                                    const float* __restrict__ dy,
                                                                    const float* __restrict__ wr,
                                                                    float* __restrict__ part) {
  __shared__ BwdTile s_tile[kBwdWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  BwdTile& T = s_tile[wv];
  const int col = lane & 31, half = lane >> 5;
  f32x16 d2 = {}, d1 = {};
  float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f;
  const int tiles = (n + kTile - 1) / kTile;
  const int stride = gridDim.x * kBwdWaves;
  const int rounds = (tiles + stride - 1) / stride;   // every wave of the block runs them all (barriers below)
  for (int rd = 0; rd < rounds; ++rd) {
    const int t = rd * stride + blockIdx.x * kBwdWaves + wv;
    const int i = t * kTile + lane;
    const bool on = t < tiles && i < n;
    float x[kIn];
#pragma unroll
    for (int q = 0; q < kIn; ++q) x[q] = on ? F[(size_t)i * kIn + q] : 0.f;
    const float g = on ? dy[i] : 0.f;   // rows past the end contribute zeros
    // the layers one unit at a time (only two units unrolled: the compiler
    // then holds two units' scalar weights instead of spilling all 1409);
    // row j of W2 serves the forward pass and dz1 in the same turn
    uint32_t on1 = 0u;
#pragma unroll 2
    for (int j = 0; j < kH; ++j) {
      float z = wr[oB1 + j];
#pragma unroll
      for (int q = 0; q < kIn; ++q) z = fmaf(wr[oW1 + j * kIn + q], x[q], z);
      on1 |= z > 0.f ? 1u << j : 0u;
      T.v[lane * kPad + j] = bf16r(fmaxf(z, 0.f));
    }
    float h1[kH], dh[kH];
#pragma unroll
    for (int m = 0; m < kH; ++m) {
      h1[m] = T.v[lane * kPad + m];
      dh[m] = 0.f;
    }
#pragma unroll 2
    for (int j = 0; j < kH; ++j) {
      const float* w = wr + oW2 + j * kH;
      float z = wr[oB2 + j];
#pragma unroll
      for (int q = 0; q < kH; ++q) z = fmaf(w[q], h1[q], z);
      const float dz2 = z > 0.f ? g * wr[oW3 + j] : 0.f;
      T.u[lane * kPad + j] = dz2;
      T.h2[lane * (kH + 2) + j] = (uint16_t)(__float_as_uint(bf16r(fmaxf(z, 0.f))) >> 16);
#pragma unroll
      for (int m = 0; m < kH; ++m) dh[m] = fmaf(dz2, w[m], dh[m]);
    }
#pragma unroll
    for (int q = 0; q < kIn; ++q) T.x[lane * kXPad + q] = x[q];
    T.dy[lane] = g;
    gb3 += g;
    __syncthreads();
#pragma unroll 8
    for (int r0 = 0; r0 < kTile; r0 += 2) {
      const int r = r0 + half;
      const float a = T.u[r * kPad + col];
      d2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a, T.v[r * kPad + col], d2, 0, 0, 0);
      gb2 += a;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kH; ++m) T.u[lane * kPad + m] = (on1 >> m) & 1u ? dh[m] : 0.f;
    __syncthreads();
#pragma unroll 8
    for (int r0 = 0; r0 < kTile; r0 += 2) {
      const int r = r0 + half;
      const float a = T.u[r * kPad + col];
      const float b = col < kIn ? T.x[r * kXPad + col] : 0.f;
      d1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, d1, 0, 0, 0);
      gb1 += a;
      gw3 = fmaf(T.dy[r], __uint_as_float((uint32_t)T.h2[r * (kH + 2) + col] << 16), gw3);
    }
    __syncthreads();
  }
  // the wave's gradient in LDS (its tile is free now), then the block's sum
  float* mine = reinterpret_cast<float*>(&T);
  static_assert(sizeof(BwdTile) >= kNP * sizeof(float), "the tile holds one gradient");
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = 8 * (i / 4) + 4 * half + i % 4;
    mine[oW2 + m * kH + col] = d2[i];
    if (col < kIn) mine[oW1 + m * kIn + col] = d1[i];
  }
  gb1 += __shfl_xor(gb1, 32, kWave);
  gb2 += __shfl_xor(gb2, 32, kWave);
  gw3 += __shfl_xor(gw3, 32, kWave);
  gb3 = wave_sum(gb3);
  if (half == 0) {
    mine[oB1 + col] = gb1;
    mine[oB2 + col] = gb2;
    mine[oW3 + col] = gw3;
  }
  if (lane == 0) mine[oB3] = gb3;
  __syncthreads();
  for (int p = threadIdx.x; p < kNP; p += kBwdWaves * kWave) {
    float a = 0.f;
#pragma unroll
    for (int v = 0; v < kBwdWaves; ++v) a += reinterpret_cast<const float*>(&s_tile[v])[p];
    part[(size_t)blockIdx.x * kNP + p] = a;
  }
}

// the blocks' gradients in FP64, fixed order: a lane per entry, the partials
// dealt to 16 waves (one thread per entry walking all partials alone: 254 us)
constexpr int kGradWaves = 16;
__global__ void __launch_bounds__(kGradWaves * kWave) k_grad_final(int nb, const float* __restrict__ part,
                                                                   float* __restrict__ grad, int accumulate) {
  __shared__ double red[kGradWaves][kWave];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int p = blockIdx.x * kWave + lane;
  double s = 0.0;
  if (p < kNP) {
#pragma unroll 8
    for (int b = wv; b < nb; b += kGradWaves) s += part[(size_t)b * kNP + p];
  }
  red[wv][lane] = s;
  __syncthreads();
  if (wv || p >= kNP) return;
  s = 0.0;
  for (int q = 0; q < kGradWaves; ++q) s += red[q][lane];
  grad[p] = accumulate ? grad[p] + (float)s : (float)s;
}

__global__ void k_adam(int n, float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

inline int nblk(long n, int t = 256) { return (int)((n + t - 1) / t); }
}  // namespace

int mlp_num_params() { return kNP; }

// level mean of log|a_ii| and the features of every row (float [n][9]);
// beta (optional) receives the omega bound 2|a_ii| / (|a_ii| + sum |a_ij|)
void mlp_features(Hierarchy& h, const Level& lv, int level, float* F, double* beta) {
  hipStream_t s = h.stream;
  double* slot = h.d_sc + kScArn + 60;
  launch_elem(lv.n, OpLogDiagSum{lv.diag, slot}, RedCtx{h.d_part, h.d_ticket}, s);
  k_features<<<nblk(lv.n), 256, 0, s>>>(lv.n, level, lv.rp, lv.ci, lv.val, slot, F, beta);
}

namespace {
// wdev with its matrices rounded to bfloat16, in scratch from tmp
const float* round_weights(Arena& tmp, const float* wdev, hipStream_t s) {
  float* wr = tmp.alloc_n<float>(kNP);
  k_round_weights<<<nblk(kNP), 256, 0, s>>>(wdev, wr);
  return wr;
}
}  // namespace

void mlp_omega(Hierarchy& h, Arena& tmp, const Level& lv, const float* F, const double* beta, const float* wdev,
               double* omega, double* wdinv, float* wdinv32, double* sig) {
  k_mlp_omega<<<nblk(lv.n), 256, 0, h.stream>>>(lv.n, F, beta, lv.diag, round_weights(tmp, wdev, h.stream), omega,
                                                wdinv, wdinv32, sig);
}

// Smoothing loss of a level and (optionally) its gradient.  Work arrays from
// `tmp`.  Returns the loss (synchronises); grad (device, kNP) when non-null.
double mlp_loss_grad(Hierarchy& h, Arena& tmp, const Level& lv, int level, const float* wdev, int S_rand,
                     uint32_t seed, const double* extra, int S_extra, const double* omega_fixed, float* grad,
                     int accumulate, bool raw_extra) {
  hipStream_t s = h.stream;
  const int n = lv.n, S = S_rand + S_extra;
  if (S < 1 || S > 64) throw Error(AMG_EINVAL, "1 to 64 error samples");
  const size_t nS = (size_t)n * S;
  double* AE = tmp.alloc_n<double>(nS);
  double* E2 = tmp.alloc_n<double>(nS);
  double* dots = tmp.alloc_n<double>(128);   // ||e_s||_A^2, then ||(I - W A) e_s||_A^2
  double* ee = dots;
  double* num = dots + S;
  const double* E = extra;   // samples taken as given
  if (S_rand > 0 || !raw_extra) {
    double* Ew = tmp.alloc_n<double>(nS);
    double* C = tmp.alloc_n<double>((size_t)lv.nc * S);
    k_err_raw<<<nblk((long)nS), 256, 0, s>>>(n, S, S_rand, seed, extra, Ew);
    k_err_restrict<<<nblk((long)lv.nc * S), 256, 0, s>>>(lv.nc, S, lv.agg_ptr, lv.agg_rows, lv.pval, Ew, C);
    k_err_project<<<nblk((long)nS), 256, 0, s>>>(n, S, raw_extra ? S_rand : S, lv.agg, lv.pval, C, Ew);
    E = Ew;
  }
  float* F = tmp.alloc_n<float>((size_t)n * kIn);
  double* beta = tmp.alloc_n<double>(n);
  double* om = tmp.alloc_n<double>(n);
  double* sig = tmp.alloc_n<double>(n);
  const float* wr = round_weights(tmp, wdev, s);
  mlp_features(h, lv, level, F, beta);
  const double* omega = omega_fixed;
  if (!omega) {
    k_mlp_omega<<<nblk(n), 256, 0, s>>>(n, F, beta, lv.diag, wr, om, nullptr, nullptr, sig);
    omega = om;
  }
  float* dy = grad && !omega_fixed ? tmp.alloc_n<float>(n) : nullptr;
  const int rpb = 256 / S;
  const int nbp = std::min((n + rpb - 1) / rpb, kProdBlocks);
  double* dpart = tmp.alloc_n<double>((size_t)S * nbp);
  k_err_product<true><<<nbp, 256, 0, s>>>(n, S, lv.rp, lv.ci, lv.val, E, omega, lv.diag, AE, E2, nullptr, nullptr,
                                          nullptr, nullptr, dpart);
  k_coldot_final<<<S, 256, 0, s>>>(nbp, dpart, ee);
  k_err_product<false><<<nbp, 256, 0, s>>>(n, S, lv.rp, lv.ci, lv.val, E2, nullptr, lv.diag, AE, nullptr, ee, beta,
                                           sig, dy, dpart);
  k_coldot_final<<<S, 256, 0, s>>>(nbp, dpart, num);
  if (dy) {
    const int tiles = (n + kTile - 1) / kTile;
    const int nb = std::min((tiles + kBwdWaves - 1) / kBwdWaves, kBwdBlocks);
    float* part = tmp.alloc_n<float>((size_t)nb * kNP);
    k_mlp_backward<<<nb, kBwdWaves * kWave, 0, s>>>(n, F, dy, wr, part);
    k_grad_final<<<nblk(kNP, kWave), kGradWaves * kWave, 0, s>>>(nb, part, grad, accumulate);
  }
  std::vector<double> hd(2 * (size_t)S);
  AMG_HIP(hipMemcpyAsync(hd.data(), dots, 2 * S * sizeof(double), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  AMG_HIP(hipGetLastError());
  double L = 0.0;
  for (int q = 0; q < S; ++q) L += hd[S + q] / hd[q];
  return L / S;
}

void mlp_adam(float* w, float* m, float* v, const float* g, int n, int step, float lr, float b1, float b2, float eps,
              hipStream_t s) {
  const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
  k_adam<<<nblk(n), 256, 0, s>>>(n, w, m, v, g, lr, b1, b2, eps, c1, c2);
}

}  // namespace amg
