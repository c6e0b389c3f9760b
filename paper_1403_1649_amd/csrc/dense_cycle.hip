// The V-cycle of the level above the coarsest as a dense operator.  With the
// coarsest inverse C, the pre-smoothing restriction S = P^T (I - A W) and the
// post-smoothing operator T = (I - W A) P the level's cycle is
//   M b = (2 W - W A W) b + T C S b,
// three dependent launches (S b, C, post-smoothing) of 4 us each whatever they
// read.  Levels of at most kDenseCycleRows rows hold M itself: one product with
// it takes 4.2 us at 779 rows and 5.4 at 1,545, in place of 13.9.  Wider levels
// whose C S is small hold that: two launches.  Both are formed once per setup
// (30 to 45 us at those sizes) from the FP64 operators, and rounded to the
// cycle's precision when stored.
#include "amg_internal.hpp"
#include "device_utils.hpp"

namespace amg {

namespace {
constexpr int kBlock = 256;

// D (nc x n): rows of S scattered over zeros, a block per row
__global__ void __launch_bounds__(kBlock) k_dc_rows(int n, const int* __restrict__ sp, const int* __restrict__ sc,
                                                    const double* __restrict__ sv, double* __restrict__ D) {
  double* row = D + (size_t)blockIdx.x * n;
  for (int j = threadIdx.x; j < n; j += kBlock) row[j] = 0.0;
  __syncthreads();
  for (int k = sp[blockIdx.x] + threadIdx.x; k < sp[blockIdx.x + 1]; k += kBlock) row[sc[k]] = sv[k];
}

// V = C D on the matrix cores: a wave per 16 x 32 tile of V, its operands eight
// steps (32 of the inner index) at a time.
constexpr int kDcCols = 32;
__global__ void __launch_bounds__(kBlock) k_dc_product(int nc, int n, const double* __restrict__ C,
                                                       const double* __restrict__ D, int ld, double* __restrict__ V,
                                                       float* __restrict__ V32) {
  const int lane = threadIdx.x & (kWave - 1);
  const int tiles = (n + kDcCols - 1) / kDcCols;
  const int tile = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  if (tile >= tiles) return;
  const int r0 = blockIdx.y * 16, c0 = tile * kDcCols;
  const int row = r0 + (lane & 15), kq = lane >> 4;
  const int j0 = c0 + (lane & 15), j1 = j0 + 16;
  f64x4 u0 = {0.0, 0.0, 0.0, 0.0}, u1 = u0;
  for (int k0 = 0; k0 < nc; k0 += 32) {
    double a[8], b0[8], b1[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int k = k0 + 4 * t + kq;
      const bool in = k < nc;
      a[t] = in && row < nc ? C[(size_t)row * nc + k] : 0.0;
      b0[t] = in && j0 < n ? D[(size_t)k * n + j0] : 0.0;
      b1[t] = in && j1 < n ? D[(size_t)k * n + j1] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      u0 = mfma_f64_16x16x4(a[t], b0[t], u0);
      u1 = mfma_f64_16x16x4(a[t], b1[t], u1);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + mfma_row(lane, i);
    if (r >= nc) continue;
    for (int h = 0; h < 2; ++h) {   // columns n .. ld - 1 are zero
      const int j = c0 + 16 * h + mfma_col(lane);
      if (j >= ld) continue;
      const double v = h ? u1[i] : u0[i];
      if (V) V[(size_t)r * ld + j] = v;
      if (V32) V32[(size_t)r * ld + j] = (float)v;
    }
  }
}

// Row i of M = 2 W - W A W + T V, a block per row, the row held in LDS
__global__ void __launch_bounds__(kBlock) k_dc_cycle(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                     const double* __restrict__ val, const double* __restrict__ wd,
                                                     const int* __restrict__ tp, const int* __restrict__ tc,
                                                     const double* __restrict__ tv, int ldv,
                                                     const double* __restrict__ V, int ld, double* __restrict__ M,
                                                     float* __restrict__ M32) {
  __shared__ double row[kDenseCycleRows];
  const int i = blockIdx.x;
  const int t0 = tp[i], t1 = tp[i + 1];
  for (int j = threadIdx.x; j < n; j += kBlock) {
    double s = 0.0;
    for (int t = t0; t < t1; ++t) s += tv[t] * V[(size_t)tc[t] * ldv + j];
    row[j] = s;
  }
  __syncthreads();
  const double wi = wd[i];
  for (int k = rp[i] + threadIdx.x; k < rp[i + 1]; k += kBlock) {   // the columns of a row are distinct
    const int j = ci[k];
    row[j] += (j == i ? 2.0 * wi : 0.0) - wi * val[k] * wd[j];
  }
  __syncthreads();
  for (int j = threadIdx.x; j < ld; j += kBlock) {
    const double v = j < n ? row[j] : 0.0;
    if (M) M[(size_t)i * ld + j] = v;
    if (M32) M32[(size_t)i * ld + j] = (float)v;
  }
}
}  // namespace

bool dense_cycle_wanted(const Level& lv, int nc, int k) {
  if (!lv.sp) return false;
  return (k > 0 && lv.n <= kDenseCycleRows) || (size_t)lv.n * nc <= kDenseCoarse;
}

void launch_dense_cycle(const Level& lv, const double* cinv, Arena& tmp, hipStream_t s) {
  const bool whole = lv.mld > 0;
  const int n = lv.n, nc = lv.nc;
  if (nc < 1) return;
  // S and T in FP64 for it where the cycle holds them in FP32
  Level lf = lv;
  if (!lf.sv) {
    lf.sv = tmp.alloc_n<double>(std::max(lv.nnz, 1));
    lf.sv32 = nullptr;
    launch_ssmooth_fill(lf, s);
  }
  if (whole && !lf.tv) {
    lf.tv = tmp.alloc_n<double>(std::max(lv.tnnz, 1));
    lf.tv32 = nullptr;
    launch_tsmooth_fill(lf, s);
  }
  double* D = tmp.alloc_n<double>((size_t)nc * n);
  k_dc_rows<<<nc, kBlock, 0, s>>>(n, lf.sp, lf.sc, lf.sv, D);
  const int ldv = whole ? n : lv.gld;
  double* V = whole ? tmp.alloc_n<double>((size_t)nc * n) : lv.gop;
  const int tiles = (std::max(n, ldv) + kDcCols - 1) / kDcCols;
  k_dc_product<<<dim3((tiles + 3) / 4, (nc + 15) / 16), kBlock, 0, s>>>(nc, n, cinv, D, ldv, V,
                                                                         whole ? nullptr : lv.gop32);
  if (whole)
    k_dc_cycle<<<n, kBlock, 0, s>>>(n, lf.rp, lf.ci, lf.val, lf.wdinv, lf.tp, lf.tc, lf.tv, ldv, V, lv.mld, lv.mop,
                                    lv.mop32);
}

}  // namespace amg
