// Coarsest-level exact solve (Algorithms 4/5, "exact solution of coarse
// grid"; Section 3 keeps that level near 600 unknowns).  The dense A_L is
// inverted once in setup by Gauss-Jordan elimination with partial pivoting,
// so each coarse solve in the cycle is one dense mat-vec (a GEMV over at most
// dense_max^2 entries) instead of two sequential triangular solves.
//
// The elimination runs as one kernel of at most 128 blocks: each block owns a
// band of columns (in LDS when the bands fit, else in the row-major work
// matrix in global memory); per pivot step the owner of
// column k picks the pivot and publishes column k, one grid barrier, then
// every block updates its band.  A single block needs no grid barrier.  The
// barrier needs all blocks resident at once, so the kernel is launched as a
// cooperative launch, which the runtime refuses (an error, not a hang) when
// the grid cannot be resident together; the grid never exceeds 128 one-CU
// workgroups of the 256 CUs.
#include <algorithm>
#include <cmath>
#include <vector>

#include "amg_internal.hpp"
#include "device_utils.hpp"

namespace amg {

namespace {
constexpr int kGJThreads = 1024;

__global__ void k_dense_zero(size_t nn, double* W) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t st = (size_t)gridDim.x * blockDim.x;
  for (; i < nn; i += st) W[i] = 0.0;
}

__global__ void k_dense_scatter(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                const double* __restrict__ val, double* __restrict__ W) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int k = rp[i]; k < rp[i + 1]; ++k) W[(size_t)i * n + ci[k]] = val[k];
}

__device__ __forceinline__ void grid_barrier(int* sync, int nblocks) {
  if (nblocks == 1) {
    __syncthreads();
    return;
  }
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) {
    const int gen = __hip_atomic_load(&sync[1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    const int arrived = __hip_atomic_fetch_add(&sync[0], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (arrived == nblocks - 1) {
      __hip_atomic_store(&sync[0], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&sync[1], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      while (__hip_atomic_load(&sync[1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == gen)
        __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  __threadfence();
}

// In-place Gauss-Jordan inversion of the n x n row-major W.  piv[k] records
// the row exchanged with row k at step k; colbuf holds 2 x n doubles.
__global__ void __launch_bounds__(kGJThreads) k_gauss_jordan(int n, int band, double* __restrict__ W,
                                                             int* __restrict__ piv,
                                                             double* __restrict__ colbuf, int* sync,
                                                             int* err) {
  __shared__ double s_rowk[1024];
  __shared__ double s_val[kGJThreads / kWave];
  __shared__ int s_idx[kGJThreads / kWave];
  const int nb = gridDim.x;
  const int c0 = blockIdx.x * band;
  const int c1 = min(n, c0 + band);
  const int w = c1 - c0;
  for (int k = 0; k < n; ++k) {
    double* cb = colbuf + (size_t)(k & 1) * n;
    const int owner = k / band;
    if ((int)blockIdx.x == owner) {
      // pivot: the largest |W[i][k]| over rows i >= k (smallest index on ties)
      double best = -1.0;
      int bi = k;
      for (int i = k + threadIdx.x; i < n; i += blockDim.x) {
        const double a = fabs(W[(size_t)i * n + k]);
        if (a > best) { best = a; bi = i; }
      }
      for (int off = kWave / 2; off > 0; off >>= 1) {
        const double ob = __shfl_xor(best, off, kWave);
        const int oi = __shfl_xor(bi, off, kWave);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
      }
      if ((threadIdx.x & (kWave - 1)) == 0) {
        s_val[threadIdx.x / kWave] = best;
        s_idx[threadIdx.x / kWave] = bi;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int q = 1; q < (int)(blockDim.x / kWave); ++q)
          if (s_val[q] > best || (s_val[q] == best && s_idx[q] < bi)) { best = s_val[q]; bi = s_idx[q]; }
        piv[k] = bi;
        if (!(best > 0.0)) atomic_or_flag(err, kErrSingular);
      }
      for (int i = threadIdx.x; i < n; i += blockDim.x) cb[i] = W[(size_t)i * n + k];
    }
    grid_barrier(sync, nb);
    const int p = __hip_atomic_load(&piv[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // column k after the exchange of rows k and p
    const double ck = cb[p];
    // exchange rows k and p inside this band, keep the (exchanged) row k
    for (int j = threadIdx.x; j < w; j += blockDim.x) {
      const int col = c0 + j;
      double a = W[(size_t)k * n + col];
      if (p != k) {
        const double b = W[(size_t)p * n + col];
        W[(size_t)p * n + col] = a;
        a = b;
      }
      s_rowk[j] = a;
    }
    __syncthreads();
    const double inv = 1.0 / ck;
    for (int e = threadIdx.x; e < n * w; e += blockDim.x) {
      const int i = e / w;
      const int j = e - i * w;
      const int col = c0 + j;
      const double ci = (i == k) ? ck : (i == p ? cb[k] : cb[i]);
      double* dst = W + (size_t)i * n + col;
      if (col == k) {
        *dst = (i == k) ? inv : -ci * inv;
      } else if (i == k) {
        *dst = s_rowk[j] * inv;
      } else {
        *dst -= ci * (s_rowk[j] * inv);
      }
    }
    __syncthreads();
  }
}

// One Gauss-Jordan step k applied to a block's LDS band (column-major,
// S[j*n + i] = W[i][c0 + j]): rows k and p exchanged, then the update with
// the pre-exchange pivot column `col` (LDS) and the staged pivot row.
__device__ __forceinline__ void gj_apply(double* S, int n, int c0, int w, int k, int p, const double* col,
                                         double* s_rowk) {
  const int tid = threadIdx.x;
  const double ck = col[p];
  for (int j = tid; j < w; j += blockDim.x) {
    double a = S[(size_t)j * n + k];
    if (p != k) {
      const double b = S[(size_t)j * n + p];
      S[(size_t)j * n + p] = a;
      a = b;
    }
    s_rowk[j] = a;
  }
  __syncthreads();
  const double inv = 1.0 / ck;
  for (int e = tid; e < w * n; e += blockDim.x) {
    const int j = e / n, i = e - j * n;
    const int colj = c0 + j;
    const double ci = (i == k) ? ck : (i == p ? col[k] : col[i]);
    double* dst = S + (size_t)j * n + i;
    if (colj == k) {
      *dst = (i == k) ? inv : -ci * inv;
    } else if (i == k) {
      *dst = s_rowk[j] * inv;
    } else {
      *dst -= ci * (s_rowk[j] * inv);
    }
  }
  __syncthreads();
}

// Gauss-Jordan with each block's band of columns resident in LDS.  The owner
// of a band runs that band's pivot steps on its own (no grid barrier: its
// columns already hold every earlier step), publishes the pivot rows and the
// pre-exchange pivot columns, and after one grid barrier the other blocks
// replay those steps on their bands.  Grid barriers: one per band.
__global__ void __launch_bounds__(kGJThreads) k_gauss_jordan_lds(int n, int band, double* __restrict__ W,
                                                                 int* __restrict__ piv,
                                                                 double* __restrict__ colbuf, int* sync,
                                                                 int* err) {
  extern __shared__ double S[];
  double* s_col = S + (size_t)band * n;
  double* s_rowk = s_col + n;
  __shared__ double s_val[kGJThreads / kWave];
  __shared__ int s_idx[kGJThreads / kWave];
  __shared__ int s_p;
  const int nb = gridDim.x;
  const int c0 = blockIdx.x * band;
  const int w = min(n, c0 + band) - c0;
  const int tid = threadIdx.x;
  for (int e = tid; e < w * n; e += blockDim.x) {
    const int i = e / w, j = e - i * w;
    S[j * n + i] = W[(size_t)i * n + c0 + j];
  }
  __syncthreads();
  for (int pb = 0; pb < nb; ++pb) {
    const int pc0 = pb * band, pc1 = min(n, pc0 + band);
    if ((int)blockIdx.x == pb) {
      for (int k = pc0; k < pc1; ++k) {
        const double* col = S + (size_t)(k - c0) * n;
        double best = -1.0;
        int bi = k;
        for (int i = k + tid; i < n; i += blockDim.x) {
          const double a = fabs(col[i]);
          if (a > best) { best = a; bi = i; }
        }
        for (int off = kWave / 2; off > 0; off >>= 1) {
          const double ob = __shfl_xor(best, off, kWave);
          const int oi = __shfl_xor(bi, off, kWave);
          if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        if ((tid & (kWave - 1)) == 0) {
          s_val[tid / kWave] = best;
          s_idx[tid / kWave] = bi;
        }
        __syncthreads();
        if (tid == 0) {
          for (int q = 1; q < (int)(blockDim.x / kWave); ++q)
            if (s_val[q] > best || (s_val[q] == best && s_idx[q] < bi)) { best = s_val[q]; bi = s_idx[q]; }
          piv[k] = bi;
          s_p = bi;
          if (!(best > 0.0)) atomic_or_flag(err, kErrSingular);
        }
        for (int i = tid; i < n; i += blockDim.x) {
          s_col[i] = col[i];
          if (nb > 1) colbuf[(size_t)k * n + i] = col[i];
        }
        __syncthreads();
        gj_apply(S, n, c0, w, k, s_p, s_col, s_rowk);
      }
    }
    if (nb > 1) {
      grid_barrier(sync, nb);
      if ((int)blockIdx.x != pb) {
        for (int k = pc0; k < pc1; ++k) {
          const int p = __hip_atomic_load(&piv[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          for (int i = tid; i < n; i += blockDim.x) s_col[i] = colbuf[(size_t)k * n + i];
          __syncthreads();
          gj_apply(S, n, c0, w, k, p, s_col, s_rowk);
        }
      }
    }
  }
  for (int e = tid; e < w * n; e += blockDim.x) {
    const int i = e / w, j = e - i * w;
    W[(size_t)i * n + c0 + j] = S[j * n + i];
  }
}

// Undo the row exchanges as column exchanges (last step first) and emit the
// float64 and float32 inverses.
__global__ void k_gj_unpermute(int n, const double* __restrict__ W, const int* __restrict__ piv,
                               double* __restrict__ inv, float* __restrict__ inv32, int* perm_tmp) {
  extern __shared__ int s_perm[];
  if (threadIdx.x == 0) {
    for (int j = 0; j < n; ++j) s_perm[j] = j;
    for (int k = n - 1; k >= 0; --k) {
      const int p = piv[k];
      const int t = s_perm[k];
      s_perm[k] = s_perm[p];
      s_perm[p] = t;
    }
  }
  __syncthreads();
  (void)perm_tmp;
  const size_t nn = (size_t)n * n;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < nn; e += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / n);
    const int j = (int)(e - (size_t)i * n);
    const double v = W[(size_t)i * n + s_perm[j]];
    inv[e] = v;
    if (inv32) inv32[e] = (float)v;
  }
}
// Batched systems: one workgroup inverts one terminal system.  Its bands of
// columns pass through LDS one after another (left-looking): a band first
// replays the pivot steps already taken (pivot rows in piv, pre-exchange pivot
// columns in cb), then takes its own steps and publishes them; a second pass
// replays the later steps on the earlier bands.  Each element sees the same
// sequence of updates as in k_gauss_jordan_lds, so the inverse is the same.
__global__ void __launch_bounds__(kGJThreads) k_gj_batched(const TermInfo* __restrict__ ti, double* __restrict__ work,
                                                           double* __restrict__ cbuf, int* __restrict__ pivbuf,
                                                           int lds_doubles, int* err) {
  extern __shared__ double S[];
  __shared__ double s_val[kGJThreads / kWave];
  __shared__ int s_idx[kGJThreads / kWave];
  __shared__ int s_p;
  const TermInfo t = ti[blockIdx.x];
  const int n = t.n;
  double* W = work + t.off;
  double* cb = cbuf + t.off;
  int* piv = pivbuf + t.row0;
  const int band = min(n, (lds_doubles - n) / (n + 1));
  double* s_col = S + (size_t)band * n;
  double* s_rowk = s_col + n;
  const int nb = (n + band - 1) / band;
  const int tid = threadIdx.x;
  auto load = [&](int c0, int w) {
    for (int e = tid; e < w * n; e += blockDim.x) {
      const int i = e / w, j = e - i * w;
      S[j * n + i] = W[(size_t)i * n + c0 + j];
    }
    __syncthreads();
  };
  auto store = [&](int c0, int w) {
    for (int e = tid; e < w * n; e += blockDim.x) {
      const int i = e / w, j = e - i * w;
      W[(size_t)i * n + c0 + j] = S[j * n + i];
    }
    __threadfence_block();
    __syncthreads();
  };
  auto replay = [&](int c0, int w, int k) {
    const int p = piv[k];
    for (int i = tid; i < n; i += blockDim.x) s_col[i] = cb[(size_t)k * n + i];
    __syncthreads();
    gj_apply(S, n, c0, w, k, p, s_col, s_rowk);
  };
  for (int pb = 0; pb < nb; ++pb) {
    const int c0 = pb * band, w = min(n, c0 + band) - c0;
    load(c0, w);
    for (int k = 0; k < c0; ++k) replay(c0, w, k);
    for (int k = c0; k < c0 + w; ++k) {
      const double* col = S + (size_t)(k - c0) * n;
      double best = -1.0;
      int bi = k;
      for (int i = k + tid; i < n; i += blockDim.x) {
        const double a = fabs(col[i]);
        if (a > best) { best = a; bi = i; }
      }
      for (int off = kWave / 2; off > 0; off >>= 1) {
        const double ob = __shfl_xor(best, off, kWave);
        const int oi = __shfl_xor(bi, off, kWave);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
      }
      if ((tid & (kWave - 1)) == 0) {
        s_val[tid / kWave] = best;
        s_idx[tid / kWave] = bi;
      }
      __syncthreads();
      if (tid == 0) {
        for (int q = 1; q < (int)(blockDim.x / kWave); ++q)
          if (s_val[q] > best || (s_val[q] == best && s_idx[q] < bi)) { best = s_val[q]; bi = s_idx[q]; }
        piv[k] = bi;
        s_p = bi;
        if (!(best > 0.0)) atomic_or_flag(err, kErrSingular);
      }
      for (int i = tid; i < n; i += blockDim.x) {
        s_col[i] = col[i];
        cb[(size_t)k * n + i] = col[i];
      }
      __threadfence_block();
      __syncthreads();
      gj_apply(S, n, c0, w, k, s_p, s_col, s_rowk);
    }
    store(c0, w);
  }
  for (int pb = 0; pb + 1 < nb; ++pb) {
    const int c0 = pb * band, w = min(n, c0 + band) - c0;
    load(c0, w);
    for (int k = c0 + w; k < n; ++k) replay(c0, w, k);
    store(c0, w);
  }
}

// Undo the row exchanges of each system as column exchanges (last step
// first); one workgroup per system.
__global__ void k_gj_unpermute_batched(const TermInfo* __restrict__ ti, const double* __restrict__ work,
                                       const int* __restrict__ pivbuf, double* __restrict__ inv,
                                       float* __restrict__ inv32) {
  extern __shared__ int s_perm[];
  const TermInfo t = ti[blockIdx.x];
  const int n = t.n;
  const int* piv = pivbuf + t.row0;
  if (threadIdx.x == 0) {
    for (int j = 0; j < n; ++j) s_perm[j] = j;
    for (int k = n - 1; k >= 0; --k) {
      const int p = piv[k];
      const int q = s_perm[k];
      s_perm[k] = s_perm[p];
      s_perm[p] = q;
    }
  }
  __syncthreads();
  const double* W = work + t.off;
  const size_t nn = (size_t)n * n;
  for (size_t e = threadIdx.x; e < nn; e += blockDim.x) {
    const int i = (int)(e / n);
    const int j = (int)(e - (size_t)i * n);
    const double v = W[(size_t)i * n + s_perm[j]];
    inv[t.off + e] = v;
    if (inv32) inv32[t.off + e] = (float)v;
  }
}

// dense copy of each terminal system's diagonal block (columns shifted to the
// system's first row)
__global__ void k_dense_scatter_batched(const TermInfo* __restrict__ ti, const int* __restrict__ rp,
                                        const int* __restrict__ ci, const double* __restrict__ val,
                                        double* __restrict__ work) {
  const TermInfo t = ti[blockIdx.x];
  double* W = work + t.off;
  for (int r = threadIdx.x; r < t.n; r += blockDim.x) {
    const int row = t.row0 + r;
    for (int k = rp[row]; k < rp[row + 1]; ++k) W[(size_t)r * t.n + (ci[k] - t.row0)] = val[k];
  }
}
// ---------------------------------------------------------------- no pivoting, blocked
// A symmetric positive definite matrix (or a diagonally dominant one) needs no
// pivoting in Gauss-Jordan elimination: every pivot is a diagonal entry of a
// Schur complement, hence positive.  One panel K of 32 columns is one launch:
// with M the inverse of the pivot block and U_J = M A_KJ,
//   A_KJ <- U_J,  A_iJ <- A_iJ - A_iK U_J,  A_KK <- M,  A_iK <- -A_iK M,
// every 32 x 32 tile by a workgroup of its own from the matrix before the
// panel, into a second buffer (the two swap), so nothing is read after it was
// written and no launch stands between pivot block and update.  The products
// are FP64 matrix-core steps (each wave one 16 x 16 quarter); the pivot block
// is inverted by one wave, by every workgroup for itself.  These
// matrices are small: what bounds the inversion is the chain of panels.  244
// unknowns: 8 panels of 50 us when pivot block (a workgroup with two barriers
// per step), its product, and two updates were four launches.
constexpr int kB = 32;

// orders a wave's own LDS writes before its lanes' later reads
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// In-place Gauss-Jordan inverse of a 16 x 16 block held by a wave in the layout
// of a matrix-core result (lane l: column l % 16, rows l / 16 + 4 i).  Returns
// whether every pivot was positive and finite.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, int2{__builtin_amdgcn_readlane(w.x, lane), __builtin_amdgcn_readlane(w.y, lane)});
}
__device__ __forceinline__ bool invert16(f64x4& a, int lane) {
  const int col = lane & 15, g = lane >> 4;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int ji = j / 4, jg = j % 4;
    const double p = lane_value(a[ji], 16 * jg + j);
    const double rj = __shfl(a[ji], 16 * jg + col, kWave);
    double c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __shfl(a[i], 16 * g + j, kWave);
    ok = ok && p > 0.0 && p < INFINITY;
    const double inv = 1.0 / p;
    const bool here = col == j;
    const double rk = here ? inv : rj * inv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double t = __builtin_fma(-c[i], rk, here ? 0.0 : a[i]);
      a[i] = i == ji && g == jg ? rk : t;
    }
  }
  return ok;
}

// The inverse of the pivot block of panel K (rows and columns c0 .. c0 + w - 1,
// identity beyond) into sM by one wave: the leading 16 x 16 block, its Schur
// complement and that one's inverse, the products on the matrix cores.  The
// chain of 32 pivots bounds it; holding all 32 columns of a row in two lanes
// took 15 us of a panel's 20; a panel now takes 13.5 (244 unknowns).
struct PivotScratch {
  double p[16][17], q[16][17];
};
__device__ __forceinline__ bool load_and_invert(const double* __restrict__ A, int n, int c0, int w, int lane,
                                                double (*sM)[kB + 1], PivotScratch& z) {
  const int col = lane & 15, g = lane >> 4;
  f64x4 a, d;
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = 2 * t + (lane >> 5), j = lane & 31;
    sM[i][j] = i < w && j < w ? A[(size_t)(c0 + i) * n + c0 + j] : (i == j ? 1.0 : 0.0);
  }
  wave_order();
  // X Y for 16 x 16 operands in LDS, added to u
  auto product = [&](auto x, auto y, f64x4 u, double sign) {
#pragma unroll
    for (int k = 0; k < 16; k += 4) u = mfma_f64_16x16x4(sign * x(col, k + g), y(k + g, col), u);
    return u;
  };
  auto block = [&](int r, int c) { return [=](int i, int j) { return sM[r + i][c + j]; }; };
  auto zp = [&](int i, int j) { return z.p[i][j]; };
  auto zq = [&](int i, int j) { return z.q[i][j]; };
  auto put = [&](auto&& at, const f64x4& u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) at(mfma_row(lane, i), mfma_col(lane)) = u[i];
  };
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = sM[mfma_row(lane, i)][col];
    d[i] = sM[16 + mfma_row(lane, i)][16 + col];
  }
  bool ok = invert16(a, lane);
  put([&](int i, int j) -> double& { return sM[i][j]; }, a);   // M11 of the leading block
  wave_order();
  put([&](int i, int j) -> double& { return z.p[i][j]; }, product(block(16, 0), block(0, 0), zero, 1.0));   // A21 M11
  put([&](int i, int j) -> double& { return z.q[i][j]; }, product(block(0, 0), block(0, 16), zero, 1.0));   // M11 A12
  wave_order();
  d = product(zp, block(0, 16), d, -1.0);   // A22 - A21 M11 A12
  ok = invert16(d, lane) && ok;
  wave_order();
  put([&](int i, int j) -> double& { return sM[16 + i][16 + j]; }, d);
  wave_order();
  const f64x4 m12 = product(zq, block(16, 16), zero, -1.0);
  const f64x4 m21 = product(block(16, 16), zp, zero, -1.0);
  put([&](int i, int j) -> double& { return sM[i][16 + j]; }, m12);
  put([&](int i, int j) -> double& { return sM[16 + i][j]; }, m21);
  wave_order();
  a = product(block(0, 16), zp, a, -1.0);   // M11 + M11 A12 M22 A21 M11
  put([&](int i, int j) -> double& { return sM[i][j]; }, a);
  wave_order();
  return ok;
}

// Buffer that holds system t before panel K: the swap ends in `inv`.
__device__ __forceinline__ bool source_is_inv(int n, int K) { return ((n + kB - 1) / kB - K) % 2 == 0; }

// Whether the operator was found unfit before the elimination (the error word,
// or null where nothing looked): the launches then end at once.
__device__ __forceinline__ bool is_refused(const int* err) { return err && (*err & kErrNotSPD); }

// dense copies of the systems' diagonal blocks (32 rows per workgroup)
__global__ void __launch_bounds__(256) k_gji_init(const TermInfo* __restrict__ ti, const int* __restrict__ rp,
                                                  const int* __restrict__ ci, const double* __restrict__ val,
                                                  double* __restrict__ inv, double* __restrict__ work,
                                                  const int* refused) {
  if (is_refused(refused)) return;
  const TermInfo t = ti[blockIdx.y];
  const int r0 = blockIdx.x * kB, rows = min(kB, t.n - r0);
  if (rows <= 0) return;
  double* W = (source_is_inv(t.n, 0) ? inv : work) + t.off + (size_t)r0 * t.n;
  for (int e = threadIdx.x; e < rows * t.n; e += 256) W[e] = 0.0;
  __syncthreads();   // the zeros are written before the entries
  const int r = threadIdx.x / 8;
  if (r >= rows) return;
  const int i = t.row0 + r0 + r;
  for (int k = rp[i] + (threadIdx.x & 7); k < rp[i + 1]; k += 8) W[(size_t)r * t.n + (ci[k] - t.row0)] = val[k];
}

// pivot blocks of panel K, one wave per system, for launches with so many
// tiles that inverting it in each costs more than a launch
__global__ void __launch_bounds__(kWave) k_gji_pivot(const TermInfo* __restrict__ ti, const double* __restrict__ inv,
                                                     const double* __restrict__ work, double* __restrict__ mbuf,
                                                     int K, int* err, const int* refused) {
  if (is_refused(refused)) return;
  const TermInfo t = ti[blockIdx.x];
  const int c0 = K * kB;
  if (c0 >= t.n) return;
  __shared__ double sM[kB][kB + 1];
  __shared__ PivotScratch z;
  const int lane = threadIdx.x;
  const double* A = (source_is_inv(t.n, K) ? inv : work) + t.off;
  if (!load_and_invert(A, t.n, c0, min(kB, t.n - c0), lane, sM, z) && lane == 0) atomic_or_flag(err, kErrNotSPD);
  for (int e = lane; e < kB * kB; e += kWave) mbuf[(size_t)blockIdx.x * kB * kB + e] = sM[e / kB][e % kB];
}

template <bool PIVOT>   // the workgroup inverts the pivot block itself (else mbuf)
__global__ void __launch_bounds__(256) k_gji_panel(const TermInfo* __restrict__ ti, double* __restrict__ inv,
                                                   double* __restrict__ work, float* __restrict__ inv32,
                                                   const double* __restrict__ mbuf, int K, int* err,
                                                   const int* refused) {
  if (is_refused(refused)) return;
  __shared__ double sM[kB][kB + 1], sA[kB][kB + 1], sT[kB][kB + 1];
  const TermInfo t = ti[blockIdx.z];
  const int n = t.n, c0 = K * kB, r0 = blockIdx.y * kB, q0 = blockIdx.x * kB;
  if (c0 >= n || r0 >= n || q0 >= n) return;
  const int w = min(kB, n - c0);
  const bool from_inv = source_is_inv(n, K);
  const double* A = (from_inv ? inv : work) + t.off;
  double* D = (from_inv ? work : inv) + t.off;
  const bool last = c0 + kB >= n;
  const bool pr = r0 == c0, pc = q0 == c0;   // in the pivot rows / columns
  const int tid = threadIdx.x, wv = tid / kWave, l = tid & (kWave - 1);
  if constexpr (PIVOT) {
    __shared__ PivotScratch z;
    if (wv == 0) {
      const bool ok = load_and_invert(A, n, c0, w, l, sM, z);
      if (pr && pc && !ok && l == 0) atomic_or_flag(err, kErrNotSPD);
    }
  } else {
    for (int e = tid; e < kB * kB; e += 256) sM[e / kB][e % kB] = mbuf[(size_t)blockIdx.z * kB * kB + e];
  }
  const int first = PIVOT ? kWave : 0, cnt = 256 - first;
  if (tid >= first) {
    for (int e = tid - first; e < kB * kB; e += cnt) {
      const int i = e / kB, j = e % kB;
      sA[i][j] = !pr && r0 + i < n && j < w ? A[(size_t)(r0 + i) * n + c0 + j] : 0.0;
      sT[i][j] = !pc && i < w && q0 + j < n ? A[(size_t)(c0 + i) * n + q0 + j] : 0.0;
    }
  }
  __syncthreads();
  const int tr = 16 * (wv >> 1), tc = 16 * (wv & 1);   // this wave's quarter
  f64x4 u = {0.0, 0.0, 0.0, 0.0};
  if (!pc) {
#pragma unroll
    for (int kk = 0; kk < kB; kk += 4) u = mfma_f64_16x16x4(sM[tr + (l & 15)][kk + (l >> 4)], sT[kk + (l >> 4)][tc + (l & 15)], u);
    __syncthreads();   // uniform: pc is the block's
#pragma unroll
    for (int i = 0; i < 4; ++i) sT[tr + mfma_row(l, i)][tc + mfma_col(l)] = u[i];
    __syncthreads();
  }
  const double (*U)[kB + 1] = pc ? sM : sT;
  f64x4 d;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = r0 + tr + mfma_row(l, i), col = q0 + tc + mfma_col(l);
    if (pr) d[i] = U[tr + mfma_row(l, i)][tc + mfma_col(l)];
    else d[i] = !pc && row < n && col < n ? A[(size_t)row * n + col] : 0.0;
  }
  if (!pr) {
#pragma unroll
    for (int kk = 0; kk < kB; kk += 4)
      d = mfma_f64_16x16x4(-sA[tr + (l & 15)][kk + (l >> 4)], U[kk + (l >> 4)][tc + (l & 15)], d);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = r0 + tr + mfma_row(l, i), col = q0 + tc + mfma_col(l);
    if (row < n && col < n) {
      D[(size_t)row * n + col] = d[i];
      if (last && inv32) inv32[t.off + (size_t)row * n + col] = (float)d[i];
    }
  }
}

}  // namespace

void launch_dense_inverse(int n, const int* rp, const int* ci, const double* val, double* work, double* inv,
                          float* inv32, int* sync, int* err, hipStream_t s) {
  const size_t nn = (size_t)n * n;
  k_dense_zero<<<(int)std::min<size_t>((nn + 255) / 256, 4096), 256, 0, s>>>(nn, work);
  k_dense_scatter<<<(n + 255) / 256, 256, 0, s>>>(n, rp, ci, val, work);
  int* piv = sync + 4;
  double* colbuf = work + nn;   // 2n doubles (global path) or n*n (LDS path)
  launch_fill_int(4, sync, 0, s);
  // LDS-resident bands when at most 128 blocks hold the matrix, else bands in
  // global memory (at most 64 blocks, band <= 1024 for the LDS pivot row)
  int dev = 0, lds_max = 0;
  AMG_HIP(hipGetDevice(&dev));
  AMG_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  const long budget = (long)lds_max - 4096;   // static LDS of the kernel
  long band = budget / 8 / (n + 1) - 1;
  if (band >= 1) {
    long nb = (n + band - 1) / band;
    band = (n + nb - 1) / nb;
    nb = (n + band - 1) / band;
    if (nb <= 128) {
      const size_t bytes = ((size_t)band * n + n + band) * sizeof(double);
      AMG_HIP(hipFuncSetAttribute((const void*)k_gauss_jordan_lds, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes));
      int bandi = (int)band;
      void* args[] = {&n, &bandi, &work, &piv, &colbuf, &sync, &err};
      AMG_HIP(hipLaunchCooperativeKernel((const void*)k_gauss_jordan_lds, dim3((unsigned)nb), dim3(kGJThreads), args,
                                         (unsigned)bytes, s));
      const int g = (int)std::min<size_t>((nn + 255) / 256, 1024);
      k_gj_unpermute<<<g, 256, n * sizeof(int), s>>>(n, work, piv, inv, inv32, nullptr);
      return;
    }
  }
  int nbg = (int)std::min<long>(64, std::max<long>(1, (long)nn / 16384));
  int bandg = (n + nbg - 1) / nbg;
  if (bandg > 1024) bandg = 1024;
  nbg = (n + bandg - 1) / bandg;
  {
    void* args[] = {&n, &bandg, &work, &piv, &colbuf, &sync, &err};
    AMG_HIP(hipLaunchCooperativeKernel((const void*)k_gauss_jordan, dim3((unsigned)nbg), dim3(kGJThreads), args, 0u, s));
  }
  const int g = (int)std::min<size_t>((nn + 255) / 256, 1024);
  k_gj_unpermute<<<g, 256, n * sizeof(int), s>>>(n, work, piv, inv, inv32, nullptr);
}

}  // namespace amg

namespace amg {

void launch_dense_inverse_batched(const Level& lv, int nterm, const TermInfo* d_term, const TermInfo* h_term,
                                  double* work, int* piv, double* inv, float* inv32, int* err, hipStream_t s) {
  if (nterm == 0) return;
  size_t total = 0;
  int nmax = 0;
  for (int t = 0; t < nterm; ++t) {
    total += (size_t)h_term[t].n * h_term[t].n;
    nmax = std::max(nmax, h_term[t].n);
  }
  double* cbuf = work + total;   // pre-exchange pivot columns, n x n per system
  launch_fill_double(total, work, 0.0, s);
  k_dense_scatter_batched<<<nterm, 256, 0, s>>>(d_term, lv.rp, lv.ci, lv.val, work);
  int dev = 0, lds_max = 0;
  AMG_HIP(hipGetDevice(&dev));
  AMG_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  const long budget = (long)lds_max - 4096;   // static LDS of the kernel
  const long need = (long)nmax * nmax + 2L * nmax;
  const long lds_d = std::min(need, budget / 8);
  if ((lds_d - nmax) / (nmax + 1) < 1) throw Error(AMG_ECOARSEN, "coarsest system too large for the LDS band");
  const size_t bytes = (size_t)lds_d * sizeof(double);
  AMG_HIP(hipFuncSetAttribute((const void*)k_gj_batched, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  k_gj_batched<<<nterm, kGJThreads, bytes, s>>>(d_term, work, cbuf, piv, (int)lds_d, err);
  k_gj_unpermute_batched<<<nterm, 256, nmax * sizeof(int), s>>>(d_term, work, piv, inv, inv32);
}

}  // namespace amg

namespace amg {

// Inverses of diagonal blocks (one per TermInfo) in inv (row-major n x n at
// each TermInfo's offset), blocked Gauss-Jordan without pivoting; inv32
// (optional) receives the float copy.  Raises kErrNotSPD on a non-positive
// pivot; the caller then redoes the inversion with pivoting.  checked: the
// operator was looked at, and a raised kErrNotSPD spares the elimination.  Scratch
// from tmp.
constexpr int kNoPivotMax = 8192;    // unknowns of a system at most
constexpr long kPivotTiles = 2048;   // tiles of a launch up to which each inverts the pivot block itself
void launch_dense_inverse_spd(int nterm, const TermInfo* d_term, const TermInfo* h_term, const int* rp, const int* ci,
                              const double* val, double* inv, float* inv32, Arena& tmp, int* err, hipStream_t s,
                              bool checked) {
  if (nterm == 0) return;
  const int* refused = checked ? err : nullptr;
  size_t total = 0;
  int nmax = 0;
  for (int t = 0; t < nterm; ++t) {
    total += (size_t)h_term[t].n * h_term[t].n;
    nmax = std::max(nmax, h_term[t].n);
  }
  if (nmax > kNoPivotMax) throw Error(AMG_ECOARSEN, "coarsest system too large for the dense inverse");
  double* work = tmp.alloc_n<double>(total);
  const int np = (nmax + kB - 1) / kB;
  // systems per launch within the grid's z (and y) limit
  constexpr int kZ = 65535;
  const bool own = (long)np * np * std::min(nterm, kZ) <= kPivotTiles;
  double* mbuf = own ? nullptr : tmp.alloc_n<double>((size_t)nterm * kB * kB);
  for (int t0 = 0; t0 < nterm; t0 += kZ) {
    const int nt = std::min(kZ, nterm - t0);
    k_gji_init<<<dim3(np, nt), 256, 0, s>>>(d_term + t0, rp, ci, val, inv, work, refused);
    for (int K = 0; K < np; ++K) {
      const dim3 g(np, np, nt);
      if (own) {
        k_gji_panel<true><<<g, 256, 0, s>>>(d_term + t0, inv, work, inv32, nullptr, K, err, refused);
      } else {
        k_gji_pivot<<<nt, kWave, 0, s>>>(d_term + t0, inv, work, mbuf, K, err, refused);
        k_gji_panel<false><<<g, 256, 0, s>>>(d_term + t0, inv, work, inv32, mbuf, K, err, refused);
      }
    }
  }
}

}  // namespace amg
