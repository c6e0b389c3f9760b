// The post-smoothing operator of a level with damped Jacobi smoothing,
//   T = (I - W A) P,  W = diag(omega_i / a_ii)  (Algorithms 4 and 5, eq.
// damped_jacobi): a cycle's corrected and post-smoothed iterate is
//   x + P e + W (b - A (x + P e)) = [x + W (b - A x)] + T e,
// and the bracket is known once the residual before the coarse correction is.
// Row i of T holds one entry per distinct aggregate among the neighbours of i
// (its own first come first listed): on a seven-point grid about 3.3 entries
// against seven of A, on coarse levels 5 to 8 against 13 to 20.
#include "amg_internal.hpp"
#include "device_utils.hpp"

namespace amg {

namespace {
constexpr int kCap = 512;   // entries of A a wave takes at a time
constexpr int kWaves = 4;

__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Flag bits set once: waves that find them set leave the word alone.
__device__ __forceinline__ void raise(int* flags, int bits) {
  if ((__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bits) != bits) atomic_or_flag(flags, bits);
}

// What both kernels below write for an entry of T, and for a row.
struct TOut {
  const double* wd;
  const double* pval;
  const int* tp;
  int* tc;
  int16_t* tc16;
  int* tbase;
  double* tv;
  float* tv32;
  int* cnt;
  int* flags;
  int shift;
  __device__ __forceinline__ void entry(int at, int J, int jbase, double v) const {
    if (tc16) tc16[at] = (int16_t)(J - jbase);
    else tc[at] = J;
    if (tv) tv[at] = v;
    if (tv32) tv32[at] = (float)v;
  }
};

// Large levels.  A wave takes 64 rows, as many at a time as hold kCap entries:
// the aggregates (and, to fill, the products a_ij P_j) of the entries go to
// LDS by coalesced loads of A; then each lane merges one row, in entry order:
// the first kRegs distinct aggregates are kept in registers (compared all at
// once), any further ones in place at the head of the row's own range.  FILL:
// the merged row is written at tp[row], each value
// (J = agg(i) ? P_i : 0) - w_i sum_j a_ij P_j.  Otherwise its length goes to
// cnt, and *flags (shifted) collects what the level's kernels have to know.
// Bound by the pass over A and the gathers of agg and P.
constexpr int kRegs = 8;
template <bool FILL>
__global__ void __launch_bounds__(kWaves * kWave) k_tsmooth_rows(int n, const int* __restrict__ rp,
                                                                 const int* __restrict__ ci,
                                                                 const double* __restrict__ val,
                                                                 const int* __restrict__ agg, TOut o) {
  __shared__ int s_j[kWaves][kCap];
  __shared__ double s_t[FILL ? kWaves : 1][FILL ? kCap : 1];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const long groups = ((long)n + kWave - 1) / kWave;
  for (long g = (long)xcd_block_index() * kWaves + wv; g < groups; g += (long)gridDim.x * kWaves) {
    const int row0 = (int)(g * kWave), row = row0 + lane;
    const int rows = min(kWave, n - row0);
    const int jbase = agg[row0];
    if constexpr (FILL)
      if (o.tc16 && lane == 0) o.tbase[g] = jbase;
    int len = 0;   // of this lane's row of T
    const int beg = rp[min(row, n)], end = rp[min(row + 1, n)];
    for (int r = 0; r < rows;) {
      const int base = __builtin_amdgcn_readlane(beg, r);
      const int take = __popcll(__ballot(lane >= r && lane < rows && end - base <= kCap));
      if (take == 0) {
        if constexpr (!FILL)
          if (lane == r) {
            o.cnt[row] = 0;
            raise(o.flags, kTLongRow << o.shift);
          }
        ++r;
        continue;
      }
      const int total = __builtin_amdgcn_readlane(end, r + take - 1) - base;
#pragma unroll
      for (int q = 0; q < kCap / kWave; ++q) {
        const int k = q * kWave + lane;
        if (k < total) {
          const int j = ci[base + k];
          s_j[wv][k] = agg[j];
          if constexpr (FILL) s_t[wv][k] = val[base + k] * o.pval[j];
        }
      }
      wave_order();
      if (lane >= r && lane < r + take) {
        const int s = beg - base, e = end - base;
        int J[kRegs];
        double t[kRegs];
        int u = 0;   // distinct aggregates found; those beyond kRegs at s_j[s + kRegs ..]
#pragma unroll
        for (int p = 0; p < kRegs; ++p) {
          J[p] = -1;
          t[p] = 0.0;
        }
        for (int k = s; k < e; ++k) {
          const int Jk = s_j[wv][k];
          double tk = 0.0;
          if constexpr (FILL) tk = s_t[wv][k];
          if (Jk < 0) continue;
          bool hit = false;
#pragma unroll
          for (int p = 0; p < kRegs; ++p) {
            const bool mine = J[p] == Jk || (!hit && p == u);   // known, or its free register
            if (mine && !hit) {
              if (J[p] != Jk) {
                J[p] = Jk;
                ++u;
              }
              t[p] += tk;
              hit = true;
            }
          }
          if (hit) continue;
          int p = kRegs;
          while (p < u && s_j[wv][s + p] != Jk) ++p;
          if constexpr (FILL) s_t[wv][s + p] = p < u ? s_t[wv][s + p] + tk : tk;
          if (p == u) s_j[wv][s + u++] = Jk;
        }
        len = u;
        if constexpr (FILL) {
          const int own = agg[row], at = o.tp[row];
          const double w = o.wd[row], pi = o.pval[row];
#pragma unroll
          for (int p = 0; p < kRegs; ++p)
            if (p < u) o.entry(at + p, J[p], jbase, (J[p] == own ? pi : 0.0) - w * t[p]);
          for (int p = kRegs; p < u; ++p) {
            const int Jp = s_j[wv][s + p];
            o.entry(at + p, Jp, jbase, (Jp == own ? pi : 0.0) - w * s_t[wv][s + p]);
          }
        } else {
          o.cnt[row] = u;
          bool far = false;
#pragma unroll
          for (int p = 0; p < kRegs; ++p) far |= p < u && (J[p] - jbase < -32768 || J[p] - jbase > 32767);
          for (int p = kRegs; p < u; ++p) {
            const int d = s_j[wv][s + p] - jbase;
            far |= d < -32768 || d > 32767;
          }
          if (far) raise(o.flags, kTFar << o.shift);
        }
      }
      wave_order();
      r += take;
    }
    if constexpr (!FILL) {
      const int total = wave_sum_int(len);
      const int bits = total > 512 ? kTGroup512 | kTGroup320 | kTGroup256 : total > 320 ? kTGroup320 | kTGroup256
                       : total > 256 ? kTGroup256 : 0;
      if (bits && lane == 0) raise(o.flags, bits << o.shift);
    }
  }
}

// Small levels (a few thousand rows of 10 to 60 entries; one lane merging a
// row took 70 to 110 us on each, a chain of LDS reads): a wave per row, a lane
// per entry (64 at a time).  The lane compares its aggregate with each of the
// row's, read from LDS for the whole wave at once, so it knows whether it is
// the aggregate's first entry, and sums the aggregate's products in entry
// order; the first entries take their places by a ballot.  The same entries,
// order and sums as above.
template <bool FILL>
__global__ void __launch_bounds__(kWaves * kWave) k_tsmooth_wave(int n, const int* __restrict__ rp,
                                                                 const int* __restrict__ ci,
                                                                 const double* __restrict__ val,
                                                                 const int* __restrict__ agg, TOut o) {
  __shared__ int s_j[kWaves][kCap];
  __shared__ double s_t[FILL ? kWaves : 1][FILL ? kCap : 1];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  for (long row = (long)blockIdx.x * kWaves + wv; row < n; row += (long)gridDim.x * kWaves) {
    const int base = rp[row], len = rp[row + 1] - base;
    if (len > kCap) {
      if constexpr (!FILL)
        if (lane == 0) {
          o.cnt[row] = 0;
          raise(o.flags, kTLongRow << o.shift);
        }
      continue;
    }
    for (int k = lane; k < len; k += kWave) {
      const int j = ci[base + k];
      s_j[wv][k] = agg[j];
      if constexpr (FILL) s_t[wv][k] = val[base + k] * o.pval[j];
    }
    wave_order();
    int own = -1, at = 0;
    double w = 0.0, pi = 0.0;
    if constexpr (FILL) {
      own = agg[row];
      at = o.tp[row];
      w = o.wd[row];
      pi = o.pval[row];
    }
    int u = 0;
    for (int k0 = 0; k0 < len; k0 += kWave) {
      const int k = k0 + lane;
      const int J = k < len ? s_j[wv][k] : -1;
      bool first = J >= 0;
      double t = 0.0;
#pragma unroll 4
      for (int p = 0; p < len; ++p) {
        const bool same = s_j[wv][p] == J;
        first = first && !(same && p < k);
        if constexpr (FILL) {
          const double tk = s_t[wv][p];
          t = same ? t + tk : t;
        }
      }
      const uint64_t bits = __ballot(first);
      if constexpr (FILL)
        if (first) o.entry(at + u + __popcll(bits & ((1ull << lane) - 1)), J, 0, (J == own ? pi : 0.0) - w * t);
      u += __popcll(bits);
    }
    if constexpr (!FILL)
      if (lane == 0) o.cnt[row] = u;
    wave_order();
  }
}

int grid_for(int n) {
  const long b = ((long)n + kWaves * kWave - 1) / (kWaves * kWave);
  return (int)(b < 1 ? 1 : b < 65536 ? b : 65536);
}
}  // namespace

template <bool FILL>
static void launch_tsmooth(int n, const int* rp, const int* ci, const double* val, const int* agg, const TOut& o,
                           hipStream_t s) {
  if (n > kTsmoothRows) {
    k_tsmooth_rows<FILL><<<grid_for(n), kWaves * kWave, 0, s>>>(n, rp, ci, val, agg, o);
  } else if (n > 0) {
    const int g = (n + kWaves - 1) / kWaves;
    k_tsmooth_wave<FILL><<<g, kWaves * kWave, 0, s>>>(n, rp, ci, val, agg, o);
  }
}

void launch_tsmooth_count(int n, const int* rp, const int* ci, const int* agg, int* cnt, int* flags, int shift,
                          hipStream_t s) {
  TOut o{};
  o.cnt = cnt;
  o.flags = flags;
  o.shift = shift;
  launch_tsmooth<false>(n, rp, ci, nullptr, agg, o, s);
}

void launch_tsmooth_fill(const Level& lv, hipStream_t s) {
  const TOut o{lv.wdinv, lv.pval, lv.tp, lv.tc, lv.tc16, lv.tbase, lv.tv, lv.tv32, nullptr, nullptr, 0};
  launch_tsmooth<true>(lv.n, lv.rp, lv.ci, lv.val, lv.agg, o, s);
}

}  // namespace amg
