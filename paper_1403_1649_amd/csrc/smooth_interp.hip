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

// S = P^T (I - A W), levels of at most kTsmoothRows rows: a wave per aggregate I.
// The entries of its rows (16 lanes a row) go to LDS, up to kSCap, as keys
// (column j, position) beside the products P_i a_ij; a hash table in LDS finds
// each column's first position, which sums the column's products in entry order
// and writes
//   s_Ij = (agg(j) = I ? P_j : 0) - w_j sum_i P_i a_ij.
// The pattern is T's transposed where A's is symmetric, but the values follow
// A itself, so a nonsymmetric operator keeps its cycle.  Bound by LDS round
// trips.  57,680 rows of 16 entries, count and fill: 23 and 60 us; comparing
// every pair of entries took 314 and 300 us, sorting the keys 75 and 91.
constexpr int kSBits = 10;
constexpr int kSCap = 1 << kSBits;
static_assert(kTsmoothRows <= 1 << 16, "column and position share a 32-bit key");
constexpr int kSMembers = 128;   // rows an aggregate may have
constexpr int kSWaves = 2;
template <bool FILL>
__global__ void __launch_bounds__(kSWaves * kWave) k_ssmooth(int nc, const int* __restrict__ agg_ptr,
                                                             const int* __restrict__ agg_rows,
                                                             const int* __restrict__ rp, const int* __restrict__ ci,
                                                             const double* __restrict__ val,
                                                             const double* __restrict__ pval,
                                                             const int* __restrict__ agg,
                                                             const double* __restrict__ wd, const int* __restrict__ sp,
                                                             int* __restrict__ sc, double* __restrict__ sv,
                                                             float* __restrict__ sv32, int* cnt, int* flags,
                                                             int shift) {
  constexpr unsigned kEmpty = ~0u;   // (column 2^22 - 1 at the last position: no key)
  __shared__ unsigned s_key[kSWaves][kSCap], s_tab[kSWaves][2 * kSCap];
  __shared__ unsigned short s_slot[kSWaves][kSCap];
  __shared__ int s_at[kSWaves][kSMembers + 1], s_beg[kSWaves][kSMembers];
  __shared__ double s_p[FILL ? kSWaves : 1][FILL ? kSMembers : 1];
  __shared__ double s_t[FILL ? kSWaves : 1][FILL ? kSCap : 1];
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int g = lane >> 4, l16 = lane & 15;
  for (long I = (long)blockIdx.x * kSWaves + wv; I < nc; I += (long)gridDim.x * kSWaves) {
    const int m0 = agg_ptr[I], members = agg_ptr[I + 1] - m0;
    // where each member's entries start, in LDS and in A
    int len = 0;
    for (int q0 = 0; q0 < min(members, kSMembers); q0 += kWave) {
      const int q = q0 + lane;
      int t = 0, b = 0;
      double pi = 0.0;
      if (q < members) {
        const int i = agg_rows[m0 + q];
        b = rp[i];
        t = rp[i + 1] - b;
        if constexpr (FILL) pi = pval[i];
      }
      int sum = t;   // inclusive scan
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(sum, d);
        if (lane >= d) sum += o;
      }
      s_at[wv][q] = len + sum - t;
      s_beg[wv][q] = b;
      if constexpr (FILL) s_p[wv][q] = pi;
      len += __builtin_amdgcn_readlane(sum, kWave - 1);
    }
    if (len > kSCap || members > kSMembers) {
      if constexpr (!FILL)
        if (lane == 0) {
          cnt[I] = 0;
          raise(flags, kSLongRow << shift);
        }
      continue;
    }
    if (lane == 0) s_at[wv][members] = len;
    wave_order();
#pragma unroll 2
    for (int q = g; q < members; q += 4) {
      const int at = s_at[wv][q], t = s_at[wv][q + 1] - at, b = s_beg[wv][q];
      for (int k = l16; k < t; k += 16) {
        s_key[wv][at + k] = (unsigned)ci[b + k] << kSBits | (unsigned)(at + k);
        if constexpr (FILL) s_t[wv][at + k] = s_p[wv][q] * val[b + k];
      }
    }
    wave_order();
    // each entry to its column's word, which keeps the least position
    int m = kWave;
    while (m < 2 * len) m <<= 1;
    for (int k = lane; k < m; k += kWave) s_tab[wv][k] = kEmpty;
    wave_order();
    for (int k = lane; k < len; k += kWave) {
      const unsigned key = s_key[wv][k];
      unsigned at = ((key >> kSBits) * 2654435761u) >> 16 & (unsigned)(m - 1);
      while (true) {   // ends: at most half the words are taken
        const unsigned old = atomicCAS(&s_tab[wv][at], kEmpty, key);
        if (old == kEmpty) break;
        if ((old ^ key) >> kSBits == 0) {
          atomicMin(&s_tab[wv][at], key);
          break;
        }
        at = (at + 1) & (unsigned)(m - 1);
      }
      s_slot[wv][k] = (unsigned short)at;
    }
    wave_order();
    if constexpr (FILL) {   // sums in place at the first position, a member's row (distinct columns) at a time
      for (int q = 0; q < members; ++q) {
        for (int k = s_at[wv][q] + lane; k < s_at[wv][q + 1]; k += kWave) {
          const int to = (int)(s_tab[wv][s_slot[wv][k]] & (kSCap - 1));
          if (to != k) s_t[wv][to] += s_t[wv][k];
        }
        wave_order();
      }
    }
    int u = 0, at = 0;
    if constexpr (FILL) at = sp[I];
    for (int k0 = 0; k0 < len; k0 += kWave) {
      const int k = k0 + lane;
      const unsigned key = k < len ? s_key[wv][k] : 0u;
      const bool first = k < len && s_tab[wv][s_slot[wv][k]] == key;
      const uint64_t bits = __ballot(first);
      if constexpr (FILL)
        if (first) {
          const int to = at + u + __popcll(bits & ((1ull << lane) - 1)), j = (int)(key >> kSBits);
          const double v = (agg[j] == I ? pval[j] : 0.0) - wd[j] * s_t[wv][k];
          sc[to] = j;
          if (sv) sv[to] = v;
          if (sv32) sv32[to] = (float)v;
        }
      u += __popcll(bits);
    }
    if constexpr (!FILL)
      if (lane == 0) cnt[I] = u;
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

void launch_ssmooth_count(const Level& lv, int* cnt, int* flags, int shift, hipStream_t s) {
  if (lv.nc < 1) return;
  k_ssmooth<false><<<(lv.nc + kSWaves - 1) / kSWaves, kSWaves * kWave, 0, s>>>(
      lv.nc, lv.agg_ptr, lv.agg_rows, lv.rp, lv.ci, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
      nullptr, cnt, flags, shift);
}

void launch_ssmooth_fill(const Level& lv, hipStream_t s) {
  if (lv.nc < 1) return;
  k_ssmooth<true><<<(lv.nc + kSWaves - 1) / kSWaves, kSWaves * kWave, 0, s>>>(
      lv.nc, lv.agg_ptr, lv.agg_rows, lv.rp, lv.ci, lv.val, lv.pval, lv.agg, lv.wdinv, lv.sp, lv.sc, lv.sv, lv.sv32,
      nullptr, nullptr, 0);
}

}  // namespace amg
