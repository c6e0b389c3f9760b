// Galerkin product by aggregate index (Section 3.1, eq. galerkin):
//   (A_{k+1})_IJ = sum_{i in G_I} sum_{j in G_J} P_iI A_ij P_jJ.
// Instead of a global sort of all (I, J) tuples, each coarse row I is built
// from its own aggregate segment G_I, in four steps:
//   1. term offsets: the entries of the fine rows, taken in segment order
//      (aggregate by aggregate, members ascending, entries in column order),
//      are numbered by a scan of the row lengths;
//   2. the terms: every entry (i, j) of a member row is the term
//      (J = agg(j), (P_iI a_ij) P_jJ) with its number in segment order; a wave
//      per coarse row stages its row's terms in LDS;
//   3. reduce: the wave takes the distinct J in ascending order (its smallest J
//      above the last one, from registers), then a lane per J sums that J's
//      terms in segment order; the (J, sum) pairs go to the head of the row's
//      term range;
//   4. a scan of the distinct counts makes the row pointers and a copy
//      compacts the rows.
// Each coarse entry is the sum of its terms in segment order, so the result
// does not depend on timing.  Rows with more terms than the first pass holds go
// to a wider one, and the rare rows beyond that to a block-per-row extraction.
#include <climits>

#include "amg_internal.hpp"
#include "device_utils.hpp"

namespace amg {

namespace {
constexpr int kBig = 256;        // threads per block on the extraction path
constexpr int kGalWaves = 2;     // waves per block of the reduce passes
constexpr int kSmallC = 8;       // terms per lane of the first reduce pass (16 to 64 lanes a row, by the average)
constexpr int kWideC = 16;       // terms per lane of the second, a wave per row
constexpr int kMaxWaveTerms = kWave * kWideC;
constexpr int kBigBlocks = 1024;  // of the extraction path, rows dealt in turn: four on a CU, whose waits overlap

// Step 1: number of terms of the k-th fine row in segment order (0 beyond the
// rows that belong to an aggregate).
__global__ void k_gal_lens(int n, const int* __restrict__ rp, const int* __restrict__ agg_ptr, int nc,
                           const int* __restrict__ agg_rows, int* __restrict__ lens) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  int len = 0;
  if (k < agg_ptr[nc]) {
    const int i = agg_rows[k];
    len = rp[i + 1] - rp[i];
  }
  lens[k] = len;
}

// The fine side of a direct reduce: A's rows, the aggregates and P.
struct GalFine {
  const int* rp;
  const int* ci;
  const double* val;
  const int* agg;
  const double* pval;
  const int* agg_rows;
};

// Steps 2 and 3 for rows of at most G C terms, G lanes per row.  Rows with more
// are appended to out_list; LAST (the wide pass) writes their terms to their
// ranges for the extraction path.  Bound by instruction issue (taking the
// distinct J one by one, and a lane per J walking all terms), which is why
// short rows share a wave, and by the chain row pointers
// -> entries -> aggregates, which four steps of members share.  Level 0 of 160^3
// 663 -> 456 us, of 128^3 338 -> 242, of 64 2-D systems (5.7 M rows) 866 -> 481,
// against a wave per row with a hash table of its J, a rank and a scan.
template <int G, int C, bool LAST>
__global__ void __launch_bounds__(kGalWaves * kWave) k_gal_rows(int nc, const int* __restrict__ agg_ptr,
                                                                const int* __restrict__ toff, int* __restrict__ tkey,
                                                                double* __restrict__ tval, int* __restrict__ ucount,
                                                                const int* __restrict__ in_list,
                                                                const int* __restrict__ in_count,
                                                                int* __restrict__ out_list,
                                                                int* __restrict__ out_count, GalFine fine) {
  constexpr int CAP = G * C, R = kWave / G * kGalWaves;   // terms and rows held
  constexpr int P = CAP + 1;                               // rows start in different LDS banks
  __shared__ int s_key[R][P];
  __shared__ double s_v[R][P];
  __shared__ int s_u[R][P];
  const int lane = threadIdx.x & (G - 1), grp = threadIdx.x / G;
  const int part = lane >> 3, l8 = lane & 7;
  int* key = s_key[grp];
  double* val = s_v[grp];
  int* uniq = s_u[grp];
  auto wave_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int count = LAST ? *in_count : nc;
  const long first = (long)xcd_block_index() * R;
  for (long base = first; base < count; base += (long)gridDim.x * R) {   // the same for the whole wave
    const bool mine_on = base + grp < count;
    const int I = !mine_on ? 0 : LAST ? in_list[base + grp] : (int)(base + grp);
    const int m0 = mine_on ? agg_ptr[I] : 0, m1 = mine_on ? agg_ptr[I + 1] : 0;
    const int t0 = mine_on ? toff[m0] : 0;
    int T = mine_on ? toff[m1] - t0 : 0;
    const bool fits = T <= CAP;
    if (!fits && lane == 0) out_list[atomicAdd(out_count, 1)] = I;
    if (fits || LAST) {
      // G / 8 members at a time, eight lanes each
      for (int mb = m0; mb < m1; mb += G) {
        const int q = mb + lane;
        int beg = 0, len = 0, off = 0;
        double pi = 0.0;
        if (q < m1) {
          const int i = fine.agg_rows[q];
          beg = fine.rp[i];
          len = fine.rp[i + 1] - beg;
          off = toff[q] - t0;
          pi = fine.pval[i];
        }
        const int cnt = min(G, m1 - mb);
        // four steps' first entries are loaded before any is used
        for (int sub = 0; sub < cnt; sub += G / 2) {
          int b[4], n[4], o[4], j[4];
          double p[4], a[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int src = min(sub + x * (G / 8) + part, G - 1);
            const bool in = sub + x * (G / 8) + part < cnt;   // past cnt: a lane with no entries
            b[x] = __shfl(beg, src, G);
            n[x] = __shfl(len, src, G);
            n[x] = in ? n[x] : 0;
            o[x] = __shfl(off, src, G);
            p[x] = __shfl(pi, src, G);
          }
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            j[x] = l8 < n[x] ? fine.ci[b[x] + l8] : -1;
            a[x] = l8 < n[x] ? fine.val[b[x] + l8] : 0.0;
          }
          int J[4];
          double pj[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            J[x] = j[x] >= 0 ? fine.agg[j[x]] : 0;
            pj[x] = j[x] >= 0 ? fine.pval[j[x]] : 0.0;
          }
          auto put = [&](int at, int Jt, double v) {
            if (fits) {
              key[at] = Jt;
              val[at] = v;
            } else {
              tkey[t0 + at] = Jt;
              tval[t0 + at] = v;
            }
          };
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            if (j[x] >= 0) put(o[x] + l8, J[x], __dmul_rn(__dmul_rn(p[x], a[x]), pj[x]));
            for (int k = l8 + 8; k < n[x]; k += 8) {
              const int jk = fine.ci[b[x] + k];
              put(o[x] + k, fine.agg[jk], __dmul_rn(__dmul_rn(p[x], fine.val[b[x] + k]), fine.pval[jk]));
            }
          }
        }
      }
    }
    const bool done = mine_on && fits;
    if (!fits) T = 0;
    wave_order();
    int J[C];
#pragma unroll
    for (int c = 0; c < C; ++c) J[c] = c * G + lane < T ? key[c * G + lane] : INT_MAX;
    int U = 0;
    for (int last = -1;;) {
      int mn = INT_MAX;
#pragma unroll
      for (int c = 0; c < C; ++c) mn = J[c] > last && J[c] < mn ? J[c] : mn;
      mn = group_min_int<G>(mn);
      if (!__any(mn != INT_MAX)) break;
      if (mn != INT_MAX) {
        last = mn;
        if (lane == 0) uniq[U] = mn;
        ++U;
      }
    }
    wave_order();
    for (int u = lane; u < U; u += G) {
      const int mine = uniq[u];
      double s = 0.0;
#pragma unroll 8
      for (int t = 0; t < T; ++t) {
        const double v = val[t];
        s = key[t] == mine ? __dadd_rn(s, v) : s;
      }
      tkey[t0 + u] = mine;
      tval[t0 + u] = s;
    }
    if (done && lane == 0) ucount[I] = U;
    wave_order();
  }
}

__device__ __forceinline__ int block_min_int(int v, int* red) {
  for (int off = kWave / 2; off > 0; off >>= 1) {
    int o = __shfl_xor(v, off, kWave);
    v = o < v ? o : v;
  }
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  int r = red[0];
  for (int w = 1; w < kBig / kWave; ++w) r = red[w] < r ? red[w] : r;
  __syncthreads();
  return r;
}

// Rows beyond the widest wave: repeatedly take the smallest J above the last
// one over the row's terms, then sum its terms (fixed thread assignment and
// reduction order).  The count pass runs before the row pointers exist, the
// fill pass writes the final row directly.
template <bool FILL>
__global__ void __launch_bounds__(kBig) k_gal_big(const int* __restrict__ agg_ptr, const int* __restrict__ toff,
                                                  const int* __restrict__ tkey, const double* __restrict__ tval,
                                                  int* __restrict__ ucount, const int* __restrict__ ovf_list,
                                                  const int* __restrict__ ovf_count, const int* __restrict__ rp_c,
                                                  int* __restrict__ ci_c, double* __restrict__ val_c) {
  __shared__ int ired[kBig / kWave];
  __shared__ double dred[kBig / kWave];
  const int count = *ovf_count;
  for (int idx = blockIdx.x; idx < count; idx += gridDim.x) {
    const int I = ovf_list[idx];
    const int t0 = toff[agg_ptr[I]], t1 = toff[agg_ptr[I + 1]];
    const int out0 = FILL ? rp_c[I] : 0;
    int last = -1, U = 0;
    while (true) {
      int mn = INT_MAX;
      for (int t = t0 + threadIdx.x; t < t1; t += kBig) {
        const int key = tkey[t];
        if (key > last && key < mn) mn = key;
      }
      mn = block_min_int(mn, ired);
      if (mn == INT_MAX) break;
      if (FILL) {
        double s = 0.0;
        for (int t = t0 + threadIdx.x; t < t1; t += kBig)
          if (tkey[t] == mn) s = __dadd_rn(s, tval[t]);
        double v[1] = {s};
        block_sum<1>(v, dred);
        if (threadIdx.x == 0) {
          ci_c[out0 + U] = mn;
          val_c[out0 + U] = v[0];
        }
      }
      ++U;
      last = mn;
    }
    if (!FILL && threadIdx.x == 0) ucount[I] = U;
    __syncthreads();
  }
}

// Step 4: rows reduced in place move to their final position (rows beyond
// the widest wave were written by the extraction path).
template <int G>
__global__ void __launch_bounds__(256) k_gal_compact(int nc, const int* __restrict__ agg_ptr,
                                                     const int* __restrict__ toff, const int* __restrict__ tkey,
                                                     const double* __restrict__ tval, const int* __restrict__ rp_c,
                                                     int* __restrict__ ci_c, double* __restrict__ val_c) {
  RowGroup<G> rg;
  for (long I0 = rg.gid; I0 < nc; I0 += rg.ngroups) {
    const int I = (int)I0;
    const int t0 = toff[agg_ptr[I]];
    if (toff[agg_ptr[I + 1]] - t0 > kMaxWaveTerms) continue;
    const int o = rp_c[I], U = rp_c[I + 1] - o;
    for (int u = rg.lane; u < U; u += G) {
      ci_c[o + u] = tkey[t0 + u];
      val_c[o + u] = tval[t0 + u];
    }
  }
}
}  // namespace

// Steps 1-3: on return ucount[I] holds the number of distinct J of every row.
void launch_galerkin_stage(const GalerkinScratch& g, int n, int nc, int nnz, const int* rp, const int* ci,
                           const double* val, const int* agg, const double* pval, const int* agg_ptr,
                           const int* agg_rows, ScanCtx& sc, hipStream_t s) {
  if (nc <= 0) return;
  k_gal_lens<<<(n + 255) / 256 > 0 ? (n + 255) / 256 : 1, 256, 0, s>>>(n, rp, agg_ptr, nc, agg_rows, g.lens);
  scan_to_ptr(g.lens, g.toff, n, sc, s);
  const GalFine fine{rp, ci, val, agg, pval, agg_rows};
  int* list1 = g.list;
  int* list2 = g.list + nc;
  launch_fill_int(2, g.ctl, 0, s);
  // the first pass holds half as many terms again as the average row
  const double avg = (double)nnz / nc;
  auto first = [&](auto lanes) {
    constexpr int G = decltype(lanes)::value, R = kWave / G * kGalWaves;
    k_gal_rows<G, kSmallC, false><<<(nc + R - 1) / R, kGalWaves * kWave, 0, s>>>(
        nc, agg_ptr, g.toff, g.tkey, g.tval, g.ucount, nullptr, nullptr, list1, g.ctl, fine);
  };
  if (avg <= 85) first(std::integral_constant<int, 16>());
  else if (avg <= 170) first(std::integral_constant<int, 32>());
  else first(std::integral_constant<int, 64>());
  k_gal_rows<kWave, kWideC, true><<<std::min(1024, (nc + kGalWaves - 1) / kGalWaves), kGalWaves * kWave, 0, s>>>(
      nc, agg_ptr, g.toff, g.tkey, g.tval, g.ucount, list1, g.ctl, list2, g.ctl + 1, fine);
  k_gal_big<false><<<std::min(kBigBlocks, nc), kBig, 0, s>>>(agg_ptr, g.toff, g.tkey, g.tval, g.ucount, list2, g.ctl + 1, nullptr,
                                        nullptr, nullptr);
}

// Step 4 once the row pointers rp_c exist.
void launch_galerkin_finish(const GalerkinScratch& g, int nc, const int* agg_ptr, const int* rp_c, int* ci_c,
                            double* val_c, hipStream_t s) {
  if (nc <= 0) return;
  const int G = group_lanes(nc, (long)nc * 16);
  with_lanes(G, [&](auto gl) {
    k_gal_compact<decltype(gl)::value><<<group_grid(nc, G), 256, 0, s>>>(nc, agg_ptr, g.toff, g.tkey, g.tval, rp_c,
                                                                         ci_c, val_c);
  });
  k_gal_big<true><<<std::min(kBigBlocks, nc), kBig, 0, s>>>(agg_ptr, g.toff, g.tkey, g.tval, nullptr, g.list + nc, g.ctl + 1, rp_c,
                                       ci_c, val_c);
}

}  // namespace amg
