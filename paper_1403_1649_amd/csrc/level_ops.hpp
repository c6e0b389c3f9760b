// Row operations on a level's operator with its tuned kernel, for the units of
// the solve phase: the typed views of a level, the launch in the layout the
// tuner chose, and the coarse-grid corrections the post-smoothing reads.
#pragma once
#include <functional>
#include <type_traits>

#include "kernels_common.hpp"

namespace amg {

struct Act {
  const int* p;
  __device__ __forceinline__ bool on() const { return p == nullptr || *p != 0; }
};

// On small levels (at most kFuseCorrectionRows rows, where a launch costs more
// than the work) the coarse-grid correction is applied where the
// post-smoothing reads the iterate, x_j + P_j (correction of aggregate agg_j),
// so it needs no pass of its own; larger levels run the prolongation as its
// own pass, which is cheaper than three extra gathers per nonzero.  V-cycle: the
// correction is c; K-cycle: coef_c c (+ coef_d d when the second inner step was
// kept).
constexpr int kFuseCorrectionRows = 65536;

template <typename T>
struct CorrV {
  const int* agg;
  const T* pval;
  const T* c;
  static constexpr bool kSmall = true;
  __device__ T at(const T* xt, int j) const { return xt[j] + pval[j] * c[agg[j]]; }
};

template <typename T>
struct CorrNone {   // correction already applied by a prolongation pass
  static constexpr bool kSmall = false;
  __device__ T at(const T* xt, int j) const { return xt[j]; }
};

template <typename T>
struct CorrK {
  const int* agg;
  const T* pval;
  const T* c;
  const T* d;
  const double* K;
  const int* F;
  static constexpr bool kSmall = true;
  __device__ T at(const T* xt, int j) const {
    const int I = agg[j];
    T xc = (T)K[kKCoefC] * c[I];
    if (F[1]) xc += (T)K[kKCoefD] * d[I];
    return xt[j] + pval[j] * xc;
  }
};

template <typename T> const T* vals(const Level& l);
template <> inline const double* vals<double>(const Level& l) { return l.val; }
template <> inline const float* vals<float>(const Level& l) { return l.val32; }
template <typename T> const T* wdinv(const Level& l);
template <> inline const double* wdinv<double>(const Level& l) { return l.wdinv; }
template <> inline const float* wdinv<float>(const Level& l) { return l.wdinv32; }
template <typename T> const Level::Tune& tune_of(const Level& l);
template <> inline const Level::Tune& tune_of<double>(const Level& l) { return l.t64; }
template <> inline const Level::Tune& tune_of<float>(const Level& l) { return l.t32; }
template <typename T> const T* sell_vals(const Level& l);
template <> inline const double* sell_vals<double>(const Level& l) { return l.sl_val; }
template <> inline const float* sell_vals<float>(const Level& l) { return l.sl_val32; }
template <typename T> const T* short_vals(const Level& l);
template <> inline const double* short_vals<double>(const Level& l) { return l.sh.val; }
template <> inline const float* short_vals<float>(const Level& l) { return l.sh.val32; }
template <typename T> const T* dia_vals(const Level& l);
template <> inline const double* dia_vals<double>(const Level& l) { return l.dia.val; }
template <> inline const float* dia_vals<float>(const Level& l) { return l.dia.val32; }
template <typename T> const T* sym_vals(const Level& l);
template <> inline const double* sym_vals<double>(const Level& l) { return l.sym.val; }
template <> inline const float* sym_vals<float>(const Level& l) { return l.sym.val32; }

inline RedCtx red(Hierarchy& h) { return RedCtx{h.d_part, h.d_ticket}; }

// An operation on the corrected iterate of a small level (CorrV, CorrK) exists
// for CSR alone: such levels are not tuned to another layout, and every kernel
// instance counts when the library is loaded (about 45 us each).
template <class Op, class = void>
struct SmallLevelOp : std::false_type {};
template <class Op>
struct SmallLevelOp<Op, std::enable_if_t<Op::kSmall>> : std::true_type {};

// A row operation on A_k with the level's tuned kernel: CSR by lanes or streamed
// (lpr 1), sliced ELL in 64-row slices or in the level's shorter slices, sliced or
// symmetric diagonals.
template <typename T, class Op>
void launch_level(const Level& lv, const Op& op, RedCtx rc, hipStream_t s) {
  const Level::Tune& t = tune_of<T>(lv);
  if constexpr (SmallLevelOp<Op>::value) {
    launch_rows<T>(lv.n, t.lpr, lv.rp, lv.ci, vals<T>(lv), op, rc, s);
  } else {
    if (t.fmt == 4 && lv.ci16)
      launch_rows16<T>(lv.n, t.lpr, lv.rp, lv.ci16, vals<T>(lv), op, rc, s);
    else if (t.fmt == 5 && sym_vals<T>(lv))
      launch_sym_dia<T>(lv.n, lv.sym, sym_vals<T>(lv), op, rc, s, t.pz);
    else if (t.fmt == 3 && dia_vals<T>(lv))
      launch_sdia<T>(lv.n, lv.dia.nslices, lv.dia.ptr, lv.dia.off, dia_vals<T>(lv), op, rc, s, t.pz);
    else if (t.fmt >= 1 && t.sh > 0 && t.sh == lv.sh.h && short_vals<T>(lv))
      launch_sell<T>(lv.n, lv.sh.nslices, lv.sh.ptr, lv.sh.col, short_vals<T>(lv), op, rc, s,
                     t.fmt == 2 ? lv.sh.dcol : nullptr, 0, lv.sh.h, lv.sh.perm);
    else if (t.fmt >= 1 && lv.sl_ptr)
      launch_sell<T>(lv.n, lv.nslices, lv.sl_ptr, lv.sl_col, sell_vals<T>(lv), op, rc, s,
                     t.fmt == 2 ? lv.sl_dcol : nullptr, t.pz);
    else if (t.lpr == 1)
      launch_stream<T>(lv.n, lv.nnz, lv.rp, lv.ci, vals<T>(lv), op, rc, s);
    else
      launch_rows<T>(lv.n, t.lpr, lv.rp, lv.ci, vals<T>(lv), op, rc, s);
  }
}

// solver.hip: the probed kernel
void probe_point(Hierarchy& h, bool selected, std::function<void(hipStream_t)> fn);

// chebyshev.hip: the polynomial smoother of level k.  Pre-smoothing from x = 0
// into xt; true: the residual b - A xt is in r as well.  Post-smoothing of the
// corrected iterate into xo.
template <typename T>
bool cheb_pre(Hierarchy& h, const Level& lv, int k, Act A, const T* b, T* xt, T* r);
template <typename T, class Corr>
void cheb_post(Hierarchy& h, const Level& lv, int k, Act A, const T* b, const T* xt, T* xo, Corr corr);

}  // namespace amg
