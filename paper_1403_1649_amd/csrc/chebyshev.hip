// The polynomial smoother of the cycle (Chebyshev, Section 5), a unit of its
// own: its kernels are loaded by the hierarchies that use it.
#include "level_ops.hpp"

namespace amg {

namespace {

// The three-term Chebyshev recurrence on M = D^-1 A over [a, b].  First step from
// an iterate x0: r = D^-1 (b - A x0), d = r / theta, x = x0 + d; each later
// step j: r -= D^-1 A d, d = c1_j d + c2_j r, x += d.  Device coefficients
// K[0] = 1 / theta, K[2j - 1] = c1_j, K[2j] = c2_j (j >= 1 counts the later
// steps); dv = 1 / a_ii.

// pre-smoothing from x0 = 0, first and second step in one pass: the gathered
// d_j = (dv_j b_j) / theta, and at row i the second step's update
template <typename T>
struct OpChebPre2 {
  static constexpr int NV = 0;
  Act a;
  const T* b;
  const T* dv;
  const double* K;
  T* r;
  T* dout;
  T* xo;
  __device__ bool active() const { return a.on(); }
  __device__ void idle() const {}
  __device__ T x(int j) const { return (T)K[0] * (dv[j] * b[j]); }
  __device__ void row(int i, T ad, double*) const {
    const T r0 = dv[i] * b[i];
    const T d0 = (T)K[0] * r0;
    const T rr = r0 - dv[i] * ad;
    const T dn = (T)K[1] * d0 + (T)K[2] * rr;
    r[i] = rr;
    dout[i] = dn;
    xo[i] = d0 + dn;
  }
  __device__ void finalize(const double*) const {}
};

// pre-smoothing of degree one from x0 = 0 with the residual: x = d, r = b - A x
template <typename T>
struct OpChebPre1Resid {
  static constexpr int NV = 0;
  Act a;
  const T* b;
  const T* dv;
  const double* K;
  T* xt;
  T* r;
  __device__ bool active() const { return a.on(); }
  __device__ void idle() const {}
  __device__ T x(int j) const { return (T)K[0] * (dv[j] * b[j]); }
  __device__ void row(int i, T ax, double*) const {
    xt[i] = (T)K[0] * (dv[i] * b[i]);
    r[i] = b[i] - ax;
  }
  __device__ void finalize(const double*) const {}
};

// a later step j (din gathered, dout written: two buffers)
template <typename T>
struct OpChebStep {
  static constexpr int NV = 0;
  Act a;
  const T* dv;
  const T* din;
  T* dout;
  T* r;
  T* xo;
  const double* K;
  int j;
  __device__ bool active() const { return a.on(); }
  __device__ void idle() const {}
  __device__ T x(int c) const { return din[c]; }
  __device__ void row(int i, T ad, double*) const {
    const T rr = r[i] - dv[i] * ad;
    const T dn = (T)K[2 * j - 1] * din[i] + (T)K[2 * j] * rr;
    r[i] = rr;
    dout[i] = dn;
    xo[i] += dn;
  }
  __device__ void finalize(const double*) const {}
};

// first post-smoothing step on the corrected iterate x0 = xt + P e
template <typename T, class Corr>
struct OpChebPost1 {
  static constexpr int NV = 0;
  Act a;
  const T* b;
  const T* xt;
  const T* dv;
  const double* K;
  T* r;
  T* dout;
  T* xo;
  Corr corr;
  static constexpr bool kSmall = Corr::kSmall;
  __device__ bool active() const { return a.on(); }
  __device__ void idle() const {}
  __device__ T x(int j) const { return corr.at(xt, j); }
  __device__ void row(int i, T ax, double*) const {
    const T rr = dv[i] * (b[i] - ax);
    const T d = (T)K[0] * rr;
    r[i] = rr;
    dout[i] = d;
    xo[i] = corr.at(xt, i) + d;
  }
  __device__ void finalize(const double*) const {}
};

// Chebyshev vectors of a level in the cycle precision: r, two d buffers
template <typename T>
struct ChebVecs {
  T* r;
  T* d0;
  T* d1;
};
template <typename T>
ChebVecs<T> cheb_vecs(const Level& lv) {
  return ChebVecs<T>{static_cast<T*>(lv.cr), static_cast<T*>(lv.cd0), static_cast<T*>(lv.cd1)};
}

}  // namespace

// Pre-smoothing by Chebyshev from x = 0 (degree m = cheb_degree); of degree one
// with the residual r_out = b - A x in the same pass (true).
template <typename T>
bool cheb_pre(Hierarchy& h, const Level& lv, int k, Act A, const T* b, T* xt, T* r_out) {
  const Level* lp = &lv;
  RedCtx rc = red(h);
  const T* dv = wdinv<T>(lv);
  const int m = h.opt.cheb_degree;
  const bool sel = k == 0 && h.opt.probe == AMG_PROBE_L0_PRESMOOTH;
  if (m == 1) {
    const OpChebPre1Resid<T> op{A, b, dv, lv.cheb, xt, r_out};
    probe_point(h, sel, [=](hipStream_t st) { launch_level<T>(*lp, op, rc, st); });
    return true;
  }
  ChebVecs<T> cv = cheb_vecs<T>(lv);
  {
    const OpChebPre2<T> op{A, b, dv, lv.cheb, cv.r, cv.d0, xt};
    probe_point(h, sel, [=](hipStream_t st) { launch_level<T>(*lp, op, rc, st); });
  }
  T* din = cv.d0;
  T* dout = cv.d1;
  for (int j = 2; j < m; ++j) {
    launch_level<T>(lv, OpChebStep<T>{A, dv, din, dout, cv.r, xt, lv.cheb, j}, rc, h.stream);
    std::swap(din, dout);
  }
  return false;
}

// Post-smoothing by Chebyshev on the corrected iterate, into xo.
template <typename T, class Corr>
void cheb_post(Hierarchy& h, const Level& lv, int k, Act A, const T* b, const T* xt, T* xo, Corr corr) {
  const Level* lp = &lv;
  RedCtx rc = red(h);
  const T* dv = wdinv<T>(lv);
  ChebVecs<T> cv = cheb_vecs<T>(lv);
  {
    const OpChebPost1<T, Corr> op{A, b, xt, dv, lv.cheb, cv.r, cv.d0, xo, corr};
    probe_point(h, k == 0 && h.opt.probe == AMG_PROBE_L0_POSTSMOOTH,
                [=](hipStream_t st) { launch_level<T>(*lp, op, rc, st); });
  }
  T* din = cv.d0;
  T* dout = cv.d1;
  for (int j = 1; j < h.opt.cheb_degree; ++j) {
    launch_level<T>(lv, OpChebStep<T>{A, dv, din, dout, cv.r, xo, lv.cheb, j}, rc, h.stream);
    std::swap(din, dout);
  }
}

template bool cheb_pre<float>(Hierarchy&, const Level&, int, Act, const float*, float*, float*);
template bool cheb_pre<double>(Hierarchy&, const Level&, int, Act, const double*, double*, double*);
#define CHEB_POST(T, Corr) \
  template void cheb_post<T, Corr<T>>(Hierarchy&, const Level&, int, Act, const T*, const T*, T*, Corr<T>);
CHEB_POST(float, CorrV)
CHEB_POST(float, CorrNone)
CHEB_POST(float, CorrK)
CHEB_POST(double, CorrV)
CHEB_POST(double, CorrNone)
CHEB_POST(double, CorrK)
#undef CHEB_POST

}  // namespace amg
