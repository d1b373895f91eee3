// Device helpers shared by every kernel translation unit of libewald (gfx950):
// complex arithmetic, phases in turns, minimum-image geometry, the pair
// potential, wave reductions, phase tables and the rho rebuild, plus the
// host-side launch helpers.  Internal; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <type_traits>

#include "ewald_internal.h"

namespace ewald {


template <typename R>
struct cplx {
  R x, y;
};

// Complex product with the FMAs written out, so that every kernel and launch
// shape rounds it the same way (left to itself the compiler may contract
// either product of each component).
template <typename R>
__device__ __forceinline__ cplx<R> cmul(cplx<R> a, cplx<R> b) {
  return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}

__device__ __forceinline__ int unpack_n(uint32_t p, int d) {
  return int(int8_t((p >> (8 * d)) & 0xffu));
}

__device__ __forceinline__ double wrap01(double x) {
  double f = x - floor(x);
  return f >= 1.0 ? 0.0 : f;
}

// Cartesian row vector -> wrapped fractional coordinates.
template <int DIM>
__device__ __forceinline__ double to_frac1(const double* r, const double* Ainv, int d) {
  double v = 0.0;
#pragma unroll
  for (int e = 0; e < DIM; ++e) v = fma(r[e], Ainv[e * 3 + d], v);
  return wrap01(v);
}

template <int DIM>
__device__ __forceinline__ void to_frac(const double* r, const double* Ainv, double* s) {
#pragma unroll
  for (int d = 0; d < DIM; ++d) s[d] = to_frac1<DIM>(r, Ainv, d);
}

// exp(2 pi i x) in turns: reduce x to the nearest quarter turn q and a
// remainder of at most half a quarter turn (exact in FP64), evaluate the
// Taylor series of cos and sin at theta = remainder * pi/2 (|theta| <= pi/4;
// the first omitted terms are below 1e-19), and rotate by i^q.  Small and
// register-light, unlike a general sincos.  Both precision forms build their
// phase tables from it in FP64 (the mixed form rounds the entries to FP32).
__device__ __forceinline__ void quarter_turns(double x, double& r, int& q) {
  x -= rint(x);
  const double y = 4.0 * x;
  const double qd = rint(y);
  r = y - qd;
  q = int(qd) & 3;
}

template <typename R>
__device__ __forceinline__ cplx<R> rotate_quarter(R c, R s, int q) {
  const R x = (q & 1) ? -s : c, y = (q & 1) ? c : s;
  return (q & 2) ? cplx<R>{-x, -y} : cplx<R>{x, y};
}

// A constant put into scalar registers where it is used (the asm takes x, the
// argument at hand, so that it is not moved out of loops).  Left to itself the
// compiler keeps the series' 17 constants in vector registers across the
// kernels' main loops: at 128 registers per lane 40 to 100 more were spilled
// (the derivative sweep with the u term at N = 1024 took 4.9 ms instead of 3.7),
// and one spill was placed at a loop's exit where no lane is active, so that
// later phases were built from a stale constant.
__device__ __forceinline__ double scalar_k(double c, double x) {
  asm("" : "+s"(c) : "v"(x));
  return c;
}

// SK: the fused kernel, which has no vector registers to spare; the others
// keep the constants as they come (a step's tables at 512 electrons take 0.2 of its
// 13 us longer with the moves to scalar registers).
template <bool SK>
__device__ __forceinline__ double series_k(double c, double x) {
  return SK ? scalar_k(c, x) : c;
}

template <bool SK>
__device__ __forceinline__ cplx<double> turn(double x) {
  double r;
  int q;
  quarter_turns(x, r, q);
  const double th = r * 1.5707963267948966, t2 = th * th;
  double sp = series_k<SK>(2.8114572543455206e-15, th);
  sp = fma(sp, t2, series_k<SK>(-7.6471637318198165e-13, th));
  sp = fma(sp, t2, series_k<SK>(1.6059043836821613e-10, th));
  sp = fma(sp, t2, series_k<SK>(-2.5052108385441720e-08, th));
  sp = fma(sp, t2, series_k<SK>(2.7557319223985893e-06, th));
  sp = fma(sp, t2, series_k<SK>(-1.9841269841269841e-04, th));
  sp = fma(sp, t2, series_k<SK>(8.3333333333333333e-03, th));
  sp = fma(sp, t2, series_k<SK>(-1.6666666666666667e-01, th));
  sp = fma(sp, t2 * th, th);
  double cp = series_k<SK>(-1.5619206968586225e-16, th);
  cp = fma(cp, t2, series_k<SK>(4.7794773323873853e-14, th));
  cp = fma(cp, t2, series_k<SK>(-1.1470745597729725e-11, th));
  cp = fma(cp, t2, series_k<SK>(2.0876756987868099e-09, th));
  cp = fma(cp, t2, series_k<SK>(-2.7557319223985891e-07, th));
  cp = fma(cp, t2, series_k<SK>(2.4801587301587302e-05, th));
  cp = fma(cp, t2, series_k<SK>(-1.3888888888888889e-03, th));
  cp = fma(cp, t2, series_k<SK>(4.1666666666666667e-02, th));
  cp = fma(cp, t2, -0.5);
  cp = fma(cp, t2, 1.0);
  return rotate_quarter<double>(cp, sp, q);
}

// Squared minimum-image distance between fractional positions a and b:
// reduce the fractional difference to [-1/2, 1/2], go Cartesian in the frame
// where the lattice rows are lower-triangular (Lrot; distances are frame
// independent), then compare with the candidate images r0 +- v_c
// (|r0 +- v|^2 = |r0|^2 + |v|^2 -+ 2 r0.v).
template <int DIM>
__device__ __forceinline__ double min_r2(const double* a, const double* b, const DevSys* __restrict__ S,
                                         int n_cand) {
  double f[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    f[d] = a[d] - b[d];
    f[d] -= rint(f[d]);
  }
  const double* L = S->Lrot;
  double r[DIM];
  if constexpr (DIM == 3) {
    r[0] = fma(f[2], L[6], fma(f[1], L[3], f[0] * L[0]));
    r[1] = fma(f[2], L[7], f[1] * L[4]);
    r[DIM - 1] = f[DIM - 1] * L[8];
  } else {
    r[0] = fma(f[1], L[3], f[0] * L[0]);
    r[DIM - 1] = f[DIM - 1] * L[4];
  }
  double r0sq = 0.0;
#pragma unroll
  for (int e = 0; e < DIM; ++e) r0sq = fma(r[e], r[e], r0sq);
  double r2 = r0sq;
  for (int c = 0; c < n_cand; ++c) {
    double dot = 0.0;
#pragma unroll
    for (int e = 0; e < DIM; ++e) dot = fma(r[e], S->cand[c][e], dot);
    r2 = fmin(r2, fma(-2.0, fabs(dot), r0sq + S->cand[c][3]));
  }
  return r2;
}

// Squared minimum-image distance in the orthogonal-sublattice frame: wrap
// each axis into the box (|x_d| <= box_d / 2); the nearest image in the coset
// offset by half box sides along the axes of its mask is at
// sum_mask (box_d/2 - |x_d|)^2 + sum_other x_d^2 = |x|^2 + cc - sum_d cw_d |x_d|
// (cw_d = box_d on the mask, else 0; cc = +inf when the frame has no coset,
// so the expression needs no branch).
// The constants a pair distance and a pair term need, by value: for kernels
// with vector registers to spare they are loaded once into vector registers
// (frame_k_vector), elsewhere read from the system tables (frame_k).
struct FrameK {
  double box[3], ibox[3], cw[3], cc;
  double rc2, alpha, scale;  // r_cut^2, alpha, 2 / r_cut^2 (pair potential)
};

__device__ __forceinline__ FrameK frame_k(const DevSys* __restrict__ S) {
  FrameK K;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    K.box[d] = S->box[d];
    K.ibox[d] = S->ibox[d];
    K.cw[d] = S->cw[0][d];
  }
  K.cc = S->cc[0];
  K.rc2 = S->rc2;
  K.alpha = S->alpha;
  K.scale = S->poly_scale;
  return K;
}

// Loaded with a lane-varying index, so that the compiler keeps them in vector
// registers rather than in the scarcer scalar ones.
__device__ __forceinline__ FrameK frame_k_vector(const DevSys* __restrict__ S) {
  int z = 0;
  asm volatile("" : "+v"(z));
  FrameK K;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    K.box[d] = S->box[d + z];
    K.ibox[d] = S->ibox[d + z];
    K.cw[d] = S->cw[0][d + z];
  }
  K.cc = S->cc[z];
  K.rc2 = (&S->rc2)[z];
  K.alpha = (&S->alpha)[z];
  K.scale = (&S->poly_scale)[z];
  return K;
}

template <int DIM>
__device__ __forceinline__ double min_r2_ortho(const double* a, const double* b, const FrameK& K) {
  double x[DIM], r0sq = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    x[d] = a[d] - b[d];
    x[d] = fma(-K.box[d], rint(x[d] * K.ibox[d]), x[d]);
    r0sq = fma(x[d], x[d], r0sq);
  }
  double t = r0sq + K.cc;
#pragma unroll
  for (int d = 0; d < DIM; ++d) t = fma(-K.cw[d], fabs(x[d]), t);
  return fmin(r0sq, t);
}

// A reference to one of two arrays chosen at compile time.
template <bool B, typename A, typename C>
__device__ __forceinline__ auto& pick_ref(A& a, C& c) {
  if constexpr (B)
    return c;
  else
    return a;
}

// Coordinates of a fractional position in the orthogonal-sublattice frame.
template <int DIM>
__device__ __forceinline__ void frame_coords(const double* s, const DevSys* __restrict__ S, double* x) {
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < DIM; ++i) v = fma(s[i], S->F[i * 3 + d], v);
    x[d] = v;
  }
}

// Minimum-image r^2 between two positions given in the kernel's geometry:
// frame coordinates (ORTHO) or fractional coordinates (general cells).
template <int DIM, bool ORTHO>
__device__ __forceinline__ double image_r2(const double* a, const double* b, const DevSys* __restrict__ S,
                                           int n_cand, const FrameK& K) {
  if (ORTHO) return min_r2_ortho<DIM>(a, b, K);
  return min_r2<DIM>(a, b, S, n_cand);
}

// A stored (fractional) position in the kernel's geometry.
template <int DIM, bool ORTHO>
__device__ __forceinline__ void geo_pos(const double* s, const DevSys* __restrict__ S, double* x) {
  if (ORTHO) {
    frame_coords<DIM>(s, S, x);
  } else {
#pragma unroll
    for (int d = 0; d < DIM; ++d) x[d] = s[d];
  }
}

// A value every lane holds alike (read from LDS at a uniform address), made
// visibly uniform for the compiler: scalar registers, and branches on it
// stay branches (not per-lane selects).
__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform_d(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ float uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform_r(double v) { return uniform_d(v); }
__device__ __forceinline__ float uniform_r(float v) { return uniform_f(v); }

// Kahan-compensated FP32 accumulator.
struct Kahan {
  float s = 0.f, c = 0.f;
  __device__ __forceinline__ void add(float v) {
    float y = v - c;
    float t = s + y;
    c = (t - s) - y;
    s = t;
  }
  __device__ __forceinline__ double value() const { return double(s) - double(c); }
};

// Pair potential phi(r) = erfc(alpha r)/r = 1/r - alpha g(alpha^2 r^2) for
// r^2 < rc2, where g(y) = erf(sqrt y)/sqrt y is entire.  On [0, r_cut] g is
// one polynomial in t = 2 r^2 / r_cut^2 - 1 (degree PD, fitted in FP64 by the
// set-up), so a pair costs one reciprocal square root and PD FMAs.
// FP64 form: everything in FP64.  Mixed form: 1/r in FP64 (it carries the
// close-pair singularity) and the bounded erf part in FP32 (degree 12 or 22)
// summed with Kahan compensation.
// FLUSH (mixed form): the compensated sum is moved to FP64 after every two
// terms (a particle's new and old distance), so that the sum does not depend
// on how many particles a thread holds.
template <bool MIXED, int PD, bool FLUSH = false>
struct PairAcc;

// 1/sqrt(x) for x in (0, r_cut^2]: the hardware estimate refined by one
// Newton step carried to second order, y (1 + e/2 + 3e^2/8) with
// e = 1 - x y^2 (remaining relative error ~5e^3/16).  Unlike the library
// rsqrt it has no zero/infinity/denormal handling, which the pair terms never
// need (coincident particles are documented as giving non-finite results).
__device__ __forceinline__ double rsqrt_pos(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Pair terms are evaluated several at a time (NE = 2 or 4): the four Horner chains interleave
// (latency hiding) and take their coefficients straight from scalar registers.
// A term enters iff r2 < r_cut^2; callers pad with r2 = r_cut^2 and q = 0.
template <int PD, bool FLUSH>
struct PairAcc<false, PD, FLUSH> {
  double s = 0.0;
  const double* __restrict__ c;  // the polynomial coefficients (system tables, or registers)
  const FrameK& K;
  __device__ __forceinline__ PairAcc(const double* c64, const float*, const FrameK& k) : c(c64), K(k) {}
  template <int NE>
  __device__ __forceinline__ void add(const double (&q)[NE], const double (&r2)[NE]) {
    double ir[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) ir[e] = rsqrt_pos(r2[e]);
    add_ir<NE>(q, r2, ir);
  }
  // the same with 1/sqrt(r2) already formed (shared with the Jastrow u term)
  template <int NE>
  __device__ __forceinline__ void add_ir(const double (&q)[NE], const double (&r2)[NE], const double (&ir)[NE]) {
    double t[NE], p[NE];
    const double scale = K.scale;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      t[e] = fma(r2[e], scale, -1.0);
      p[e] = c[PD];
    }
#pragma unroll
    for (int i = PD - 1; i >= 0; --i) {
      const double ci = c[i];
#pragma unroll
      for (int e = 0; e < NE; ++e) p[e] = fma(p[e], t[e], ci);
    }
    const double rc2 = K.rc2, alpha = K.alpha;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const double phi = fma(-alpha, p[e], ir[e]);
      s = fma(r2[e] < rc2 ? q[e] : 0.0, phi, s);
    }
  }
  __device__ __forceinline__ double value() const { return s; }
};

template <int PD, bool FLUSH>
struct PairAcc<true, PD, FLUSH> {
  static constexpr int PF = PD == 16 ? 12 : 22;
  double inv = 0.0;
  Kahan erfpart;
  const float* __restrict__ c;  // the FP32 polynomial coefficients (system tables, or registers)
  const FrameK& K;
  __device__ __forceinline__ PairAcc(const double*, const float* c32, const FrameK& k) : c(c32), K(k) {}
  template <int NE>
  __device__ __forceinline__ void add(const double (&q)[NE], const double (&r2)[NE]) {
    double ir[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) ir[e] = rsqrt_pos(r2[e]);
    add_ir<NE>(q, r2, ir);
  }
  template <int NE>
  __device__ __forceinline__ void add_ir(const double (&q)[NE], const double (&r2)[NE], const double (&ir)[NE]) {
    float t[NE], p[NE];
    const float scale = float(K.scale);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      t[e] = fmaf(float(r2[e]), scale, -1.0f);
      p[e] = c[PF];
    }
#pragma unroll
    for (int i = PF - 1; i >= 0; --i) {
      const float ci = c[i];
#pragma unroll
      for (int e = 0; e < NE; ++e) p[e] = fmaf(p[e], t[e], ci);
    }
    const double rc2 = K.rc2;
    const float alpha = float(K.alpha);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const double qe = r2[e] < rc2 ? q[e] : 0.0;
      inv = fma(qe, ir[e], inv);
      erfpart.add(float(qe) * (alpha * p[e]));
      if (FLUSH && (e & 1)) {
        inv -= erfpart.value();
        erfpart = Kahan{};
      }
    }
  }
  __device__ __forceinline__ double value() const { return inv - erfpart.value(); }
};

// ---------------------------------------------------------------------------
// Jastrow two-body polynomial term u (Sec. 2.3, Eq. (8)), in powers of
// t = r / L_u with the coefficients of the pair's spin channel,
// c_m = u_c0[m] + s u_dc[m] (s = 0 for equal labels, 1 for unequal ones).
// FP64 in both precision forms.

// u at two arguments (a moved particle's new and old position against one
// partner), sharing the channel blend.
__device__ __forceinline__ void u_two(const DevSys* __restrict__ S, double s, double ta, double tb, double& ua,
                                      double& ub) {
  double pa = 0.0, pb = 0.0;
#pragma unroll
  for (int m = UDEG; m >= 0; --m) {
    const double c = fma(s, S->u_dc[m], S->u_c0[m]);
    pa = fma(pa, ta, c);
    pb = fma(pb, tb, c);
  }
  ua = pa;
  ub = pb;
}

// u and its first and second derivatives with respect to t at one argument,
// and u at a second one (Horner with derivative chains).
__device__ __forceinline__ void u_der_two(const DevSys* __restrict__ S, double s, double ta, double tb, double& ua,
                                          double& d1, double& d2, double& ub) {
  double p = 0.0, p1 = 0.0, p2 = 0.0, pb = 0.0;
#pragma unroll
  for (int m = UDEG; m >= 0; --m) {
    const double c = fma(s, S->u_dc[m], S->u_c0[m]);
    p2 = fma(p2, ta, p1);
    p1 = fma(p1, ta, p);
    p = fma(p, ta, c);
    pb = fma(pb, tb, c);
  }
  ua = p;
  d1 = p1;
  d2 = 2.0 * p2;
  ub = pb;
}

// u of one pair at r^2 with 1/r given (energy sums); 0 beyond L_u or when
// the pair does not take part.
__device__ __forceinline__ double u_pair(const DevSys* __restrict__ S, bool take, bool unequal, double r2,
                                         double ir) {
  double u, unused;
  u_two(S, unequal ? 1.0 : 0.0, r2 * ir * S->u_icut, 0.0, u, unused);
  return (take && r2 < S->u_cut2) ? u : 0.0;
}

// Change of U in a move against one partner (new minus old), and for UD the
// partner's share of grad_k U (in the geometry's frame axes: x is the
// minimum-image displacement of the new position from the partner) and of
// lap_k U at the new position.
template <int DIM>
struct UOut {
  double d = 0.0;
  double g[DIM] = {};
  double l = 0.0;
};

template <int DIM, bool UD>
__device__ __forceinline__ void u_move_term(const DevSys* __restrict__ S, bool ok, bool unequal, double r2n,
                                            double irn, double r2o, double iro, const double* xn, UOut<DIM>& out) {
  const double s = unequal ? 1.0 : 0.0, ic = S->u_icut, uc2 = S->u_cut2;
  const double tn = r2n * irn * ic, to = r2o * iro * ic;
  const bool inn = ok && r2n < uc2, ino = ok && r2o < uc2;
  double un, uo;
  if (UD) {
    double d1, d2;
    u_der_two(S, s, tn, to, un, d1, d2, uo);
    const double dur = inn ? d1 * ic * irn : 0.0;  // u'(r) / r
#pragma unroll
    for (int d = 0; d < DIM; ++d) out.g[d] = fma(dur, xn[d], out.g[d]);
    out.l += inn ? fma(d2, ic * ic, double(DIM - 1) * dur) : 0.0;
  } else {
    u_two(S, s, tn, to, un, uo);
  }
  out.d += (inn ? un : 0.0) - (ino ? uo : 0.0);
}

// A vector in a frame's axes (rows of E) in Cartesian axes.
template <int DIM>
__device__ __forceinline__ void frame_to_cart(const double* x, const double* E, double* out) {
#pragma unroll
  for (int e = 0; e < DIM; ++e) {
    double v = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) v = fma(x[d], E[d * 3 + e], v);
    out[e] = v;
  }
}

// Minimum-image displacement a - b (as min_r2, which gives the same r^2) in
// the lower-triangular frame's axes; returns r^2.
template <int DIM>
__device__ __forceinline__ double min_disp(const double* a, const double* b, const DevSys* __restrict__ S,
                                           int n_cand, double* x) {
  double f[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    f[d] = a[d] - b[d];
    f[d] -= rint(f[d]);
  }
  const double* L = S->Lrot;
  double r[DIM];
  if constexpr (DIM == 3) {
    r[0] = fma(f[2], L[6], fma(f[1], L[3], f[0] * L[0]));
    r[1] = fma(f[2], L[7], f[1] * L[4]);
    r[DIM - 1] = f[DIM - 1] * L[8];
  } else {
    r[0] = fma(f[1], L[3], f[0] * L[0]);
    r[DIM - 1] = f[DIM - 1] * L[4];
  }
  double r0sq = 0.0;
#pragma unroll
  for (int e = 0; e < DIM; ++e) r0sq = fma(r[e], r[e], r0sq);
  double r2 = r0sq;
#pragma unroll
  for (int e = 0; e < DIM; ++e) x[e] = r[e];
  for (int c = 0; c < n_cand; ++c) {
    double dot = 0.0;
#pragma unroll
    for (int e = 0; e < DIM; ++e) dot = fma(r[e], S->cand[c][e], dot);
    const double t = fma(-2.0, fabs(dot), r0sq + S->cand[c][3]);
    if (t < r2) {
      r2 = t;
      const double sg = dot >= 0.0 ? 1.0 : -1.0;
#pragma unroll
      for (int e = 0; e < DIM; ++e) x[e] = fma(-sg, S->cand[c][e], r[e]);
    }
  }
  return r2;
}

// The same in the orthogonal-sublattice frame (as min_r2_ortho): the coset
// image moves each masked axis by half a box side towards zero.
template <int DIM>
__device__ __forceinline__ double min_disp_ortho(const double* a, const double* b, const FrameK& K, double* x) {
  double r0sq = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    x[d] = a[d] - b[d];
    x[d] = fma(-K.box[d], rint(x[d] * K.ibox[d]), x[d]);
    r0sq = fma(x[d], x[d], r0sq);
  }
  double t = r0sq + K.cc;
#pragma unroll
  for (int d = 0; d < DIM; ++d) t = fma(-K.cw[d], fabs(x[d]), t);
  if (t < r0sq) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) x[d] -= copysign(0.5 * K.cw[d], x[d]);
    return t;
  }
  return r0sq;
}

template <int DIM, bool ORTHO>
__device__ __forceinline__ double image_disp(const double* a, const double* b, const DevSys* __restrict__ S,
                                             int n_cand, const FrameK& K, double* x) {
  if (ORTHO) return min_disp_ortho<DIM>(a, b, K, x);
  return min_disp<DIM>(a, b, S, n_cand, x);
}

// Real-space part of a move of particle k from so to sn, summed over the
// mobile particles j != k (positions pos, charges q) and the fixed ions:
// sum_j q_j [phi(sn - s_j) - phi(so - s_j)].  Threads take j = tid, tid + NT, ...
// PPR particles (2 PPR pair terms) per round: 2 for workgroups of up to 512
// threads, 1 for 1024 (one particle per thread at N = 1024).  Indices are
// clamped rather than branched on, so every load is in bounds and the loop
// body has no divergent control flow.  UJ: also the Jastrow u term of the
// mobile pairs into uo (UD: with its gradient, in the lower-triangular
// frame's axes, and Laplacian at the new position).
// A layered 2D system (S->n_layers = 2) adds (z_1 - z_0)^2 to r^2 for the
// partners in the other plane.  sub_k >= 0: particle sub_k is taken at
// sub_s instead of its stored position (a move accepted in the same launch).
template <int DIM, bool MIXED, int PD, int NT, bool UJ = false, bool UD = false>
__device__ __forceinline__ double real_move(const double* sn, const double* so, int k, const double* pos,
                                            const double* q, int n, const DevSys* __restrict__ S,
                                            UOut<DIM>* uo = nullptr, int sub_k = -1,
                                            const double* sub_s = nullptr) {
  constexpr int PPR = NT >= 1024 ? 1 : 2;
  const FrameK K = frame_k(S);
  PairAcc<MIXED, PD> pr(S->p64, S->p32, K);
  const int n_cand = S->n_cand;
  const double rc2 = S->rc2;
  const int sk = UJ ? S->spin[k] : 0;
  const bool lay = DIM == 2 && S->n_layers > 1;
  const int n0 = S->n0, lk = k >= n0 ? 1 : 0;
  const double dz2 = S->dz2;
  for (int j0 = threadIdx.x; j0 < n; j0 += PPR * NT) {
    double qq[2 * PPR], r2[2 * PPR], ir[2 * PPR];
    double xn[UD ? PPR : 1][DIM] = {};  // zero for masked partners (their weight is zero too)
    bool okc[PPR];
    int sj[PPR];
#pragma unroll
    for (int c = 0; c < PPR; ++c) {
      const int j = j0 + c * NT;
      const bool ok = j < n && j != k;
      const int jj = j < n ? j : n - 1;
      double pj[DIM];
#pragma unroll
      for (int d = 0; d < DIM; ++d) pj[d] = jj == sub_k ? sub_s[d] : pos[jj * DIM + d];
      const double qj = ok ? q[jj] : 0.0;
      if (UD)
        r2[2 * c] = ok ? min_disp<DIM>(sn, pj, S, n_cand, xn[UD ? c : 0]) : rc2;
      else
        r2[2 * c] = ok ? min_r2<DIM>(sn, pj, S, n_cand) : rc2;
      r2[2 * c + 1] = ok ? min_r2<DIM>(so, pj, S, n_cand) : rc2;
      if (lay && ok && (jj >= n0 ? 1 : 0) != lk) {
        r2[2 * c] += dz2;
        r2[2 * c + 1] += dz2;
      }
      qq[2 * c] = qj;
      qq[2 * c + 1] = -qj;
      okc[c] = ok;
      if (UJ) sj[c] = S->spin[jj];
    }
#pragma unroll
    for (int e = 0; e < 2 * PPR; ++e) ir[e] = rsqrt_pos(r2[e]);
    pr.template add_ir<2 * PPR>(qq, r2, ir);
    if (UJ)
#pragma unroll
      for (int c = 0; c < PPR; ++c)
        u_move_term<DIM, UD>(S, okc[c], sj[c] != sk, r2[2 * c], ir[2 * c], r2[2 * c + 1], ir[2 * c + 1],
                             xn[UD ? c : 0], *uo);
  }
  const int nfix = S->n_fixed;
  for (int j0 = threadIdx.x; j0 < nfix; j0 += PPR * NT) {
    double qq[2 * PPR], r2[2 * PPR];
#pragma unroll
    for (int c = 0; c < PPR; ++c) {
      const int j = j0 + c * NT;
      const bool ok = j < nfix;
      const int jj = ok ? j : nfix - 1;
      double sj[DIM];
#pragma unroll
      for (int d = 0; d < DIM; ++d) sj[d] = S->fixed_s[jj * DIM + d];
      const double qj = ok ? S->fixed_q[jj] : 0.0;
      r2[2 * c] = ok ? min_r2<DIM>(sn, sj, S, n_cand) : rc2;
      r2[2 * c + 1] = ok ? min_r2<DIM>(so, sj, S, n_cand) : rc2;
      if (lay && ok && S->fixed_layer[jj] != lk) {
        r2[2 * c] += dz2;
        r2[2 * c + 1] += dz2;
      }
      qq[2 * c] = qj;
      qq[2 * c + 1] = -qj;
    }
    pr.template add<2 * PPR>(qq, r2);
  }
  return pr.value();
}

// Real-space part of a move inside the fused sweep.  Thread t owns the
// particles j = t + c NT (c < PPR) and keeps their positions (in the
// kernel's geometry: frame or fractional coordinates, as sn and so) and
// charges in registers (ps, pq); it alone updates them when they move.  Particles beyond
// PPR NT (larger systems than the launch shape covers) are read from the LDS
// copy, again only by their owner t = j mod NT.  XTRA = false: the batch has
// no such particles and no fixed ions, and those loops are left out (at 1024
// threads their mere presence costs scalar-register reloads on every move).
// UJ: also the Jastrow u term of the mobile pairs into uo (psp: the spin
// labels of the thread's own particles, sk: the moved particle's); UD: with
// its gradient (in the geometry's frame axes) and Laplacian at the new
// position.
// LAY (a layered system when `lay`): partners in the other plane (mobile
// j >= n0 against k, or an ion's plane) are dz2 further apart in r^2.
template <int DIM, bool MIXED, int PD, int NT, int PPR, bool ORTHO, bool XTRA, bool UJ = false, bool UD = false,
          bool LAY = false, bool FLUSH = false>
__device__ __forceinline__ double real_move_own(const double* sn, const double* so, int k,
                                                const double (&ps)[PPR][DIM], const double (&pq)[PPR],
                                                const double* lpos, const double* lq, int n,
                                                const DevSys* __restrict__ S, const double* c64,
                                                const float* c32, const FrameK& K,
                                                const int* psp = nullptr, int sk = 0,
                                                UOut<DIM>* uo = nullptr, bool lay = false, int n0 = 0,
                                                double dz2 = 0.0) {
  PairAcc<MIXED, PD, FLUSH> pr(c64, c32, K);
  const int n_cand = S->n_cand;
  const double rc2 = S->rc2;
  const int lk = k >= n0 ? 1 : 0;
  // the own particles c < NC; a wave evaluates only the c for which some
  // lane holds a particle (the count is the same for every lane of the
  // wave), so small walkers in a large workgroup skip the empty ones
  auto own = [&](auto nc) {
    constexpr int NC = decltype(nc)::value;
    double qq[2 * NC], r2[2 * NC], ir[2 * NC];
    double xn[UD ? NC : 1][DIM] = {};  // zero for masked partners (their weight is zero too)
    bool okc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = threadIdx.x + c * NT;
      const bool ok = j < n && j != k;
      if (UD)
        r2[2 * c] = ok ? image_disp<DIM, ORTHO>(sn, ps[c], S, n_cand, K, xn[UD ? c : 0]) : rc2;
      else
        r2[2 * c] = ok ? image_r2<DIM, ORTHO>(sn, ps[c], S, n_cand, K) : rc2;
      r2[2 * c + 1] = ok ? image_r2<DIM, ORTHO>(so, ps[c], S, n_cand, K) : rc2;
      if (LAY && lay && ok && (j >= n0 ? 1 : 0) != lk) {
        r2[2 * c] += dz2;
        r2[2 * c + 1] += dz2;
      }
      qq[2 * c] = pq[c];
      qq[2 * c + 1] = -pq[c];
      okc[c] = ok;
    }
#pragma unroll
    for (int e = 0; e < 2 * NC; ++e) ir[e] = rsqrt_pos(r2[e]);
    pr.template add_ir<2 * NC>(qq, r2, ir);
    if (UJ)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        u_move_term<DIM, UD>(S, okc[c], psp[c] != sk, r2[2 * c], ir[2 * c], r2[2 * c + 1], ir[2 * c + 1],
                             xn[UD ? c : 0], *uo);
  };
  static_assert(PPR == 1 || PPR == 2, "own particles per thread: 1 or 2");
  {
    const int wbase = uniform_i(int(threadIdx.x) & ~63);  // the wave's first thread
    const int cw = n > wbase ? min(PPR, (n - wbase + NT - 1) / NT) : 0;
    if (cw >= PPR)
      own(std::integral_constant<int, PPR>{});
    else if (PPR > 1 && cw == 1)
      own(std::integral_constant<int, 1>{});
  }
  if (!XTRA) return pr.value();
  for (int j = threadIdx.x + PPR * NT; j < n; j += NT) {
    double qq[2], r2[2], ir[2];
    double xn[DIM] = {};
    const bool ok = j != k;
    double xj[DIM];
    geo_pos<DIM, ORTHO>(lpos + j * DIM, S, xj);
    if (UD)
      r2[0] = ok ? image_disp<DIM, ORTHO>(sn, xj, S, n_cand, K, xn) : rc2;
    else
      r2[0] = ok ? image_r2<DIM, ORTHO>(sn, xj, S, n_cand, K) : rc2;
    r2[1] = ok ? image_r2<DIM, ORTHO>(so, xj, S, n_cand, K) : rc2;
    if (LAY && lay && ok && (j >= n0 ? 1 : 0) != lk) {
      r2[0] += dz2;
      r2[1] += dz2;
    }
    qq[0] = lq[j];
    qq[1] = -lq[j];
    ir[0] = rsqrt_pos(r2[0]);
    ir[1] = rsqrt_pos(r2[1]);
    pr.template add_ir<2>(qq, r2, ir);
    if (UJ) u_move_term<DIM, UD>(S, ok, S->spin[j] != sk, r2[0], ir[0], r2[1], ir[1], xn, *uo);
  }
  const int nfix = S->n_fixed;
  for (int j0 = threadIdx.x; j0 < nfix; j0 += 2 * NT) {
    double qq[4], r2[4];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int j = j0 + c * NT;
      const bool ok = j < nfix;
      const int jj = ok ? j : nfix - 1;
      double sj[DIM];
      geo_pos<DIM, ORTHO>(S->fixed_s + jj * DIM, S, sj);
      const double qj = ok ? S->fixed_q[jj] : 0.0;
      r2[2 * c] = ok ? image_r2<DIM, ORTHO>(sn, sj, S, n_cand, K) : rc2;
      r2[2 * c + 1] = ok ? image_r2<DIM, ORTHO>(so, sj, S, n_cand, K) : rc2;
      if (LAY && lay && ok && S->fixed_layer[jj] != lk) {
        r2[2 * c] += dz2;
        r2[2 * c + 1] += dz2;
      }
      qq[2 * c] = qj;
      qq[2 * c + 1] = -qj;
    }
    pr.template add<4>(qq, r2);
  }
  return pr.value();
}

// A double moved between the lanes of a row of 16 by a DPP pattern in which every
// lane has a source (no previous value to preserve).
template <int CTRL>
__device__ __forceinline__ double dpp_all(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// Sums of N values over each row of 16 lanes, stored at p[0 .. N - 1] (p: the
// row's place).  Four values go through the row together: a lane hands its
// neighbour the values that it does not keep, so after two exchanges lane
// l of a row holds the sum of value l % 4 over its quad, and two rotations add
// the quads.  That is 75 issue cycles for four values (46 for two) against 37
// for each by itself.
template <int N>
__device__ __forceinline__ void row_sums(const double (&v)[N], int lane, double* p) {
  const bool odd = lane & 1, upper = lane & 2;
  auto pair = [&](double a, double b) { return (odd ? b : a) + dpp_all<0xB1>(odd ? a : b); };  // quad_perm [1,0,3,2]
  auto rest = [&](double x) {
    x += dpp_all<0x124>(x);  // row_ror 4
    x += dpp_all<0x128>(x);  // row_ror 8
    return x;
  };
  constexpr int N4 = N & ~3;
#pragma unroll
  for (int i = 0; i < N4; i += 4) {
    const double ab = pair(v[i], v[i + 1]), cd = pair(v[i + 2], v[i + 3]);
    const double x = rest((upper ? cd : ab) + dpp_all<0x4E>(upper ? ab : cd));  // quad_perm [2,3,0,1]
    if ((lane & 15) < 4) p[i + (lane & 3)] = x;
  }
  if constexpr (N - N4 >= 2) {
    double x = pair(v[N4], v[N4 + 1]);
    x = rest(x + dpp_all<0x4E>(x));
    if ((lane & 15) < 2) p[N4 + (lane & 1)] = x;
  }
  if constexpr ((N & 1) != 0) {
    double x = v[N - 1];
    x += dpp_all<0xB1>(x);
    x = rest(x + dpp_all<0x4E>(x));
    if ((lane & 15) == 0) p[N - 1] = x;
  }
}

// Sum NV values over a workgroup of NT threads; the result is valid in the
// first wave.  red must hold NV * NT / 16 doubles.  Rows of 16 lanes by DPP, then
// one lane per value over the rows: a butterfly of shuffles goes through LDS
// six times per value, one after the other.
template <int NV, int NT = BLOCK>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* red) {
  static_assert(NV <= 64, "one lane per value");
  const int lane = threadIdx.x & 63;
  row_sums<NV>(v, lane, red + (threadIdx.x >> 4) * NV);
  __syncthreads();
  if (threadIdx.x < 64) {
    double t = 0.0;
    if (lane < NV)
#pragma unroll
      for (int r = 0; r < NT / 16; ++r) t += red[r * NV + lane];
#pragma unroll
    for (int i = 0; i < NV; ++i)
      v[i] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(t), i),
                              __builtin_amdgcn_readlane(__double2loint(t), i));
  }
}

// Phase tables: per dimension d one row of tbl = 2 nm + 1 complex entries,
// exp(2 pi i n s_d) at [nm + n] for n = -nm..nm; a table of one position is
// DIM rows.
template <typename R>
__device__ __forceinline__ cplx<R> tab_at(const cplx<R>* tab, int row, int idx, int tbl) {
  return tab[row * tbl + idx];
}

// FP64 entries as one 16-byte read (every table base in LDS is 16-byte aligned).
__device__ __forceinline__ cplx<double> ld_entry(const cplx<double>* tab, int i) {
  const double2 v = reinterpret_cast<const double2*>(tab)[i];
  return {v.x, v.y};
}

template <>
__device__ __forceinline__ cplx<double> tab_at<double>(const cplx<double>* tab, int row, int idx, int tbl) {
  return ld_entry(tab, row * tbl + idx);
}

// FP32 entries as one 8-byte read.
template <>
__device__ __forceinline__ cplx<float> tab_at<float>(const cplx<float>* tab, int row, int idx, int tbl) {
  const float2 v = reinterpret_cast<const float2*>(tab)[row * tbl + idx];
  return {v.x, v.y};
}

// An entry at a byte offset into a 16-byte aligned LDS table, as one read.
template <typename R>
__device__ __forceinline__ cplx<R> ld_at_byte(const cplx<R>* tab, uint32_t byte_off) {
  using V = typename std::conditional<sizeof(R) == 8, double2, float2>::type;
  const V v = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(tab) + byte_off);
  return {v.x, v.y};
}

// One row, by one thread: powers of exp(2 pi i s) formed by repeated FP64
// multiplication (the paper's buffered powers, Sec. 5.2), with an exact
// restart every 8 powers so the rounding error stays below ~8 ulp; stored in R.
template <typename R, bool SK>
__device__ __forceinline__ void fill_row(cplx<R>* row, double s, int nm) {
  const cplx<double> u = turn<SK>(s);
  cplx<double> c = {1.0, 0.0};
  row[nm] = {R(1), R(0)};
  for (int m = 1; m <= nm; ++m) {
    c = (m & 7) == 0 ? turn<SK>(double(m) * s) : cmul(c, u);
    row[nm + m] = {R(c.x), R(c.y)};
    row[nm - m] = {R(c.x), R(-c.y)};
  }
}

// Coordinate r of (a, b) read as one array of 2 DIM values, with the index
// resolved by selects (a runtime index into register arrays would place
// them in scratch memory).
template <int DIM>
__device__ __forceinline__ double pick_coord(const double (&a)[DIM], const double (&b)[DIM], int r) {
  double v = 0.0;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    v = r == d ? a[d] : v;
    v = r == DIM + d ? b[d] : v;
  }
  return v;
}

// First phase of segment `pn` from the tables.
template <int DIM, typename R>
__device__ __forceinline__ cplx<R> anchor(const cplx<R>* tab, uint32_t pn, int nm) {
  const int tbl = 2 * nm + 1;
  cplx<R> e = cmul(tab_at(tab, 0, nm + unpack_n(pn, 0), tbl), tab_at(tab, 1, nm + unpack_n(pn, 1), tbl));
  if (DIM == 3) e = cmul(e, tab_at(tab, 2, nm + unpack_n(pn, 2), tbl));
  return e;
}

// Phases along a segment: e_0 = the anchor, e_1 = e_0 u, then the three-term
// recurrence e_{j+1} = 2 Re(u) e_j - e_{j-1} for u = exp(2 pi i s_last)
// (|u| = 1): two FMAs per slot instead of a complex multiply.  Rounding errors
// grow at most linearly along the segment (they propagate through Chebyshev
// polynomials of the second kind, |U_j(cos phi)| <= j + 1).
template <typename R>
struct SegWalk {
  cplx<R> cur, prev;
  R c2;
  cplx<R> u;
  __device__ __forceinline__ SegWalk(cplx<R> a, cplx<R> u_) : cur(a), prev(a), c2(R(2) * u_.x), u(u_) {}
  // u_ and c2_ = 2 Re u_ precomputed (e.g. wave-uniform, in scalar registers)
  __device__ __forceinline__ SegWalk(cplx<R> a, cplx<R> u_, R c2_) : cur(a), prev(a), c2(c2_), u(u_) {}
  __device__ __forceinline__ void step(int j) {  // e_j -> e_{j+1}; j is a compile-time index in unrolled loops
    if (j == 0) {
      prev = cur;
      cur = cmul(cur, u);
    } else {
      const cplx<R> nx = {fma(c2, cur.x, -prev.x), fma(c2, cur.y, -prev.y)};
      prev = cur;
      cur = nx;
    }
  }
};

// ---------------------------------------------------------------------------
// rho from the positions: rho(G) = rho_fix(G) + sum_p q_p exp(i G.r_p), FP64.
//
// The sum is a matrix product over the particles.  A column piece (n_1, n_2;
// 4 Q consecutive n_3 centred on the half-integer c) has
//   rho(c + x) = sum_p A_p exp(i x th_p),  A_p = q_p exp(i (n_1, n_2, c).th_p),
//   x = +-(h + 1/2), h = 0 .. 2Q - 1,
// and the four real sums of (Re A, Im A) times (cos, sin)((h + 1/2) th) give
// the two entries c +- (h + 1/2): two multiply-adds per entry and particle,
// where a walk along the column costs eight operations.  The sums run on the
// FP64 matrix instruction with four 4 x 4 x 4 blocks (rows: 16 column pieces;
// columns: cos and sin of two h; depth: four particles): its 16 cycles for 256
// multiply-adds are what the vector unit takes (4.4 cycles for 64), without
// padding to 16 columns, and its operands come one per lane, so that the
// LDS reads (48 bytes per row and particle, 8 per block column) stay below
// the arithmetic, which broadcasting the 2 Q phases of a particle to every
// lane of a vector loop would not.  (16 x 16 x 4 blocks measured 84 cycles for
// 1024 multiply-adds, a fifth slower.  Matrix and vector FP64 share the unit:
// run together their times add.)
// Bound by FP64 issue.  At N = 1024 (254 columns, 3960 entries) 1024 rebuilds by
// the per-step calls take 0.84 ms with their accepts (1.66 ms by walking the
// columns, eight operations per entry), 1024 energies 1.55 ms (2.1 ms).  Few
// particles go by segments instead (walk_sums below).
//
// Lanes (operand A: piece l % 16, particle l / 16; operand B: column l % 4,
// particle l / 16; result: column l % 4, piece 4 (l / 4 % 4) + l / 16).
// Columns 2t and 2t + 1 of a block are cos and sin of one h, so a lane's
// neighbour holds the other half of the pair: even lanes end with the entry
// c + (h + 1/2), odd ones with c - (h + 1/2).
//
// Waves: NW per workgroup, gw of them (a power of two) share the pieces'
// groups, NS groups per wave and pass (the longest with the shortest, the
// groups being sorted by length), and NW / gw of them share the particles.
// Their sums meet in `rc` (LDS, rc_bytes of it, 1 KB per segment of the groups'
// longest pieces at the least; the tables' own may serve, such a pass being the only
// one), in a fixed order: where every share's sums fit, all waves then take a
// part of the entries, else one share after the other adds its own.  (Small systems
// wait for this end, not for arithmetic: by groups, a bilayer of 40 electrons, 30 walkers,
// took 17.5 us per energy call so, 29.0 one share after the other, its loads in
// between; by segments 10.)
// Each pass takes the particles `tile` at a time (a multiple of four) through LDS
// phase tables at `tabs` (S->ph_stride bytes per particle), from the fractional
// coordinates frac(p, d).  `sink(idx, v, w)`
// receives each entry once: slot idx, the sum v without the fixed ions, w its
// weights from grp_w (WGT; else unused).  All threads must call it.
typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ cplx<double> lds_entry(const char* p) {
  const f64x2 v = *reinterpret_cast<const f64x2*>(p);
  return {v.x, v.y};
}

// One run of at most 8 entries of a phase-table row: entry m is
// scale exp(2 pi i (m + off) s), m = m0 .. min(m0 + 8, m1) - 1, powers from an
// exactly reduced start (error below ~8 ulp).
template <bool SK>
__device__ __forceinline__ void fill_run(char* row, double s, double off, int m0, int m1, double scale) {
  const cplx<double> u = turn<SK>(s);
  cplx<double> c = turn<SK>((double(m0) + off) * s);
  c.x *= scale;
  c.y *= scale;
  const int e = min(m0 + 8, m1);
  for (int m = m0; m < e; ++m) {
    *reinterpret_cast<f64x2*>(row + 16 * m) = f64x2{c.x, c.y};
    c = cmul(c, u);
  }
}

// The phase tables of particles p0 .. p0 + np - 1 (up to the next multiple of
// four, empty ones, all zero): per particle the rows exp(i n th_d), n = 0 .. nmax[d], of
// the leading dimensions (the first carries the charge) and
// exp(i (h + 1/2) th_last), h = 0 .. ph_hn - 1.
template <int DIM, int NT, bool SK, typename Pos>
__device__ __forceinline__ void fill_tables(const DevSys* __restrict__ S, const Pos& frac, const double* q, int p0,
                                            int np, int turn_at, char* tabs) {
  const int runs = S->ph_runs;  // of the longest row
  const int stride = S->ph_stride;
  const int np_pad = (np + 3) & ~3;
  // another wave starts each time, as a tile seldom has work for all of them
  for (int e = (threadIdx.x + 8 * turn_at) & (NT - 1); e < np_pad * DIM * runs; e += NT) {
    const int row = e / runs, m0 = 8 * (e - row * runs);
    const int pp = row / DIM, d = row - pp * DIM;
    const bool last = d == DIM - 1;
    const int off = last ? S->ph_ou : (d == 0 ? 0 : S->ph_o1);
    const int m1 = last ? S->ph_hn : S->nmax[d] + 1;
    if (m0 >= m1) continue;
    char* t = tabs + pp * stride + off;
    if (pp < np)
      fill_run<SK>(t, frac(p0 + pp, d), last ? 0.5 : 0.0, m0, m1, d == 0 ? q[p0 + pp] : 1.0);
    else
      for (int m = m0; m < min(m0 + 8, m1); ++m) *reinterpret_cast<f64x2*>(t + 16 * m) = f64x2{0.0, 0.0};
  }
}

__device__ __forceinline__ double flip_sign(double v, uint32_t mask) {
  return __hiloint2double(__double2hiint(v) ^ int(mask), __double2loint(v));
}

template <int DIM, int NW, int NS, bool WGT, bool SK, typename Pos, typename Sink>
__device__ __forceinline__ void rho_build(const DevSys* __restrict__ S, const Pos& frac, const double* q, int n,
                                          char* tabs, int tile, cplx<double>* rc, int rc_bytes, int gw, int g_lo,
                                          int g_hi, Sink&& sink) {
  static_assert(NS == 1 || NS == 2, "groups per wave and pass");
  static_assert(GRP_QMAX == 6, "the block columns' reads are written out");
  constexpr int NT = NW * 64;
  const int lane = threadIdx.x & 63, wave = uniform_i(int(threadIdx.x) >> 6);
  const int nks = NW / gw, wg = wave & (gw - 1), ks = wave / gw;
  const int stride = S->ph_stride, ou = S->ph_ou;
  char* const tabs1 = tabs + tile * stride;  // the tables of one tile are filled while the other's are read
  const double2* gwt = reinterpret_cast<const double2*>(S->grp_w);
  const int at0 = 64 * S->grp_off[g_lo], cnt = 64 * (g_hi < S->n_grp ? S->grp_off[g_hi] : S->n_ent) - at0;
  const bool slabs = nks > 1 && nks * cnt * int(sizeof(cplx<double>)) <= rc_bytes;  // uniform
  for (int gp = g_lo; gp < g_hi; gp += NS * gw) {
    int grp[NS], Q[NS], o0[NS], o1[NS], oc[NS];
    uint32_t s1[NS], sc[NS];
    double ax[NS][GRP_QMAX], ay[NS][GRP_QMAX];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int g = gp + (t == 0 ? wg : 2 * gw - 1 - wg);
      grp[t] = g < g_hi ? g : g_lo;
      Q[t] = g < g_hi ? S->grp_q[grp[t]] : 0;
      const uint32_t pk = S->grp_col[grp[t] * 16 + (lane & 15)];
      o0[t] = 16 * int(pk & 0xff);
      o1[t] = S->ph_o1 + 16 * int((pk >> 8) & 0xff);
      oc[t] = ou + 16 * int((pk >> 16) & 0xff);
      s1[t] = (pk << 7) & 0x80000000u;  // bit 24: n_2 < 0
      sc[t] = (pk << 6) & 0x80000000u;  // bit 25: the centre is negative
#pragma unroll
      for (int i = 0; i < GRP_QMAX; ++i) ax[t][i] = ay[t][i] = 0.0;
    }
    fill_tables<DIM, NT, SK>(S, frac, q, 0, min(tile, n), 0, tabs);
#pragma unroll
    for (int t = 0; t < NS; ++t) Q[t] = uniform_i(Q[t]);
    __syncthreads();
    for (int p0 = 0, b = 0; p0 < n; p0 += tile, b ^= 1) {
      const int left = n - p0;
      if (left > tile) fill_tables<DIM, NT, SK>(S, frac, q, p0 + tile, min(tile, left - tile), p0 + tile, b ? tabs : tabs1);
      const int np_pad = (min(tile, left) + 3) & ~3;
      // uniform branches on the groups' lengths (Q[1] <= Q[0]: they are
      // sorted); written as a switch, or as loops for every pair of lengths,
      // the accumulators were copied from register to register around the
      // branches (1024 rebuilds 1.02 ms)
      if (Q[0] > 0) {
        const char* base = (b ? tabs1 : tabs) + (4 * ks + (lane >> 4)) * stride;
        for (int p = 4 * ks; p < np_pad; p += 4 * nks, base += 4 * nks * stride) {
          const double* bu = reinterpret_cast<const double*>(base + ou + 8 * (lane & 3));
          double bq[GRP_QMAX];
          bq[0] = bu[0];
          bq[1] = bu[4];
          if (Q[0] > 2) {
            bq[2] = bu[8];
            bq[3] = bu[12];
          }
          if (Q[0] > 4) {
            bq[4] = bu[16];
            bq[5] = bu[20];
          }
          cplx<double> a[NS];
#pragma unroll
          for (int t = 0; t < NS; ++t) {  // (an absent second group repeats the first piece's entries)
            a[t] = lds_entry(base + o0[t]);
            if (DIM == 3) {
              cplx<double> e1 = lds_entry(base + o1[t]);
              e1.y = flip_sign(e1.y, s1[t]);
              a[t] = cmul(a[t], e1);
            }
            cplx<double> ec = lds_entry(base + oc[t]);
            ec.y = flip_sign(ec.y, sc[t]);
            a[t] = cmul(a[t], ec);
          }
#pragma unroll
          for (int i = 0; i < GRP_QMAX; ++i)
#pragma unroll
            for (int t = 0; t < NS; ++t)
              if (i < Q[t]) {
                ax[t][i] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[t].x, bq[i], ax[t][i], 0, 0, 0);
                ay[t][i] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[t].y, bq[i], ay[t][i], 0, 0, 0);
              }
        }
      }
      __syncthreads();
    }
    const bool odd = lane & 1;
    auto entry = [&](int t, int i) {  // this lane's entry of block column i
      const double x = ax[t][i], y = ay[t][i];
      const double nx = dpp_all<0xB1>(x), ny = dpp_all<0xB1>(y);  // the neighbour's (quad_perm [1,0,3,2])
      return cplx<double>{odd ? nx + y : x - ny, odd ? ny - x : y + nx};
    };
    if (slabs) {  // uniform
#pragma unroll
      for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int i = 0; i < GRP_QMAX; ++i)
          if (i < Q[t]) rc[ks * cnt + (S->grp_off[grp[t]] + i) * 64 - at0 + lane] = entry(t, i);
      __syncthreads();
      // a thread's entries two at a time (loads may not pass the sinks' stores;
      // asking for them before the first tile took registers and was slower)
      for (int e0 = threadIdx.x; e0 < cnt; e0 += 2 * NT) {
        int idx[2];
        double2 w[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int e = e0 + c * NT;
          idx[c] = e < cnt ? S->grp_slot[at0 + e] : -1;
          if (WGT) w[c] = e < cnt ? gwt[at0 + e] : double2{0.0, 0.0};
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          if (idx[c] < 0) continue;
          cplx<double> v = rc[e0 + c * NT];
          for (int k2 = 1; k2 < nks; ++k2) {  // uniform
            const cplx<double> o = rc[k2 * cnt + e0 + c * NT];
            v.x += o.x;
            v.y += o.y;
          }
          sink(idx[c], v, w[c]);
        }
      }
      __syncthreads();
    } else {
      for (int k2 = 0; k2 < nks; ++k2) {  // uniform: the particle shares in a fixed order
        if (k2 == ks) {
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            const int at = 64 * S->grp_off[grp[t]] + lane;
            if (k2 + 1 < nks) {
#pragma unroll
              for (int i = 0; i < GRP_QMAX; ++i)
                if (i < Q[t]) {
                  cplx<double> v = entry(t, i);
                  cplx<double>* r = rc + at - at0 + 64 * i;
                  *r = k2 > 0 ? cplx<double>{v.x + r->x, v.y + r->y} : v;
                }
            } else {
              int idx[GRP_QMAX];
#pragma unroll
              for (int i = 0; i < GRP_QMAX; ++i) idx[i] = i < Q[t] ? S->grp_slot[at + 64 * i] : -1;
#pragma unroll
              for (int i = 0; i < GRP_QMAX; ++i)
                if (i < Q[t]) {
                  cplx<double> v = entry(t, i);
                  if (k2 > 0) {
                    const cplx<double> r = rc[at - at0 + 64 * i];
                    v.x += r.x;
                    v.y += r.y;
                  }
                  if (idx[i] >= 0) sink(idx[i], v, WGT ? gwt[at + 64 * i] : double2{0.0, 0.0});
                }
            }
          }
        }
        if (nks > 1) __syncthreads();
      }
    }
  }
}

// rho of few particles at one segment's four slots, on the vector unit, from the
// same phase tables (those of particles p_lo .. p_hi - 1, all of them in LDS): the
// segment is a column piece of Q = 1, 16 FP64 operations per particle.
// A thread per segment needs no groups and no meeting of shares, which for few
// particles cost more than the matrix instructions save.
template <int DIM>
__device__ __forceinline__ void walk_sums(const DevSys* __restrict__ S, uint32_t an, const char* tabs, int p_lo,
                                          int p_hi, cplx<double> (&v)[SEG]) {
  static_assert(SEG == 4, "two half-integer offsets either side of the centre");
  const int stride = S->ph_stride, ou = S->ph_ou;
  const int n1 = DIM == 3 ? unpack_n(an, 1) : 0, c2 = 2 * unpack_n(an, DIM - 1) + SEG - 1;  // twice the centre
  const int o0 = 16 * unpack_n(an, 0), o1 = S->ph_o1 + 16 * abs(n1), oc = ou + 16 * ((abs(c2) - 1) / 2);
  const uint32_t s1 = n1 < 0 ? 0x80000000u : 0u, sc = c2 < 0 ? 0x80000000u : 0u;
  double xc[2] = {}, xs[2] = {}, yc[2] = {}, ys[2] = {};  // sums of (Re, Im) A times (cos, sin)((h + 1/2) th)
  const char* base = tabs + p_lo * stride;
#pragma unroll 2
  for (int p = p_lo; p < p_hi; ++p, base += stride) {
    cplx<double> a = lds_entry(base + o0);
    if (DIM == 3) {
      cplx<double> e1 = lds_entry(base + o1);
      e1.y = flip_sign(e1.y, s1);
      a = cmul(a, e1);
    }
    cplx<double> ec = lds_entry(base + oc);
    ec.y = flip_sign(ec.y, sc);
    a = cmul(a, ec);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const cplx<double> u = lds_entry(base + ou + 16 * h);
      xc[h] = fma(a.x, u.x, xc[h]);
      xs[h] = fma(a.x, u.y, xs[h]);
      yc[h] = fma(a.y, u.x, yc[h]);
      ys[h] = fma(a.y, u.y, ys[h]);
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    v[1 - h] = {xc[h] + ys[h], yc[h] - xs[h]};
    v[2 + h] = {xc[h] - ys[h], yc[h] + xs[h]};
  }
}

// Waves that share the groups of column pieces in rho_build: the fewest whose
// NS groups each cover them in one pass, so that the others share the particles.
__host__ __device__ __forceinline__ int rho_waves(int n_grp, int ns, int nw) {
  int gw = 1;
  while (gw < nw && ns * gw < n_grp) gw *= 2;
  return gw;
}

// ---------------------------------------------------------------------------
// launch helpers

inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

inline int last_launch() {
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : int(e);
}

// Kernels asking for more than 64 KiB of LDS must raise their limit first
// (gfx950 has 160 KiB per workgroup processor).
template <typename F>
int allow_lds(F* kernel, size_t bytes) {
  if (bytes <= 65536) return 0;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  return e == hipSuccess ? 0 : int(e);
}

inline int even(int x) { return (x + 1) & ~1; }
inline size_t up16(size_t x) { return (x + 15) & ~size_t(15); }

constexpr size_t RUN_LDS_BUDGET = 160 * 1024;  // LDS per workgroup on gfx950
// LDS that each of per_cu workgroups on a CU may take: it is given out in blocks of
// 1280 bytes (a third of 160 KB to the byte lets two workgroups run, not three).
inline size_t lds_share(int per_cu) { return RUN_LDS_BUDGET / 1280 / size_t(per_cu) * 1280; }
constexpr int RUN_NO_FIT = -1;                 // the fused kernel's LDS does not fit: use the per-step kernels

// Particles per phase-table tile of rho_build with its tiles within `bytes` of
// LDS: a multiple of four (a matrix instruction takes four particles), at least
// four.  One tile where it holds the largest walker of up to 2 TILE_MAX particles,
// else two of up to TILE_MAX each.
inline int rho_tile(const LaunchBatch& b, size_t bytes) {
  const int most = (b.max_particles + 3) & ~3;
  if (most <= 2 * TILE_MAX && size_t(most) * size_t(b.max_ph) <= bytes) return most;
  return std::max(4, std::min(std::min(TILE_MAX, most), int(bytes / (2 * size_t(b.max_ph))) & ~3));
}
inline size_t rho_lds(const LaunchBatch& b, int tile) {
  return (b.max_particles <= tile ? 1 : 2) * size_t(tile) * size_t(b.max_ph);
}

// Workgroups of this kernel that fit on one CU by registers (4 SIMDs, 512
// VGPRs per lane each); the fused kernel sizes its LDS so as not to lower it.
template <typename F>
int blocks_per_cu(F* kernel, int nt) {
  hipFuncAttributes a{};
  if (hipFuncGetAttributes(&a, reinterpret_cast<const void*>(kernel)) != hipSuccess || a.numRegs <= 0) return 1;
  const int vgpr = (a.numRegs + 7) & ~7;
  const int waves_per_simd = std::min(8, 512 / vgpr);
  return std::max(1, 4 * waves_per_simd / (nt / 64));
}

}  // namespace ewald
