// Device-side helpers of the TU-fRG library: complex arithmetic and the
// regulator functions whose divided differences are the loop kernels.
//
// Loops (Sec. 3.1 of the paper, generalised to the temperature and Omega
// regulators): with an odd function J_Lambda(e) and K = dJ/dLambda,
//   L-(e1, e2) =  (K(e1) + K(e2)) / (e1 + e2)    (particle-particle)
//   L+(e1, e2) = -(K(e1) - K(e2)) / (e1 - e2)    (particle-hole)
// Temperature flow (Lambda = T): J = tanh(e / 2T) / 2, the Fermi-function
// combination 1 - 2 f(e).  Omega scheme at T = 0 (propagator times
// w^2 / (w^2 + Omega^2)): J = e (2|e| + Omega) / (4 (|e| + Omega)^2).
// At coinciding arguments the divided difference is the mean of K' over the
// interval: K' and its derivatives at the middle (Omega scheme in FP64: the two-point
// Gauss-Legendre rule).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tufrg {

enum { CUT_TEMPERATURE = 0, CUT_OMEGA = 1, CUT_SHELL = 2 };

// The momentum-shell scheme (Sec. 3.1 regulator) takes its bubbles at a fixed
// temperature: its divided differences are those of the temperature scheme,
// evaluated at Lambda = T, and the loop kernels carry a shell factor.
__host__ __device__ constexpr int dd_scheme(int scheme) { return scheme == CUT_SHELL ? CUT_TEMPERATURE : scheme; }

// Shell factor of a band value: the loop kernel of a pair is the fixed-T
// divided difference times a_m b_n + b_m a_n, with chi = e^2 / (e^2 + Lambda^2)
// and (a, b) = (d chi / d Lambda, chi) for the loop (deriv) or
// (chi, chi) / sqrt 2 for the bubble.
template <typename T>
__device__ inline void shell_ab(T e, T lam, int deriv, T &a, T &b) {
  const T e2 = e * e, d = e2 + lam * lam;
  const T chi = e2 / d;
  if (deriv) {
    a = -T(2) * lam * e2 / (d * d);
    b = chi;
  } else {
    a = b = chi * T(0.70710678118654752440);
  }
}

template <typename T>
struct cx {
  T re, im;
};

template <typename T>
__host__ __device__ inline cx<T> cmake(T r, T i) {
  cx<T> z;
  z.re = r;
  z.im = i;
  return z;
}

template <typename T>
__host__ __device__ inline cx<T> cadd(cx<T> a, cx<T> b) {
  return cmake(a.re + b.re, a.im + b.im);
}

template <typename T>
__host__ __device__ inline cx<T> cmul(cx<T> a, cx<T> b) {
  return cmake(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}

// acc += a * b
template <typename T>
__host__ __device__ inline void cfma(cx<T> &acc, cx<T> a, cx<T> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}

// acc += a * conj(b)
template <typename T>
__host__ __device__ inline void cfmaconj(cx<T> &acc, cx<T> a, cx<T> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(a.im, b.re, acc.im);
  acc.im = fma(-a.re, b.im, acc.im);
}

// Fast reciprocal: hardware estimate refined by Newton steps (FP64) or the
// 1-ulp hardware reciprocal (FP32).
__device__ inline double rcp_fast(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return r;
}
__device__ inline float rcp_fast(float d) { return __builtin_amdgcn_rcpf(d); }

// 1 / x to about half an ulp (FP64: one), hardware estimate and Newton steps
__device__ inline double rcp_newton(double x) { return rcp_fast(x); }
__device__ inline float rcp_newton(float x) {
  const float r = rcp_fast(x);
  return fmaf(fmaf(-x, r, 1.f), r, r);
}

// 1 / x: exact division in FP64, the hardware reciprocal in FP32
__device__ inline double rdiv(double x) { return 1.0 / x; }
__device__ inline float rdiv(float x) { return __builtin_amdgcn_rcpf(x); }

// sech^2(x) and tanh(x) from s = exp(-2|x|), stable for every x.
template <typename T>
__device__ inline void sech2_tanh(T x, T &sech2, T &th) {
  T ax = fabs(x);
  T s = exp(T(-2) * ax);
  T inv = T(1) / (T(1) + s);
  sech2 = T(4) * s * inv * inv;
  th = copysign((T(1) - s) * inv, x);
}

// J or K = dJ/dLambda at energy e (deriv selects K).
template <typename T>
__device__ inline T cut_val(T e, T lam, int scheme, int deriv) {
  if (scheme == CUT_TEMPERATURE) {
    T x = e / (T(2) * lam);
    T s2, th;
    sech2_tanh(x, s2, th);
    if (deriv) return -e * s2 / (T(4) * lam * lam);
    return T(0.5) * th;
  }
  T a = fabs(e);
  T d = a + lam;
  if (deriv) return -e * (T(3) * a + lam) * rdiv(T(4) * d * d * d);
  return e * (T(2) * a + lam) * rdiv(T(4) * d * d);
}

// d/de of cut_val.
template <typename T>
__device__ inline T cut_der(T e, T lam, int scheme, int deriv) {
  if (scheme == CUT_TEMPERATURE) {
    T x = e / (T(2) * lam);
    T s2, th;
    sech2_tanh(x, s2, th);
    if (deriv) return -s2 * (T(1) - T(2) * x * th) / (T(4) * lam * lam);
    return s2 / (T(4) * lam);
  }
  T a = fabs(e);
  T d = a + lam;
  T d2 = d * d;
  if (deriv) return (T(3) * e * e - T(4) * a * lam - lam * lam) * rdiv(T(4) * d2 * d2);
  return lam * (T(3) * a + lam) * rdiv(T(4) * d2 * d);
}

template <typename T>
__device__ inline T gl2_mean(T a, T b, T lam, int scheme, int deriv) {
  const T c = T(0.57735026918962576451);  // 1/sqrt(3)
  T m = T(0.5) * (a + b), h = T(0.5) * (b - a);
  return T(0.5) * (cut_der(m - c * h, lam, scheme, deriv) + cut_der(m + c * h, lam, scheme, deriv));
}

// Mean of f = cut_der over [x, y] from its middle m: f(m) + d^2 / 24 f''(m) +
// d^4 / 1920 f''''(m), d = x - y.  At the switch widths the last term is 2.6e-15 of f
// in FP64 and 2e-7 with the Omega scheme in FP32 (with the temperature scheme it is
// below FP32 rounding and left out), the next one below 1e-8 of that.  One
// exponential or reciprocal instead of the two of the two-point rule, which took
// 603 us where one takes 553 (FP32 Rashba loops, 13 form factors, L 24): near
// Lambda = 1 a fifth to a half of the waves of a loop kernel hold such a pair.
// Written so that the rounding stays below that rule's, which averages two
// evaluations (600 000 pairs, largest error relative to the largest f, that rule's
// and this one's: FP64 1.4e-15 and 6.7e-16, FP32 2.9e-7 and 2.4e-7, Omega 3.8e-7 and
// 2.3e-7): sech^2 as 4 z, z = p - p^2 with p = 1 / (1 + e^{2|u|}), in
// which an error of p falls out where sech^2 is largest; with the Omega scheme the
// polynomial of K' in |m| / D and not in Lambda / D, without its cancellation.
template <typename T>
__device__ inline T mid_mean(T x, T y, T lam, int scheme, int deriv) {
  const T m = T(0.5) * (x + y), d = x - y, w = d * d * T(1.0 / 24.0);
  if (scheme == CUT_TEMPERATURE) {
    // derivatives in u = e / 2T, r = 1 / 2T, s = sech^2 u, t = tanh u
    const T il = rcp_newton(lam), u = fabs(m) * (T(0.5) * il), w4 = w * (T(0.25) * il * il);
    const T ex = exp(T(-2) * u), p = ex * rcp_newton(T(1) + ex), z = fma(-p, p, p);
    if (deriv) {
      // f = -s (1 - 2 u t) r^2, second derivative -(12 s - 18 s^2 + u t s (24 s - 8)) r^2,
      // fourth -s (80 - 600 s + 600 s^2 + u t (-32 + 480 s - 720 s^2)) r^2, times 0.3 w4^2
      const T ut = u * fma(T(-2), p, T(1));
      T g = fma(ut, fma(T(96), z, T(-8)), fma(T(-72), z, T(12)));
      if (sizeof(T) == 8)
        g = fma(w4, fma(ut, fma(fma(T(-3456), z, T(576)), z, T(-9.6)), fma(fma(T(2880), z, T(-720)), z, T(24))), g);
      const T il2 = sizeof(T) == 8 ? il * il : rcp_newton(lam * lam);
      return -(z * il2) * fma(w4, g, fma(T(-2), ut, T(1)));
    }
    // f = s r / 2, second derivative (4 s - 6 s^2) r / 2, fourth (16 s - 120 s^2 + 120 s^3) r / 2
    T g = fma(T(-24), z, T(4));
    if (sizeof(T) == 8) g = fma(w4, fma(fma(T(576), z, T(-144)), z, T(4.8)), g);
    return z * il * fma(w4, g, T(1));
  }
  // D = |e| + Lambda, g = Lambda / D, h = |e| / D = 1 - g:
  // f = (3 - 10 g + 6 g^2) / 4 D^2 = (6 h^2 - 2 h - 1) / 4 D^2 (of K) or (3 g - 2 g^2) / 4 D (of J)
  const T i = rcp_newton(fabs(m) + lam), g = lam * i, w2 = w * i * i;
  if (deriv) {
    const T h = fabs(m) * i;
    const T f2 = fma(fma(T(120), g, T(-120)), g, T(18)), f4 = fma(fma(T(1512), g, T(-1080)), g, T(108));
    return T(0.25) * (i * i) * fma(w2, fma(w2, f4, f2), fma(fma(T(6), h, T(-2)), h, T(-1)));
  }
  const T f2 = fma(T(-24), g, T(18)), f4 = fma(T(-216), g, T(108));
  return T(0.25) * i * g * fma(w2, fma(w2, f4, f2), fma(T(-2), g, T(3)));
}

// Relative width below which the divided difference switches to the mean of
// the derivative.  FP64: 1e-3; FP32: 2e-2 (cancellation in the quotient costs
// about eps / width = 3e-6 at the switch; a wider switch sends more lanes, and
// with them whole waves, through the slower branch: at 5e-2 the Rashba loop ran
// 6 % slower with the same error).
template <typename T>
struct degen_rel;
template <>
struct degen_rel<double> {
  static constexpr double v = 1e-3;
};
template <>
struct degen_rel<float> {
  static constexpr float v = 2e-2f;
};

// Mean of K' over [x, y], x and y closer than the switch.
template <typename T>
__device__ inline T near_mean(T x, T y, T lam, int scheme, int deriv) {
  if (sizeof(T) == 8 && scheme == CUT_OMEGA) return gl2_mean(x, y, lam, scheme, deriv);
  return mid_mean(x, y, lam, scheme, deriv);
}

// x - y = d too small for the quotient.  Omega scheme: K' is even with a kink at 0;
// around 0 the quotient (K(|x|) + K(|y|)) / (|x| + |y|) has no cancellation.
template <typename T>
__device__ inline bool near_degenerate(T d, T x, T y, T lam, int scheme) {
  if (scheme == CUT_OMEGA && x * y < T(0)) return false;
  const T scale = scheme == CUT_TEMPERATURE ? lam : lam + fabs(x) + fabs(y);
  return !(fabs(d) > degen_rel<T>::v * scale);
}

// (g(x) - g(y)) / (x - y) given gx = g(x), gy = g(y).
template <typename T>
__device__ inline T divided_difference(T x, T y, T gx, T gy, T lam, int scheme, int deriv) {
  const T d = x - y;
  if (!near_degenerate(d, x, y, lam, scheme)) return (gx - gy) * rcp_fast(d);
  return near_mean(x, y, lam, scheme, deriv);
}

}  // namespace tufrg
