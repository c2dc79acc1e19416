// Face integral and barycentric moments of a triangle from its centred vertex phases through the fitted
// symmetric polynomials (face_poly.h), and the binary64 sine / cosine they are combined with.
//
// With d_0 + d_1 + d_2 = 0, p = d_0^2 + d_0 d_1 + d_1^2, E = d_0 d_1 (d_0 + d_1), w = E^2:
//   J = A + i E B,   Y_k = alpha + beta d_k + gamma d_k^2,   beta = i bi + E br,   gamma = gr + i E gi,
//   alpha = (J - 2 p gamma) / 3,
// A, B, bi, br, gr, gi polynomials in (p, w). Valid for max |d_k| <= FaceFit64::M / FaceFit32::M.
#pragma once

#include "face_poly.h"
#include "pft_device.h"

namespace pft {

// The binary64 coefficients in constant memory. A binary64 instruction takes no 64-bit literal, and the coefficients
// of a face term (54 in the forward, 110 in the adjoint) fit neither register file, so each face reads them through
// the scalar cache: fit64() once per face, whose empty asm keeps the loads inside the face loop (hoisted out of it
// they spilled 86 vector registers). A scalar source costs a binary64 instruction nothing.
__constant__ const double kFit64Row[] = {PFT_FIT64_ROW};
using Fit64 = const __attribute__((address_space(4))) double*;
__device__ __forceinline__ Fit64 fit64() {
  Fit64 t = (Fit64)kFit64Row;
  asm volatile("" : "+s"(t));
  return t;
}

// a * b + c with c in scalar registers. (The compiler's own choice, v_fmac_f64, first copies the coefficient into the
// destination with two v_mov_b32: 1.3 times the instructions of a Horner sum.)
__device__ __forceinline__ double fma64s(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}

// sum_a C::c[a] x^a, binary64.
template <class C>
__device__ __forceinline__ double horner64(Fit64 t, double x) {
  constexpr int N = sizeof(C::c) / sizeof(C::c[0]);
  double s = t[C::at + N - 1];
#pragma unroll
  for (int a = N - 2; a >= 0; --a) s = fma64s(s, x, t[C::at + a]);
  return s;
}

// sin x and cos x for |x| <= kSinCosMax64: x reduced by the nearest multiple n of pi/2 (pi/2 as a double plus its
// remainder, both products exact in the fused multiply-add: the reduced argument carries one rounding), polynomials
// on [-pi/4, pi/4]. Beyond, n times pi/2's second remainder would be felt: the callers take the library function
// there (sincos_any64), which costs twice the instructions everywhere.
constexpr double kSinCosMax64 = 268435456.0;  // 2^28
__device__ __forceinline__ void sincos64(Fit64 t, double x, double* s, double* c) {
  const double n = rint(x * 0.63661977236758134308);
  double r = fma(-n, 1.5707963267948965580, x);
  r = fma(-n, 6.123233995736766036e-17, r);
  const double z = r * r;
  const double sr = r + r * z * horner64<SinCos64::S>(t, z);
  const double cr = 1.0 + z * (z * horner64<SinCos64::C>(t, z) - 0.5);
  const int q = (int)n;
  const double a = (q & 1) ? cr : sr, b = (q & 1) ? sr : cr;
  *s = (q & 2) ? -a : a;
  *c = ((q + 1) & 2) ? -b : b;
}
__device__ __forceinline__ void sincos_any64(Fit64 t, double x, double* s, double* c) {
  if (__builtin_expect(!(fabs(x) <= kSinCosMax64), 0))
    sincos(x, s, c);
  else
    sincos64(t, x, s, c);
}

// C0 + C1 w (+ C2 w^2 + C3 w^3), each a polynomial in p, binary64.
template <class C0, class... C>
__device__ __forceinline__ double poly64(Fit64 t, double p, double w) {
  if constexpr (sizeof...(C) == 0)
    return horner64<C0>(t, p);
  else
    return poly64<C...>(t, p, w) * w + horner64<C0>(t, p);
}

// A and B of J = A + i E B, and J itself, binary64, max |d_k| <= F::M: FaceFit64, or FaceFit64S of two thirds of its
// coefficients for half its range.
template <class F>
__device__ __forceinline__ void face_ab64(Fit64 t, double p, double w, double& A, double& B) {
  if constexpr (F::M < FaceFit64::M) {
    A = poly64<typename F::A0, typename F::A1, typename F::A2>(t, p, w);
  } else {
    A = poly64<typename F::A0, typename F::A1, typename F::A2, typename F::A3>(t, p, w);
  }
  B = poly64<typename F::B0, typename F::B1, typename F::B2>(t, p, w);
}
template <class F>
__device__ __forceinline__ void face_integral_fit64(Fit64 t, double d0, double d1, double& jr, double& ji) {
  const double s = d0 + d1;
  const double E = d0 * d1 * s;
  double B;
  face_ab64<F>(t, d0 * s + d1 * d1, E * E, jr, B);
  ji = E * B;
}

// Whether every phase |d_k| <= |Q| rho (as in fit_range_test_needed) of a Q is within FaceFit64S.
__device__ __forceinline__ bool short_phases64(double q2, double rho) {
  return sqrt(q2) * rho <= 0.999 * FaceFit64S::M;
}

// beta and gamma's parts: beta = i bi + E br, gamma = gr + i E gi.
template <class F>
__device__ __forceinline__ void face_beta_gamma64(Fit64 t, double p, double w, double& bi, double& br, double& gr, double& gi) {
  if constexpr (F::M < FaceFit64::M) {
    bi = poly64<typename F::bi0, typename F::bi1, typename F::bi2>(t, p, w);
    br = poly64<typename F::br0, typename F::br1>(t, p, w);
    gr = poly64<typename F::gr0, typename F::gr1, typename F::gr2>(t, p, w);
    gi = poly64<typename F::gi0, typename F::gi1>(t, p, w);
  } else {
    bi = poly64<typename F::bi0, typename F::bi1, typename F::bi2, typename F::bi3>(t, p, w);
    br = poly64<typename F::br0, typename F::br1, typename F::br2>(t, p, w);
    gr = poly64<typename F::gr0, typename F::gr1, typename F::gr2>(t, p, w);
    gi = poly64<typename F::gi0, typename F::gi1, typename F::gi2>(t, p, w);
  }
}

// J and the complex moments Y_0, Y_1 (Y_2 = J - Y_0 - Y_1), binary64, max |d_k| <= FaceFit64::M.
__device__ __forceinline__ void bary_moments_fit64(Fit64 t, double d0, double d1, double* yr, double* yi, double& jr,
                                                   double& ji) {
  const double s = d0 + d1;
  const double p = d0 * s + d1 * d1, E = d0 * d1 * s, w = E * E;
  double B, bi, br, gr, gi;
  face_ab64<FaceFit64>(t, p, w, jr, B);
  ji = E * B;
  face_beta_gamma64<FaceFit64>(t, p, w, bi, br, gr, gi);
  br *= E;
  gi *= E;
  const double ar = (jr - 2.0 * p * gr) * (1.0 / 3.0), ai = (ji - 2.0 * p * gi) * (1.0 / 3.0);
  yr[0] = ar + d0 * (br + d0 * gr);
  yi[0] = ai + d0 * (bi + d0 * gi);
  yr[1] = ar + d1 * (br + d1 * gr);
  yi[1] = ai + d1 * (bi + d1 * gi);
}

// sum_a C::c[a] x^a in binary32 by fused multiply-adds whose addend is the instruction's literal. (Left to
// itself the compiler keeps a loop's coefficients in scalar registers, and a scalar source halves the issue
// rate of a vector instruction on this target: 99 460 faces x 64 000 Q, 5.80 ms against 5.66 ms.)
template <class C, int A>
__device__ __forceinline__ float horner_lit_from(float s, float x) {
  if constexpr (A < 0) {
    return s;
  } else {
    float r;
    asm("v_fmaak_f32 %0, %1, %2, %3" : "=v"(r) : "v"(s), "v"(x), "n"(__builtin_bit_cast(int, C::c[A])));
    return horner_lit_from<C, A - 1>(r, x);
  }
}
template <class C>
__device__ __forceinline__ float horner_lit(float x) {
  constexpr int N = sizeof(C::c) / sizeof(C::c[0]);
  return horner_lit_from<C, N - 2>(C::c[N - 1], x);
}

// The six functions of the binary32 moments, max |d_k| <= FaceFit32M::M (32 operations).
struct Moments32 {
  float A, B, bi, br, gr, gi;
};
__device__ __forceinline__ Moments32 face_moments32(float p, float w) {
  Moments32 m;
  m.A = horner_lit<FaceFit32M::A1>(p) * w + horner_lit<FaceFit32M::A0>(p);
  m.B = horner_lit<FaceFit32M::B1>(p) * w + horner_lit<FaceFit32M::B0>(p);
  m.bi = horner_lit<FaceFit32M::bi1>(p) * w + horner_lit<FaceFit32M::bi0>(p);
  m.br = FaceFit32M::br1::c[0] * w + horner_lit<FaceFit32M::br0>(p);
  m.gr = horner_lit<FaceFit32M::gr1>(p) * w + horner_lit<FaceFit32M::gr0>(p);
  m.gi = horner_lit<FaceFit32M::gi0>(p);
  return m;
}

// The face origin phase Q.g / (2 pi) reduced to [-1/2, 1/2] turn, by binary64 multiply-adds onto 1.5 * 2^20: the sum's
// low 32 mantissa bits are the phase in units of 2^-32 turn modulo one turn, so no rounding to the nearest turn and no
// conversion from binary64 is needed (4 of the 6 binary64 instructions of the plain form; each remaining one rounds at
// 2^-33 turn). |Q.g| / (2 pi) must stay below 2^19 turns (wide_phases32 tests it per wavefront; beyond, the plain
// form).
__device__ __forceinline__ float origin_turns(const double* Q, const double* gt) {
  const double v = fma(Q[2], gt[2], fma(Q[1], gt[1], fma(Q[0], gt[0], 1572864.0)));
  return (float)(int)(uint32_t)__double_as_longlong(v) * 2.3283064365386963e-10f;  // 2^-32
}
__device__ __forceinline__ float origin_turns_plain(const double* Q, const double* gt) {
  const double ph = Q[0] * gt[0] + Q[1] * gt[1] + Q[2] * gt[2];
  return (float)(ph - rint(ph));
}
constexpr double kWidePhase32 = 3.2e6;                                // 2^19 turns = 3.29e6 rad
__device__ __forceinline__ bool wide_phases32(double q2, double R) {  // |g| <= R; NaN counts as beyond
  return __any(!(sqrt(q2) * R <= kWidePhase32));
}

// Whether an origin phase Q.g of a wavefront can exceed the range of sincos64: |g| <= R, the mesh's radius (q2
// the lane's |Q|^2). NaN counts as beyond.
__device__ __forceinline__ bool big_phases64(double q2, double R) {
  return __any(!(sqrt(q2) * R <= 0.999 * kSinCosMax64));
}

}  // namespace pft
