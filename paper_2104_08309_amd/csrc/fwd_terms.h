// Per-(Q, face) terms of the forward transform, binary64 and FP32-compensated
// forms, shared by the single-mesh and batched kernels (formulas in pft_device.h).
#pragma once

#include "face_moments.h"
#include "moment_poly.h"
#include "pft_device.h"

namespace pft {

// ---------------------------------------------------------------------------
// binary64 per-(Q, face) term T_m (see pft_device.h for the formula)
// ---------------------------------------------------------------------------
// sin(x) / x for |x| < kSincNear64 (Taylor series), where the quotient of a sine from vertex phase products loses relative
// accuracy.
constexpr double kSincNear64 = 0.1;
__device__ __forceinline__ double sinc_near64(double x) {
  const double x2 = x * x;
  return 1.0 + x2 * (-1.0 / 6.0 + x2 * (1.0 / 120.0 + x2 * (-1.0 / 5040.0 + x2 * (1.0 / 362880.0))));
}

// J beyond the fitted range by the edge terms (as the FP32C form below): J = i / (2 p) sum_k d_k
// sinc((d_{k+1} - d_{k+2}) / 2) exp(-i d_k / 2). One division serves the three sincs and 1 / (2 p).
__device__ __forceinline__ void face_integral_far64(Fit64 t, double d0, double d1, double& jr, double& ji) {
  const double s = d0 + d1;
  double s0, c0, s1, c1;
  sincos_any64(t, 0.5 * d0, &s0, &c0);
  sincos_any64(t, 0.5 * d1, &s1, &c1);
  // exp(i d_2 / 2) = conj(exp(i d_0 / 2) exp(i d_1 / 2))
  const double c2 = c0 * c1 - s0 * s1, s2 = -(s0 * c1 + c0 * s1);
  // half-differences of the edges opposite the vertices, and their sines
  const double x0 = 0.5 * (s + d1), x1 = -0.5 * (s + d0), x2 = 0.5 * (d0 - d1);
  const bool n0 = fabs(x0) < kSincNear64, n1 = fabs(x1) < kSincNear64, n2 = fabs(x2) < kSincNear64;
  const double r0 = n0 ? 1.0 : x0, r1 = n1 ? 1.0 : x1, r2 = n2 ? 1.0 : x2, p2 = 2.0 * (d0 * s + d1 * d1);
  const double r01 = r0 * r1, r2p = r2 * p2;
  const double inv = 1.0 / (r01 * r2p);
  const double i01 = inv * r2p, i2p = inv * r01;  // 1 / (r0 r1), 1 / (r2 2 p)
  double g0 = (s1 * c2 - c1 * s2) * (i01 * r1), g1 = (s2 * c0 - c2 * s0) * (i01 * r0),
         g2 = (s0 * c1 - c0 * s1) * (i2p * p2);
  if (n0 | n1 | n2) {
    g0 = n0 ? sinc_near64(x0) : g0;
    g1 = n1 ? sinc_near64(x1) : g1;
    g2 = n2 ? sinc_near64(x2) : g2;
  }
  // d_k times the sinc of the edge opposite vertex k
  const double a0 = d0 * g0, a1 = d1 * g1, a2 = -s * g2, h = i2p * r2;
  jr = h * (a0 * s0 + a1 * s1 + a2 * s2);
  ji = h * (a0 * c0 + a1 * c1 + a2 * c2);
}

// Whether a centred vertex phase of a wavefront can exceed the range of FaceFit64, as fit_range_test_needed.
__device__ __forceinline__ bool fit_range_test_needed64(float qmax, double rho) {
  return (double)qmax * rho > 0.999 * FaceFit64::M;
}

// One face against a thread's NQ Q points, binary64: adds T = -i (Q.N) exp(iQ.g) J to xr, xi. J by the fitted
// polynomials where the largest centred vertex phase is at most FaceFit64::M (no quotient, nothing cancels near the
// face normal), by the edge terms beyond; the choice is per lane, and a lane whose pairs are all beyond forms no
// polynomials (116 faces x 200 000 Q, phases to 8: 198 -> 176 us with that and the one division; prism over a 60-gon, phases
// to 20: 561 -> 492). A face without area (N = 0, finite J) gives 0. CHECK: test the phases against the range (left out
// where no phase of the wavefront can exceed it, 5 120 faces x 64 000 Q with gradient 3.08 -> 3.05 ms); big
// (wavefront-uniform): some origin phase may exceed kSinCosMax64.
template <int NQ, bool CHECK>
__device__ __forceinline__ void fwd_face_f64(const Face64& f, const double (*Q)[3], bool big, double* xr, double* xi) {
  const Fit64 t = fit64();
  double d0[NQ], d1[NQ], jr[NQ], ji[NQ];
  bool far[NQ];
  bool any = false, all = true;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    d0[k] = Q[k][0] * f.u0[0] + Q[k][1] * f.u0[1] + Q[k][2] * f.u0[2];
    d1[k] = Q[k][0] * f.u1[0] + Q[k][1] * f.u1[1] + Q[k][2] * f.u1[2];
    if (CHECK) {
      far[k] = fmax(fabs(d0[k]), fmax(fabs(d1[k]), fabs(d0[k] + d1[k]))) > FaceFit64::M;
      any |= far[k];
      all &= far[k];
      jr[k] = ji[k] = 0.0;
    }
  }
  if (!CHECK || !all) {
#pragma unroll
    for (int k = 0; k < NQ; ++k) face_integral_fit64<FaceFit64>(t, d0[k], d1[k], jr[k], ji[k]);
  }
  if (CHECK && any) {
#pragma unroll
    for (int k = 0; k < NQ; ++k)
      if (far[k]) face_integral_far64(t, d0[k], d1[k], jr[k], ji[k]);
  }
  double sf[NQ], cf[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const double phi = Q[k][0] * f.g[0] + Q[k][1] * f.g[1] + Q[k][2] * f.g[2];
    if (__builtin_expect(big, 0))
      sincos_any64(t, phi, &sf[k], &cf[k]);
    else
      sincos64(t, phi, &sf[k], &cf[k]);
  }
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const double QN = Q[k][0] * f.N[0] + Q[k][1] * f.N[1] + Q[k][2] * f.N[2];
    xr[k] += QN * (cf[k] * ji[k] + sf[k] * jr[k]);
    xi[k] += QN * (sf[k] * ji[k] - cf[k] * jr[k]);
  }
}

// ---------------------------------------------------------------------------
// FP32-compensated per-(Q, face) term
// ---------------------------------------------------------------------------
// T = -i (Q.N) exp(iQ.g) J, J the face integral normalised by twice the area, a symmetric function of the
// centred vertex phases d_k = Q.u_k (d_0 + d_1 + d_2 = 0) alone. In binary32 on the record's face-local
// quantities (Face32), with the phases as p_k = d_k / (4 pi) (half-phases in turns, p_2 = -s, s = p_0 + p_1):
//
// * largest |d_k| <= FaceFit32::M: J = A(P, w) + i E B(P, w), two fitted polynomials in P = p_0^2 + p_0 p_1 +
//   p_1^2 and w = E^2, E = p_0 p_1 s (face_poly.h; fit error 2.3e-8 of J(0) = 1/2). No quotient, so nothing
//   cancels and Q along the face normal is an ordinary point; one sine and one cosine (of the face origin
//   phase) are the only transcendental instructions.
// * beyond: the divided differences of exp over the pairs of vertices, each an edge term sinc exp(i midpoint
//   phase). -i (d_j - d_k) J is the difference of the two other edges' terms; weighting the three relations
//   by the differences themselves gives the symmetric form
//     J = i / (2 p) sum_k d_k E_k,   E_k the term of the edge opposite vertex k (midpoint phase -d_k / 2,
//                                    half-difference (d_{k+1} - d_{k+2}) / 2),  p = d_0^2 + d_0 d_1 + d_1^2
//   (the 3D section's edge sum with the weights expressed in the phases). p >= 3/4 max d_k^2, so |d_k| / (2 p)
//   stays below 1 / M here: nothing is divided by a small number.
//
// The choice is per lane, on the pair's own phases, so a Q's value does not depend on the other Q of its
// wavefront.
//
// The face origin phase r = Q.g / (2 pi) (turns). In an edge-sharing order (Face32::flags) a face's edge 0 is
// its predecessor's edge 1, the same segment: its midpoint phase is t = r - p_2 = r + s. t is carried in a
// register, reduced to [-1/2, 1/2] turn: r = t - s, and the phase passed on is that of the face's own edge 1,
// r - p_0 = t - (s + p_0), formed from t so that each step adds one rounding of t (at most 2^-25 turn). The
// chain is re-anchored every kAnchor faces: there, and at every face that does not follow its predecessor across
// an edge, r is formed in binary64 and reduced to [-1/2, 1/2] before it is rounded to binary32.
//
// Cost and bound: FP32 vector issue (99 460 faces x 64 000 Q: 8.33 -> 5.54 ms a call against the form that summed
// the three edge terms of every pair, with 5 transcendentals; 5 120 x 262 144: 1.65 -> 1.12 ms). Per pair 9 operations for Q.N, p_0, p_1, 6 for s, P, E, w, 14 for the
// polynomials, 5 for the phase chain, 6 for the complex product and the sums, 2 transcendentals.
#ifndef PFT_ANCHOR
#define PFT_ANCHOR kTileF32
#endif
constexpr int kAnchor = PFT_ANCHOR;  // faces between binary64 origin phases in a chain (divides kTileF32)
static_assert(kTileF32 % kAnchor == 0, "the anchor interval divides the face tile");

// Largest |p_k| in the range of FaceFit32.
constexpr float kFitMax32 = (float)(FaceFit32::M / 12.566370614359172954);

// The face integral J = sum_n i^n h_n(d) / (n+2)! (normalised by twice the area) in
// binary32 from the polynomial P of exp(ix) fitted on [-P::M, P::M]: J = sum_n i^n
// a_n n! h_n(d) / (n+2)!, within P's fit error / 2 of the exact J for every
// triangle with max |d_k| <= P::M (the simplex average of the fit error).
template <class P>
__device__ __forceinline__ void face_integral_poly(float d0, float d1, float& jr, float& ji) {
  static_assert(P::N >= 5, "the first five terms are written out");
  const float d2 = -d0 - d1;
  const float e2 = d0 * d1 + d2 * (d0 + d1);
  const float e3 = d0 * d1 * d2;
  // H_0 = 1, H_1 = 0, H_2 = -e2, H_3 = e3, H_4 = e2^2, H_n = -e2 H_{n-2} + e3 H_{n-3}
  const float H2 = -e2, H3 = e3, H4 = e2 * e2;
  jr = P::cj[0] - P::cj[2] * H2;
  jr += P::cj[4] * H4;
  ji = -P::cj[3] * H3;
  float Hm3 = H2, Hm2 = H3, Hm1 = H4;
#pragma unroll
  for (int n = 5; n <= P::N; ++n) {
    const float H = -e2 * Hm2 + e3 * Hm3;
    const float c = P::cj[n];
    if ((n & 3) == 1) {
      ji += c * H;
    } else if ((n & 3) == 2) {
      jr -= c * H;
    } else if ((n & 3) == 3) {
      ji -= c * H;
    } else {
      jr += c * H;
    }
    Hm3 = Hm2;
    Hm2 = Hm1;
    Hm1 = H;
  }
}

// What one thread carries from face to face within a face range: the midpoint phase of the previous record's
// edge 1, in turns reduced to [-1/2, 1/2].
template <int NQ>
struct FwdCarry {
  float t[NQ];
  bool prev;             // there is a previous record in this range (uniform)
  __device__ __forceinline__ void reset() { prev = false; }
};

// Where a thread's origin phases come from. QLowLds: the Q as binary32 pairs Q = hi + lo with hi = (float)Q (the
// binary32 Q of the edge arithmetic) and lo = (float)(Q - hi), i.e. Q to 48 bits (relative error <= 2^-48), the low
// parts in a wavefront's slice of LDS (64 * 3 * NQ floats, lane-major so a wavefront's access is one conflict-free
// row) instead of nine registers: only the anchors, the chain starts and the small-|Q| fan read them. Each lane reads
// only what it wrote itself.
template <int NQ>
struct QLowLds {
  float* lo;  // this wavefront's slice
  int lane;
  __device__ __forceinline__ void set(int k, const double* Q, float hx, float hy, float hz) {
    lo[(k * 3 + 0) * 64 + lane] = (float)(Q[0] - (double)hx);
    lo[(k * 3 + 1) * 64 + lane] = (float)(Q[1] - (double)hy);
    lo[(k * 3 + 2) * 64 + lane] = (float)(Q[2] - (double)hz);
  }
  __device__ __forceinline__ double qd(float hi, int k, int j) const {
    return (double)hi + (double)lo[(k * 3 + j) * 64 + lane];
  }
  __device__ __forceinline__ float turns(int k, float hx, float hy, float hz, const double* gt) const {
    const double Q[3] = {qd(hx, k, 0), qd(hy, k, 1), qd(hz, k, 2)};
    return origin_turns_plain(Q, gt);
  }
};

// QReg: the binary64 Q themselves, for lists of few faces without a chain, where every pair forms its origin phase.
// wide: beyond the fixed-point range (per Q, so a Q's value does not depend on its wavefront; any_wide uniform).
template <int NQ>
struct QReg {
  double Q[NQ][3];
  bool wide[NQ];
  bool any_wide;
  __device__ __forceinline__ float turns(int k, float, float, float, const double* gt) const {
    float r = origin_turns(Q[k], gt);
    if (__builtin_expect(any_wide, 0)) r = wide[k] ? origin_turns_plain(Q[k], gt) : r;
    return r;
  }
};

// Orders a wavefront's LDS accesses around a tile it stages for itself: its stores are complete before
// any lane reads, and its earlier reads before it overwrites (a wavefront's LDS instructions execute in
// order; the fence also keeps the compiler from moving accesses across it).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Largest |Q| over the wavefront's lanes (every lane gets the same value).
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// Whether a centred vertex phase of a wavefront can exceed the fitted range: |d_k| <= |Q| rho for a face whose
// vertices lie within rho of its centroid. A wavefront that passes this test never meets a phase beyond
// FaceFit32::M (1e-3 of margin for rounding) and skips the per-lane test; each lane's value is the same either
// way.
__device__ __forceinline__ bool fit_range_test_needed(float qmax, double rho) {
  return (double)qmax * rho > 0.999 * FaceFit32::M;
}

// The face term beyond the fitted range (edge terms, above): T / (Q.N) = 1 / (16 pi^2 P) sum_k p_k c_k exp(2 pi i t_k)
// with t_k = r - p_k and c_k = 2 pi sinc of x_k = p_{k+1} - p_{k+2} (in turns, sin(2 pi x_k) from the exponentials
// already formed: x_k = t_{k+2} - t_{k+1}).
__device__ __forceinline__ void face_edge_term_fp32c(float r, float p0, float p1, float s, float P,
                                                     float& Tr, float& Ti) {
  constexpr float kInv16Pi2 = 0.0063325739776461107152f;
  const float p[3] = {p0, p1, -s};
  float c[3], cs[3], sn[3], t[3], x[3];
  bool wide = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    t[k] = r - p[k];
    x[k] = p[(k + 1) % 3] - p[(k + 2) % 3];
    c[k] = sinc2pi_poly(x[k]);
    wide |= fabsf(x[k]) > kSincPolyMax;
  }
  // the transcendentals in one run, as in the fitted form (12 faces x 128^3 Q: 72.6 -> 69.4 us)
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cs[k] = cos_turns(t[k]);
    sn[k] = sin_turns(t[k]);
  }
  const float rP = rcp_f(P);
  __builtin_amdgcn_sched_barrier(0);
  if (wide) {
    float rx[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) rx[k] = rcp_f(x[k]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int i = (k + 1) % 3, j = (k + 2) % 3;
      c[k] = fabsf(x[k]) > kSincPolyMax ? (sn[j] * cs[i] - sn[i] * cs[j]) * rx[k] : c[k];
    }
  }
  const float a0 = p[0] * c[0], a1 = p[1] * c[1], a2 = p[2] * c[2];
  const float co = kInv16Pi2 * rP;
  Tr = co * (a0 * cs[0] + a1 * cs[1] + a2 * cs[2]);
  Ti = co * (a0 * sn[0] + a1 * sn[1] + a2 * sn[2]);
}

// One face record against a thread's NQ Q points: adds each term to tr[k], ti[k]. CHECK: test each pair's phases
// against the fitted range; anchor: form the origin phase in binary64 even when the face is linked. `c` holds the
// previous record's edge-1 midpoint phase and gets this one's (SHARE only).
template <int NQ, bool SHARE, bool CHECK, class QL>
__device__ __forceinline__ void fwd_face_fp32c(const Face32& f, const float* qx, const float* qy, const float* qz,
                                               const QL& ql, float* tr, float* ti, bool anchor, FwdCarry<NQ>& c) {
  float QN[NQ], p0[NQ], p1[NQ], s[NQ], P[NQ], r[NQ], Tr[NQ], Ti[NQ];
  bool far[NQ];
  bool any = false, all = true;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    QN[k] = qx[k] * f.N[0] + qy[k] * f.N[1] + qz[k] * f.N[2];
    p0[k] = qx[k] * f.u0[0] + qy[k] * f.u0[1] + qz[k] * f.u0[2];
    p1[k] = qx[k] * f.u1[0] + qy[k] * f.u1[1] + qz[k] * f.u1[2];
    s[k] = p0[k] + p1[k];
    P[k] = p0[k] * s[k] + p1[k] * p1[k];
    if (CHECK) {
      far[k] = fmaxf(fabsf(p0[k]), fmaxf(fabsf(p1[k]), fabsf(s[k]))) > kFitMax32;
      any |= far[k];
      all &= far[k];
    }
  }
  const bool linked = SHARE && c.prev && (__builtin_amdgcn_readfirstlane(f.flags) & kFaceLinked) != 0u;
  if (linked && !anchor) {
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      r[k] = c.t[k] - s[k];
      c.t[k] = c.t[k] - (s[k] + p0[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      r[k] = ql.turns(k, qx[k], qy[k], qz[k], f.gt);
      if (SHARE) c.t[k] = r[k] - p0[k];
    }
  }
  if (!CHECK || !all) {  // some pair of this lane is in the fitted range
    float jr[NQ], ji[NQ], cf[NQ], sf[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const float E = p0[k] * p1[k] * s[k];
      const float w = E * E;
      jr[k] = horner_lit<FaceFit32::A1>(P[k]) * w + horner_lit<FaceFit32::A0>(P[k]);
      ji[k] = E * (horner_lit<FaceFit32::B1>(P[k]) * w + horner_lit<FaceFit32::B0>(P[k]));
    }
    // The face's transcendental instructions back to back: every switch between transcendental and ordinary
    // vector instructions costs issue cycles on this target.
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      cf[k] = cos_turns(r[k]);
      sf[k] = sin_turns(r[k]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      Tr[k] = cf[k] * ji[k] + sf[k] * jr[k];
      Ti[k] = sf[k] * ji[k] - cf[k] * jr[k];
    }
  }
  if (CHECK && __builtin_expect(any, 0)) {  // one branch per face for the lanes with a pair beyond it
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      float Xr, Xi;
      face_edge_term_fp32c(r[k], p0[k], p1[k], s[k], P[k], Xr, Xi);
      Tr[k] = far[k] ? Xr : Tr[k];
      Ti[k] = far[k] ? Xi : Ti[k];
    }
  }
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    tr[k] = fmaf(QN[k], Tr[k], tr[k]);
    ti[k] = fmaf(QN[k], Ti[k], ti[k]);
    if (SHARE) c.t[k] = c.t[k] - rintf(c.t[k]);
  }
  c.prev = true;
}

// One LDS tile of FP32C face records against the NQ Q points of a thread (plain binary32 sums inside the tile).
// SHARE: the records are in an edge-sharing order; `c` carries the shared edge's midpoint phase across faces and
// tiles of one face range (reset it at the range's start). The origin phase is formed in binary64 at every
// kAnchor-th face of a tile (of kTileF32 faces).
template <int NQ, bool SHARE, bool CHECK, class QL>
__device__ __forceinline__ void fwd_tile_fp32c(const Face32* tile, int nt, const float* qx, const float* qy,
                                               const float* qz, const QL& ql, float* tr, float* ti,
                                               FwdCarry<NQ>& c) {
  for (int j = 0; j < nt; ++j)
    fwd_face_fp32c<NQ, SHARE, CHECK>(tile[j], qx, qy, qz, ql, tr, ti, (j % kAnchor) == 0, c);
}

__device__ __forceinline__ void kahan_add(float& sum, float& comp, float x) {
  const float y = x - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

}  // namespace pft
