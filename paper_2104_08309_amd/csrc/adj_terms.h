// Per-(Q, face) terms of the adjoint (barycentric moments of each face),
// binary64 and FP32-compensated forms, shared by the single-mesh and batched
// kernels. The formulas are stated at the top of bwd3d.hip.
#pragma once

#include <type_traits>

#include "face_moments.h"
#include "pft_device.h"

namespace pft {

// ---------------------------------------------------------------------------
// binary64
// ---------------------------------------------------------------------------
PFT_HD __forceinline__ double dsinc_series(double x) {
  // d/dx sin(x)/x = sum_k (-1)^k 2k x^(2k-1) / (2k+1)!, |x| < 0.5
  const double x2 = x * x;
  return x * (-1.0 / 3.0 + x2 * (1.0 / 30.0 + x2 * (-1.0 / 840.0 + x2 * (1.0 / 45360.0 +
             x2 * (-1.0 / 3991680.0 + x2 * (1.0 / 518918400.0))))));
}

// Barycentric moments of a triangle from its centred vertex phases d0 + d1 + d2 = 0 (d_k = Q.(v_k - g)):
//   Y_k = sum_n i^n h_n(d0, d1, d2, d_k) / (n+3)!   (k = 0, 1),
//   J   = sum_n i^n h_n(d0, d1, d2) / (n+2)!         (so Y_2 = J - Y_0 - Y_1).
// They come from the fitted symmetric polynomials (face_moments.h) for max |d_k| <= kSeriesMaxPhase and from the
// edge form below beyond.
static_assert(FaceFit64::M == kSeriesMaxPhase && FaceFit32M::M == kSeriesMaxPhase, "fitted range of the moments");

// Edge form of the barycentric moments (|Q.(v - g)| beyond the series range):
// the moment of corner k relative to exp(iQ.g), normalised by 2A, is
// X_k * inv with inv = 1/|P|^2 (P = Q x N), and S is the face's edge sum, so
// that X_0 + X_1 + X_2 = i S and the normalised face integral is i S inv. The
// moments come from the closed-form Q-derivative of the edge sum.
__device__ __forceinline__ void edge_moments_f64(Fit64 t, const Face64& f, const double* G, double Px, double Py,
                                                 double Pz, double q0, double q1, double inv, double* Xr, double* Xi,
                                                 double& Sr, double& Si) {
  const double q2 = -q0 - q1;
  const double p0 = 0.5 * q0, p1 = 0.5 * q1, p2 = 0.5 * q2;
  double s0, c0, s1, c1;
  sincos_any64(t, p0, &s0, &c0);
  sincos_any64(t, p1, &s1, &c1);
  const double c2 = c0 * c1 - s0 * s1;
  const double s2 = -(s0 * c1 + c0 * s1);
  const double pi0 = Px * f.u0[0] + Py * f.u0[1] + Pz * f.u0[2];
  const double pi1 = Px * f.u1[0] + Py * f.u1[1] + Pz * f.u1[2];
  const double pi2 = -pi0 - pi1;
  const double w[3] = {pi1 - pi0, pi2 - pi1, pi0 - pi2};
  const double eta[3] = {p1 - p0, p2 - p1, p0 - p2};
  const double sn[3] = {s1 * c0 - c1 * s0, s2 * c1 - c2 * s1, s0 * c2 - c0 * s2};
  const double cs[3] = {c1 * c0 + s1 * s0, c2 * c1 + s2 * s1, c0 * c2 + s0 * s2};
  // e_l = exp(-i psi_{l+2})
  const double er[3] = {c2, c0, c1};
  const double ei[3] = {-s2, -s0, -s1};
  double ar[3], ai[3], br[3], bi[3], cr[3], ci[3];
  Sr = 0.0;
  Si = 0.0;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const double x = eta[l];
    double sg, dsg;
    if (fabs(x) < 0.1) {
      const double x2 = x * x;
      sg = 1.0 + x2 * (-1.0 / 6.0 + x2 * (1.0 / 120.0 + x2 * (-1.0 / 5040.0 + x2 * (1.0 / 362880.0))));
    } else {
      sg = sn[l] / x;
    }
    dsg = fabs(x) < 0.5 ? dsinc_series(x) : (cs[l] - sg) / x;
    cr[l] = sg * er[l];
    ci[l] = sg * ei[l];
    ar[l] = w[l] * cr[l];
    ai[l] = w[l] * ci[l];
    br[l] = w[l] * dsg * er[l];
    bi[l] = w[l] * dsg * ei[l];
    Sr += ar[l];
    Si += ai[l];
  }
  // Gram matrix of the edges, G = {d0.d0, d1.d1, d2.d2, d0.d1, d1.d2, d2.d0}
  const double Gm[3][3] = {{G[0], G[3], G[5]}, {G[3], G[1], G[4]}, {G[5], G[4], G[2]}};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kp = (k + 1) % 3, km = (k + 2) % 3;
    double xr = -0.5 * Si, xi = 0.5 * Sr;  // (i/2) S
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      xr += Gm[kp][l] * cr[l];
      xi += Gm[kp][l] * ci[l];
    }
    xr += 0.5 * (br[km] - br[k]);
    xi += 0.5 * (bi[km] - bi[k]);
    xr += 0.5 * ai[kp];   // -(i/2) a_{k+1}
    xi -= 0.5 * ar[kp];
    const double s = 2.0 * w[kp] * inv;
    Xr[k] = xr - s * Sr;
    Xi[k] = xi - s * Si;
  }
}

// The edge form's moments of one pair: X_k / |P|^2 for k = 0, 1 and the face integral J = i S / |P|^2. A record of a
// zero-area face (thr < 0) keeps its vertices, so its phases can lead here with P = 0: its moments are 0.
__device__ __forceinline__ void far_moments_f64(Fit64 t, const Face64& f, const double* G, const double* Q, double d0,
                                                double d1, double* yr, double* yi, double& jr, double& ji) {
  const double Px = Q[1] * f.N[2] - Q[2] * f.N[1];
  const double Py = Q[2] * f.N[0] - Q[0] * f.N[2];
  const double Pz = Q[0] * f.N[1] - Q[1] * f.N[0];
  const double inv = f.thr < 0.0 ? 0.0 : 1.0 / (Px * Px + Py * Py + Pz * Pz);
  double Xr[3], Xi[3], Sr, Si;
  edge_moments_f64(t, f, G, Px, Py, Pz, d0, d1, inv, Xr, Xi, Sr, Si);
  for (int k = 0; k < 2; ++k) yr[k] = Xr[k] * inv, yi[k] = Xi[k] * inv;
  jr = -Si * inv;
  ji = Sr * inv;
}

// One face against a thread's P Q points, binary64: with z = conj(g) exp(iQ.g), adds Re z(Y_0 - Y_2), Re z(Y_1 - Y_2)
// and Re(z J) to S (adj_block_sum turns their sums into the corners' Re(z Y_k)). With Y_k = alpha + beta d_k + gamma
// d_k^2, Y_0 - Y_2 = (d_0 - d_2)(beta - gamma d_1) and Y_1 - Y_2 = (d_1 - d_2)(beta - gamma d_0): three real
// combinations of the six fitted functions serve all corners and alpha drops out. The edge
// form beyond the fitted range; the choice is per lane. A zero-area face (N = 0; its phases need not be 0) gives finite
// weights that the vertex gather multiplies by N = 0. Bound by binary64 issue, about 160 instructions per pair against some 300 of
// the series in n (5 120 faces x 64 000 Q: kernel 3.41 -> 2.41 ms under the profiler, and fitting step 3.22 -> 3.08 ms
// with the differences in place of the corners); with P = 2 a coefficient is
// read once for two pairs (3 and 4 points: 9 % and 0.5 % slower fitting step, fewer wavefronts in flight).
// SHORT (uniform): every phase of the wavefront's Q is within FaceFit64S, two thirds of the coefficients and no range
// test (20 480 faces x 16 384 Q with phases to 0.7, transform and adjoint: 3.17 -> 2.92 ms). The forward has no such
// choice: a Q's value there must not depend on its wavefront, and forming both where a wavefront's Q lie on both sides
// cost more than it saved (5 120 faces x 64 000 Q, phases to 2.1: 3.15 -> 3.23 ms).
template <int P, bool SHORT>
__device__ __forceinline__ void adj_face_f64(const Face64& f, const double* G, const double (*Q)[3], const double* gr,
                                             const double* gi, bool big, double* S) {
  const Fit64 t = fit64();
  // the P points side by side: a coefficient is read once for all of them
  double d0[P], d1[P], zr[P], zi[P], A[P], B[P], bi[P], br[P], cr[P], ci[P];
  bool any = false;
#pragma unroll
  for (int k = 0; k < P; ++k) {
    d0[k] = Q[k][0] * f.u0[0] + Q[k][1] * f.u0[1] + Q[k][2] * f.u0[2];
    d1[k] = Q[k][0] * f.u1[0] + Q[k][1] * f.u1[1] + Q[k][2] * f.u1[2];
    const double phi = Q[k][0] * f.g[0] + Q[k][1] * f.g[1] + Q[k][2] * f.g[2];
    double sf, cf;
    if (__builtin_expect(big, 0))
      sincos_any64(t, phi, &sf, &cf);
    else
      sincos64(t, phi, &sf, &cf);
    zr[k] = gr[k] * cf + gi[k] * sf;
    zi[k] = gr[k] * sf - gi[k] * cf;
  }
#pragma unroll
  for (int k = 0; k < P; ++k) {
    const double s = d0[k] + d1[k];
    const double p = d0[k] * s + d1[k] * d1[k], E = d0[k] * d1[k] * s, w = E * E;
    if (!SHORT) any |= fmax(fabs(d0[k]), fmax(fabs(d1[k]), fabs(s))) > FaceFit64::M;
    using F = std::conditional_t<SHORT, FaceFit64S, FaceFit64>;
    face_ab64<F>(t, p, w, A[k], B[k]);
    face_beta_gamma64<F>(t, p, w, bi[k], br[k], cr[k], ci[k]);
    const double er = zr[k] * E, ei = zi[k] * E;
    const double a = zr[k] * A[k] - ei * B[k];           // Re(z J)
    const double b = er * br[k] - zi[k] * bi[k];         // Re(z beta)
    const double c = zr[k] * cr[k] - ei * ci[k];         // Re(z gamma)
    A[k] = a;
    B[k] = (d0[k] + s) * (b - c * d1[k]);
    bi[k] = (d1[k] + s) * (b - c * d0[k]);
  }
  if (!SHORT && any) {
#pragma unroll
    for (int k = 0; k < P; ++k)
      if (fmax(fabs(d0[k]), fmax(fabs(d1[k]), fabs(d0[k] + d1[k]))) > FaceFit64::M) {
        double yr[2], yi[2], jr, ji;
        far_moments_f64(t, f, G, Q[k], d0[k], d1[k], yr, yi, jr, ji);
        const double R0 = zr[k] * yr[0] - zi[k] * yi[0], R1 = zr[k] * yr[1] - zi[k] * yi[1];
        A[k] = zr[k] * jr - zi[k] * ji;
        const double R2 = A[k] - R0 - R1;
        B[k] = R0 - R2;
        bi[k] = R1 - R2;
      }
  }
#pragma unroll
  for (int k = 0; k < P; ++k) {
    S[0] += B[k];
    S[1] += bi[k];
    S[2] += A[k];
  }
}

// ---------------------------------------------------------------------------
// FP32-compensated
// ---------------------------------------------------------------------------
// sin(x)/x for |x| < 1 (Taylor series to x^10)
__device__ __forceinline__ float sinc_series_f(float x) {
  const float x2 = x * x;
  return 1.0f + x2 * (-1.0f / 6.0f + x2 * (1.0f / 120.0f + x2 * (-1.0f / 5040.0f + x2 * (1.0f / 362880.0f +
         x2 * (-1.0f / 39916800.0f)))));
}

// d/dx sin(x)/x for |x| < 1 (Taylor series to x^11)
__device__ __forceinline__ float dsinc_series_f(float x) {
  const float x2 = x * x;
  return x * (-1.0f / 3.0f + x2 * (1.0f / 30.0f + x2 * (-1.0f / 840.0f + x2 * (1.0f / 45360.0f +
             x2 * (-1.0f / 3991680.0f + x2 * (1.0f / 518918400.0f))))));
}

// Edge form of the barycentric moments in binary32, as edge_moments_f64:
// moment k (normalised by 2A, relative to exp(iQ.g)) = X_k * inv, inv = 1/|P|^2,
// and the face integral i S inv. Sinc and its derivative use their Taylor
// series for |x| < 1 (the hardware sine loses relative accuracy at small
// arguments) and quotients beyond.
__device__ __forceinline__ void edge_moments_fp32c(const Face32B& f, float Px, float Py, float Pz, float q0, float q1,
                                                   float inv, float* Xr, float* Xi, float& Sr, float& Si) {
  const float w0 = Px * f.d0[0] + Py * f.d0[1] + Pz * f.d0[2];
  const float w1 = Px * f.d1[0] + Py * f.d1[1] + Pz * f.d1[2];
  const float w[3] = {w0, w1, -w0 - w1};
  const float p0 = q0 * (0.5f * kInv2PiF), p1 = q1 * (0.5f * kInv2PiF), p2 = -p0 - p1;  // psi_k in turns
  const float s0 = sin_turns(p0), c0 = cos_turns(p0);
  const float s1 = sin_turns(p1), c1 = cos_turns(p1);
  const float c2 = c0 * c1 - s0 * s1;
  const float s2 = -(s0 * c1 + c0 * s1);
  const float eta[3] = {p1 - p0, p2 - p1, p0 - p2};  // turns
  const float cs[3] = {c1 * c0 + s1 * s0, c2 * c1 + s2 * s1, c0 * c2 + s0 * s2};
  const float er[3] = {c2, c0, c1};
  const float ei[3] = {-s2, -s0, -s1};
  float ar[3], ai[3], br[3], bi[3], cr[3], ci[3];
  Sr = 0.0f;
  Si = 0.0f;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const float xt = eta[l];
    const float x = kTwoPiF * xt;                  // radians
    const float rx = rcp_f(xt) * kInv2PiF;         // 1/x
    const bool near0 = fabsf(x) < 1.0f;
    const float sg = near0 ? sinc_series_f(x) : sin_turns(xt) * rx;
    const float dsg = near0 ? dsinc_series_f(x) : (cs[l] - sg) * rx;
    cr[l] = sg * er[l];
    ci[l] = sg * ei[l];
    ar[l] = w[l] * cr[l];
    ai[l] = w[l] * ci[l];
    const float wd = w[l] * dsg;
    br[l] = wd * er[l];
    bi[l] = wd * ei[l];
    Sr += ar[l];
    Si += ai[l];
  }
  const float Gm[3][3] = {{f.G[0], f.G[3], f.G[5]}, {f.G[3], f.G[1], f.G[4]}, {f.G[5], f.G[4], f.G[2]}};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int kp = (k + 1) % 3, km = (k + 2) % 3;
    float xr = -0.5f * Si, xi = 0.5f * Sr;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      xr += Gm[kp][l] * cr[l];
      xi += Gm[kp][l] * ci[l];
    }
    xr += 0.5f * (br[km] - br[k]);
    xi += 0.5f * (bi[km] - bi[k]);
    xr += 0.5f * ai[kp];
    xi -= 0.5f * ar[kp];
    const float s = 2.0f * w[kp] * inv;
    Xr[k] = xr - s * Sr;
    Xi[k] = xi - s * Si;
  }
}

// The edge form's moments of one pair in binary32: Y_0, Y_1 and J relative to exp(iQ.g).
__device__ __forceinline__ void far_moments_fp32c(const Face32B& f, float qx, float qy, float qz, float d0, float d1,
                                                  float* yr, float* yi, float& jr, float& ji) {
  const float Px = qy * f.N[2] - qz * f.N[1];
  const float Py = qz * f.N[0] - qx * f.N[2];
  const float Pz = qx * f.N[1] - qy * f.N[0];
  const float inv = rcp_f(fmaxf(Px * Px + Py * Py + Pz * Pz, 1e-30f));
  float Xr[3], Xi[3], Sr, Si;
  edge_moments_fp32c(f, Px, Py, Pz, d0, d1, inv, Xr, Xi, Sr, Si);
  for (int k = 0; k < 2; ++k) yr[k] = Xr[k] * inv, yi[k] = Xi[k] * inv;
  jr = -Si * inv;
  ji = Sr * inv;
}

// One face against a thread's P Q points in binary32, the sums of adj_face_f64. Bound by FP32 issue: per pair 12
// operations for the phases and their symmetric functions, 32 for the six fitted functions, 17 for the products and
// sums, 2 transcendentals and 3 binary64 multiply-adds (origin_turns); the one-variable recurrences it replaced took
// some 15 more (5 120 faces x 262 144 Q: fitting step 3.21 -> 3.09 ms; 6 400 x 91 125 with grad_Q 3.67 -> 3.26 ms). An empty face has an all-zero record: finite
// weights, times N = 0 in the vertex gather.
template <int P>
__device__ __forceinline__ void adj_face_fp32c(const Face32B& f, const float* qx, const float* qy, const float* qz,
                                               const double (*Qd)[3], const float* gr, const float* gi, bool wide,
                                               float* S) {
  float d0[P], d1[P], zr[P], zi[P], a[P], D0[P], D1[P], r[P], cf[P], sf[P];
  bool any = false;
#pragma unroll
  for (int k = 0; k < P; ++k) r[k] = wide ? origin_turns_plain(Qd[k], f.gt) : origin_turns(Qd[k], f.gt);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < P; ++k) {
    cf[k] = cos_turns(r[k]);
    sf[k] = sin_turns(r[k]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < P; ++k) {
    zr[k] = gr[k] * cf[k] + gi[k] * sf[k];
    zi[k] = gr[k] * sf[k] - gi[k] * cf[k];
    d0[k] = qx[k] * f.u0[0] + qy[k] * f.u0[1] + qz[k] * f.u0[2];
    d1[k] = qx[k] * f.u1[0] + qy[k] * f.u1[1] + qz[k] * f.u1[2];
    const float s = d0[k] + d1[k];
    const float p = d0[k] * s + d1[k] * d1[k], E = d0[k] * d1[k] * s, w = E * E;
    any |= fmaxf(fabsf(d0[k]), fmaxf(fabsf(d1[k]), fabsf(s))) > (float)FaceFit32M::M;
    const Moments32 m = face_moments32(p, w);
    const float er = zr[k] * E, ei = zi[k] * E;
    a[k] = zr[k] * m.A - ei * m.B;                 // Re(z J)
    const float b = er * m.br - zi[k] * m.bi;      // Re(z beta)
    const float c = zr[k] * m.gr - ei * m.gi;      // Re(z gamma)
    D0[k] = (d0[k] + s) * (b - c * d1[k]);
    D1[k] = (d1[k] + s) * (b - c * d0[k]);
  }
  if (__builtin_expect(any, 0)) {
#pragma unroll
    for (int k = 0; k < P; ++k)
      if (fmaxf(fabsf(d0[k]), fmaxf(fabsf(d1[k]), fabsf(d0[k] + d1[k]))) > (float)FaceFit32M::M) {
        float yr[2], yi[2], jr, ji;
        far_moments_fp32c(f, qx[k], qy[k], qz[k], d0[k], d1[k], yr, yi, jr, ji);
        const float R0 = zr[k] * yr[0] - zi[k] * yi[0], R1 = zr[k] * yr[1] - zi[k] * yi[1];
        a[k] = zr[k] * jr - zi[k] * ji;
        const float R2 = a[k] - R0 - R1;
        D0[k] = R0 - R2;
        D1[k] = R1 - R2;
      }
  }
#pragma unroll
  for (int k = 0; k < P; ++k) {
    S[0] += D0[k];
    S[1] += D1[k];
    S[2] += a[k];
  }
}

// ---------------------------------------------------------------------------
// Wavefront sum in binary64 (shuffles through the LDS crossbar).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum over a block of NT threads in binary64 and a fixed order; every thread
// must call it and every thread gets the total. lds holds NT / 64 doubles.
template <int NT>
__device__ __forceinline__ double block_total(double v, double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_total(v);
  __syncthreads();
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) t += lds[w];
  return t;
}

// ---------------------------------------------------------------------------
// binary64 adjoint, one block's share: `nt` face records in LDS (with their
// edge Gram matrices) against the reordered Q records [qb, qe), P Q per
// thread per pass. Each thread adds its weights for face j to its own
// binary64 slots acc[3 j + k][thread] (zeroed by the caller); adj_block_sum
// reduces the slots once the range is done.
// ---------------------------------------------------------------------------
template <int P>
__device__ __forceinline__ void adj_tile_f64(const Face64* tile, const double (*gtile)[8], int nt, int64_t qb,
                                             int64_t qe, const QRec64* __restrict__ rec, const MeshInfo& info,
                                             double (*acc)[kBlock]) {
  const int tid = threadIdx.x;
  for (int64_t q0 = qb; q0 < qe; q0 += (int64_t)kBlock * P) {
    double Qd[P][3];
    double hr[P], hi[P];
    bool big = false, brief = true;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int64_t qi = q0 + (int64_t)p * kBlock + tid;
      Qd[p][0] = Qd[p][1] = Qd[p][2] = 0.0;
      hr[p] = hi[p] = 0.0;
      if (qi < qe) {
        const QRec64 r = rec[qi];
        Qd[p][0] = r.q[0];
        Qd[p][1] = r.q[1];
        Qd[p][2] = r.q[2];
        hr[p] = r.hr;
        hi[p] = r.hi;
      }
      const double q2 = Qd[p][0] * Qd[p][0] + Qd[p][1] * Qd[p][1] + Qd[p][2] * Qd[p][2];
      big |= big_phases64(q2, info.R);
      brief &= short_phases64(q2, info.rho);
    }
    brief = __all(brief) != 0;
#pragma unroll 1
    for (int j = 0; j < nt; ++j) {
      double S[3] = {0.0, 0.0, 0.0};
      if (brief)
        adj_face_f64<P, true>(tile[j], gtile[j], Qd, hr, hi, big, S);
      else
        adj_face_f64<P, false>(tile[j], gtile[j], Qd, hr, hi, big, S);
#pragma unroll
      for (int k = 0; k < 3; ++k) acc[3 * j + k][tid] += S[k];
    }
  }
}

// ---------------------------------------------------------------------------
// FP32C adjoint, one block's share: `nt` face records in LDS against the
// reordered Q records [qb, qe), P Q per thread per pass. Each thread adds
// its weights for face j to its own binary32 slots acc[3 j + k][thread] (zeroed
// by the caller); adj_block_sum32 reduces the slots once the range is done, so
// no cross-lane traffic happens per face.
// ---------------------------------------------------------------------------
template <int P>
__device__ __forceinline__ void adj_tile_fp32c(const Face32B* tile, int nt, int64_t qb, int64_t qe,
                                               const QRec32* __restrict__ rec, double R, float (*acc)[kBlock]) {
  const int tid = threadIdx.x;
  for (int64_t q0 = qb; q0 < qe; q0 += (int64_t)kBlock * P) {
    double Qd[P][3];
    float qx[P], qy[P], qz[P], hr[P], hi[P];
    bool wide = false;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int64_t qi = q0 + (int64_t)p * kBlock + tid;
      Qd[p][0] = Qd[p][1] = Qd[p][2] = 0.0;
      hr[p] = hi[p] = 0.0f;
      if (qi < qe) {
        const QRec32 r = rec[qi];
        Qd[p][0] = r.q[0];
        Qd[p][1] = r.q[1];
        Qd[p][2] = r.q[2];
        hr[p] = r.hr;
        hi[p] = r.hi;
      }
      qx[p] = (float)Qd[p][0];
      qy[p] = (float)Qd[p][1];
      qz[p] = (float)Qd[p][2];
      wide |= wide_phases32(Qd[p][0] * Qd[p][0] + Qd[p][1] * Qd[p][1] + Qd[p][2] * Qd[p][2], R);
    }
#pragma unroll 1
    for (int j = 0; j < nt; ++j) {
      float S[3] = {0.0f, 0.0f, 0.0f};
      adj_face_fp32c<P>(tile[j], qx, qy, qz, Qd, hr, hi, wide, S);
      // private slots: a plain read-modify-write (an LDS atomic add is far slower)
#pragma unroll
      for (int k = 0; k < 3; ++k) acc[3 * j + k][tid] += S[k];
    }
  }
}

// Sum of the per-thread slots of adj_tile_fp32c / adj_tile_f64 for each of the nt faces, in binary64 and a fixed
// order; wave w handles faces w, w + 4, ... and lane 0 writes the corner weights out[3 j + k]: from the sums D_0, D_1
// of Re z(Y_0 - Y_2), Re z(Y_1 - Y_2) and a of Re(z J) = Re z(Y_0 + Y_1 + Y_2). Call after a barrier.
template <typename T>
__device__ __forceinline__ void adj_block_sum(T (*acc)[kBlock], int nt, double* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int j = wave; j < nt; j += kBlock / 64) {
    double x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[k] = 0.0;
#pragma unroll
      for (int i = 0; i < kBlock / 64; ++i) x[k] += (double)acc[3 * j + k][lane + 64 * i];
      x[k] = wave_total(x[k]);
    }
    if (lane == 0) {
      const double R2 = (x[2] - x[0] - x[1]) * (1.0 / 3.0);
      out[3 * j] = R2 + x[0];
      out[3 * j + 1] = R2 + x[1];
      out[3 * j + 2] = R2;
    }
  }
}

}  // namespace pft
