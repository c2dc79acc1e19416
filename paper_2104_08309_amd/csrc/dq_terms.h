// Per-(Q, face) terms of grad_Q F, binary64 and FP32-compensated forms.
//
// grad_Q F = i * volume integral of r exp(iQ.r). With the field
// x_a (-iQ/|Q|^2) exp(iQ.r), whose divergence is x_a exp(iQ.r) - iQ_a exp(iQ.r)/|Q|^2,
// the divergence theorem turns the volume integral into face integrals of
// r exp(iQ.r) plus (iQ/|Q|^2) F; r is linear on a face, r = sum_k lambda_k v_k,
// so the face integral of r exp(iQ.r) is sum_k v_k times the barycentric
// moment of corner k (the moments of the vertex adjoint). In coordinates
// centred on the mesh centre t, with c_m = (Q.N_m) exp(iQ.g_m) and the moments
// Y_k normalised by 2A relative to exp(iQ.g_m) (J = Y_0 + Y_1 + Y_2):
//   A = sum_m c_m sum_k (v_k - t) Y_k,   B = sum_m c_m J,
//   F_c = -i B / |Q|^2,   grad F_c = (A + iQ B / |Q|^2) / |Q|^2,
//   grad F = exp(iQ.t) (grad F_c + i t F_c).
// The two parts cancel as (|Q| R)^-2 at small |Q| R; there the tetrahedra
// (t, a, b, c) give F_c and grad F_c directly by their series.
#pragma once

#include "adj_terms.h"

namespace pft {

// Tetrahedron with one vertex at the origin and vertex phases x = (x_a, x_b, x_c):
//   S   = sum_n i^n h_n(x_a, x_b, x_c) / (n+3)!,
//   T_k = sum_n i^n h_n(x_a, x_b, x_c, x_k) / (n+4)!   (node k doubled),
// so the integral of exp(iQ.r) over it is 6|T| S and that of lambda_k exp(iQ.r)
// is 6|T| T_k. H_n = h_n(x_a, x_b, x_c) = e1 H_{n-1} - e2 H_{n-2} + e3 H_{n-3} and
// h_n(x, x_k) = H_n + x_k h_{n-1}(x, x_k). Both terms of index n are below
// m^n / n! (m = max |x|); four terms are added per step until that bound on
// the next index is below 1e-18 (the sums are near 1/6 and 1/24 here).
PFT_HD inline void tet_moments_f64(const double* x, double& sr, double& si, double* tr, double* ti) {
  const double e1 = x[0] + x[1] + x[2];
  const double e2 = x[0] * x[1] + x[0] * x[2] + x[1] * x[2];
  const double e3 = x[0] * x[1] * x[2];
  const double m = fmax(fabs(x[0]), fmax(fabs(x[1]), fabs(x[2])));
  const double m4 = (m * m) * (m * m);
  double Hm3 = 0.0, Hm2 = 0.0, Hm1 = 1.0;  // H_{n-3}, H_{n-2}, H_{n-1} at n = 1
  double a[3] = {1.0, 1.0, 1.0};           // h_{n-1}(x, x_k) at n = 1
  sr = 1.0 / 6.0;
  si = 0.0;
  for (int k = 0; k < 3; ++k) tr[k] = 1.0 / 24.0, ti[k] = 0.0;
  double mn = m;  // m^n at the start of each step
  for (int n = 1; n < 85; n += 4) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double H = e1 * Hm1 - e2 * Hm2 + e3 * Hm3;
      const double cs = inv_fact(n + r + 3), ct = inv_fact(n + r + 4);
#pragma unroll
      for (int k = 0; k < 3; ++k) a[k] = H + x[k] * a[k];
      // i^(n+r) with n = 1 (mod 4): +i, -1, -i, +1
      if (r == 0) {
        si += cs * H;
        for (int k = 0; k < 3; ++k) ti[k] += ct * a[k];
      } else if (r == 1) {
        sr -= cs * H;
        for (int k = 0; k < 3; ++k) tr[k] -= ct * a[k];
      } else if (r == 2) {
        si -= cs * H;
        for (int k = 0; k < 3; ++k) ti[k] -= ct * a[k];
      } else {
        sr += cs * H;
        for (int k = 0; k < 3; ++k) tr[k] += ct * a[k];
      }
      Hm3 = Hm2;
      Hm2 = Hm1;
      Hm1 = H;
    }
    mn *= m4;
    if (mn * inv_fact(n + 4) < 1e-18) break;
  }
}

// Small |Q| R: the tetrahedron (o, a, b, c) of face F (o an apex relative to t) adds 6|T| S to F and
// i sum_k v_k 6|T| T_k to grad F, both about o (dq_apex moves them to t).
PFT_HD __forceinline__ void dq_tet_f64(const Face64& F, const double* Q, double* Gr, double* Gi, double& Fr,
                                       double& Fi, const double* o) {
  double v[3][3];
  for (int c = 0; c < 3; ++c) {
    v[0][c] = F.g[c] + F.u0[c] - o[c];
    v[1][c] = F.g[c] + F.u1[c] - o[c];
    v[2][c] = F.g[c] - F.u0[c] - F.u1[c] - o[c];
  }
  const double six_v = F.N[0] * v[0][0] + F.N[1] * v[0][1] + F.N[2] * v[0][2];
  double x[3];
  for (int k = 0; k < 3; ++k) x[k] = Q[0] * v[k][0] + Q[1] * v[k][1] + Q[2] * v[k][2];
  double sr, si, tr[3], ti[3];
  tet_moments_f64(x, sr, si, tr, ti);
  Fr += six_v * sr;
  Fi += six_v * si;
  for (int c = 0; c < 3; ++c) {
    const double mr = v[0][c] * tr[0] + v[1][c] * tr[1] + v[2][c] * tr[2];
    const double mi = v[0][c] * ti[0] + v[1][c] * ti[1] + v[2][c] * ti[2];
    Gr[c] -= six_v * mi;  // i (mr + i mi)
    Gi[c] += six_v * mr;
  }
}

// The fan sums about an apex o, moved to coordinates about t: F = exp(iQ.o) F_o and
// grad F = exp(iQ.o) (grad F_o + i o F_o).
PFT_HD __forceinline__ void dq_apex(const double* Q, const double* o, double* Gr, double* Gi, double& Fr,
                                    double& Fi) {
  double so, co;
  sincos(Q[0] * o[0] + Q[1] * o[1] + Q[2] * o[2], &so, &co);
  for (int c = 0; c < 3; ++c) {
    const double ur = Gr[c] - o[c] * Fi, ui = Gi[c] + o[c] * Fr;
    Gr[c] = co * ur - so * ui;
    Gi[c] = co * ui + so * ur;
  }
  const double fr = co * Fr - so * Fi;
  Fi = co * Fi + so * Fr;
  Fr = fr;
}

// binary64 surface term of face f: A += c sum_k (v_k - t) Y_k, B += c J. (A zero-area face has N = 0 and finite
// moments: it adds 0.)
__device__ __forceinline__ void dq_term_f64(const Face64& f, const double* G, const double* Q, bool big, double* Ar,
                                            double* Ai, double& Br, double& Bi) {
  const Fit64 t = fit64();
  double sf, cf;
  const double phi = Q[0] * f.g[0] + Q[1] * f.g[1] + Q[2] * f.g[2];
  if (__builtin_expect(big, 0))
    sincos_any64(t, phi, &sf, &cf);
  else
    sincos64(t, phi, &sf, &cf);
  const double QN = Q[0] * f.N[0] + Q[1] * f.N[1] + Q[2] * f.N[2];
  const double q0 = Q[0] * f.u0[0] + Q[1] * f.u0[1] + Q[2] * f.u0[2];
  const double q1 = Q[0] * f.u1[0] + Q[1] * f.u1[1] + Q[2] * f.u1[2];
  double yr[2], yi[2], jr, ji;
  bary_moments_fit64(t, q0, q1, yr, yi, jr, ji);
  if (fmax(fabs(q0), fmax(fabs(q1), fabs(q0 + q1))) > FaceFit64::M) far_moments_f64(t, f, G, Q, q0, q1, yr, yi, jr, ji);
  const double cr = QN * cf, ci = QN * sf;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    // v_2 - t, v_0 - v_2 and v_1 - v_2 (Y_2 = J - Y_0 - Y_1)
    const double p2 = f.g[c] - f.u0[c] - f.u1[c];
    const double e0 = 2.0 * f.u0[c] + f.u1[c];
    const double e1 = f.u0[c] + 2.0 * f.u1[c];
    const double vr = p2 * jr + e0 * yr[0] + e1 * yr[1];
    const double vi = p2 * ji + e0 * yi[0] + e1 * yi[1];
    Ar[c] += cr * vr - ci * vi;
    Ai[c] += cr * vi + ci * vr;
  }
  Br += cr * jr - ci * ji;
  Bi += cr * ji + ci * jr;
}

// FP32C surface term of face f (record of the FP32C adjoint), the same sums in binary32 as
//   sum_k (v_k - t) Y_k = g J + u_0 (Y_0 - Y_2) + u_1 (Y_1 - Y_2),
// with the differences in the adjoint's form (d_0 - d_2)(beta - gamma d_1), (d_1 - d_2)(beta - gamma d_0). (An empty
// face has an all-zero record: N = 0 makes its terms 0.)
__device__ __forceinline__ void dq_term_fp32c(const Face32B& f, float qx, float qy, float qz, const double* Qd,
                                              bool wide, float* Ar, float* Ai, float& Br, float& Bi) {
  const float r = wide ? origin_turns_plain(Qd, f.gt) : origin_turns(Qd, f.gt);
  const float cf = cos_turns(r), sf = sin_turns(r);
  const float QN = qx * f.N[0] + qy * f.N[1] + qz * f.N[2];
  const float d0 = qx * f.u0[0] + qy * f.u0[1] + qz * f.u0[2];
  const float d1 = qx * f.u1[0] + qy * f.u1[1] + qz * f.u1[2];
  const float s = d0 + d1;
  const float p = d0 * s + d1 * d1, E = d0 * d1 * s, w = E * E;
  const Moments32 m = face_moments32(p, w);
  float jr = m.A, ji = E * m.B;
  const float br = E * m.br, gi = E * m.gi;
  const float t0 = d0 + s, t1 = d1 + s;
  float ur = t0 * (br - m.gr * d1), ui = t0 * (m.bi - gi * d1);   // Y_0 - Y_2
  float vr = t1 * (br - m.gr * d0), vi = t1 * (m.bi - gi * d0);   // Y_1 - Y_2
  if (__builtin_expect(fmaxf(fabsf(d0), fmaxf(fabsf(d1), fabsf(s))) > (float)FaceFit32M::M, 0)) {
    float yr[2], yi[2];
    far_moments_fp32c(f, qx, qy, qz, d0, d1, yr, yi, jr, ji);
    const float y2r = jr - yr[0] - yr[1], y2i = ji - yi[0] - yi[1];
    ur = yr[0] - y2r;
    ui = yi[0] - y2i;
    vr = yr[1] - y2r;
    vi = yi[1] - y2i;
  }
  // times c = (Q.N) exp(iQ.g)
  const float cr = QN * cf, ci = QN * sf;
  const float Jr = cr * jr - ci * ji, Ji = cr * ji + ci * jr;
  const float Ur = cr * ur - ci * ui, Ui = cr * ui + ci * ur;
  const float Vr = cr * vr - ci * vi, Vi = cr * vi + ci * vr;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    Ar[c] += f.g[c] * Jr + f.u0[c] * Ur + f.u1[c] * Vr;
    Ai[c] += f.g[c] * Ji + f.u0[c] * Ui + f.u1[c] * Vi;
  }
  Br += Jr;
  Bi += Ji;
}

}  // namespace pft
