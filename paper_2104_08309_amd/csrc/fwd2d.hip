// Forward 2D transform of a polygon (one or more closed contours), binary64.
//
// 2D section of the paper: with the field F = -iQ exp(iQ.r)/Q^2 (whose
// divergence is exp(iQ.r)), the area integral becomes a sum over contour
// edges of the flux through each edge (eq. line_integral_generic), whose
// exponential difference is written in midpoint form as
//   (exp(iQ.r_{l+1}) - exp(iQ.r_l)) / (Q.d_l) = i exp(iQ.m_l) sinc(Q.d_l/2),
// and with (Q.n_l)|d_l| = Qx dy - Qy dx for the outward normal of a
// counter-clockwise edge (eq. line_normal):
//   F(Q) = -(i/|Q|^2) sum_l (Qx dy_l - Qy dx_l) exp(iQ.m_l) sinc(Q.d_l/2).
// Coordinates are relative to the vertex mean t; F gets exp(iQ.t) at the end.
// For |Q| R < tau0 the area is summed as the fan of triangles (t, r_l, r_{l+1})
// through their simplex series, which is exact at Q = 0 (signed area).
//
// The sines are the binary64 kernels' own (face_moments.h) up to their range, and sinc is the same polynomial without a
// division up to pi/4; a polygon of one contour and at most one LDS tile needs no prologue launches, every block forms
// the centre and the edges itself. 64 edges x 128^2 Q: 17.6 -> 11.0 us a call,
// x 2^18 Q: 99 -> 53. Short lists are bound by latency (one launch; the host's call takes as long), long ones by
// binary64 issue.
#include "face_moments.h"
#include "pft_device.h"

namespace pft {
namespace {

// Block layout: kBlock / GROUPS Q points x GROUPS edge groups; the thread of (Q, group g) sums the edges
// g, g + GROUPS, ... of each LDS tile, and the groups' sums are added in the order g = 0, 1, ..., so that a polygon of a
// few dozen edges still gives every CU several waves: eight groups. Two where the Q alone do that, for fewer blocks and
// less idling on polygons of few edges (2^18 Q, eight -> two: 4 edges 26.1 -> 11.7 us, 64 edges 61 -> 53, 256 edges
// 157 -> 149); not with the prologue, where it loses (1 000 edges 497 -> 525).
constexpr int kGroups2D = 8, kGroups2DLong = 2;
constexpr int64_t kLongNq2D = 1 << 17;

// WIDE: phases beyond the range of sincos64, through the library's functions.
template <bool WIDE>
__device__ __forceinline__ void edge_term_2d(Fit64 fit, const Edge2D& e, double Qx, double Qy, double& xr, double& xi) {
  const double dx = e.b[0] - e.a[0], dy = e.b[1] - e.a[1];
  const double mx = 0.5 * (e.a[0] + e.b[0]), my = 0.5 * (e.a[1] + e.b[1]);
  const double eta = 0.5 * (Qx * dx + Qy * dy);
  const double z = eta * eta;
  double sinc, sm, cm;
  if (z <= 0.61685027506808487) {  // |eta| <= pi/4, where S is the fit of (sin x - x) / x^3
    sinc = 1.0 + z * horner64<SinCos64::S>(fit, z);
  } else if (WIDE) {
    sinc = sin(eta) / eta;
  } else {
    sincos64(fit, eta, &sm, &cm);
    sinc = sm / eta;
  }
  const double ph = Qx * mx + Qy * my;
  if (WIDE)
    sincos(ph, &sm, &cm);
  else
    sincos64(fit, ph, &sm, &cm);
  const double wgt = (Qx * dy - Qy * dx) * sinc;
  // -i * wgt * exp(i Q.m)
  xr += wgt * sm;
  xi -= wgt * cm;
}

// Triangle (t, a, b) of the fan by its simplex series: 2 |T| sum_n i^n h_n(0, Q.a, Q.b) / (n+2)!, to n = 6: with
// |Q.a|, |Q.b| < kTau02D the next term is under 8 tau^7 / 9! = 2.3e-19. (The loop to convergence that this was divides
// once a term: one such Q in a wavefront took 64 edges x 2^14 random Q from 10.5 to 19 us.)
static_assert(kTau02D <= 0.01, "the series below is cut for it");
__device__ __forceinline__ void fan_term_2d(const Edge2D& e, double Qx, double Qy, double& xr, double& xi) {
  const double two_a = e.a[0] * e.b[1] - e.a[1] * e.b[0];
  const double xa = Qx * e.a[0] + Qy * e.a[1];
  const double xb = Qx * e.b[0] + Qy * e.b[1];
  // h_n = e1 h_{n-1} - e2 h_{n-2}
  const double e1 = xa + xb, e2 = xa * xb;
  const double h2 = e1 * e1 - e2, h3 = e1 * h2 - e2 * e1;
  const double h4 = e1 * h3 - e2 * h2, h5 = e1 * h4 - e2 * h3, h6 = e1 * h5 - e2 * h4;
  xr += two_a * (0.5 + (h2 * (-1.0 / 24.0) + (h4 * (1.0 / 720.0) + h6 * (-1.0 / 40320.0))));
  xi += two_a * (e1 * (1.0 / 6.0) + (h3 * (-1.0 / 120.0) + h5 * (1.0 / 5040.0)));
}

// The centre t and radius R of a contour of nv <= kTileE vertices, and its edges about t in LDS. Each wavefront reads
// all vertices, so the sums need no barrier. Ends with a barrier.
__device__ __forceinline__ void own_edges(const double* verts, int nv, Edge2D* tile, double* t, double& R) {
  static_assert(kTileE == kBlock, "a vertex per thread");
  const int tid = threadIdx.x, lane = tid & 63;
  double px[kTileE / 64], py[kTileE / 64], sx = 0.0, sy = 0.0, r2 = 0.0;
#pragma unroll
  for (int k = 0; k < kTileE / 64; ++k) {
    const int i = k * 64 + lane;
    px[k] = i < nv ? verts[2 * i] : 0.0;
    py[k] = i < nv ? verts[2 * i + 1] : 0.0;
    sx += px[k];
    sy += py[k];
  }
  for (int d = 32; d > 0; d >>= 1) {
    sx += __shfl_xor(sx, d);
    sy += __shfl_xor(sy, d);
  }
  t[0] = sx / (double)nv;
  t[1] = sy / (double)nv;
  double ax = 0.0, ay = 0.0;
#pragma unroll
  for (int k = 0; k < kTileE / 64; ++k) {
    px[k] -= t[0];
    py[k] -= t[1];
    if (k * 64 + lane < nv) r2 = fmax(r2, px[k] * px[k] + py[k] * py[k]);
    if (k == tid / 64) {
      ax = px[k];
      ay = py[k];
    }
  }
  for (int d = 32; d > 0; d >>= 1) r2 = fmax(r2, __shfl_xor(r2, d));
  R = sqrt(r2);
  if (tid < nv) {
    Edge2D& e = tile[tid];
    Edge2D& p = tile[tid > 0 ? tid - 1 : nv - 1];
    e.a[0] = p.b[0] = ax;
    e.a[1] = p.b[1] = ay;
  }
  __syncthreads();
}

// OWN: `verts` is one contour of at most kTileE vertices; the edges and the centre come from it. Else from `edges` and
// `info`, the prologue's.
template <bool OWN, int GROUPS>
__global__ __launch_bounds__(kBlock) void fwd2d_kernel(const double* verts, const Edge2D* edges, int64_t ne,
                                                       const MeshInfo* info, const double* q, int64_t nq, double tau0,
                                                       double* out) {
  __shared__ Edge2D tile[kTileE];
  constexpr int kQ2D = kBlock / GROUPS;
  __shared__ double2 part[GROUPS][kQ2D];
  const int lq = threadIdx.x % kQ2D, grp = threadIdx.x / kQ2D;
  const int64_t qi = (int64_t)blockIdx.x * kQ2D + lq;
  const bool active = qi < nq;
  const double Qx = active ? q[2 * qi] : 0.0;
  const double Qy = active ? q[2 * qi + 1] : 0.0;
  const double Q2 = Qx * Qx + Qy * Qy;
  const Fit64 fit = fit64();
  double t[2], R;
  if constexpr (OWN) {
    own_edges(verts, (int)ne, tile, t, R);
  } else {
    t[0] = info[0].t[0];
    t[1] = info[0].t[1];
    R = info[0].R;
  }
  const bool small = active && sqrt(Q2) * R < tau0, wide = big_phases64(Q2, R);
  double xr = 0.0, xi = 0.0;
  for (int64_t t0 = 0; t0 < ne; t0 += kTileE) {
    const int nt = (int)min((int64_t)kTileE, ne - t0);
    if constexpr (!OWN) {
      __syncthreads();
      for (int i = threadIdx.x; i < nt * 2; i += kBlock)
        reinterpret_cast<uint4*>(tile)[i] = reinterpret_cast<const uint4*>(edges + t0)[i];
      __syncthreads();
    }
    if (small) {
      for (int j = grp; j < nt; j += GROUPS) fan_term_2d(tile[j], Qx, Qy, xr, xi);
    } else if (__builtin_expect(wide, 0)) {
      for (int j = grp; j < nt; j += GROUPS) edge_term_2d<true>(fit, tile[j], Qx, Qy, xr, xi);
    } else {
      for (int j = grp; j < nt; j += GROUPS) edge_term_2d<false>(fit, tile[j], Qx, Qy, xr, xi);
    }
  }
  part[grp][lq] = make_double2(xr, xi);
  __syncthreads();
  if (grp != 0 || !active) return;
  xr = xi = 0.0;
  for (int g = 0; g < GROUPS; ++g) {
    xr += part[g][lq].x;
    xi += part[g][lq].y;
  }
  if (!small) {
    xr /= Q2;
    xi /= Q2;
  }
  double st, ct;
  sincos_any64(fit, Qx * t[0] + Qy * t[1], &st, &ct);
  out[2 * qi] = ct * xr - st * xi;
  out[2 * qi + 1] = ct * xi + st * xr;
}

}  // namespace

namespace {
template <bool OWN, int GROUPS>
hipError_t launch(const double* verts, const Edge2D* edges, int64_t ne, const MeshInfo* info, const double* q,
                  int64_t nq, double tau0, double* out, hipStream_t s) {
  const int64_t blocks = (nq + kBlock / GROUPS - 1) / (kBlock / GROUPS);
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  fwd2d_kernel<OWN, GROUPS><<<(unsigned)blocks, kBlock, 0, s>>>(verts, edges, ne, info, q, nq, tau0, out);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_fwd2d(const Edge2D* edges, int64_t ne, const MeshInfo* info, const double* q, int64_t nq, double tau0,
                        double* out, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  return launch<false, kGroups2D>(nullptr, edges, ne, info, q, nq, tau0, out, s);
}

hipError_t launch_fwd2d_own(const double* verts, int64_t nv, const double* q, int64_t nq, double tau0, double* out,
                            hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  if (nv < 1 || nv > kTileE) return hipErrorInvalidValue;
  return nq < kLongNq2D ? launch<true, kGroups2D>(verts, nullptr, nv, nullptr, q, nq, tau0, out, s)
                        : launch<true, kGroups2DLong>(verts, nullptr, nv, nullptr, q, nq, tau0, out, s);
}

}  // namespace pft
