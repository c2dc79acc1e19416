// Forward 3D transform of a closed triangle mesh: F(Q) for a list of Q.
//
// Layout: Q-tiles of QPT Q per thread, each wavefront of a block on its own
// share of the faces, faces streamed through LDS tiles and broadcast to the
// wavefront. Each block's sums over its face range are binary64 partials; the
// finish kernel adds a Q's partials in a fixed order and applies
// exp(i Q.t) / |Q|^2. The faces are split when there are too few Q to fill
// the GPU (the split is part of the one-dimensional block index).
//
// Two arithmetic forms:
//  * fwd3d_fp64_kernel  -- IEEE binary64 throughout.
//  * fwd3d_fp32c_kernel -- the face integral in binary32 from its centred
//    vertex phases (fwd_terms.h), the face origin phase Q.g reduced in
//    binary64 and evaluated in turns, the sum over faces blocked per LDS tile
//    and compensated (Kahan) across tiles. With the records in an edge-sharing
//    order (Face32::flags) the origin phase follows the shared edges.
#include "fwd_terms.h"

namespace pft {
namespace {

// The tetrahedron fan about an apex o (relative to t) gives the integral of exp(iQ.(r - o)); times
// exp(iQ.o) it is relative to t like the surface sums.
__device__ __forceinline__ void apex_phase(const double* Q, const double* o, double& xr, double& xi) {
  double so, co;
  sincos(Q[0] * o[0] + Q[1] * o[1] + Q[2] * o[2], &so, &co);
  const double r = co * xr - so * xi;
  xi = co * xi + so * xr;
  xr = r;
}

// Face range of split `sp`: from the split table when the splits follow region boundaries, else equal
// ranges.
__device__ __forceinline__ void split_faces(const FwdArgs& a, int64_t sp, int64_t& b, int64_t& e) {
  if (a.split_face) {
    b = a.split_face[sp];
    e = a.split_face[sp + 1];
  } else {
    b = sp * a.faces_per_split;
    e = min(a.nf, b + a.faces_per_split);
  }
}

// (Q-tile, split) of a forward block. The grid is one-dimensional and its blocks go to the dies in turn (block b
// to die b mod kXcds), so the block index is read as (die, rank on the die) and the k-th group of `splits` blocks a
// die receives holds every split of one Q-tile: a Q-tile's Q and permutation entries are fetched into that die's L2
// once and served from there to its other splits (the Q-tile count is padded to a multiple of kXcds; the padding
// blocks exit at once).
__device__ __forceinline__ void fwd_block(const FwdArgs& a, uint32_t& qtile, uint32_t& sp) {
  const uint32_t rank = blockIdx.x / kXcds;
  qtile = blockIdx.x % kXcds + kXcds * (rank / (uint32_t)a.splits);
  sp = rank % (uint32_t)a.splits;
}

// The last of a block's wavefronts to come here returns true, with the others' LDS writes visible.
__device__ __forceinline__ bool last_wave(uint32_t* done) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  int last = 0;
  if ((threadIdx.x & 63) == 0) last = atomicAdd(done, 1u) == (uint32_t)(kFwdSplitWaves - 1) ? 1 : 0;
  if (__builtin_amdgcn_readfirstlane(last) == 0) return false;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return true;
}

// The binary64 forward, in the FP32C forward's layout (below): QPT Q per lane, each wavefront of a block on its own
// quarter of the split's faces through its own LDS tile. Bound by binary64 issue: about 95 binary64 instructions
// per pair (two Horner sums of 42 coefficients, one sine and cosine) against some 290 with the edge terms'
// library sines and divisions (5 120 faces x 64 000 Q: kernel 3.3 -> 1.35 ms under the profiler). QPT = 2: a record
// read from LDS (96 B) and a coefficient read through the scalar cache serve two pairs (1 and 4 Q per lane: 1 % and
// -0.6 % on the fitting step; 3: 3 %).
template <int QPT>
__global__ __launch_bounds__(kFwdBlock, kFwdWaves64) void fwd3d_fp64_kernel(FwdArgs a) {
  constexpr int kQT = fwd_qtile(QPT);
  __shared__ Face64 tiles[kFwdSplitWaves][kTileF64];
  __shared__ uint32_t done;
  static_assert(sizeof(Face64) * kTileF64 >= sizeof(double2) * QPT * 64, "a wavefront's partials fit its tile");
  uint32_t qtile, sp;
  fwd_block(a, qtile, sp);
  if ((int64_t)qtile * kQT >= a.nq) return;  // padding of the Q-tile count (whole block)
  if (threadIdx.x == 0) done = 0u;
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
  Face64* tile = tiles[w];
  // the split's region (centre o relative to t, radius) when the splits follow regions, else the mesh
  const double4 geo = a.split_geo ? a.split_geo[sp] : make_double4(0.0, 0.0, 0.0, a.info[0].R);
  int64_t f_begin, f_end;
  split_faces(a, sp, f_begin, f_end);
  {  // this wavefront's share
    const int64_t per = (f_end - f_begin + kFwdSplitWaves - 1) / kFwdSplitWaves;
    const int64_t b = min(f_end, f_begin + w * per);
    f_end = min(f_end, b + per);
    f_begin = b;
  }
  double Q[QPT][3], xr[QPT], xi[QPT];
  bool small[QPT];
  bool any_small = false, surface = false, big = false;
  float qmax = 0.0f;
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int64_t qi = (int64_t)qtile * kQT + k * 64 + lane;
    Q[k][0] = Q[k][1] = Q[k][2] = 0.0;
    if (qi < a.nq) load_q3(a.q, a.qdtype, a.perm ? (int64_t)a.perm[qi] : qi, Q[k]);
    const double Q2 = Q[k][0] * Q[k][0] + Q[k][1] * Q[k][1] + Q[k][2] * Q[k][2];
    small[k] = qi < a.nq && sqrt(Q2) * geo.w < a.tau0;
    any_small |= small[k];
    surface |= qi < a.nq && !small[k];
    big |= big_phases64(Q2, a.info[0].R);
    qmax = fmaxf(qmax, (float)sqrt(Q2));
    xr[k] = xi[k] = 0.0;
  }
  const bool check = __builtin_amdgcn_readfirstlane((int)fit_range_test_needed64(
                         wave_max(qmax), fmax(a.info[0].rho, a.info[0].fan_rho))) != 0;
  // A wavefront of small Q alone takes the fan in the loop, QPT Q to a face's record and vertices, and no surface
  // sums (few Q: the lane-per-face fan below).
  const bool fans = !__any(surface) && __popcll(__ballot(small[0])) > kFanShared;
  const double o[3] = {geo.x, geo.y, geo.z};
  for (int64_t t0 = f_begin; t0 < f_end && (fans || __any(surface)); t0 += kTileF64) {
    const int nt = (int)min((int64_t)kTileF64, f_end - t0);
    wave_lds_fence();
    {
      const uint4* src = reinterpret_cast<const uint4*>(a.f64 + t0);
      uint4* dst = reinterpret_cast<uint4*>(tile);
      for (int i = lane; i < nt * (int)(sizeof(Face64) / 16); i += 64) dst[i] = src[i];
    }
    wave_lds_fence();
    if (fans) {
      for (int j = 0; j < nt; ++j)
#pragma unroll
        for (int k = 0; k < QPT; ++k) {
          double t[2] = {0.0, 0.0};
          tet_term_f64(tile[j], Q[k], t[0], t[1], o);
          add_term(xr[k], t[0]);
          add_term(xi[k], t[1]);
        }
    } else if (check)
      for (int j = 0; j < nt; ++j) fwd_face_f64<QPT, true>(tile[j], Q, big, xr, xi);
    else
      for (int j = 0; j < nt; ++j) fwd_face_f64<QPT, false>(tile[j], Q, big, xr, xi);
  }
  if (__any(any_small)) {  // small-|Q| lanes: the tetrahedron fan about the apex instead
    const auto term = [&](int64_t f, const double* q, double* t) { tet_term_f64(a.f64[f], q, t[0], t[1], o); };
#pragma unroll
    for (int k = 0; k < QPT; ++k) {
      double x[2] = {xr[k], xi[k]};
      if (!fans) fan_sum<2>(small[k], f_begin, f_end, Q[k], term, x);
      if (small[k] && a.split_geo) apex_phase(Q[k], o, x[0], x[1]);
      xr[k] = x[0];
      xi[k] = x[1];
    }
  }
  // this wavefront's partials into its own tile (it reads no more records)
  wave_lds_fence();
  double2* red = reinterpret_cast<double2*>(tiles[w]);
#pragma unroll
  for (int k = 0; k < QPT; ++k) red[k * 64 + lane] = make_double2(xr[k], xi[k]);
  if (!last_wave(&done)) return;
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int64_t qi = (int64_t)qtile * kQT + k * 64 + lane;
    double2 v = reinterpret_cast<const double2*>(tiles[0])[k * 64 + lane];
    for (int u = 1; u < kFwdSplitWaves; ++u) {
      const double2 x = reinterpret_cast<const double2*>(tiles[u])[k * 64 + lane];
      v.x += x.x;
      v.y += x.y;
    }
    if (qi < a.nq) store_stream(a.partial + (int64_t)sp * a.nq + qi, v);
  }
}

// The FP32C forward. A block holds one Q-tile of kQT = 64 QPT Q, the same in each of its
// kFwdSplitWaves wavefronts (lane l holds the tile's Q l, l + 64, ...; QPT per thread, so each face
// record read from LDS serves QPT independent instruction streams), and one face split (fwd_block).
// Each wavefront takes its own contiguous share of the split's faces and streams them through its own
// LDS tile of kTileF32 records, with wavefront-local ordering only: no block barrier after the start.
// A wavefront that is done leaves its binary64 partials in its own tile and counts itself done; the
// last of the block's wavefronts adds their partials of each Q in wavefront order and writes them (one
// partial per Q and block), and the others exit at once. SHARE: the records are in an
// edge-sharing order and each face takes its origin phase from its predecessor in the wavefront's range
// (binary32 instead of the binary64 dot product). Small-|Q| lanes (|Q| R < tau0, R the split's radius) take
// the binary64 tetrahedron fan about the split's apex.
template <bool SHARE, int QPT>
__global__ __launch_bounds__(kFwdBlock, fwd_waves(QPT)) void fwd3d_fp32c_kernel(FwdArgs a) {
  constexpr int kQT = fwd_qtile(QPT);
  __shared__ Face32 tiles[kFwdSplitWaves][kTileF32];
  __shared__ float qlo[kFwdSplitWaves][3 * QPT * 64];
  __shared__ uint32_t done;  // wavefronts of the block that have left their partials
  static_assert(sizeof(Face32) * kTileF32 >= sizeof(double2) * QPT * 64, "a wavefront's partials fit its tile");
  uint32_t qtile, sp;
  fwd_block(a, qtile, sp);
  if ((int64_t)qtile * kQT >= a.nq) return;  // padding of the Q-tile count (whole block)
  if (threadIdx.x == 0) done = 0u;
  __syncthreads();
  // the wavefront index as a wavefront-uniform (scalar) value, so the face range and tile addresses
  // derived from it stay in scalar registers
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & 63);
  Face32* tile = tiles[w];
  const double4 geo = a.split_geo ? a.split_geo[sp] : make_double4(0.0, 0.0, 0.0, a.info[0].R);
  const double R = geo.w;
  const double o[3] = {geo.x, geo.y, geo.z};
  int64_t f_begin, f_end;
  split_faces(a, sp, f_begin, f_end);
  {  // this wavefront's share
    const int64_t per = (f_end - f_begin + kFwdSplitWaves - 1) / kFwdSplitWaves;
    const int64_t b = min(f_end, f_begin + w * per);
    f_end = min(f_end, b + per);
    f_begin = b;
  }
  const int64_t qbase = (int64_t)qtile * kQT + lane;
  QLowLds<QPT> ql;
  ql.lo = qlo[w];
  ql.lane = lane;
  float qx[QPT], qy[QPT], qz[QPT], Q2[QPT];
  bool small[QPT], active[QPT];
  bool any_small = false;
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int64_t qi = qbase + (int64_t)k * 64;
    active[k] = qi < a.nq;
    double Qd[3] = {0.0, 0.0, 0.0};
    if (active[k]) load_q3(a.q, a.qdtype, a.perm ? (int64_t)a.perm[qi] : qi, Qd);
    qx[k] = (float)Qd[0];
    qy[k] = (float)Qd[1];
    qz[k] = (float)Qd[2];
    ql.set(k, Qd, qx[k], qy[k], qz[k]);
    Q2[k] = qx[k] * qx[k] + qy[k] * qy[k] + qz[k] * qz[k];
    const double Q2d = Qd[0] * Qd[0] + Qd[1] * Qd[1] + Qd[2] * Qd[2];
    small[k] = qi < a.nq && sqrt(Q2d) * R < a.tau0;
    any_small |= small[k];
  }
  float qmax = 0.0f;
#pragma unroll
  for (int k = 0; k < QPT; ++k) qmax = fmaxf(qmax, sqrtf(Q2[k]));
  const bool check = __builtin_amdgcn_readfirstlane((int)fit_range_test_needed(wave_max(qmax), fmax(a.info[0].rho, a.info[0].fan_rho))) != 0;
  float sr[QPT], si[QPT], cr[QPT], ci[QPT];
#pragma unroll
  for (int k = 0; k < QPT; ++k) sr[k] = si[k] = cr[k] = ci[k] = 0.0f;
  FwdCarry<QPT> carry;  // shared edge's phase from the previous face (SHARE)
  carry.reset();         // no previous face at the start of the range
  for (int64_t t0 = f_begin; t0 < f_end; t0 += kTileF32) {
    const int nt = (int)min((int64_t)kTileF32, f_end - t0);
    // the wavefront's previous tile has been read (its LDS reads were issued in order before these
    // writes); its writes are complete before any lane reads the tile
    wave_lds_fence();
    {
      const uint4* src = reinterpret_cast<const uint4*>(a.f32 + t0);
      uint4* d = reinterpret_cast<uint4*>(tile);
      for (int i = lane; i < nt * (int)(sizeof(Face32) / 16); i += 64) d[i] = src[i];
    }
    wave_lds_fence();
    float tr[QPT], ti[QPT];
#pragma unroll
    for (int k = 0; k < QPT; ++k) tr[k] = ti[k] = 0.0f;
    if (check)
      fwd_tile_fp32c<QPT, SHARE, true>(tile, nt, qx, qy, qz, ql, tr, ti, carry);
    else
      fwd_tile_fp32c<QPT, SHARE, false>(tile, nt, qx, qy, qz, ql, tr, ti, carry);
#pragma unroll
    for (int k = 0; k < QPT; ++k) {
      kahan_add(sr[k], cr[k], tr[k]);
      kahan_add(si[k], ci[k], ti[k]);
    }
  }
  // small-|Q| lanes: the binary64 tetrahedron fan over the range's faces, after the surface sums (the
  // rare wavefronts that hold such a lane pay for it; the others keep no binary64 sums live above)
  double xr[QPT], xi[QPT];
#pragma unroll
  for (int k = 0; k < QPT; ++k) xr[k] = xi[k] = 0.0;
  if (__any(any_small)) {
    const auto term = [&](int64_t f, const double* q, double* t) { tet_term_f64(a.f64[f], q, t[0], t[1], o); };
#pragma unroll
    for (int k = 0; k < QPT; ++k) {
      const double Qd[3] = {ql.qd(qx[k], k, 0), ql.qd(qy[k], k, 1), ql.qd(qz[k], k, 2)};
      double x[2] = {0.0, 0.0};
      fan_sum<2>(small[k], f_begin, f_end, Qd, term, x);
      if (small[k] && a.split_geo) apex_phase(Qd, o, x[0], x[1]);
      xr[k] = x[0];
      xi[k] = x[1];
    }
  }
  // this wavefront's partials into its own tile (it reads no more records)
  wave_lds_fence();
  double2* red = reinterpret_cast<double2*>(tiles[w]);
#pragma unroll
  for (int k = 0; k < QPT; ++k)
    red[k * 64 + lane] = small[k] ? make_double2(xr[k], xi[k])
                                  : make_double2((double)sr[k] - (double)cr[k],
                                                 (double)si[k] - (double)ci[k]);
  // count this wavefront done once its partials are visible to the block; the last one adds them all
  if (!last_wave(&done)) return;
  // the lane index anew (from the lane mask, not threadIdx), so no Q index is kept live across the loop
  const int l = (int)__lane_id();
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int64_t qi = (int64_t)qtile * kQT + k * 64 + l;
    double2 v = reinterpret_cast<const double2*>(tiles[0])[k * 64 + l];
    for (int u = 1; u < kFwdSplitWaves; ++u) {
      const double2 x = reinterpret_cast<const double2*>(tiles[u])[k * 64 + l];
      v.x += x.x;
      v.y += x.y;
    }
    if (qi < a.nq) store_stream(a.partial + (int64_t)sp * a.nq + qi, v);
  }
}

// F and |F|^2 of one Q from its centred sum x: exp(i Q.t), and 1/|Q|^2 unless the small-|Q| fan gave x.
__device__ __forceinline__ void write_transform(const FwdArgs& a, int out_c128, int64_t dst, const double* Q, double xr,
                                                double xi) {
  const MeshInfo mi = a.info[0];
  const double Q2 = Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2];
  const bool small = sqrt(Q2) * mi.R < a.tau0;
  if (!small) {
    xr /= Q2;
    xi /= Q2;
  }
  double st, ct;
  sincos_any64(fit64(), Q[0] * mi.t[0] + Q[1] * mi.t[1] + Q[2] * mi.t[2], &st, &ct);
  double Fr = ct * xr - st * xi;
  double Fi = ct * xi + st * xr;
  if (!out_c128 && fp32c_phase_out_of_range(sqrt(Q2), mi)) Fr = Fi = quiet_nan();  // beyond the FP32C phase range
  if (out_c128) {
    if (a.out) static_cast<double2*>(a.out)[dst] = make_double2(Fr, Fi);
    if (a.intensity) static_cast<double*>(a.intensity)[dst] = Fr * Fr + Fi * Fi;
  } else {
    if (a.out) static_cast<float2*>(a.out)[dst] = make_float2((float)Fr, (float)Fi);
    if (a.intensity) static_cast<float*>(a.intensity)[dst] = (float)(Fr * Fr + Fi * Fi);
  }
}

// The FP32C forward of a mesh of few faces (at most one LDS tile): each thread holds one Q in the list order, walks all
// faces and writes F itself. No face splits, so no partial sums and no finish launch, and no Q order: at a dozen faces
// the split form's wavefronts loaded, reduced and finished each Q for three faces each (12 faces x 2^21 Q of |Q| about
// 9: 187 -> 88 us a call; x 128^3 grid: 127 -> 69; two Q a thread instead of one: 91). Bound by issue: of the faces'
// polynomials and phases for small faces, of the edge terms' transcendentals for large ones.
// The faces are summed in binary32 in as many runs as the split form has wavefronts, and the runs in binary64, as there
// (one binary32 sum of 32 faces doubled the error of F at phases of some radians, 5.3e-8 -> 1.07e-7; the runs cost nothing
// that can be measured: 12 faces x 128^3, 68.8 and 68.2 us a call).
__global__ __launch_bounds__(kBlock, 8) void fwd3d_few_fp32c_kernel(FwdArgs a) {
  __shared__ Face32 tile[kTileF32];
  const int nt = (int)a.nf;
  for (int i = threadIdx.x; i < nt * (int)(sizeof(Face32) / 16); i += kBlock)
    reinterpret_cast<uint4*>(tile)[i] = reinterpret_cast<const uint4*>(a.f32)[i];
  __syncthreads();
  const double R = a.info[0].R;
  const int64_t qi = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  QReg<1> ql;
  ql.Q[0][0] = ql.Q[0][1] = ql.Q[0][2] = 0.0;
  if (qi < a.nq) load_q3(a.q, a.qdtype, qi, ql.Q[0]);
  const double* Q = ql.Q[0];
  const float qx[1] = {(float)Q[0]}, qy[1] = {(float)Q[1]}, qz[1] = {(float)Q[2]};
  const double qabs = sqrt(Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2]);
  const bool small = qi < a.nq && qabs * R < a.tau0;
  ql.wide[0] = !(qabs * R <= kWidePhase32);
  ql.any_wide = __any(ql.wide[0]) != 0;
  FwdCarry<1> carry;
  carry.reset();
  const double rho = fmax(a.info[0].rho, a.info[0].fan_rho);
  const bool check = __builtin_amdgcn_readfirstlane((int)fit_range_test_needed(wave_max((float)qabs), rho)) != 0;
  double x[2] = {0.0, 0.0};
  const int per = (nt + kFwdSplitWaves - 1) / kFwdSplitWaves;
  for (int j = 0; j < nt; j += per) {
    float tr[1] = {0.0f}, ti[1] = {0.0f};
    const int n = min(per, nt - j);
    if (check)
      fwd_tile_fp32c<1, false, true>(tile + j, n, qx, qy, qz, ql, tr, ti, carry);
    else
      fwd_tile_fp32c<1, false, false>(tile + j, n, qx, qy, qz, ql, tr, ti, carry);
    x[0] += (double)tr[0];
    x[1] += (double)ti[0];
  }
  if (__any(small))
    fan_sum<2>(small, 0, nt, Q,
               [&](int64_t f, const double* q, double* t) { tet_term_f64(a.f64[f], q, t[0], t[1], kZeroOrigin); }, x);
  if (qi < a.nq) write_transform(a, 0, qi, Q, x[0], x[1]);
}

// Sum the splits in order, apply exp(i Q.t) and 1/|Q|^2, write F and |F|^2 at
// the caller's index of the visited Q.
__global__ __launch_bounds__(256) void fwd3d_finish_kernel(FwdArgs a, int out_c128) {
  const int64_t qi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (qi >= a.nq) return;
  const int64_t dst = a.perm ? (int64_t)a.perm[qi] : qi;
  double Q[3];
  load_q3(a.q, a.qdtype, dst, Q);
  double xr, xi;
  fwd_partial_sum(a, qi, xr, xi);
  write_transform(a, out_c128, dst, Q, xr, xi);
}

}  // namespace

static hipError_t fwd_grid(const FwdArgs& a, unsigned* blocks) {
  const int64_t qtiles = (a.nq + fwd_qtile(a.qpt) - 1) / fwd_qtile(a.qpt);
  const int64_t n = (qtiles + kXcds - 1) / kXcds * kXcds * a.splits;
  if (n > 0x7fffffff) return hipErrorInvalidConfiguration;
  *blocks = (unsigned)n;
  return hipSuccess;
}

hipError_t launch_fwd3d_fp64(const FwdArgs& a, hipStream_t s) {
  unsigned blocks = 0;
  if (hipError_t e = fwd_grid(a, &blocks)) return e;
  if (a.qpt == 1)
    fwd3d_fp64_kernel<1><<<blocks, kFwdBlock, 0, s>>>(a);
  else if (a.qpt == kQPT64)
    fwd3d_fp64_kernel<kQPT64><<<blocks, kFwdBlock, 0, s>>>(a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_fwd3d_fp32c(const FwdArgs& a, hipStream_t s) {
  unsigned blocks = 0;
  if (hipError_t e = fwd_grid(a, &blocks)) return e;
#define PFT_FWD3D(SH, QP) fwd3d_fp32c_kernel<SH, QP><<<blocks, kFwdBlock, 0, s>>>(a)
  if (a.qpt == 1)
    a.share_edges ? PFT_FWD3D(true, 1) : PFT_FWD3D(false, 1);
  else if (a.qpt == kQPT)
    a.share_edges ? PFT_FWD3D(true, kQPT) : PFT_FWD3D(false, kQPT);
  else if (a.qpt == kQPTLarge)
    a.share_edges ? PFT_FWD3D(true, kQPTLarge) : PFT_FWD3D(false, kQPTLarge);
  else
    return hipErrorInvalidValue;
#undef PFT_FWD3D
  return hipGetLastError();
}

hipError_t launch_fwd3d_few_fp32c(const FwdArgs& a, hipStream_t s) {
  if (a.nf > kTileF32) return hipErrorInvalidValue;
  const int64_t blocks = (a.nq + kBlock - 1) / kBlock;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  fwd3d_few_fp32c_kernel<<<(unsigned)blocks, kBlock, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_fwd3d_finish(const FwdArgs& a, int out_c128, hipStream_t s) {
  fwd3d_finish_kernel<<<(unsigned)((a.nq + 255) / 256), 256, 0, s>>>(a, out_c128);
  return hipGetLastError();
}

}  // namespace pft
