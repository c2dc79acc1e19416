// Q ordering.
//
// Each Q is evaluated independently, so the kernels may visit the Q list in any
// order. Their cost per (Q, face) follows the worst lane of a wavefront: the
// edge form beyond the fitted phase range runs whenever one lane needs it. Wavefronts of nearby Q waste less
// work than wavefronts spanning a grid row or a random set. The Q points are
// sorted by mesh, then by the Morton code of their cells (5 bits per axis). One
// list: cells of the box of its Q, or of the span of most of them (list_span)
// where a few outlying Q make the box four times as wide. Batch: cells of each
// list's own span. The forward reads Q through the permutation and writes F back
// to the caller's order, the adjoints gather Q with their centred cotangents into
// QRec records.
//
// The sort is a stable radix sort by 8-bit digits, three launches a pass
// (digit counts per tile, their scan, the scatter), two passes for one mesh.
// It is bound by launches and their tails on short lists: against the library
// sort, whose merge-based path below 1e5 keys took 14 launches, ordering 91 125 Q
// takes 36 us instead of 75, 1.4e6 Q of 64 meshes about 125 instead of 230 (which
// sorted 36-bit keys, 10 bits per axis). Long lists are bound by the scattered
// writes: 4e6 random Q 104 us (202 with the tiles of short lists; library 137).
#include "pft_device.h"

namespace pft {
namespace {

constexpr int kBoxBlocks = 256;

// The span along an axis of all but about 3 % of a list's Q: kSpanSample of them, one from each stretch of the list (at a
// scrambled place in it, so that the period of a grid list does not show), less kSpanTrim at either end, widened to what
// the whole sample of an even list would span. Its cost does not depend on the list's length. {lowest, width}; {0, 0}
// for a list of one wavefront or less; not finite where that many Q are not. A block of kSpanSample threads calls it.
// Cells of a common box put two thirds of the wavefronts of such lists back into the list order (12 lists of 24 000 Q,
// short and long by turns, two in each at 30 times the range: binary64 adjoint 1.36 ms, 1.00 with spans; 48 lists of
// 5 000 to 40 000 and one such Q each: FP32C adjoint 1.78 -> 1.45 ms; without such Q the same to 1 % either way).
constexpr int kSpanSample = 256;
constexpr int kSpanTrim = 4;
__device__ __forceinline__ void list_span(const void* q, int qdtype, int64_t b, int64_t n, int axis, float2* out) {
  __shared__ alignas(16) float x[kSpanSample];
  __shared__ float end[2];
  const int tid = threadIdx.x;
  if (n <= 64) {
    if (tid == 0) *out = make_float2(0.0f, 0.0f);
    return;
  }
  uint32_t h = (uint32_t)tid * 2654435769u;
  h = (h ^ (h >> 15)) * 2246822519u;
  h ^= h >> 13;
  double Q[3];
  load_q3(q, qdtype, b + (tid * n + (int64_t)(((uint64_t)h * (uint64_t)n) >> 32)) / kSpanSample, Q);
  const float v = (float)Q[axis];
  x[tid] = v == v ? v : INFINITY;  // a NaN goes last
  __syncthreads();
  const float mine = x[tid];
  int below = 0, upto = 0;  // of the sample: less than mine, at most mine
#pragma unroll 8
  for (int i = 0; i < kSpanSample / 4; ++i) {
    const float4 u = reinterpret_cast<const float4*>(x)[i];
    below += (u.x < mine) + (u.y < mine) + (u.z < mine) + (u.w < mine);
    upto += (u.x <= mine) + (u.y <= mine) + (u.z <= mine) + (u.w <= mine);
  }
  // the sample's values at the two places (the threads of equals of such a value write the same)
  constexpr int kLo = kSpanTrim, kHi = kSpanSample - 1 - kSpanTrim;
  if (below <= kLo && kLo < upto) end[0] = mine;
  if (below <= kHi && kHi < upto) end[1] = mine;
  __syncthreads();
  if (tid != 0) return;
  const float w = end[1] - end[0], wide = w * ((float)kSpanSample / (float)(kSpanSample - 2 * kSpanTrim));
  *out = make_float2(end[0] - 0.5f * (wide - w), wide);
}

__global__ __launch_bounds__(kSpanSample) void batch_span_kernel(const void* q, int qdtype, const int64_t* q_off,
                                                                 float2* span) {
  const int64_t b = q_off[blockIdx.x];
  list_span(q, qdtype, b, q_off[blockIdx.x + 1] - b, (int)blockIdx.y, span + (int64_t)blockIdx.x * 3 + blockIdx.y);
}

// Box of every stride-th Q from `first` (each thread's own part of a list), kAhead of them in flight.
template <class T>
__device__ __forceinline__ void box_of(const T* q, int64_t nq, int64_t first, int64_t stride, double* lo, double* hi) {
  constexpr int kAhead = 4;
  for (int64_t i = first; i < nq; i += kAhead * stride) {
    T Q[kAhead][3];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t j = 3 * min(i + u * stride, nq - 1);
      for (int k = 0; k < 3; ++k) Q[u][k] = q[j + k];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      for (int k = 0; k < 3; ++k) {
        lo[k] = fmin(lo[k], (double)Q[u][k]);
        hi[k] = fmax(hi[k], (double)Q[u][k]);
      }
  }
}

// One list: the partial boxes of its Q (blocks 0 .. gridDim.x - 4) and its span per axis (the last three blocks).
__global__ __launch_bounds__(256) void qbox_partial_kernel(const void* q, int qdtype, int64_t nq, double* partial,
                                                           float2* span) {
  static_assert(kSpanSample == 256, "blocks of both kinds");
  __shared__ double red[6][256];
  const int tid = threadIdx.x, boxes = (int)gridDim.x - 3;
  if ((int)blockIdx.x >= boxes) {
    list_span(q, qdtype, 0, nq, (int)blockIdx.x - boxes, span + (blockIdx.x - boxes));
    return;
  }
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + tid, stride = (int64_t)boxes * blockDim.x;
  if (qdtype == PFT_F64)
    box_of(static_cast<const double*>(q), nq, first, stride, lo, hi);
  else
    box_of(static_cast<const float*>(q), nq, first, stride, lo, hi);
  for (int k = 0; k < 3; ++k) {
    red[k][tid] = lo[k];
    red[3 + k][tid] = hi[k];
  }
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s)
      for (int k = 0; k < 3; ++k) {
        red[k][tid] = fmin(red[k][tid], red[k][tid + s]);
        red[3 + k][tid] = fmax(red[3 + k][tid], red[3 + k][tid + s]);
      }
    __syncthreads();
  }
  if (tid < 6) partial[blockIdx.x * 6 + tid] = red[tid][0];
}

// spread the low 10 bits of x to every third bit
__device__ __forceinline__ uint64_t spread3(uint32_t x) {
  uint64_t v = x & 0x3ffu;
  v = (v | (v << 16)) & 0x30000ffull;
  v = (v | (v << 8)) & 0x300f00full;
  v = (v | (v << 4)) & 0x30c30c3ull;
  v = (v | (v << 2)) & 0x9249249ull;
  return v;
}

__device__ __forceinline__ int64_t mesh_of(const int64_t* q_off, int64_t n_meshes, int64_t i) {
  if (!q_off) return 0;
  int64_t lo = 0, hi = n_meshes;  // last mesh with q_off[mesh] <= i
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) / 2;
    if (q_off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// Sort tiles: 256 ROUNDS items per block, each wavefront a contiguous quarter of it. 4 rounds on short lists (16: 14 us a
// scatter of 91 125, which are 23 blocks), 16 on long ones, whose scatter then has runs of a digit to write in one piece.
constexpr int kSortBlock = 256;
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortRounds = 4, kSortRoundsLong = 16;
constexpr int64_t kSortLong = 3 << 19;  // short and long tiles: 1e6 random Q 70 and 73 us, a grid of them 57 and 72; 1.5e6
                                        // 95 and 81, 72 and 80; 2e6 119 and 87, 87 and 86
constexpr int kDigits = 256;
inline int sort_rounds(int64_t nq) { return nq >= kSortLong ? kSortRoundsLong : kSortRounds; }
inline int64_t sort_tiles(int64_t nq) {
  const int64_t tile = (int64_t)kSortBlock * sort_rounds(nq);
  return (nq + tile - 1) / tile;
}

// First item of this wavefront's part of the block's tile.
template <int ROUNDS>
__device__ __forceinline__ int64_t sort_first() {
  return (int64_t)blockIdx.x * (kSortBlock * ROUNDS) + (int64_t)(threadIdx.x >> 6) * (64 * ROUNDS);
}

// Keys of the tile's Q (mesh, then Morton code of `bits` bits per axis) and the counts of their lowest digit. One list:
// cells of the box of all Q, whose partial boxes every block reduces for itself, or of the list's span. BATCH: of each
// list's span.
template <bool BATCH, int ROUNDS>
__global__ __launch_bounds__(kSortBlock) void qkey_kernel(const void* q, int qdtype, int64_t nq,
                                                          const double* box_partial, int n_partial, const float2* span,
                                                          const int64_t* q_off, int64_t n_meshes, int bits,
                                                          uint32_t* keys, uint32_t* counts) {
  __shared__ uint32_t hist[kDigits];
  const int tid = threadIdx.x;
  hist[tid] = 0u;
  double lo[3], ext[3];
  if constexpr (!BATCH) {
    __shared__ double red[6][kSortBlock];
    const float2 own[3] = {span[0], span[1], span[2]};
    for (int k = 0; k < 6; ++k)
      red[k][tid] = tid < n_partial ? box_partial[tid * 6 + k] : (k < 3 ? INFINITY : -INFINITY);
    __syncthreads();
    for (int h = kSortBlock / 2; h > 0; h >>= 1) {
      if (tid < h)
        for (int k = 0; k < 3; ++k) {
          red[k][tid] = fmin(red[k][tid], red[k][tid + h]);
          red[3 + k][tid] = fmax(red[3 + k][tid], red[3 + k][tid + h]);
        }
      __syncthreads();
    }
    for (int k = 0; k < 3; ++k) {
      lo[k] = red[k][0];
      ext[k] = red[3 + k][0] - lo[k];
      if (ext[k] > 4.0 * (double)own[k].y) {
        lo[k] = (double)own[k].x;
        ext[k] = (double)own[k].y;
      }
    }
  } else {
    __syncthreads();
  }
  const double cells = (double)(1u << bits);
  const int64_t i0 = sort_first<ROUNDS>() + (tid & 63);
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = i0 + r * 64;
    if (i >= nq) break;
    double Q[3];
    load_q3(q, qdtype, i, Q);
    int64_t mesh = 0;
    if constexpr (BATCH) {
      mesh = mesh_of(q_off, n_meshes, i);
      for (int k = 0; k < 3; ++k) {
        const float2 s = span[mesh * 3 + k];
        lo[k] = (double)s.x;
        ext[k] = (double)s.y;
      }
    }
    uint32_t code = 0;
    for (int k = 0; k < 3; ++k) {
      double u = ext[k] > 0.0 ? (Q[k] - lo[k]) / ext[k] * cells : 0.0;
      u = fmin(fmax(u, 0.0), cells - 1.0);  // NaN coordinates map to 0 (fmax returns the non-NaN operand)
      code |= (uint32_t)spread3((uint32_t)u) << k;
    }
    const uint32_t key = (uint32_t)((uint64_t)mesh << (3 * bits)) | code;
    keys[i] = key;
    atomicAdd(&hist[key & (kDigits - 1)], 1u);
  }
  __syncthreads();
  counts[(int64_t)tid * gridDim.x + blockIdx.x] = hist[tid];
}

// Counts of the digit at `shift` per tile, digit-major.
template <int ROUNDS>
__global__ __launch_bounds__(kSortBlock) void sort_count_kernel(const uint32_t* keys, int64_t n, int shift,
                                                                uint32_t* counts) {
  __shared__ uint32_t hist[kDigits];
  hist[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t i0 = sort_first<ROUNDS>() + (threadIdx.x & 63);
  for (int r = 0; r < ROUNDS; ++r)
    if (i0 + r * 64 < n) atomicAdd(&hist[(keys[i0 + r * 64] >> shift) & (kDigits - 1)], 1u);
  __syncthreads();
  counts[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = hist[threadIdx.x];
}

// Exclusive sum over a block's threads (kSortBlock of them; part holds kSortWaves words); total is every thread's.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* part, uint32_t& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;  // inclusive over the wavefront, then over the wavefronts
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  __syncthreads();  // part is free
  if (lane == 63) part[w] = x;
  __syncthreads();
  uint32_t base = 0;
  total = 0;
  for (int u = 0; u < kSortWaves; ++u) {
    if (u < w) base += part[u];
    total += part[u];
  }
  return base + x - v;
}

// Exclusive scan in place of each digit's counts over the tiles (a block per digit), and the digits' totals.
__global__ __launch_bounds__(kSortBlock) void sort_scan_kernel(uint32_t* counts, int64_t tiles, uint32_t* totals) {
  __shared__ uint32_t part[kSortWaves];
  uint32_t* row = counts + (int64_t)blockIdx.x * tiles;
  uint32_t base = 0;
  for (int64_t i0 = 0; i0 < tiles; i0 += kSortBlock) {
    const int64_t i = i0 + threadIdx.x;
    uint32_t total;
    const uint32_t x = block_scan(i < tiles ? row[i] : 0u, part, total);
    if (i < tiles) row[i] = base + x;
    base += total;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = base;
}

// One stable pass: every item to the place its digit's scanned count gives (vals NULL: an item's value is its index;
// keys_out NULL: the last pass). STAGED (long lists): the tile is put in order in LDS first, so that a digit's items go
// out side by side; written one by one, 4e6 random Q took 56 us a scatter.
template <int ROUNDS, bool STAGED>
__global__ __launch_bounds__(kSortBlock) void sort_scatter_kernel(const uint32_t* keys, const uint32_t* vals, int64_t n,
                                                                  int shift, const uint32_t* counts,
                                                                  const uint32_t* totals, uint32_t* keys_out,
                                                                  uint32_t* vals_out) {
  constexpr int kStage = STAGED ? kSortBlock * ROUNDS : 1;
  __shared__ uint32_t part[kSortWaves];
  __shared__ uint32_t place[kSortWaves][kDigits];  // next place of each digit in each wavefront's part
  __shared__ uint32_t base[STAGED ? kDigits : 1];  // place in the list less place in the tile, per digit
  __shared__ uint32_t skey[kStage], sval[kStage];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int u = 0; u < kSortWaves; ++u) place[u][tid] = 0u;
  __syncthreads();
  const int64_t i0 = sort_first<ROUNDS>() + lane;
  uint32_t key[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = i0 + r * 64;
    key[r] = i < n ? keys[i] : 0u;
    if (i < n) atomicAdd(&place[w][(key[r] >> shift) & (kDigits - 1)], 1u);
  }
  __syncthreads();
  {
    uint32_t total;
    uint32_t at = block_scan(totals[tid], part, total) + counts[(int64_t)tid * gridDim.x + blockIdx.x];
    if constexpr (STAGED) {
      uint32_t mine = 0u;
      for (int u = 0; u < kSortWaves; ++u) mine += place[u][tid];
      const uint32_t in_tile = block_scan(mine, part, total);
      base[tid] = at - in_tile;
      at = in_tile;
    }
    for (int u = 0; u < kSortWaves; ++u) {
      const uint32_t c = place[u][tid];
      place[u][tid] = at;
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = i0 + r * 64;
    const bool valid = i < n;
    const uint32_t d = (key[r] >> shift) & (kDigits - 1);
    uint64_t peers = __ballot(valid);  // the lanes of this round with the same digit
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint64_t m = __ballot((d >> k) & 1u);
      peers &= ((d >> k) & 1u) ? m : ~m;
    }
    const int rank = __popcll(peers & ((1ull << lane) - 1ull));
    uint32_t at = 0u;
    if (valid) at = place[w][d] + (uint32_t)rank;
    // the wavefront's reads of this round come before the update of the next round's places
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (valid && rank == 0) place[w][d] += (uint32_t)__popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (valid) {
      const uint32_t v = vals ? vals[i] : (uint32_t)i;
      if constexpr (STAGED) {
        skey[at] = key[r];
        sval[at] = v;
      } else {
        if (keys_out) keys_out[at] = key[r];
        vals_out[at] = v;
      }
    }
  }
  if constexpr (STAGED) {
    __syncthreads();
    const int m = (int)min((int64_t)kStage, n - (int64_t)blockIdx.x * kStage);
    for (int j = tid; j < m; j += kSortBlock) {
      const uint32_t k = skey[j], at = base[(k >> shift) & (kDigits - 1)] + (uint32_t)j;
      if (keys_out) keys_out[at] = k;
      vals_out[at] = sval[j];
    }
  }
}

__global__ __launch_bounds__(256) void qrec32_kernel(const void* q, int qdtype, const float2* grad_out, int64_t nq,
                                                     const uint32_t* perm, const MeshInfo* info,
                                                     const int64_t* q_off, int64_t n_meshes, QRec32* rec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nq) return;
  const int64_t j = perm ? (int64_t)perm[i] : i;
  double Q[3];
  load_q3(q, qdtype, j, Q);
  const float2 g = grad_out[j];
  const MeshInfo& mi = info[mesh_of(q_off, n_meshes, j)];
  double hr, hi;
  centred_cotangent((double)g.x, (double)g.y, Q, mi.t, hr, hi);
  // beyond the FP32C phase range: a NaN cotangent, so every vertex gradient is NaN
  if (fp32c_phase_out_of_range(sqrt(Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2]), mi)) hr = hi = quiet_nan();
  QRec32 r;
  r.q[0] = Q[0];
  r.q[1] = Q[1];
  r.q[2] = Q[2];
  r.hr = (float)hr;
  r.hi = (float)hi;
  rec[i] = r;
}

__global__ __launch_bounds__(256) void qrec64_kernel(const void* q, int qdtype, const double2* grad_out, int64_t nq,
                                                     const uint32_t* perm, const MeshInfo* info,
                                                     const int64_t* q_off, int64_t n_meshes, QRec64* rec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nq) return;
  const int64_t j = perm ? (int64_t)perm[i] : i;
  double Q[3];
  load_q3(q, qdtype, j, Q);
  const double2 g = grad_out[j];
  QRec64 r;
  centred_cotangent(g.x, g.y, Q, info[mesh_of(q_off, n_meshes, j)].t, r.hr, r.hi);
  r.q[0] = Q[0];
  r.q[1] = Q[1];
  r.q[2] = Q[2];
  r.pad = 0.0;
  rec[i] = r;
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

int64_t qorder_counts(int64_t nq) { return sort_tiles(nq) * kDigits + kDigits; }

namespace {
template <int ROUNDS, bool STAGED>
hipError_t sort_by_key(const void* q, int qdtype, int64_t nq, const int64_t* d_q_off, int64_t n_meshes, int boxes,
                       const QOrderScratch& w, hipStream_t s) {
  int mesh_bits = 0;
  while (mesh_bits < 32 && ((int64_t)1 << mesh_bits) < n_meshes) ++mesh_bits;
  const int bits = std::min(5, (32 - mesh_bits) / 3);  // Morton bits per axis
  const int passes = std::max(1, (mesh_bits + 3 * bits + 7) / 8);
  const unsigned tiles = (unsigned)sort_tiles(nq);
  const uint32_t* vals = nullptr;
  uint32_t *from = w.keys, *to = w.keys2, *totals = w.counts + (int64_t)tiles * kDigits;
  for (int p = 0; p < passes; ++p) {
    const bool last = p + 1 == passes;
    if (p == 0 && d_q_off)
      qkey_kernel<true, ROUNDS><<<tiles, kSortBlock, 0, s>>>(q, qdtype, nq, nullptr, 0, w.span, d_q_off, n_meshes, bits,
                                                             from, w.counts);
    else if (p == 0)
      qkey_kernel<false, ROUNDS><<<tiles, kSortBlock, 0, s>>>(q, qdtype, nq, w.box_partial, boxes, w.span, nullptr, 1,
                                                              bits, from, w.counts);
    else
      sort_count_kernel<ROUNDS><<<tiles, kSortBlock, 0, s>>>(from, nq, 8 * p, w.counts);
    sort_scan_kernel<<<kDigits, kSortBlock, 0, s>>>(w.counts, tiles, totals);
    // the values end in w.perm: passes before the last alternate so that they do
    uint32_t* out = (passes - 1 - p) % 2 == 0 ? w.perm : w.vals;
    sort_scatter_kernel<ROUNDS, STAGED><<<tiles, kSortBlock, 0, s>>>(from, vals, nq, 8 * p, w.counts, totals,
                                                                     last ? nullptr : to, out);
    vals = out;
    std::swap(from, to);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_qorder(const void* q, int qdtype, int64_t nq, const int64_t* d_q_off, int64_t n_meshes,
                         const QOrderScratch& w, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  const int nb = (int)std::min<int64_t>(kBoxBlocks, (nq + 255) / 256);
  static_assert(kDigits == kSortBlock, "a thread per digit");
  static_assert(kBoxBlocks <= kSortBlock, "a block reduces all partial boxes in one step");
  if (d_q_off)
    batch_span_kernel<<<dim3((unsigned)n_meshes, 3), kSpanSample, 0, s>>>(q, qdtype, d_q_off, w.span);
  else
    qbox_partial_kernel<<<nb + 3, 256, 0, s>>>(q, qdtype, nq, w.box_partial, w.span);
  return sort_rounds(nq) == kSortRounds ? sort_by_key<kSortRounds, false>(q, qdtype, nq, d_q_off, n_meshes, nb, w, s)
                                        : sort_by_key<kSortRoundsLong, true>(q, qdtype, nq, d_q_off, n_meshes, nb, w, s);
}

hipError_t launch_qrec32_gather(const void* q, int qdtype, const void* grad_out, int64_t nq, const uint32_t* perm,
                                const MeshInfo* info, const int64_t* d_q_off, int64_t n_meshes, QRec32* rec,
                                hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  qrec32_kernel<<<grid_for(nq), 256, 0, s>>>(q, qdtype, static_cast<const float2*>(grad_out), nq, perm, info,
                                             d_q_off, n_meshes, rec);
  return hipGetLastError();
}

hipError_t launch_qrec64_gather(const void* q, int qdtype, const void* grad_out, int64_t nq, const uint32_t* perm,
                                const MeshInfo* info, const int64_t* d_q_off, int64_t n_meshes, QRec64* rec,
                                hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  qrec64_kernel<<<grid_for(nq), 256, 0, s>>>(q, qdtype, static_cast<const double2*>(grad_out), nq, perm, info,
                                             d_q_off, n_meshes, rec);
  return hipGetLastError();
}

}  // namespace pft
