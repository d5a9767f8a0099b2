// Jagged (CSR) event kernels for gfx950: pair-offset scan, offset checks,
// and the one-launch per-event reduction -- each event's total 4-vector,
// its mass and the masses of all its particle pairs (the pair mass of
// GenVectorX Fig. 1 applied to every i < j inside an event) -- with its
// reverse mode.
//
// Work decomposition of the reduction.  Each wavefront takes its own tile of
// consecutive events and walks it in event-aligned chunks of at most
// `lds_particles` particles, staging each particle once, converted, in its
// own slice of LDS (no workgroup barrier: the wavefronts of a workgroup never
// share data).  Four lanes per event sum its particles, one residue class of
// the particle index modulo 4 each, combined in a fixed order; the
// chunk's pairs -- contiguous in the output too -- are dealt out as equal
// contiguous runs, one per lane, each lane stepping its run in lexicographic
// order across event boundaries, so every lane has the same work whatever the
// event sizes.  In the compensated mode each lane also sums K_ij over its run
// per event, and the partial sums of an event that spans runs are combined
// across lanes by a segmented scan keyed by event: deterministic for a
// tiling, never dependent on timing.  The same kernel can choose, per event,
// the pair whose mass lies closest to a target (a candidate per run and
// event, combined by the same scheme under a total order) instead of storing
// pair masses.
// The reverse mode stages one particle per thread of a workgroup (below).
// Events of many particles, whose pairs are too many for one wavefront or
// one workgroup's staging, are left to a second launch in either direction,
// which shares their pairs, or the events, out evenly (k_event_dense,
// k_event_bwd_dense);
// on collider-sized events it only reads the pair offsets.
#include "glv_device.h"
#include "glv_launch.h"
#include "glv_share.h"

namespace glv {
namespace {

__device__ __forceinline__ int64_t npairs(int64_t c) { return c * (c - 1) / 2; }

// ------------------------------------------------------------ pair offsets

// Exclusive scan of n_e (n_e - 1)/2.  Up to kScanOnce events in one launch:
// workgroup b sums the pair counts before its tile itself (k_po_once).  More
// events in three launches, with pair_offsets itself holding the per-tile
// totals between them (no scratch):
//   1. workgroup b sums the pair counts of its kScanTile events and writes the
//      total to pair_offsets[end_b], end_b = min((b + 1) kScanTile, ne);
//   2. one workgroup turns those totals into running totals in place and sets
//      pair_offsets[0] = 0;
//   3. workgroup b scans its own events from pair_offsets[b kScanTile] and
//      writes pair_offsets[e + 1] for its events except the last one, whose
//      value step 2 left in place -- so no entry one workgroup reads is
//      written by another.
// Tiles of 2048 events (512 workgroups of 8 wavefronts on 2^20 events) keep
// enough loads in flight: 12.9 us for the three launches on 2^20 events against
// 17.6 with 4096 events by four wavefronts.  One launch takes 2.8 us on 1,000
// events (three: 7.6), 9.0 on 32,000 (10.1) and 12.8 on 64,000 (10.0, but two
// launches and the gaps between them more).
constexpr int kScanThreads = 512;
constexpr int kScanPer = 4;
constexpr int kScanTile = kScanThreads * kScanPer;
constexpr int64_t kScanOnce = 1 << 16;

// Exclusive prefix over the workgroup of one int64 per thread; *total gets
// the workgroup's sum.  ws holds one int64 per wavefront.
__device__ __forceinline__ int64_t block_excl_scan(int64_t x, int64_t* ws, int64_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int64_t v = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int64_t y = __shfl_up(v, d);
    if (lane >= d) v += y;
  }
  if (lane == 63) ws[wid] = v;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wid) before += ws[w];
    all += ws[w];
  }
  __syncthreads();
  *total = all;
  return before + v - x;
}

__global__ __launch_bounds__(kScanThreads) void k_po_tile_totals(const int64_t* __restrict__ off,
                                                                 int64_t* __restrict__ po, int64_t ne) {
  __shared__ int64_t ws[kScanThreads / 64];
  const int64_t b0 = (int64_t)blockIdx.x * kScanTile;
  int64_t sum = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const int64_t e = b0 + j * kScanThreads + threadIdx.x;
    if (e < ne) sum += npairs(off[e + 1] - off[e]);
  }
  int64_t total;
  block_excl_scan(sum, ws, &total);
  if (threadIdx.x == 0) po[min(b0 + kScanTile, ne)] = total;
}

__global__ __launch_bounds__(1024) void k_po_scan_totals(int64_t* __restrict__ po, int64_t ne, int64_t ntiles) {
  __shared__ int64_t ws[1024 / 64];
  if (threadIdx.x == 0) po[0] = 0;
  int64_t carry = 0;
  for (int64_t base = 0; base < ntiles; base += 1024) {
    const int64_t b = base + threadIdx.x;
    const int64_t at = min((b + 1) * kScanTile, ne);
    const int64_t v = (b < ntiles) ? po[at] : 0;
    int64_t total;
    const int64_t ex = block_excl_scan(v, ws, &total);
    if (b < ntiles) po[at] = carry + ex + v;
    carry += total;
  }
}

// pair_offsets[e + 1] for the events [b0, end) of a tile whose first pair is
// `base` (the last event's left out unless `last`).
__device__ __forceinline__ void scan_tile(const int64_t* __restrict__ off, int64_t* __restrict__ po, int64_t b0,
                                          int64_t ne, int64_t base, bool last, int64_t* c, int64_t* ws) {
  const int64_t end = min(b0 + kScanTile, ne);
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const int idx = j * kScanThreads + threadIdx.x;
    const int64_t e = b0 + idx;
    c[idx] = (e < ne) ? npairs(off[e + 1] - off[e]) : 0;
  }
  __syncthreads();
  int64_t run = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) run += c[threadIdx.x * kScanPer + k];
  int64_t total;
  int64_t pre = base + block_excl_scan(run, ws, &total);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    pre += c[threadIdx.x * kScanPer + k];
    c[threadIdx.x * kScanPer + k] = pre;  // inclusive: pair_offsets[e + 1]
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    const int idx = j * kScanThreads + threadIdx.x;
    const int64_t e = b0 + idx;
    if (e + (last ? 0 : 1) < end) po[e + 1] = c[idx];
  }
}

__global__ __launch_bounds__(kScanThreads) void k_po_tile_scan(const int64_t* __restrict__ off,
                                                               int64_t* __restrict__ po, int64_t ne) {
  __shared__ int64_t c[kScanTile];
  __shared__ int64_t ws[kScanThreads / 64];
  const int64_t b0 = (int64_t)blockIdx.x * kScanTile;
  scan_tile(off, po, b0, ne, (blockIdx.x == 0) ? 0 : po[b0], false, c, ws);
}

// One launch: the workgroup first sums the pair counts of all earlier events
// (at most kScanOnce, 128 per thread, read from L2), then scans its tile.
__global__ __launch_bounds__(kScanThreads) void k_po_once(const int64_t* __restrict__ off, int64_t* __restrict__ po,
                                                          int64_t ne) {
  __shared__ int64_t c[kScanTile];
  __shared__ int64_t ws[kScanThreads / 64];
  const int64_t b0 = (int64_t)blockIdx.x * kScanTile;
  int64_t before = 0;
#pragma unroll 16
  for (int64_t e = threadIdx.x; e < b0; e += kScanThreads) before += npairs(off[e + 1] - off[e]);
  int64_t base = 0;
  if (b0) block_excl_scan(before, ws, &base);
  if (b0 == 0 && threadIdx.x == 0) po[0] = 0;
  scan_tile(off, po, b0, ne, base, true, c, ws);
}

__global__ __launch_bounds__(256) void k_validate_offsets(const int64_t* __restrict__ off, int64_t ne,
                                                          int64_t np, long long* bad) {
  long long cnt = 0;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e <= ne; e += stride) {
    int64_t v = off[e];
    if (e == 0 && v != 0) ++cnt;
    if (e == ne && v != np) ++cnt;
    if (e < ne && off[e + 1] < v) ++cnt;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) cnt += __shfl_xor(cnt, d);
  if ((threadIdx.x & 63) == 0 && cnt) atomicAdd((unsigned long long*)bad, (unsigned long long)cnt);
}

// --------------------------------------------------------------- helpers

// i of the pair with in-event rank r among n particles (lexicographic i < j):
// the largest i with R(i) = i (2n - i - 1)/2 <= r.
__device__ __forceinline__ int64_t row_start(int64_t i, int64_t n) { return i * (2 * n - i - 1) / 2; }

__device__ __forceinline__ void decode_pair(int64_t r, int64_t n, int64_t* pi, int64_t* pj) {
  double b = (double)(2 * n - 1);
  int64_t i = (int64_t)((b - sqrt(b * b - 8.0 * (double)r)) * 0.5);
  if (i < 0) i = 0;
  if (i > n - 2) i = n - 2;
  while (i > 0 && row_start(i, n) > r) --i;
  while (i < n - 2 && row_start(i + 1, n) <= r) ++i;
  *pi = i;
  *pj = i + 1 + (r - row_start(i, n));
}

// Decode for events staged in LDS (2 <= n <= 4096).  With b = 2n - 1 the
// row is the floor of the root x = (b - sqrt(b^2 - 8r))/2 of R(x) = r.  In
// FP32 b^2 - 8r (< 2^27, one rounding by the fused multiply-add) is off by at
// most 4 and is at least 9, so the hardware square root (1 ulp) puts the
// estimate within one row of the answer: one step down and one step up fix it.
// Products stay below 2^25, so 24-bit multiplies are exact.
__device__ __forceinline__ int row_start32(int i, int n) { return (int)(__umul24(i, 2 * n - i - 1) >> 1); }

__device__ __forceinline__ void decode_pair_small(int r, int n, int* pi, int* pj) {
  const float b = (float)(2 * n - 1);
  const float d = fmaf(b, b, -8.0f * (float)r);
  int i = (int)((b - __builtin_amdgcn_sqrtf(fmaxf(d, 0.0f))) * 0.5f);
  i = max(0, min(i, n - 2));
  if (row_start32(i, n) > r) --i;
  if (i < n - 2 && row_start32(i + 1, n) <= r) ++i;
  *pi = i;
  *pj = i + 1 + (r - row_start32(i, n));
}

// Per event of a chunk: first particle and first pair, relative to the chunk.
struct EvRec {
  int o;
  int p;
};

__device__ __forceinline__ int search_le(const int64_t* a, int lo, int hi, int64_t key) {
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= key)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Per-particle staged records in LDS, read with 16-byte LDS loads:
//   cart[t] = (px, py, pz, E)                       every mode
//   leg[2t] = (pt, eta, phi, M), leg[2t+1] = (mT, delta, mT - pt, M^2)
//                                                    compensated mode
template <typename T>
struct V4 {
  typedef T type __attribute__((ext_vector_type(4)));
};

// The total of an event's records rec[lo..hi) is ((P0 + P1) + (P2 + P3)), P_r
// the sum from zero, component-wise and in index order, of the records
// lo + r, lo + r + 4, ...  Forward and reverse mode both give each event a
// quad of lanes, one residue each, and combine the quad's sums in this order
// (lane ^ 1, then lane ^ 2), so that their totals agree bit for bit.
// residue_sum adds P_r to acc (two records read per LDS wait); with a
// non-null `legs` (compensated mode) it also adds the residue's sum of M^2
// (the mass is the fourth component of leg[2t]) to *m2.
template <typename V>
__device__ __forceinline__ void residue_sum(const V* rec, int lo, int hi, int r, double acc[4],
                                            const V* legs = nullptr, double* m2 = nullptr) {
  int t = lo + r;
  for (; t + 4 < hi; t += 8) {
    const V r0 = rec[t], r1 = rec[t + 4];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = (acc[k] + (double)r0[k]) + (double)r1[k];
    if (legs) {
      const double m0 = (double)legs[2 * t][3], m1 = (double)legs[2 * t + 8][3];
      *m2 = (*m2 + m0 * m0) + m1 * m1;
    }
  }
  if (t < hi) {
    const V r0 = rec[t];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += (double)r0[k];
    if (legs) {
      const double m0 = (double)legs[2 * t][3];
      *m2 += m0 * m0;
    }
  }
}

// Compensated pair mass and K = E_i E_j - p_i.p_j (as double) from two legs,
// with the FP64 redo of an FP32 pair whose error bound is too large.
template <typename T>
__device__ __forceinline__ T comp_pair(const LegC<T>& a, const LegC<T>& b, T ma, T mb, double* kout,
                                       unsigned* fb) {
  T k;
  if constexpr (sizeof(T) == 4) {
    bool redo;
    T m2 = comp_pair_m2<T>(a, b, &k, &redo);
    if (redo) {
      LegC<double> da = comp_leg<double, true>(a.pt, a.eta, a.phi, ma);
      LegC<double> db = comp_leg<double, true>(b.pt, b.eta, b.phi, mb);
      double kd;
      double m2d = comp_pair_m2<double, true>(da, db, &kd, nullptr);
      *kout = kd;
      ++*fb;
      return (T)sqrt(m2d);
    }
    *kout = (double)k;
    return sqrt_budgeted(m2);
  } else {
    T m2 = comp_pair_m2<T>(a, b, &k, nullptr);
    *kout = (double)k;
    return d_sqrt(m2);
  }
}

// Marks an event of the tiled FP32 compensated reduction that holds a pair
// needing the FP64 redo: written to the event's mass (or, without event
// masses, to its first pair mass) for k_event_dense to find.  A quiet NaN
// with a payload that arithmetic does not produce; should an input NaN carry
// it, the event is merely recomputed.
constexpr unsigned kRedoMarkBits = 0x7fd2e6b1u;
__device__ __forceinline__ float redo_mark() { return __builtin_bit_cast(float, kRedoMarkBits); }
__device__ __forceinline__ bool is_redo_mark(float x) { return __builtin_bit_cast(unsigned, x) == kRedoMarkBits; }

// Cross-lane moves within a wavefront (GFX9 DPP controls): shift right by d
// lanes within each row of 16 lanes, lane 15 of each row to the next row,
// lane 31 to rows 2 and 3, and the whole wavefront right by one lane.  A lane
// whose source does not exist, or whose row is masked off, receives `old`.
constexpr int kDppRowShr = 0x110;
constexpr int kDppRowBcast15 = 0x142;
constexpr int kDppRowBcast31 = 0x143;
constexpr int kDppWaveShr1 = 0x138;
// Within each quad of lanes: lane ^ 1 and lane ^ 2 (quad_perm [1,0,3,2] and
// [2,3,0,1]).
constexpr int kDppQuadXor1 = 0xb1;
constexpr int kDppQuadXor2 = 0x4e;

template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i32(int x, int old) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xf, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x) {  // old = +0
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)dpp_i32<CTRL, ROWS>((int)(unsigned)b, 0);
  const unsigned hi = (unsigned)dpp_i32<CTRL, ROWS>((int)(unsigned)(b >> 32), 0);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_scan_step(double& x, int key) {
  const double y = dpp_f64<CTRL, ROWS>(x);
  const int ky = dpp_i32<CTRL, ROWS>(key, -1);  // -1: never a key
  x = (ky == key) ? x + y : x;
}

// Inclusive segmented sum over a full wavefront: keys do not decrease with the
// lane, and each lane receives the sum of x over the lanes at or below it with
// its key.  Sums within rows by shifts of 1, 2, 4 and 8, then the running row
// totals carried across rows (lane 15 into rows 1 and 3, lane 31 into rows 2
// and 3); a source with another key adds nothing (keys are monotone, so the
// lanes between agree too).  No LDS traffic; all 64 lanes must be active.
__device__ __forceinline__ double seg_scan_wave(double x, int key) {
  seg_scan_step<kDppRowShr + 1, 0xf>(x, key);
  seg_scan_step<kDppRowShr + 2, 0xf>(x, key);
  seg_scan_step<kDppRowShr + 4, 0xf>(x, key);
  seg_scan_step<kDppRowShr + 8, 0xf>(x, key);
  seg_scan_step<kDppRowBcast15, 0xa>(x, key);
  seg_scan_step<kDppRowBcast31, 0xc>(x, key);
  return x;
}

// A best-pair candidate (distance, in-event rank (-1: none), mass) and the
// strict order that picks it: any candidate over none, then the smaller
// distance, then the lower rank.  A total order, so that any grouping of a
// minimum gives the same candidate.
template <typename T>
__device__ __forceinline__ bool cand_better(double d, int r, double od, int orr) {
  return r >= 0 && (orr < 0 || d < od || (d == od && r < orr));
}

template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_t(T x) {  // old = +0
  if constexpr (sizeof(T) == 8)
    return dpp_f64<CTRL, ROWS>(x);
  else
    return __builtin_bit_cast(T, dpp_i32<CTRL, ROWS>(__builtin_bit_cast(int, x), 0));
}

template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ void best_scan_step(double& d, int& r, T& m, int key) {
  const double yd = dpp_f64<CTRL, ROWS>(d);
  const int yr = dpp_i32<CTRL, ROWS>(r, -1);
  const T ym = dpp_t<CTRL, ROWS, T>(m);
  const int ky = dpp_i32<CTRL, ROWS>(key, -1);
  const bool take = ky == key && cand_better<T>(yd, yr, d, r);
  d = take ? yd : d;
  r = take ? yr : r;
  m = take ? ym : m;
}

// Inclusive segmented minimum of candidates over a full wavefront, the network
// of seg_scan_wave.
template <typename T>
__device__ __forceinline__ void best_scan_wave(double& d, int& r, T& m, int key) {
  best_scan_step<kDppRowShr + 1, 0xf, T>(d, r, m, key);
  best_scan_step<kDppRowShr + 2, 0xf, T>(d, r, m, key);
  best_scan_step<kDppRowShr + 4, 0xf, T>(d, r, m, key);
  best_scan_step<kDppRowShr + 8, 0xf, T>(d, r, m, key);
  best_scan_step<kDppRowBcast15, 0xa, T>(d, r, m, key);
  best_scan_step<kDppRowBcast31, 0xc, T>(d, r, m, key);
}

// Deterministic workgroup sum of one double per thread (fixed tree).
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double r = 0.0;
  for (int w = 0; w < nw; ++w) r += red[w];
  __syncthreads();
  return r;
}

template <typename T>
__device__ __forceinline__ void store_out(T* p, int64_t i, T v) {
  __builtin_nontemporal_store(v, p + i);
}

// ---------------------------------------------------------------- forward

struct FwdOut {
  void* total[4];
  void* event_m;
  void* pair_m;
};

template <typename T, int COORDS, int MODE>
struct FwdArgs {
  Cols4<T> p;
  const int64_t* off;
  const int64_t* poff;
  T* total[4];
  T* event_m;
  T* pair_m;
  int64_t* best_rank;  // per-event best pair (fused selection), or NULL
  T* best_m;
  double target;
  unsigned long long* fallback;
  int64_t ne;
  int epb;         // events per wavefront tile
  int cap;         // particles staged per chunk (per wavefront)
  int small;       // events of more particles are left to the second launch (see small_events)
  int qcap;        // pairs evaluated per round (per wavefront)
  int wave_bytes;  // LDS bytes per wavefront
};

// Orders the LDS accesses of the lanes of one wavefront.  The waves of a
// workgroup work independently, so the forward reduction needs no workgroup
// barrier: LDS operations of one wavefront are performed in program order, and
// the fences keep the compiler from moving LDS accesses across this point.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The value of x held by lane `lane` (uniform), for a 64-bit x.
__device__ __forceinline__ int64_t readlane64(int64_t x, int lane) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(uint64_t)x, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)((uint64_t)x >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double lane_value(double x, int lane) {
  return __builtin_bit_cast(double, readlane64(__builtin_bit_cast(int64_t, x), lane));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}

// Last c in [lo, hi) with a[c] <= key (a non-decreasing, a[lo] <= key).
__device__ __forceinline__ int search_le32(const int* a, int lo, int hi, int key) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a[mid] <= key)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The largest events of the first launch.  Where pairs are evaluated it
// depends on their mean number per event, which both launches read: on
// small events the tail of the sizes is better done beside its neighbours
// (up to kDenseFrom particles) than by waking the second launch, and once most
// events are large that launch takes all but the smallest (kDenseLow).  The
// line lies where the two cross for Poisson sizes, by type, mode and number of
// events: with few events the first launch's small tiles spread them as well as
// the second's shares do, and with very many its wavefronts fill the GPU with
// less work per pair.  All but the smallest in the second launch / all in the
// first, plain FP32 of 26 particles 1.24 at 1,000 events, 0.81 at 10,000, 0.98 at
// 100,000, 1.16 at 270,000; FP64 1.19, 0.84, 1.02 and 1.00; compensated FP32 of 24
// 0.97, 0.61, 0.97 and 1.10; compensated FP64 of 20 1.20, 0.87, 0.93 and 0.94;
// best pair FP64 of 32 0.69, 0.74, 1.22 and (200,000) 1.36; compensated best pair
// FP32 of 32 0.64, 0.61, 1.16 and (200,000) 1.20, FP64 0.65, 0.64, 0.96 and 1.04.
// (Best pairs cross at 40 particles from 65,000 events on with the sizes of
// untuned calls; smaller tilings that are given cross earlier, so the line is at
// 36: 100,000 events of 40 at (64, 64, 128, 1024) 434 us in the first launch, 221 in
// the second.)
constexpr int kDenseFrom = 48;
constexpr int kDenseLow = 12;
constexpr int64_t kShareByEvents = 1 << 18;  // see my_share

// That line in pairs per event.
template <typename T, int MODE, bool BEST>
__device__ __forceinline__ int64_t dense_line(int64_t ne) {
  constexpr bool f64 = sizeof(T) == 8, comp = MODE == GLV_COMPENSATED;
  if (ne <= 4096) return BEST ? 480 : comp ? (f64 ? 270 : 290) : 370;
  if (ne <= 49152) return BEST ? 480 : comp ? (f64 ? 170 : 250) : 290;
  if (ne < kShareByEvents) return BEST ? (comp && f64 ? 480 : 640) : comp ? (f64 ? 170 : 290) : 340;
  return BEST ? 640 : comp ? (f64 ? 200 : 400) : f64 ? 340 : 480;
}

template <typename T, int MODE, bool BEST>
__device__ __forceinline__ int small_events(const int64_t* poff, int64_t ne, int small) {
  return poff[ne] >= ne * dense_line<T, MODE, BEST>(ne) ? min(small, kDenseLow) : small;
}

// LDS of one wavefront of the forward reduction (cap particles, qcap pairs):
//   cart[cap]  (px, py, pz, E)             staged Cartesian records
//   leg[2 cap] (pt, eta, phi, M), (mT, delta, mT - pt, M^2) per particle,
//              adjacent (one address for both reads)   compensated mode
//   pm[qcap]   pair masses of a round (stored from here, coalesced); not for
//              FP32 compensated masses
//   kev[epb+1] K of each of the chunk's events with pairs in a round
//              (compensated event mass)
//   bm[epb+1], br[epb+1]  best pair of each of the chunk's events with
//              pairs in a round: mass and in-event rank (-1: none)
//              (fused best-pair selection)
//   eo, en, ep [epb + 1] int               the chunk's events with pairs:
//              first particle, size, first pair (chunk-relative), then a
//              sentinel (np, 0, nq)
template <typename T, int MODE>
struct WaveLds {
  typename V4<T>::type* cart;
  typename V4<T>::type* leg;
  T* pm;
  double* kev;
  T* bm;
  int* br;
  int* eo;
  int* en;
  int* ep;
};

template <typename T, int MODE, bool BEST>
__host__ __device__ __forceinline__ size_t wave_lds_bytes(int cap, int qcap, int epb) {
  size_t b = (size_t)cap * 4 * sizeof(T);
  if (MODE == GLV_COMPENSATED) b += (size_t)cap * 8 * sizeof(T) + (size_t)(epb + 1) * sizeof(double);
  if (BEST)
    b += (size_t)(epb + 1) * (sizeof(T) + sizeof(int));  // each event's best of a round
  else if (sizeof(T) == 8 || MODE == GLV_PLAIN)
    b += (size_t)qcap * sizeof(T);  // staged pair masses
  b += 3 * (size_t)(epb + 1) * sizeof(int);
  return (b + 31) & ~(size_t)31;
}

template <typename T, int MODE, bool BEST>
__device__ __forceinline__ WaveLds<T, MODE> carve_wave_lds(unsigned char* p, int cap, int qcap, int epb) {
  WaveLds<T, MODE> w;
  w.cart = reinterpret_cast<typename V4<T>::type*>(p);
  p += (size_t)cap * 4 * sizeof(T);
  if constexpr (MODE == GLV_COMPENSATED) {
    w.leg = reinterpret_cast<typename V4<T>::type*>(p);
    p += (size_t)cap * 8 * sizeof(T);
    w.kev = reinterpret_cast<double*>(p);
    p += (size_t)(epb + 1) * sizeof(double);
  } else {
    w.leg = nullptr;
    w.kev = nullptr;
  }
  w.pm = reinterpret_cast<T*>(p);
  w.bm = reinterpret_cast<T*>(p);
  if (BEST) {
    p += (size_t)(epb + 1) * sizeof(T);
    w.br = reinterpret_cast<int*>(p);
    p += (size_t)(epb + 1) * sizeof(int);
  } else {
    w.br = nullptr;
    if (sizeof(T) == 8 || MODE == GLV_PLAIN) p += (size_t)qcap * sizeof(T);
  }
  w.eo = reinterpret_cast<int*>(p);
  w.en = w.eo + (epb + 1);
  w.ep = w.en + (epb + 1);
  return w;
}

// Particles of a chunk held in registers between their load and their
// staging: lane t of the wavefront keeps particles t, t + 64, ...; FP64 keeps
// one per lane (64 particles), FP32 two, or three for plain masses, whose
// chunks hold up to 160 (2^20 Poisson(8) events 105 -> 101 us, 2^19 of 14 119 ->
// 115; compensated 179 -> 195).  Two in FP64: 190 -> 199.  Particles of larger
// chunks past these are loaded when staged.
template <typename T, int MODE, bool BEST>
struct Prefetch {
  static constexpr int kSlots = sizeof(T) == 8 ? 1 : MODE == GLV_PLAIN && !BEST ? 3 : 2;
  T v[kSlots][4];
};

template <typename T, int MODE, bool BEST>
__device__ __forceinline__ void prefetch_chunk(const Cols4<T>& p, int64_t base, int np, int lane,
                                               Prefetch<T, MODE, BEST>* r) {
#pragma unroll
  for (int s = 0; s < Prefetch<T, MODE, BEST>::kSlots; ++s) {
    const int t = lane + 64 * s;
    if (t < np) {
#pragma unroll
      for (int k = 0; k < 4; ++k) r->v[s][k] = __builtin_nontemporal_load(p.c[k] + base + t);
    }
  }
}

// Converts one particle and writes its staged records (slot t).
template <typename T, int COORDS, int MODE>
__device__ __forceinline__ void stage_one(const WaveLds<T, MODE>& W, int t, T c0, T c1, T c2, T c3) {
  using R4 = typename V4<T>::type;
  T v[4];
  if constexpr (MODE == GLV_COMPENSATED) {  // (pt, eta, phi, M)
    const LegC<T> L = comp_leg_cart<T>(c0, c1, c2, c3, v);
    W.leg[2 * t] = R4{c0, c1, c2, c3};
    W.leg[2 * t + 1] = R4{L.mt, L.delta, L.dmt, L.m2};
  } else {
    to_cart<COORDS, T, true>(c0, c1, c2, c3, v);
  }
  W.cart[t] = R4{v[0], v[1], v[2], v[3]};
}

// Compensated leg terms of a staged particle, from its two leg records at q;
// *mass receives M.
template <typename T>
__device__ __forceinline__ LegC<T> staged_leg(const typename V4<T>::type* q, T* mass) {
  const typename V4<T>::type a = q[0];
  const typename V4<T>::type b = q[1];
  LegC<T> L;
  L.pt = a[0];
  L.eta = a[1];
  L.phi = a[2];
  *mass = a[3];
  L.mt = b[0];
  L.delta = b[1];
  L.dmt = b[2];
  L.m2 = b[3];
  return L;
}

// The chunk of a wavefront's tile that starts at the first event at or after
// `from` that belongs to this launch (n <= small): [*ca, *cb), the longest run
// of consecutive such events whose particles fit in cap slots (small <= cap)
// and whose pairs number at most pcap (the first event always belongs to it).
// *ca = nev: none left.
__device__ __forceinline__ void next_chunk(int from, int nev, uint64_t valid, bool mine, int64_t olo, int64_t ohi,
                                           int cap, int small, int64_t plo, int64_t phi, int64_t pcap, int* ca,
                                           int* cb) {
  const uint64_t after = from >= 64 ? 0ull : (valid & (~0ull << from));
  const uint64_t ours = __ballot(mine && (ohi - olo) <= (int64_t)small);
  const int a = (ours & after) ? (int)__builtin_ctzll(ours & after) : nev;
  int b = a;
  if (a < nev) {
    const int64_t base = readlane64(olo, a), pbase = readlane64(plo, a);
    const uint64_t ge = valid & (~0ull << a);
    const uint64_t fits = __ballot(mine && (ohi - base <= (int64_t)cap) && (phi - pbase <= pcap)) & ours & ge;
    // the first event always opens the chunk (its pairs then take several rounds)
    const uint64_t stop = ge & ~fits & ~(1ull << a);
    b = stop ? (int)__builtin_ctzll(stop) : nev;
  }
  *ca = a;
  *cb = b;
}

// Wavefronts per SIMD the compiler must leave room for (its register budget):
// five for the FP32 compensated reduction and the plain best pair, which
// otherwise take 107 and 101 VGPRs and four wavefronts (a few bytes then
// spill; on 2^20 events FP32 compensated 233 -> 218 us, fused best pair
// 205 -> 198 us); none for the FP64 compensated mode and the compensated best
// pair, which would spill more (the FP32 one measured 257 -> 292 us); the
// plain reductions fit six anyway.
template <typename T, int MODE, bool BEST>
constexpr int fwd_waves() {
  return (MODE == GLV_COMPENSATED && (sizeof(T) == 8 || BEST)) ? 1 : 5;
}

// The forward reduction.  Each wavefront of a workgroup independently takes a
// tile of epb consecutive events (one per lane for their offsets) and walks it
// in chunks of consecutive events holding at most cap particles; the next
// chunk's particles are loaded into registers while the current one is
// reduced, so that their latency hides behind its arithmetic:
//   1. stage: the chunk's particles are converted once and written to the
//      wave's LDS;
//   2. totals: four lanes per event, each summing one residue class of the
//      particle index modulo 4 in index order, combined as
//      ((P0 + P1) + (P2 + P3)) (the plain event mass from that total; in the
//      compensated mode also the sum of M^2);
//   3. pairs, in rounds: lane L takes the contiguous pairs [L m, (L + 1) m)
//      of the round, locates the first by a binary search over the chunk's
//      events with pairs and the square-root decode of its rank, then steps
//      to the lexicographic successor -- every lane the same number of pairs
//      whatever the event sizes, and a handful of integer operations per
//      step.  Masses go to the wave's LDS, in rounds of 64 m pairs with m odd
//      (which spreads one LDS store instruction's lanes over distinct banks),
//      and from there to pair_m with coalesced stores; those of the FP32
//      compensated mode, whose evaluation hides the scattered stores (189 us
//      against 231 staged on 2^20 Poisson(8) events), are stored by their lane.
//      FP32 plain masses stored by their lane cost 120 us instead of 103, and
//      on 2^19 events of 14 particles, whose runs of pairs are longer than a
//      64-byte segment, 212 instead of 117.  Compensated mode and best pair:
//      rounds of qcap, a chunk holding at most one round of pairs unless a
//      single event has more.  In the compensated mode
//      each lane also sums K = E_i E_j - p_i.p_j of its pairs per event: an
//      event inside one run takes the lane's sum, an event spanning runs the
//      scan of their tails (keyed by event over the lanes) plus the head of
//      the run where it ends; the event's lane adds its K per round:
//      deterministic for a tiling.
// Events with more than `small` particles are left to k_event_dense.  In
// the FP32 compensated mode a pair whose error bound asks for FP64 makes its
// K a NaN; the event's lane then writes a marker -- a quiet NaN with a fixed
// payload -- into the event mass (or, without event masses, into the event's
// first pair mass), and k_event_dense recomputes the event.
template <typename T, int COORDS, int MODE, bool BEST>
__global__ __launch_bounds__(kMaxBlock, (fwd_waves<T, MODE, BEST>())) void k_event_reduce(FwdArgs<T, COORDS, MODE> A) {
  extern __shared__ __align__(32) unsigned char lds[];
  constexpr bool kComp = MODE == GLV_COMPENSATED;
  constexpr bool kDefer = kComp && (sizeof(T) == 4);
  constexpr int kSlots = Prefetch<T, MODE, BEST>::kSlots;
  constexpr bool kStageMasses = (sizeof(T) == 8 || !kComp) && !BEST;
  using R4 = typename V4<T>::type;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nwaves = blockDim.x >> 6;
  const int epb = A.epb, cap = A.cap, qcap = A.qcap;
  const WaveLds<T, MODE> W = carve_wave_lds<T, MODE, BEST>(lds + (size_t)wid * A.wave_bytes, cap, qcap, epb);

  const int64_t e0 = ((int64_t)blockIdx.x * nwaves + wid) * epb;
  if (e0 >= A.ne) return;  // the whole wavefront: no workgroup barrier follows
  const int nev = (int)min((int64_t)epb, A.ne - e0);
  const bool want_pairs = !BEST && A.pair_m != nullptr;
  // FP32 compensated: K is summed whenever pairs are evaluated (a NaN sum marks the redo)
  const bool want_k = kComp && (A.event_m != nullptr || (kDefer && (want_pairs || BEST)));
  const bool need_po = want_pairs || want_k || BEST;
  const bool want_sums = A.total[0] != nullptr || A.event_m != nullptr;

  // this lane's event of the tile
  const bool mine = lane < nev;
  int64_t olo = 0, ohi = 0, plo = 0, phi = 0;
  if (mine) {
    olo = A.off[e0 + lane];
    ohi = A.off[e0 + lane + 1];
    if (need_po) {
      plo = A.poff[e0 + lane];
      phi = A.poff[e0 + lane + 1];
    }
  }
  const uint64_t valid = (nev >= 64) ? ~0ull : ((1ull << nev) - 1);
  const int small = need_po ? small_events<T, MODE, BEST>(A.poff, A.ne, A.small) : A.small;
  // where the rounds hold per-pair partials (compensated, best pair), a chunk
  // takes at most one round of pairs, so that no round runs nearly empty
  // (FP32 compensated 252 -> 241 us, best pair 254 -> 225 us on 2^20
  // Poisson(8) events); an event with more pairs alone takes several rounds
  const int64_t pcap = (kComp || BEST) && need_po ? (int64_t)qcap : ((int64_t)1 << 62);
  unsigned fb = 0;

  int ca, cb;
  next_chunk(0, nev, valid, mine, olo, ohi, cap, small, plo, phi, pcap, &ca, &cb);
  Prefetch<T, MODE, BEST> pre;
  if (ca < nev) {
    const int64_t b0 = readlane64(olo, ca);
    prefetch_chunk(A.p, b0, (int)(readlane64(ohi, cb - 1) - b0), lane, &pre);
  }
  while (ca < nev) {
    const int64_t base = readlane64(olo, ca);
    const int np = (int)(readlane64(ohi, cb - 1) - base);
    const int64_t q0 = need_po ? readlane64(plo, ca) : 0;
    const int nq = need_po ? (int)(readlane64(phi, cb - 1) - q0) : 0;
    const bool in_chunk = lane >= ca && lane < cb;
    const int lo_rel = (int)(olo - base), n_e = (int)(ohi - olo);

    // the chunk's events with pairs, compacted, then the sentinel
    const bool has_pairs = in_chunk && n_e >= 2;
    const uint64_t hp = __ballot(has_pairs);
    const int ncp = __builtin_popcountll(hp);
    const int my_c = __builtin_popcountll(hp & ((1ull << lane) - 1));  // this event among those with pairs
    if (need_po) {
      if (has_pairs) {
        const int c = my_c;
        W.eo[c] = lo_rel;
        W.en[c] = n_e;
        W.ep[c] = (int)(plo - q0);
      }
      if (lane == 0) {
        W.eo[ncp] = np;
        W.en[ncp] = 0;
        W.ep[ncp] = nq;
      }
    }

    // 1. stage the chunk's particles: those held in registers, then any
    //    beyond them straight from memory
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
      const int t = lane + 64 * s;
      if (t < np) stage_one<T, COORDS, MODE>(W, t, pre.v[s][0], pre.v[s][1], pre.v[s][2], pre.v[s][3]);
    }
    for (int t = lane + 64 * kSlots; t < np; t += 64) {
      const int64_t gi = base + t;
      stage_one<T, COORDS, MODE>(W, t, A.p.c[0][gi], A.p.c[1][gi], A.p.c[2][gi], A.p.c[3][gi]);
    }
    wave_sync();

    // the next chunk's particles into registers, in flight from here on
    int na, nb;
    next_chunk(cb, nev, valid, mine, olo, ohi, cap, small, plo, phi, pcap, &na, &nb);
    if (na < nev) {
      const int64_t b1 = readlane64(olo, na);
      prefetch_chunk(A.p, b1, (int)(readlane64(ohi, nb - 1) - b1), lane, &pre);
    }

    // 2. totals: four lanes per event, one residue sum each (residue_sum),
    //    combined across the lane quad in the fixed order, 16 events per
    //    pass; the plain event mass from the total; in the compensated mode
    //    also the sum of M^2, handed to the event's lane
    double msum = 0.0;
    if (want_sums) {
      const int nk = cb - ca;  // events in the chunk
      const int rr = lane & 3;
      const R4* legs = nullptr;
      if constexpr (kComp) legs = W.leg;
      for (int c0 = 0; c0 < nk; c0 += 16) {
        const int c = c0 + (lane >> 2);
        const bool act = c < nk;
        const int src = min(ca + c, 63);
        const int glo = __shfl(lo_rel, src), gn = __shfl(n_e, src);
        const int lo = act ? glo : 0, hi = act ? glo + gn : 0;
        double tot[4] = {0, 0, 0, 0}, ms = 0.0;
        residue_sum(W.cart, lo, hi, rr, tot, legs, &ms);
        // (P0 + P1) + (P2 + P3): partner lane ^ 1, then lane ^ 2, of the quad
#pragma unroll
        for (int k = 0; k < 4; ++k) tot[k] = tot[k] + dpp_f64<kDppQuadXor1, 0xf>(tot[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) tot[k] = tot[k] + dpp_f64<kDppQuadXor2, 0xf>(tot[k]);
        if constexpr (kComp) {
          ms = ms + dpp_f64<kDppQuadXor1, 0xf>(ms);
          ms = ms + dpp_f64<kDppQuadXor2, 0xf>(ms);
        }
        if (act && rr == 0) {
          const int64_t e = e0 + ca + c;
          T tt[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) tt[k] = (T)tot[k];
          if (A.total[0]) {
#pragma unroll
            for (int k = 0; k < 4; ++k) store_out(A.total[k], e, tt[k]);
          }
          if constexpr (!kComp) {
            if (A.event_m) store_out(A.event_m, e, mass_of(tt));
          }
        }
        if constexpr (kComp) {
          // the event lanes of this pass take their quad's sum of M^2
          const int q = lane - ca - c0;
          const double mq = __shfl(ms, min(max(q, 0), 15) << 2);
          if (q >= 0 && q < 16 && in_chunk) msum = mq;
        }
      }
    }

    // 3. pairs, in rounds
    double ks = 0.0;  // the event lane's sum of K (compensated)
    double ebd = 0.0;  // the event lane's best pair (ebr < 0: none yet)
    int ebr = -1;
    T ebm = T(0);
    if (need_po) {
      // the records the pair loop reads per particle: the compensated legs
      // (two records each) or the Cartesian vectors
      constexpr int kStride = kComp ? 2 : 1;
      const R4* const recs = kComp ? W.leg : W.cart;
      const int rcap = kStageMasses ? 64 * (((qcap >> 6) - 1) | 1) : qcap;
      T* const pout = want_pairs ? A.pair_m + q0 : nullptr;
      for (int r0 = 0; r0 < nq; r0 += rcap) {
        const int qn = min(rcap, nq - r0);
        // pairs per lane, odd where the masses pass through LDS
        const int m = kStageMasses ? (((qn + 63) >> 6) | 1) : ((qn + 63) >> 6);
        int k = r0 + lane * m;
        const int kend = min(k + m, r0 + qn);
        // the run's K partials of events it shares with other runs: the head
        // (the end of an event begun before the run) and the tail (the start
        // of an event that goes on after it); events wholly inside the run go
        // to kev directly
        double head = 0.0, tail = 0.0;
        double hd = 0.0, td = 0.0;  // best pair: the head's and the tail's candidates
        int hr = -1, tr = -1;
        T hm = T(0), tm = T(0);
        bool has_head = false, has_tail = false, first_seg = true, began_before = false;
        int head_c = 0, cur_c = ncp;  // cur_c: the run's current event (after a closing pair: the next)
        const bool ran = k < kend;
        if (k < kend) {
          int c = search_le32(W.ep, 0, ncp, k);
          const int o = W.eo[c], n = W.en[c];
          int i, j;
          decode_pair_small(k - W.ep[c], n, &i, &j);
          int cn = c + 1;
          int on = W.eo[cn], nn = W.en[cn];  // the next event with pairs (or the sentinel)
          // the staged records of the pair's two particles and the end of
          // their event, stepped directly (kStride records per particle)
          const R4* qa = recs + kStride * (o + i);
          const R4* qb = recs + kStride * (o + j);
          const R4* qe = recs + kStride * (o + n);
          double kacc = 0.0;
          int rk = k - W.ep[c];  // in-event rank of pair k
          cur_c = c;
          began_before = rk > 0;
          double bdist = 0.0;    // the run's best so far (brk < 0: none)
          int brk = -1;
          T bmass = T(0);
          for (; k < kend; ++k) {
            T mk;
            if constexpr (kComp) {
              T ma, mb;
              const LegC<T> la = staged_leg<T>(qa, &ma), lb = staged_leg<T>(qb, &mb);
              double kd;
              if constexpr (kDefer) {
                bool redo;
                float kf;
                mk = sqrt_budgeted(comp_pair_m2<float>(la, lb, &kf, &redo));
                kd = (double)(redo ? __builtin_nanf("") : kf);
              } else {
                mk = comp_pair<T>(la, lb, ma, mb, &kd, &fb);
              }
              kacc += kd;
            } else {
              const R4 ra = *qa, b = *qb;
              T w[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) w[q] = ra[q] + b[q];
              mk = mass_of(w);
            }
            if constexpr (BEST) {
              // ranks grow along the run, so a tie keeps the earlier pair
              const double d = fabs((double)mk - A.target);
              if (d == d && (brk < 0 || d < bdist)) {
                bdist = d;
                brk = rk;
                bmass = mk;
              }
              ++rk;
            } else if constexpr (kStageMasses) {
              W.pm[k - r0] = mk;
            } else if (want_pairs) {
              pout[k] = mk;
            }
            // lexicographic successor within the chunk
            const int seg_c = cur_c;  // pair k's event
            bool fin = false;
            qb += kStride;
            if (qb == qe) {  // the row's last partner: the next row
              qa += kStride;
              if (qa + kStride == qe) {  // the event's last pair: the next event
                fin = true;
                qa = recs + kStride * on;
                qe = qa + kStride * nn;
                cur_c = cn;
                cn = min(cn + 1, ncp);
                on = W.eo[cn];
                nn = W.en[cn];
              }
              qb = qa + kStride;
            }
            if (fin || k + 1 == kend) {  // the run's partials at its last pair of the event
              // the head ends an event begun in an earlier run, the tail starts
              // one that goes on in the next run; an event wholly inside the
              // run goes to its slot directly
              const bool is_head = fin && first_seg && began_before;
              if constexpr (kComp) {
                if (is_head)
                  head = kacc;
                else if (fin)
                  W.kev[seg_c] = kacc;
                else
                  tail = kacc;
                kacc = 0.0;
              }
              if constexpr (BEST) {
                if (is_head) {
                  hd = bdist;
                  hr = brk;
                  hm = bmass;
                } else if (fin) {
                  W.bm[seg_c] = bmass;
                  W.br[seg_c] = brk;
                } else {
                  td = bdist;
                  tr = brk;
                  tm = bmass;
                }
                brk = -1;
                rk = 0;
              }
              if (is_head) {
                has_head = true;
                head_c = seg_c;
              }
              has_tail = !fin;
              first_seg = false;
            }
          }
        }
        // Each shared event's K (best pair): the tails of the runs it spans,
        // combined by a segmented scan keyed by event, then with the head of
        // the run where it ends; an event that goes on into the next round
        // takes the scan at the round's last run.  Keys grow with the lane: 2e
        // for a tail on event e, 2e + 1 for a run whose last event e closed in
        // it (cur_c is then e + 1), past every event for a run without pairs.
        const int key = has_tail ? 2 * cur_c : (ran ? 2 * cur_c - 1 : 2 * ncp + 1);
        if constexpr (BEST) {
          double sd = has_tail ? td : 0.0;
          int sr = has_tail ? tr : -1;
          T sm = has_tail ? tm : T(0);
          best_scan_wave<T>(sd, sr, sm, key);
          const double pd = dpp_f64<kDppWaveShr1, 0xf>(sd);
          const int pr = dpp_i32<kDppWaveShr1, 0xf>(sr, -1);
          const T pmv = dpp_t<kDppWaveShr1, 0xf, T>(sm);
          const int pk = dpp_i32<kDppWaveShr1, 0xf>(key, -1);
          if (has_head) {
            // the earlier runs' best, unless the head's is strictly better
            const bool from_prev = pk == 2 * head_c;
            double bd = from_prev ? pd : 0.0;
            int brr = from_prev ? pr : -1;
            T bmv = from_prev ? pmv : T(0);
            if (cand_better<T>(hd, hr, bd, brr)) {
              brr = hr;
              bmv = hm;
            }
            W.bm[head_c] = bmv;
            W.br[head_c] = brr;
          }
          if (has_tail && kend == r0 + qn) {
            W.bm[cur_c] = sm;
            W.br[cur_c] = sr;
          }
        }
        if constexpr (kComp) {
          if (want_k) {
            const double sc = seg_scan_wave(has_tail ? tail : 0.0, key);
            const double sp = dpp_f64<kDppWaveShr1, 0xf>(sc);
            const int kp = dpp_i32<kDppWaveShr1, 0xf>(key, -1);
            if (has_head) W.kev[head_c] = (kp == 2 * head_c ? sp : 0.0) + head;
            if (has_tail && kend == r0 + qn) W.kev[cur_c] = sc;
          }
        }
        wave_sync();
        if (kStageMasses && want_pairs) {
          T* out = A.pair_m + q0 + r0;
          for (int t = lane; t < qn; t += 64) store_out(out, t, W.pm[t]);
        }
        if constexpr (kComp) {
          if (want_k && in_chunk && n_e >= 2) {
            const int plo_rel = (int)(plo - q0), phi_rel = (int)(phi - q0);
            if (max(plo_rel, r0) < min(phi_rel, r0 + qn)) ks += W.kev[my_c];  // pairs in this round
          }
        }
        if constexpr (BEST) {
          if (in_chunk && n_e >= 2) {
            const int plo_rel = (int)(plo - q0), phi_rel = (int)(phi - q0);
            if (max(plo_rel, r0) < min(phi_rel, r0 + qn)) {  // pairs in this round (in rank order)
              const int r = W.br[my_c];
              if (r >= 0) {
                const T bmv = W.bm[my_c];
                const double d = fabs((double)bmv - A.target);
                if (ebr < 0 || d < ebd) {
                  ebd = d;
                  ebr = r;
                  ebm = bmv;
                }
              }
            }
          }
        }
        wave_sync();
      }
    }
    bool marked = false;  // FP32 compensated: a pair of the event asked for the FP64 redo
    if constexpr (kComp) {
      if (want_k && in_chunk) {
        marked = kDefer && (ks != ks) && n_e >= 2;
        if (A.event_m) {
          T em = (T)sqrt(msum + 2.0 * ks);
          if constexpr (kDefer) {
            if (marked) em = redo_mark();
          }
          store_out(A.event_m, e0 + lane, em);
        } else if (!BEST) {
          if constexpr (kDefer) {
            // without event masses the mark goes to the event's first pair
            // mass, after this wavefront's own stores of the chunk's masses
            if (__ballot(marked)) {
              // every earlier store of the wavefront completes first
              __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
              if (marked) A.pair_m[plo] = redo_mark();
            }
          }
        }
      }
    }
    if constexpr (BEST) {
      // without event masses a redo mark goes to the event's best mass
      if (in_chunk) {
        const bool mark_here = marked && A.event_m == nullptr;
        A.best_rank[e0 + lane] = ebr;
        store_out(A.best_m, e0 + lane, mark_here ? redo_mark() : (ebr >= 0 ? ebm : (T)__builtin_nan("")));
      }
    }
    wave_sync();
    ca = na;
    cb = nb;
  }
  if constexpr (kComp && sizeof(T) == 4) {
    if (A.fallback) {
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) fb += __shfl_xor(fb, d);
      if (lane == 0 && fb) atomicAdd(A.fallback, (unsigned long long)fb);
    }
  }
}

// ------------------------------------- forward, events of many particles
//
// Events of more than `small` particles, which k_event_reduce leaves out.
// Two launches share the work by events' pairs, so that neither a few large
// events nor a few events in all leave the chip idle:
//   * plain pair masses: the pairs of all events (pair_offsets is their scan)
//     are cut into equal runs, one per workgroup, an event's pairs falling
//     to as many workgroups as its size asks for;
//   * K sums (compensated event mass) and the best pair need one result per
//     event: a workgroup takes every event whose first pair lies in its run.
// (From kShareByEvents events on the events are dealt out instead, and one that
// is larger than all others together is one workgroup's in any mode.)
// A workgroup finds its first event by interpolation or a search of
// pair_offsets, reads the sizes of several thousand events at a time
// (scan_share) and lists the ones that are its business.  It stages runs of
// listed events (dense_cap particles) in LDS, converted once per workgroup, and
// deals the staged events' pairs to its wavefronts as equal runs of the folded
// pairs (Folded), 64 per step, so that the masses go out as runs of consecutive
// addresses straight from registers and a step's bookkeeping is the same for
// every lane.  What bounds it: VALU issue for two thirds of it (54 instructions
// per 64 FP32 pairs, staging and totals included: 39 us), then waits on the
// stores and on LDS: 57 us on 4,096 FP32 events of 96 particles on average, up to
// 1,024 (2.8e7 pairs); 27 ms with one workgroup per event, 72 us with unfolded
// rows and streaming stores.
// An event that does not fit dense_cap slots is walked in tiles of half as many
// rows by half as many columns, one row per wavefront.

// Particles staged per chunk (LDS: 16 KB of records in FP64, 8 KB in FP32, 24 KB
// with the legs of the compensated mode in either).
template <typename T, int MODE>
constexpr int dense_cap() {
  return (MODE == GLV_COMPENSATED && sizeof(T) == 8) ? 256 : 512;
}
constexpr int kDenseEvents = 64;  // events per chunk (one lane each)
constexpr int kDenseMinPairs = 2048;  // pairs a workgroup takes at least, of few events

template <int MODE, bool BEST>
constexpr bool dense_owned() {  // events stay with one workgroup
  return MODE == GLV_COMPENSATED || BEST;
}
template <int MODE, bool BEST>
constexpr int dense_block() {
  return MODE != GLV_COMPENSATED && BEST ? 512 : 256;
}

// Workgroups of the large-event launches: what the GPU holds at once (four of
// 256 threads per CU, three with the registers of the compensated mode, or two
// of 512), so that on small events, where they only read the pair offsets,
// they take one round.  No variant uses scratch memory where that can be
// helped: it made the same scan take 14 us instead of 6 on 2^19 events.
template <int MODE, bool BEST>
constexpr int dense_grid() {
  return MODE == GLV_COMPENSATED ? 768 : BEST ? 512 : 1024;
}

// Slices of events a workgroup of those launches reads at once: 4,096 events, or
// 3,072, or 2,048 in the compensated mode, whose registers have no room for
// more (twelve slices: 44 bytes of scratch memory, and best pairs of 100,000
// FP64 events of 8 particles take 66 us instead of 63).
template <int MODE, bool BEST>
constexpr int dense_slices() {
  return MODE == GLV_COMPENSATED || BEST ? 8 : 12;
}

// The events a workgroup of the large-event launches has to do among B
// consecutive ones: first particle, size, first pair, and 2 (index in the
// slice) + flag.
template <int B>
struct EventList {
  int64_t lo[B], po[B];
  int n[B], e[B];
  int cnt[B / 64];
};

// Lists the threads' events with `mine`, in order, event `index` of the slice;
// returns their number.
template <int B>
__device__ __forceinline__ int list_events(EventList<B>& L, bool mine, int index, int64_t lo, int n, int64_t po,
                                           bool flag) {
  const int lane = (int)threadIdx.x & 63, wid = (int)threadIdx.x >> 6;
  const uint64_t mk = __ballot(mine);
  __syncthreads();  // the previous list is no longer read
  if (lane == 0) L.cnt[wid] = __builtin_popcountll(mk);
  __syncthreads();
  int at = 0, all = 0;
#pragma unroll
  for (int w = 0; w < B / 64; ++w) {
    const int c = L.cnt[w];
    at += w < wid ? c : 0;
    all += c;
  }
  if (mine) {
    at += __builtin_popcountll(mk & ((1ull << lane) - 1));
    L.lo[at] = lo;
    L.n[at] = n;
    L.po[at] = po;
    L.e[at] = (index << 1) | (flag ? 1 : 0);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(all);
}

// The share of the calling workgroup in the large-event launches: the pairs of
// all events, whose scan is pair_offsets, cut into one equal run [q0, q1) per
// workgroup, of at least min_pairs.  Neighbouring runs go to workgroups of the
// same XCD (dispatched round-robin over the eight), whose L2 then serves the
// pair offsets both read.  From kShareByEvents events on the events themselves
// are dealt out (dealt_event), and every pair offset is read once: 5.0 us
// against 6.9 on 2^19 small FP64 events, 6.9 against 15.0 on 2^21, where shares of
// pairs need windows of several times their events.  Large events, also
// neighbouring ones, then go to many workgroups, but each one whole to its own
// (2^18 events, 1,000 neighbours of 100 particles among them: forward 112 us, best
// pair 119, reverse mode 299; 939, 1895 and 3066 where a workgroup took a run of
// 256 events; 54, 49 and 102 with shares of pairs, one event fewer.  One event of
// 3,000 particles: 3.0 ms, 83 us with shares).
// GRID, the number of workgroups, is a constant of each kernel: the divisions by
// it were a third of the instructions of a launch that finds nothing.
template <int GRID>
__device__ __forceinline__ int share_index() {
  static_assert(GRID % 8 == 0, "one run of shares per XCD");
  return (int)((blockIdx.x & 7) * (GRID / 8) + (blockIdx.x >> 3));
}
template <int GRID>
__device__ __forceinline__ Share my_share(int64_t nq, int64_t min_pairs) {
  return pair_share(nq, min_pairs, GRID, share_index<GRID>());
}

// An event e with poff[e] <= q at most `within` events before the last such
// one, by probing 1024 evenly spread pair offsets per round.
template <int B>
__device__ __forceinline__ int64_t search_share(const int64_t* __restrict__ poff, int64_t ne, int64_t q,
                                                int64_t within, int* cnt) {
  constexpr int kProbes = 1024 / B;
  const int tid = (int)threadIdx.x;
  int64_t lo = 0, hi = ne;
  while (hi - lo > within) {
    const int64_t step = (hi - lo + 1023) >> 10;
    int c = 0;
#pragma unroll
    for (int k = 0; k < kProbes; ++k) {
      const int64_t at = lo + step * (tid + B * k);
      c += __builtin_popcountll(__ballot(at < hi && poff[min(at, ne)] <= q));
    }
    __syncthreads();
    if ((tid & 63) == 0) cnt[tid >> 6] = c;
    __syncthreads();
    c = 0;
#pragma unroll
    for (int w = 0; w < B / 64; ++w) c += cnt[w];
    const int64_t top = lo + step * __builtin_amdgcn_readfirstlane(c);  // c >= 1: poff[lo] <= q
    lo = top - step;
    hi = min(hi, top);
  }
  return lo;
}

struct Nothing {};  // what peek returns where the pair offsets tell all

// What a thread sees of its events of a window, one per slice: event e of slice
// sl is wins + at + sl STEP.
template <int SLICES, int STEP, typename Seen>
struct Window {
  // the low words do where the window holds fewer than 2^32 pairs (half the
  // registers); the list looks at the whole offsets
  unsigned po[SLICES], pe[SLICES];
  Seen seen[SLICES];

  // Slices past the window's last event are not read.
  template <typename Peek>
  __device__ __forceinline__ void read(const int64_t* __restrict__ poff, int64_t wins, int at, int last, Peek peek) {
#pragma unroll
    for (int sl = 0; sl < SLICES; ++sl) {
      po[sl] = pe[sl] = 0;
      seen[sl] = {};
      if (sl > 0 && sl * STEP > last) continue;
      const int t = min(sl * STEP + at, last);
      const unsigned* const low = reinterpret_cast<const unsigned*>(poff + wins);
      po[sl] = low[2 * t];
      pe[sl] = low[2 * t + 2];
      seen[sl] = peek(wins + t);
    }
    // nothing of a slice is looked at, and waited for, before all are on their way
    if constexpr (!__is_same(Seen, Nothing)) {
#pragma unroll
      for (int sl = 0; sl < SLICES; ++sl) asm volatile("" : "+v"(seen[sl]));
    }
  }

  // Bit sl: the thread's event of slice sl is picked, or has to be looked at whole.
  template <typename Pick>
  __device__ __forceinline__ unsigned picked(int64_t at0, int64_t at1, int64_t end, int at, int last, Pick pick) const {
    const bool wide = at1 - at0 >= ((int64_t)1 << 32);
    unsigned some = 0;
#pragma unroll
    for (int sl = 0; sl < SLICES; ++sl) {
      const int64_t q = at0 + (unsigned)(po[sl] - (unsigned)at0);
      if (sl * STEP + at <= last && (wide || (q < end && pick(seen[sl], q, (int64_t)(unsigned)(pe[sl] - po[sl])))))
        some |= 1u << sl;
    }
    return some;
  }
};

// Calls body(win, listed) with the whole workgroup for every slice of B events
// that has events e with pick(peek(e), po, d) in its share (first pair po, d
// pairs; peek reads what else tells), listed in L in order with their index
// from event wins on and flag(d).  The pair offsets of up to kSlices slices are
// read at once, first around the place where the share would begin if all events
// had the same number of pairs, so that where no event is the workgroup's
// business, as on small events, the scan costs one memory latency; a share that
// begins outside is searched for.  Such a launch takes 5.6 us on 4,096 FP64
// events and 6.0 on 100,000, FP32 compensated 5.4 and 6.3; with windows of all
// slices and 2,048 pairs to a share 6.8, 7.8, 11.0 and 10.1.
template <int B, int GRID, int kSlices, typename Peek, typename Pick, typename Flag, typename Body>
__device__ __forceinline__ void scan_share(const int64_t* __restrict__ off, const int64_t* __restrict__ poff,
                                           int64_t ne, EventList<B>& L, Share* share, Peek peek, Pick pick, Flag flag,
                                           Body body) {
  constexpr int64_t kWin = (int64_t)kSlices * B;
  // few pairs fill fewer workgroups, but only where one window holds all events:
  // the place of such shares is not known before the number of pairs (20,000
  // events of 8 particles, all outputs, FP32 17.6 -> 14.9 us, FP64 20.0 -> 17.1)
  const int64_t min_pairs = ne > kWin ? 64 : kDenseMinPairs;
  using Seen = decltype(peek((int64_t)0));
  const int tid = (int)threadIdx.x;
  const bool dealt = ne >= kShareByEvents;
  int64_t wins = 0;  // the window's first event
  int tries = 0;
  bool more = true;
  int64_t win = kWin;  // events of a window, whole slices
  if (!dealt) {
    // Where equal events would put the share.  For sizes drawn alike the place is
    // off by 0.4 sqrt(ne) events (Poisson sizes of 8) to 0.9 (a long tail), one
    // standard deviation; the window has 2 sqrt(ne) on either side.
    if (ne > kWin) {
      const int need = (int)ne / GRID + (int)(4.0f * __builtin_amdgcn_sqrtf((float)ne));
      win = B * min(kSlices, 1 + need / B);
    }
    wins = ne * share_index<GRID>() / GRID - (win - ne / GRID) / 2;
    wins = max((int64_t)0, min(wins, ne - win));
    tries = 2;
  }
  while (more) {
    const int64_t span = dealt ? kWin * GRID : win;  // events the window reaches over
    const int64_t wend = min(wins + span, ne);
    const int64_t at0 = poff[wins], at1 = poff[wend], nq = poff[ne];
    const int last = (int)(wend - wins) - 1;
    unsigned some;
    if (dealt) {
      const int at = dealt_event<B>(tid, share_index<GRID>(), GRID);
      Window<kSlices, B * GRID, Seen> w;
      w.read(poff, wins, at, last, peek);
      *share = whole_share(nq);
      some = w.picked(at0, at1, nq, at, last, pick);
    } else {
      Window<kSlices, B, Seen> w;
      w.read(poff, wins, tid, last, peek);
      if (tries) {
        *share = my_share<GRID>(nq, min_pairs);
        if (share->q0 >= share->q1) return;
        if (at0 > share->q0 || at1 <= share->q0) {  // begins elsewhere
          if (--tries && share->q1 - share->q0 == min_pairs) {  // few pairs: shares larger than the grid's equal ones
            wins = (int64_t)((double)ne * (double)share->q0 / (double)nq) - win / 2;
            wins = max((int64_t)0, min(wins, ne - win));
          } else {
            wins = search_share<B>(poff, ne, share->q0, win / 4, L.cnt);
            tries = 0;
          }
          continue;
        }
        tries = 0;
      }
      some = w.picked(at0, at1, share->q1, tid, last, pick);
    }
    more = wend < ne && at1 < share->q1;
    if (__syncthreads_or(some != 0)) {
#pragma unroll 1
      for (int sl = 0; sl < kSlices; ++sl) {
        bool mine = (some >> sl) & 1u;
        if (!__syncthreads_or(mine)) continue;
        const int index = dealt ? dealt_event<B>(tid, share_index<GRID>(), GRID) + sl * (B * GRID) : tid + sl * B;
        const int64_t e = wins + index;
        int64_t first = 0, n = 0, po = 0, d = 0;
        if (mine) {
          first = off[e];
          n = off[e + 1] - first;
          po = poff[e];
          d = npairs(n);
          mine = po < share->q1 && pick(peek(e), po, d);
        }
        const int listed = list_events<B>(L, mine, index, first, (int)n, po, mine && flag(d));
        body(wins, listed);
      }
    }
    wins += span;
  }
}

// Inclusive sum over the lanes at or below this one.
__device__ __forceinline__ int wave_incl_sum(int x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  return x;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

// Sum over the wavefront by lane moves: rows of 16 lanes, then across rows.
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_f64<kDppRowShr + 1, 0xf>(v);
  v += dpp_f64<kDppRowShr + 2, 0xf>(v);
  v += dpp_f64<kDppRowShr + 4, 0xf>(v);
  v += dpp_f64<kDppRowShr + 8, 0xf>(v);
  v += dpp_f64<kDppRowBcast15, 0xa>(v);
  v += dpp_f64<kDppRowBcast31, 0xc>(v);
  return lane_value(v, 63);
}

// A best-pair candidate by the bits of its distance (which order as unsigned
// integers; ~0: none), then its rank.
template <typename T, typename R>
struct Cand {
  unsigned long long d;
  R r;
  T m;
  __device__ __forceinline__ void offer(unsigned long long od, R orr, T om) {
    if (od < d || (od == d && orr < r)) {
      d = od;
      r = orr;
      m = om;
    }
  }
};

template <typename T, typename R>
__device__ __forceinline__ void wave_best(Cand<T, R>& c) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    const unsigned long long od = __shfl_xor(c.d, d);
    const R orr = __shfl_xor(c.r, d);
    const T om = __shfl_xor(c.m, d);
    c.offer(od, orr, om);
  }
}

// Total (and sum of M^2) of a staged event of more than kQuadMax particles,
// by one wavefront: 256 strided partial sums, a butterfly per 64 of them, the
// four results added in order.
constexpr int kQuadMax = 128;
template <typename V>
__device__ __forceinline__ void tree_sum(const V* rec, int n, int lane, double tot[4], const V* legs, double* m2) {
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    double acc[4] = {0, 0, 0, 0}, ms = 0.0;
    for (int t = w * 64 + lane; t < n; t += 256) {
      const V r = rec[t];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] += (double)r[k];
      if (legs) {
        const double m = (double)legs[2 * t][3];
        ms += m * m;
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) tot[k] += wave_sum(acc[k]);
    if (legs) *m2 += wave_sum(ms);
  }
}

// The pairs of an event of n particles (2 <= n <= 512) folded into a rectangle
// of rows of equal length w: row i of the pairs followed by the row that
// completes it, n - 1 - i (n even, w = n - 1) or n - 2 - i (n odd, w = n).
// Position `at` goes through it 64 at a time with one comparison per step,
// whatever the rows' lengths; (i, i + 1 + y) is the pair there.
struct Folded {
  int n, w, c;     // c - i: the completing row
  int rows, rest;  // 64 positions: so many rows and the rest
  int at, i0, x;
  __device__ __forceinline__ Folded(int n_, int f) : n(n_), at(f) {
    w = n - 1 + (n & 1);
    c = n - 1 - (n & 1);
    rows = 64 / w;
    rest = 64 - rows * w;
    // the row: exact, as (f + 1/2) / w stays 1 / (2 w) > 2^-10 from an integer
    // and the quotient, at most 256, is off by less than 2^-13
    i0 = (int)(((float)f + 0.5f) * __builtin_amdgcn_rcpf((float)w));
    x = f - (int)__umul24(i0, w);
  }
  __device__ __forceinline__ void step() {
    at += 64;
    x += rest;
    const bool over = x >= w;
    x = over ? x - w : x;
    i0 += rows + (over ? 1 : 0);
  }
  __device__ __forceinline__ void pair(int* i, int* y) const {
    const int len = n - 1 - i0;
    const bool first = x < len;
    *i = first ? i0 : c - i0;
    *y = first ? x : x - len;
  }
};

template <typename T, int COORDS, int MODE, bool BEST>
__global__ __launch_bounds__((dense_block<MODE, BEST>()),
                             (MODE == GLV_COMPENSATED ? 3 : 4)) void k_event_dense(FwdArgs<T, COORDS, MODE> A) {
  constexpr bool kComp = MODE == GLV_COMPENSATED;
  constexpr bool kDefer = kComp && sizeof(T) == 4;
  constexpr bool kOwn = dense_owned<MODE, BEST>();
  constexpr int B = dense_block<MODE, BEST>();
  constexpr int NW = B / 64;
  constexpr int kCap = dense_cap<T, MODE>();
  constexpr int kHalf = kCap / 2;
  using R4 = typename V4<T>::type;
  __shared__ R4 cart[kCap];
  __shared__ R4 leg[kComp ? 2 * kCap : 1];
  __shared__ EventList<B> L;                               // flag: redo only
  __shared__ double kpart[kComp ? NW * kDenseEvents : 1];  // K of an event from each wavefront
  __shared__ double kmsum[kComp ? kDenseEvents : 1];       // an event's sum of M^2
  __shared__ unsigned long long bd[BEST ? NW * kDenseEvents : 1];  // best pair from each wavefront
  __shared__ int64_t br[BEST ? NW * kDenseEvents : 1];
  __shared__ T bm[BEST ? NW * kDenseEvents : 1];
  __shared__ double red[16];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);

  const bool want_pairs = !BEST && (!kComp || A.pair_m != nullptr);  // plain: pairs are all that brings it here
  const bool want_k = kComp && A.event_m != nullptr;
  const bool want_sums = A.total[0] != nullptr || A.event_m != nullptr;
  unsigned fb = 0;

  // mass of the pair of staged particles i, j
  auto pair_of = [&](int i, int j, double* kd) -> T {
    if constexpr (kComp) {
      T ma, mb;
      const LegC<T> la = staged_leg<T>(leg + 2 * i, &ma), lb = staged_leg<T>(leg + 2 * j, &mb);
      return comp_pair<T>(la, lb, ma, mb, kd, &fb);
    } else {
      const R4 a = cart[i], b = cart[j];
      T w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = a[k] + b[k];
      return pair_mass_of(w);
    }
  };
  auto stage = [&](int slot, int64_t gi) {
    T v[4];
    const T c0 = A.p.c[0][gi], c1 = A.p.c[1][gi], c2 = A.p.c[2][gi], c3 = A.p.c[3][gi];
    if constexpr (kComp) {
      const LegC<T> L = comp_leg_cart<T>(c0, c1, c2, c3, v);
      leg[2 * slot] = R4{c0, c1, c2, c3};
      leg[2 * slot + 1] = R4{L.mt, L.delta, L.dmt, L.m2};
    } else {
      to_cart<COORDS, T, true>(c0, c1, c2, c3, v);
    }
    cart[slot] = R4{v[0], v[1], v[2], v[3]};
  };
  auto finish_total = [&](int64_t e, const double* tot) {
    T tt[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tt[k] = (T)tot[k];
    if (A.total[0]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) A.total[k][e] = tt[k];
    }
    if constexpr (!kComp) {
      if (A.event_m) A.event_m[e] = mass_of(tt);
    }
  };
  auto offer = [&](auto& c, T m, auto r) {
    const double d = fabs((double)m - A.target);
    if (d == d) c.offer((unsigned long long)__double_as_longlong(d), r, m);
  };

  Share sh;
  const int64_t small_pairs = npairs(small_events<T, MODE, BEST>(A.poff, A.ne, A.small));
  // the event's place for a redo mark (without event masses or best pairs: its
  // first pair mass, looked at by picked(); what is read here is then unused, but
  // read without a branch, so that all slices' reads are in flight together)
  const T* const marks = A.event_m ? A.event_m : BEST ? A.best_m : reinterpret_cast<const T*>(A.poff);
  auto peek = [&](int64_t e) {
    if constexpr (kDefer)
      return marks[e];
    else
      return Nothing{};
  };
  // whether an event (first pair po, d pairs) is this workgroup's business
  auto picked = [&](auto seen, int64_t po, int64_t d) -> bool {
    if (kOwn ? po < sh.q0 : po + d <= sh.q0) return false;
    if constexpr (kDefer) {
      if (d > 0 && d <= small_pairs) {
        if (!A.event_m && !BEST) return is_redo_mark(A.pair_m[po]);
        return is_redo_mark(seen);
      }
    }
    return d > small_pairs;
  };
  auto redo_only = [&](int64_t d) { return d <= small_pairs; };

  auto work = [&](int64_t win, int total_listed) {
    const int64_t q0 = sh.q0, q1 = sh.q1;
    for (int li = 0; li < total_listed;) {
      // chunk: one lane per event from li on (each wavefront forms it alike)
      const bool have = li + lane < total_listed;
      int64_t clo = 0, cpo = 0;
      int cn = 0, ce = 0;
      if (have) {
        clo = L.lo[li + lane];
        cn = L.n[li + lane];
        cpo = L.po[li + lane];
        ce = L.e[li + lane];
      }
      const int cn32 = min(cn, kCap + 1);
      const int incl = wave_incl_sum(cn32, lane);
      const int nc = __builtin_popcountll(__ballot(have && incl <= kCap));
      if (nc == 0) {
        // one event of more than kCap particles, in tiles
        const int64_t hlo = L.lo[li], hn = L.n[li], hpo = L.po[li], he = win + (L.e[li] >> 1);
        const int64_t hq = npairs(hn);
        const int64_t r0 = kOwn ? 0 : max((int64_t)0, q0 - hpo), r1 = kOwn ? hq : min(hq, q1 - hpo);
        double msum = 0.0;
        if (r0 == 0 && want_sums) {  // 256 strided partial sums, as tree_sum
          double acc[4] = {0, 0, 0, 0}, ms = 0.0;
          if (tid < 256) {
            for (int64_t i = hlo + tid; i < hlo + hn; i += 256) {
              T v[4];
              to_cart<COORDS, T, true>(A.p.c[0][i], A.p.c[1][i], A.p.c[2][i], A.p.c[3][i], v);
#pragma unroll
              for (int k = 0; k < 4; ++k) acc[k] += (double)v[k];
              if constexpr (kComp) ms += (double)A.p.c[3][i] * (double)A.p.c[3][i];
            }
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[k] = block_sum(acc[k], red);
          if constexpr (kComp) msum = block_sum(ms, red);
          if (tid == 0) finish_total(he, acc);
        }
        int64_t i0, i1, jt;
        decode_pair(r0, hn, &i0, &jt);
        decode_pair(r1 - 1, hn, &i1, &jt);
        double kacc = 0.0;
        Cand<T, int64_t> best{~0ull, 0, T(0)};
        T* const pout = want_pairs ? A.pair_m + hpo : nullptr;
        for (int64_t ta = i0; ta <= i1; ta += kHalf) {
          const int64_t tae = min(i1 + 1, ta + kHalf);  // rows [ta, tae)
          for (int64_t tb = ta + 1; tb < hn; tb += kHalf) {
            const int64_t tbe = min(hn, tb + kHalf);  // columns [tb, tbe)
            __syncthreads();
            for (int t = tid; t < kCap; t += B) {
              const int64_t g = t < kHalf ? ta + t : tb + (t - kHalf);
              if (g < (t < kHalf ? tae : tbe)) stage(t, hlo + g);
            }
            __syncthreads();
            for (int64_t i = ta + wid; i < tae; i += NW) {
              const int64_t rs = row_start(i, hn) - i - 1;  // rank of (i, j) is rs + j
              const int64_t jb = max(max(tb, i + 1), r0 - rs), je = min(tbe, r1 - rs);
              for (int64_t j = jb + lane; j < je; j += 64) {
                double kd;
                const T m = pair_of((int)(i - ta), kHalf + (int)(j - tb), &kd);
                if constexpr (kComp) kacc += kd;
                if (want_pairs) store_out(pout, rs + j, m);
                if constexpr (BEST) offer(best, m, rs + j);
              }
            }
          }
        }
        if constexpr (kComp) {
          if (want_k) {
            kacc = block_sum(kacc, red);
            if (tid == 0) A.event_m[he] = (T)sqrt(msum + 2.0 * kacc);
          }
        }
        if constexpr (BEST) {
          wave_best(best);
          __syncthreads();
          if (lane == 0) {
            bd[wid] = best.d;
            br[wid] = best.r;
            bm[wid] = best.m;
          }
          __syncthreads();
          if (tid == 0) {
            for (int w = 1; w < NW; ++w) best.offer(bd[w], br[w], bm[w]);
            const bool found = best.d != ~0ull;
            A.best_rank[he] = found ? best.r : -1;
            A.best_m[he] = found ? best.m : (T)__builtin_nan("");
          }
        }
        __syncthreads();
        ++li;
        continue;
      }
      const bool in = lane < nc;
      const int slot0 = in ? incl - cn32 : kCap;  // first slot of this lane's event
      const int np = __shfl(incl, nc - 1);
      int r0 = 0, cq = 0;  // the event's first rank and number of pairs here
      if (in) {
        const int q = (int)npairs(cn);
        const int64_t a = kOwn ? 0 : max((int64_t)0, q0 - cpo), b = kOwn ? q : min((int64_t)q, q1 - cpo);
        r0 = (int)a;
        cq = (int)(b - a);
      }
      const int qincl = wave_incl_sum(cq, lane);
      const int p0 = in ? qincl - cq : 0x7fffffff;  // first pair of this lane's event in the chunk
      const int ptot = __shfl(qincl, nc - 1);

      // stage: each slot's event by a binary search over the lanes' first slots
      for (int t0 = 0; t0 < np; t0 += B) {
        const int t = t0 + tid;
        int c = 0;
#pragma unroll
        for (int d = kDenseEvents / 2; d > 0; d >>= 1) {
          const int s = __shfl(slot0, c + d);
          c = s <= t ? c + d : c;
        }
        const int64_t plo = __shfl(clo, c);
        const int ps = __shfl(slot0, c);
        if (t < np) stage(t, plo + (t - ps));
      }
      if constexpr (kComp) {
        for (int t = tid; t < NW * kDenseEvents; t += B) kpart[t] = 0.0;
      }
      if constexpr (BEST) {
        for (int t = tid; t < NW * kDenseEvents; t += B) bd[t] = ~0ull;
      }
      __syncthreads();

      // totals: events of at most kQuadMax particles by a quad of lanes, 16
      // events per wavefront, the others by one wavefront each
      if (want_sums) {
        const R4* legs = nullptr;
        if constexpr (kComp) legs = leg;
        for (int c0 = wid * 16; c0 < nc; c0 += NW * 16) {
          const int c = c0 + (lane >> 2), src = min(c, 63);
          const int s0 = __shfl(slot0, src), n0 = __shfl(cn32, src), rr0 = __shfl(r0, src), e0 = __shfl(ce, src);
          const bool act = c < nc && n0 <= kQuadMax && rr0 == 0;
          double tot[4] = {0, 0, 0, 0}, ms = 0.0;
          residue_sum(cart, act ? s0 : 0, act ? s0 + n0 : 0, lane & 3, tot, legs, &ms);
#pragma unroll
          for (int k = 0; k < 4; ++k) tot[k] = tot[k] + dpp_f64<kDppQuadXor1, 0xf>(tot[k]);
#pragma unroll
          for (int k = 0; k < 4; ++k) tot[k] = tot[k] + dpp_f64<kDppQuadXor2, 0xf>(tot[k]);
          if constexpr (kComp) {
            ms = ms + dpp_f64<kDppQuadXor1, 0xf>(ms);
            ms = ms + dpp_f64<kDppQuadXor2, 0xf>(ms);
          }
          if (act && (lane & 3) == 0) {
            if constexpr (kComp) kmsum[c] = ms;
            if (!(e0 & 1)) finish_total(win + (e0 >> 1), tot);
          }
        }
        uint64_t wide = __ballot(in && cn32 > kQuadMax && r0 == 0);
        for (int turn = 0; wide; ++turn, wide &= wide - 1) {
          if (turn % NW != wid) continue;
          const int c = (int)__builtin_ctzll(wide);
          const int s0 = __builtin_amdgcn_readlane(slot0, c), n0 = __builtin_amdgcn_readlane(cn32, c);
          const int e0 = __builtin_amdgcn_readlane(ce, c);
          double tot[4] = {0, 0, 0, 0}, ms = 0.0;
          tree_sum(cart + s0, n0, lane, tot, legs ? legs + 2 * s0 : legs, &ms);
          if (lane == 0) {
            if constexpr (kComp) kmsum[c] = ms;
            if (!(e0 & 1)) finish_total(win + (e0 >> 1), tot);
          }
        }
      }

      // pairs: each wavefront a contiguous run of the chunk's, whole steps of
      // 64 but for the last
      const int share = ((ptot + B - 1) / B) * 64;
      const int ka = wid * share, kb = min(ka + share, ptot);
      for (int c = (int)__builtin_popcountll(__ballot(p0 <= ka)) - 1, k = ka; k < kb; ++c) {
        const int s0 = __builtin_amdgcn_readlane(slot0, c), n0 = __builtin_amdgcn_readlane(cn32, c);
        const int pb = __builtin_amdgcn_readlane(p0, c);
        const int rb = __builtin_amdgcn_readlane(r0, c);
        const int ke = min(kb, pb + __builtin_amdgcn_readlane(cq, c));
        T* const pout = want_pairs ? A.pair_m + readlane64(cpo, c) : nullptr;
        double kacc = 0.0;
        Cand<T, int> best{~0ull, 0, T(0)};
        const int fe = rb + (ke - pb);
        Folded f(n0, rb + (k - pb) + lane);
        for (; f.at < fe; f.step()) {
          int i, y;
          f.pair(&i, &y);
          const unsigned r = (unsigned)row_start32(i, n0) + (unsigned)y;  // its rank
          double kd;
          const T m = pair_of(s0 + i, s0 + i + 1 + y, &kd);
          if constexpr (kComp) kacc += kd;
          if (want_pairs)  // a 32-bit offset: at most kCap particles
            *reinterpret_cast<T*>(reinterpret_cast<char*>(pout) + r * (unsigned)sizeof(T)) = m;
          if constexpr (BEST) offer(best, m, (int)r);
        }
        if constexpr (kComp) {
          if (want_k) {
            kacc = wave_sum(kacc);
            if (lane == 0) kpart[wid * kDenseEvents + c] = kacc;
          }
        }
        if constexpr (BEST) {
          wave_best(best);
          if (lane == 0) {
            bd[wid * kDenseEvents + c] = best.d;
            br[wid * kDenseEvents + c] = best.r;
            bm[wid * kDenseEvents + c] = best.m;
          }
        }
        k = ke;
      }
      __syncthreads();
      if constexpr (kOwn) {
        if (wid == 0 && in) {
          const int64_t ev = win + (ce >> 1);
          if constexpr (kComp) {
            if (want_k) {
              double ks = 0.0;
              for (int w = 0; w < NW; ++w) ks += kpart[w * kDenseEvents + lane];
              A.event_m[ev] = (T)sqrt(kmsum[lane] + 2.0 * ks);
            }
          }
          if constexpr (BEST) {
            Cand<T, int64_t> best{~0ull, 0, T(0)};
            for (int w = 0; w < NW; ++w) {
              const int t = w * kDenseEvents + lane;
              if (bd[t] != ~0ull) best.offer(bd[t], br[t], bm[t]);
            }
            const bool found = best.d != ~0ull;
            A.best_rank[ev] = found ? best.r : -1;
            A.best_m[ev] = found ? best.m : (T)__builtin_nan("");
          }
        }
        __syncthreads();  // kpart, kmsum and the candidates are free again
      }
      li += nc;
    }
  };
  scan_share<B, dense_grid<MODE, BEST>(), dense_slices<MODE, BEST>()>(A.off, A.poff, A.ne, L, &sh, peek, picked, redo_only, work);
  if constexpr (kDefer) {
    if (A.fallback) {
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) fb += __shfl_xor(fb, d);
      if (lane == 0 && fb) atomicAdd(A.fallback, (unsigned long long)fb);
    }
  }
}

// Without pairs to evaluate (no pair offsets then), the events of more than
// cap particles: the workgroup scans the offsets for them and sums each one
// whole, from global memory; on collider-sized events it only reads the
// offsets.
constexpr int kBigBlock = 256;
// Events each thread sizes per pass (kBigScan coalesced slices of kBigBlock
// events): all their offsets are read at once, so the scan of 2^20 events
// takes one or two memory latencies per workgroup with a grid that fits the
// GPU.
constexpr int kBigScan = 4;

// Sizes of events base + k kBigBlock + threadIdx.x, k < kBigScan, or -1 past
// the last event.
__device__ __forceinline__ void scan_sizes(const int64_t* off, int64_t ne, int64_t base, int64_t n[kBigScan]) {
  int64_t lo[kBigScan], hi[kBigScan];
#pragma unroll
  for (int k = 0; k < kBigScan; ++k) {
    const int64_t e = base + k * kBigBlock + threadIdx.x;
    lo[k] = 0;
    hi[k] = -1;
    if (e < ne) {
      lo[k] = off[e];
      hi[k] = off[e + 1];
    }
  }
#pragma unroll
  for (int k = 0; k < kBigScan; ++k) n[k] = hi[k] - lo[k];
}

// Calls event(e) with the whole workgroup for every event with picked(n).
template <typename Pick, typename Event>
__device__ __forceinline__ void scan_events(const int64_t* off, int64_t ne, Pick picked, Event event) {
  __shared__ int64_t list[kBigBlock];
  __shared__ int count;
  const int64_t step = (int64_t)gridDim.x * kBigBlock * kBigScan;
  for (int64_t base = (int64_t)blockIdx.x * kBigBlock * kBigScan; base < ne; base += step) {
    int64_t n[kBigScan];
    scan_sizes(off, ne, base, n);
    unsigned bigm = 0;  // bit k: event k of this thread
#pragma unroll
    for (int k = 0; k < kBigScan; ++k)
      if (n[k] >= 0 && picked(n[k])) bigm |= 1u << k;
#pragma unroll 1
    for (int k = 0; k < kBigScan; ++k) {
      const bool big = (bigm >> k) & 1u;
      if (!__syncthreads_or(big)) continue;
      if (threadIdx.x == 0) count = 0;
      __syncthreads();
      if (big) list[atomicAdd(&count, 1)] = base + k * kBigBlock + threadIdx.x;
      __syncthreads();
      const int nbig = count;
      for (int b = 0; b < nbig; ++b) event(list[b]);
      __syncthreads();
    }
  }
}

template <typename T, int COORDS, int MODE>
__global__ __launch_bounds__(kBigBlock) void k_event_totals_big(FwdArgs<T, COORDS, MODE> A) {
  __shared__ double red[16];
  scan_events(A.off, A.ne, [&](int64_t n) { return n > A.cap; }, [&](int64_t e) {
    const int64_t lo = A.off[e], hi = A.off[e + 1];
    double acc[4] = {0, 0, 0, 0};
    for (int64_t i = lo + threadIdx.x; i < hi; i += kBigBlock) {
      T v[4];
      to_cart<COORDS>(A.p.c[0][i], A.p.c[1][i], A.p.c[2][i], A.p.c[3][i], v);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] += (double)v[k];
    }
    T tot[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tot[k] = (T)block_sum(acc[k], red);
    if (threadIdx.x == 0) {
      if (A.total[0]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) A.total[k][e] = tot[k];
      }
      if (MODE != GLV_COMPENSATED && A.event_m) A.event_m[e] = mass_of(tot);
    }
  });
}

// --------------------------------------------------------------- backward

template <typename T, int COORDS>
struct BwdArgs {
  Cols4<T> p;
  const int64_t* off;
  const int64_t* poff;
  const T* gt[4];
  const T* gem;
  const T* gpair;
  const T* tot[4];  // the forward's event totals, or null: recomputed
  T* gp[4];
  int64_t ne;
  int epb;         // events per wavefront tile
  int cap;         // particles staged per chunk (per wavefront)
  int qcap;        // pair upstreams staged per chunk (per wavefront)
};

// An event the tiled backward leaves to the second launch: more than
// cap particles or, with pair upstreams, more than qcap pairs.
__device__ __forceinline__ bool bwd_big(int64_t n, int cap, int qcap, bool pairs) {
  return n > cap || (pairs && npairs(n) > (int64_t)qcap);
}

// LDS-staged backward.  A workgroup takes tiles of epb consecutive events and
// walks each in chunks of consecutive events with at most cap particles (one
// per thread: cap <= block) and, when pair upstreams are given, at most qcap
// pairs:
//   * thread t converts particle t of the chunk once, keeps its Cartesian
//     vector and Jacobian pieces (cos phi, sin phi, sinh eta, cosh eta) in
//     registers and stages the vector in LDS for its partners; the chunk's
//     pair upstreams -- contiguous in grad_pair -- are copied to LDS, two
//     loads in flight per thread; one lane per event records its particles'
//     event;
//   * pair phase: each pair's upstream g_ij becomes c_ij = g_ij / |m_ij| in
//     place, computed once, by one of its two legs: particle a of an event of
//     n takes the partners a + 1, ..., a + d cyclically, d = (n - 1) / 2
//     rounded down, plus a + n/2 when n is even and a < n/2 -- every pair
//     once, about n/2 per particle, whatever the particle's place;
//   * in the same phase a quad of threads per event sums the event's vectors
//     V as the forward does (or the event's lane, which loaded its g_total
//     and g_m with the chunk, takes V from the forward's totals), and
//     g_total + g_m dm(V)/dV, the upstream every particle of the event
//     receives from the event outputs, is staged;
//   * thread t sums the pair terms c_ij (v_i + v_j) = c_ij v_i + c_ij v_j
//     (dm(w)/dw = (-P, E) / |m|, the same 4-vector for both legs of a pair)
//     of its own pairs while evaluating them, then walks the partners that
//     evaluated its other pairs (b = a - d cyclically, stepping the pair
//     indices incrementally), adds the event's upstream and applies its own
//     conversion Jacobian.
// Every sum has a fixed order and no atomics are needed.  Six wavefronts per
// SIMD (what the LDS of the default tiling allows): the compiler keeps the
// registers within that (a few bytes spilled in FP64), 318 -> 309 us on 2^20
// events against its own choice of five.
template <typename T, int COORDS>
__global__ __launch_bounds__(kMaxBlock, 6) void k_event_reduce_bwd(BwdArgs<T, COORDS> A) {
  extern __shared__ __align__(32) unsigned char lds[];
  using R4 = typename V4<T>::type;
  const int epb = A.epb, cap = A.cap;  // cap <= blockDim.x
  const bool pairs = A.gpair != nullptr;
  const bool want_v = A.gem != nullptr;
  const int qcap = pairs ? A.qcap : 0;
  const int tid = (int)threadIdx.x;
  const bool want_u = want_v || A.gt[0] != nullptr;
  // LDS: cart[cap], s_ut[epb] (R4), s_g[qcap + 2] (T; qcap is even, one
  //      slot of slack), s_gm[epb rounded up to even] (T), s_off[epb+1],
  //      s_poff[epb+1] (int64), ch[epb+1] (EvRec), ev_of[cap] (uint16)
  R4* cart = reinterpret_cast<R4*>(lds);
  R4* s_ut = cart + cap;
  T* s_g = reinterpret_cast<T*>(s_ut + epb);
  T* s_gm = s_g + A.qcap + 2;
  int64_t* s_off = reinterpret_cast<int64_t*>(s_gm + ((epb + 1) & ~1));
  int64_t* s_poff = s_off + (epb + 1);
  EvRec* ch = reinterpret_cast<EvRec*>(s_poff + (epb + 1));
  unsigned short* ev_of = reinterpret_cast<unsigned short*>(ch + (epb + 1));
  // event lanes: event t of a chunk belongs to thread (t % nw) * 64 + t / nw,
  // spread over the workgroup's nw wavefronts (the block is a power of two
  // >= 64 and a chunk has at most epb <= block events); tev is the inverse
  const int nw = (int)blockDim.x >> 6;
  const int tev = (tid & 63) * nw + (tid >> 6);
  const int64_t ntiles = (A.ne + epb - 1) / epb;

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t e0 = tile * epb;
    const int nev = (int)min((int64_t)epb, A.ne - e0);
    for (int i = tid; i <= nev; i += blockDim.x) {
      s_off[i] = A.off[e0 + i];
      if (pairs) s_poff[i] = A.poff[e0 + i];
    }
    __syncthreads();
    int ca = 0;
    while (ca < nev) {
      if (bwd_big(s_off[ca + 1] - s_off[ca], cap, qcap, pairs)) {  // the second launch's event
        ++ca;
        continue;
      }
      // largest cb with at most cap particles (and qcap pairs) from ca
      int cb = search_le(s_off, ca + 1, nev + 1, s_off[ca] + cap);
      if (pairs) cb = min(cb, search_le(s_poff, ca + 1, nev + 1, s_poff[ca] + qcap));
      const int nch = cb - ca;
      const int64_t pbase = s_off[ca];
      const int64_t q0 = pairs ? s_poff[ca] : 0;
      const int np = (int)(s_off[cb] - pbase);
      const int nq = pairs ? (int)(s_poff[cb] - q0) : 0;
      const bool mine = tid < np;
      const int64_t gi = pbase + tid;
      // loads first: own particle, the first pair upstreams
      T c[4] = {0, 0, 0, 0};
      if (mine) {
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = A.p.c[k][gi];
      }
      // pair upstreams per thread in flight (two: 317 against 325 us for four
      // on 2^20 events, whose registers cost occupancy)
      constexpr int kG = 2;
      T gv[kG];
#pragma unroll
      for (int r = 0; r < kG; ++r) {
        const int idx = tid + r * (int)blockDim.x;
        gv[r] = (idx < nq) ? A.gpair[q0 + idx] : T(0);
      }
      // the event lane's upstreams (g_total, g_m), staged with the rest
      const bool evl = want_u && tev < nch;
      const bool given_v = want_v && A.tot[0] != nullptr;  // the forward's totals: no sum here
      T gtv[4] = {0, 0, 0, 0}, gmv = 0, tv[4] = {0, 0, 0, 0};
      if (evl) {
        const int64_t e = e0 + ca + tev;
        if (A.gt[0]) {
#pragma unroll
          for (int k = 0; k < 4; ++k) gtv[k] = A.gt[k][e];
        }
        if (want_v) gmv = A.gem[e];
        if (given_v) {
#pragma unroll
          for (int k = 0; k < 4; ++k) tv[k] = A.tot[k][e];
        }
      }
      for (int t = tid; t <= nch; t += blockDim.x)
        ch[t] = EvRec{(int)(s_off[ca + t] - pbase), pairs ? (int)(s_poff[ca + t] - q0) : 0};
      for (int t = tid; t < nch; t += blockDim.x) {
        const int lo = (int)(s_off[ca + t] - pbase), hi = (int)(s_off[ca + t + 1] - pbase);
        for (int i = lo; i < hi; ++i) ev_of[i] = (unsigned short)t;
      }
#pragma unroll
      for (int r = 0; r < kG; ++r) {
        const int idx = tid + r * (int)blockDim.x;
        if (idx < nq) s_g[idx] = gv[r];
      }
      // upstreams past the first kG per thread (pairs_per_round > kG block)
      for (int base = kG * (int)blockDim.x; base < nq; base += kG * (int)blockDim.x) {
#pragma unroll
        for (int r = 0; r < kG; ++r) {
          const int idx = base + tid + r * (int)blockDim.x;
          gv[r] = (idx < nq) ? A.gpair[q0 + idx] : T(0);
        }
#pragma unroll
        for (int r = 0; r < kG; ++r) {
          const int idx = base + tid + r * (int)blockDim.x;
          if (idx < nq) s_g[idx] = gv[r];
        }
      }
      if (evl) {
        if (given_v) {  // g_total + g_m dm(V)/dV at once, from the forward's V
          T ud[4];
          dmass<T>(tv, gmv, ud);
          s_ut[tev] = R4{ud[0] + gtv[0], ud[1] + gtv[1], ud[2] + gtv[2], ud[3] + gtv[3]};
        } else {
          s_ut[tev] = R4{gtv[0], gtv[1], gtv[2], gtv[3]};
        }
        s_gm[tev] = gmv;
      }
      LegJ<T> L = to_cart_j<COORDS, T, true>(c[0], c[1], c[2], c[3]);
      if (mine) cart[tid] = R4{L.v[0], L.v[1], L.v[2], L.v[3]};
      __syncthreads();

      // four lanes per event (events spread over the wavefronts like the
      // event lanes): the upstream every particle's 4-vector receives from
      // the event outputs, g_total + g_m dm(V)/dV, with V summed as the
      // forward sums it (the same residue sums, combined in the same order)
      if (want_v && !given_v) {
        const int rr = tid & 3;
        const int qe = ((tid & 63) >> 2) * nw + (tid >> 6);
        for (int c0 = 0; c0 < nch; c0 += (int)blockDim.x >> 2) {
          const int c = c0 + qe;
          const bool act = c < nch;
          int lo = 0, hi = 0;
          if (act) {
            lo = ch[c].o;
            hi = ch[c + 1].o;
          }
          double vt[4] = {0, 0, 0, 0};
          residue_sum(cart, lo, hi, rr, vt);
#pragma unroll
          for (int k = 0; k < 4; ++k) vt[k] = vt[k] + dpp_f64<kDppQuadXor1, 0xf>(vt[k]);
#pragma unroll
          for (int k = 0; k < 4; ++k) vt[k] = vt[k] + dpp_f64<kDppQuadXor2, 0xf>(vt[k]);
          if (act && rr == 0) {
            T tot[4], ud[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) tot[k] = (T)vt[k];
            dmass<T>(tot, s_gm[c], ud);
            const R4 gt4 = s_ut[c];
            s_ut[c] = R4{ud[0] + gt4[0], ud[1] + gt4[1], ud[2] + gt4[2], ud[3] + gt4[3]};
          }
        }
      }

      // Pair ranks inside an event: pair (b, a), b < a, sits at
      // R(b) + a - b - 1, which grows by n - b - 2 with b; pair (a, b), b > a,
      // at R(a) + b - a - 1, consecutive from R(a) = a (2n - a - 1) / 2.
      int ev = 0, n = 0, ai = 0;
      EvRec rc{0, 0};
      if (mine) {
        ev = ev_of[tid];
        rc = ch[ev];
        n = ch[ev + 1].o - rc.o;
        ai = tid - rc.o;
      }
      const int qrow = rc.p + (int)(__umul24(ai, 2 * n - ai - 1) >> 1);
      // S = sum of c_ab v_b and C = sum of c_ab over the partners b: the
      // thread's own pairs as it evaluates them, then (after the barrier) the
      // pairs its partners evaluated -- an order fixed by the event alone
      T S[4] = {0, 0, 0, 0}, C = 0;
      const int cnt = ((n - 1) >> 1) + ((n & 1) == 0 && 2 * ai < n ? 1 : 0);
      if (pairs) {
        if (mine) {
          int qlo = rc.p + ai - 1, qhi = qrow;
          for (int t = 0, b = ai + 1; t < cnt; ++t, ++b) {
            const bool wrap = b >= n;
            const int bb = wrap ? b - n : b;
            const int q = wrap ? qlo : qhi;
            const T g = s_g[q];
            const R4 vj = cart[rc.o + bb];
            T w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = L.v[k] + vj[k];
            const T cf = pair_coef<T>(w, g);
            s_g[q] = cf;
#pragma unroll
            for (int k = 0; k < 4; ++k) S[k] += cf * vj[k];
            C += cf;
            if (wrap)
              qlo += n - bb - 2;
            else
              ++qhi;
          }
        }
      }
      if (pairs || want_u) __syncthreads();  // s_g and s_ut complete

      if (mine) {
        T u[4] = {0, 0, 0, 0};
        if (want_u) {
          const R4 ut = s_ut[ev];
#pragma unroll
          for (int k = 0; k < 4; ++k) u[k] = ut[k];
        }
        if (pairs && n > 1) {
          // the pairs evaluated by the partners b = a - d (cyclically),
          // d = 1, ..., n - 1 - cnt: pair (b, a) at R(b) + a - b - 1 while
          // b < a (R(b - 1) = R(b) - (n - b)), pair (a, b) at R(a) + b - a - 1
          // once b wraps to n - 1, n - 2, ...
          const int inc = n - 1 - cnt;
          int b = ai - 1, qlo = qrow - (n - ai), qhi = qrow + n - 2 - ai;
          for (int t = 0; t < inc; ++t) {
            const bool below = b >= 0;
            const int bb = below ? b : b + n;
            const T cs = s_g[below ? qlo : qhi];
            const R4 vj = cart[rc.o + bb];
#pragma unroll
            for (int k = 0; k < 4; ++k) S[k] += cs * vj[k];
            C += cs;
            if (below)
              qlo -= n - b - 1;
            else
              --qhi;
            --b;
          }
          // sum of c_ab (v_a + v_b) = C v_a + S, with dm/dw = (-P, E) / |m|
#pragma unroll
          for (int k = 0; k < 3; ++k) u[k] -= C * L.v[k] + S[k];
          u[3] += C * L.v[3] + S[3];
        }
        T g[4];
        chain_coords<COORDS, T>(L, c[0], c[3], u, g);
#pragma unroll
        for (int k = 0; k < 4; ++k) store_out(A.gp[k], gi, g[k]);
      }
      __syncthreads();
      ca = cb;
    }
  }
}

// Backward of the events k_event_reduce_bwd leaves out when there are no
// pair upstreams (more than cap particles): every particle's share of the
// event outputs.
template <typename T, int COORDS>
__global__ __launch_bounds__(kBigBlock) void k_event_reduce_bwd_big(BwdArgs<T, COORDS> A) {
  __shared__ double red[16];
  scan_events(A.off, A.ne, [&](int64_t n) { return n > A.cap; }, [&](int64_t e) {
    const int64_t lo = A.off[e], hi = A.off[e + 1];
    T ut[4] = {0, 0, 0, 0};
    if (A.gem) {
      T tot[4];
      if (A.tot[0]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) tot[k] = A.tot[k][e];
      } else {
        double acc[4] = {0, 0, 0, 0};
        for (int64_t i = lo + threadIdx.x; i < hi; i += kBigBlock) {
          T v[4];
          to_cart<COORDS>(A.p.c[0][i], A.p.c[1][i], A.p.c[2][i], A.p.c[3][i], v);
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[k] += (double)v[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) tot[k] = (T)block_sum(acc[k], red);
      }
      dmass<T>(tot, A.gem[e], ut);
    }
    if (A.gt[0]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) ut[k] += A.gt[k][e];
    }
    for (int64_t i = lo + threadIdx.x; i < hi; i += kBigBlock) {
      const T c0 = A.p.c[0][i], c3 = A.p.c[3][i];
      const LegJ<T> L = to_cart_j<COORDS, T>(c0, A.p.c[1][i], A.p.c[2][i], c3);
      T g[4];
      chain_coords<COORDS, T>(L, c0, c3, ut, g);
#pragma unroll
      for (int k = 0; k < 4; ++k) store_out(A.gp[k], i, g[k]);
    }
    __syncthreads();
  });
}

// ------------------------------------ backward, events of many particles
//
// With pair upstreams, the events k_event_reduce_bwd leaves out.  Each event
// is cut into blocks of 32 particles, which stand at equal distances in the
// event's run of pairs, and a workgroup takes the blocks that stand in its
// equal share of all pairs, its wavefronts in turn.  A block is summed by one
// wavefront, without atomics or workgroup barriers, and a large event spreads
// over many.
//
// A block: lane l of either half of the wavefront owns particle a0 + (l & 31)
// and goes through the event's partners 64 at a time, the halves taking 32
// partners each.  The partners' Cartesian vectors are converted by the lanes
// and staged in the wavefront's LDS; their pair upstreams come in batches of
// kBatch partners per half: rows (b, a0..a0+31) of partners before the block
// lie over the lanes, those after it along the lanes' own rows and are read
// as 64- or 128-byte pieces; both are laid out in LDS as one row per lane.
// The next batch's upstreams and the next partners are in flight while a
// batch is evaluated.  Every ordered pair's c = g/|m| is evaluated by the lane
// that needs it: twice per pair, where a shared evaluation would need a second
// pass over the batch and sums across wavefronts.  Bound by VALU issue for two
// thirds of it (55 instructions per 64 ordered FP32 pairs: 79 us), then by waits
// on the upstreams: 111 us on the events named at k_event_dense (44 ms with one
// workgroup per event; 202 us with blocks of 64 particles whose partners the
// workgroup staged).
//
// Workgroups: what the GPU holds at once, as for the forward (four per CU, three
// with the registers and LDS of FP64; at 1,024 in FP64 the rest started when the
// first were done: 8.0 -> 5.5 us on 2^19 small events, and 93 -> 70 us on 200 of 300
// particles).
template <typename T>
constexpr int bwd_dense_grid() {
  return sizeof(T) == 4 ? 1024 : 768;
}
template <typename T>
constexpr int batch_cols() {
  return sizeof(T) == 4 ? 16 : 8;
}

// Pair (i, j) of an event of n sits at row_at(i) + j; rows_on(d, left) is
// row_at(i + d) - row_at(i) for left = n - i.
__device__ __forceinline__ int64_t row_at(int64_t i, int64_t n) { return row_start(i, n) - i - 1; }
__device__ __forceinline__ unsigned rows_on(unsigned d, unsigned left) {
  return __umul24(d, left) - d - (__umul24(d, d + 1) >> 1);
}

template <typename T, int COORDS>
__global__ __launch_bounds__(256, (sizeof(T) == 4 ? 4 : 3)) void k_event_bwd_dense(BwdArgs<T, COORDS> A) {
  using R4 = typename V4<T>::type;
  constexpr int B = 256, NW = 4;
  constexpr int kC = batch_cols<T>(), kPitch = kC + 1;
  constexpr int kRows = 32 / kC;  // rows of a block a half reads per load after the block
  __shared__ R4 carts[NW][64];
  __shared__ R4 owns[NW][64];  // a block's particles: Jacobian pieces, (c0, c3), until the end
  __shared__ T tiles[NW][64 * kPitch];
  __shared__ EventList<B> L;
  const int tid = (int)threadIdx.x, lane = tid & 63, half = lane >> 5, al = lane & 31;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  R4* const cart = carts[wid];
  T* const tile = tiles[wid];
  const bool want_v = A.gem != nullptr;
  const bool sum_v = want_v && A.tot[0] == nullptr;

  // One block: particles [a0, a0 + 32) of the event at lo with n particles
  // and upstreams g.
  auto block = [&](int64_t ev, int64_t lo, int n, const T* g, int a0) {
    const int a = min(a0 + al, n - 1);  // past the event: its last particle again, not stored
    const int64_t ai = lo + a;
    R4* const own = owns[wid] + 2 * al;
    T v[4] = {A.p.c[0][ai], A.p.c[1][ai], A.p.c[2][ai], A.p.c[3][ai]};  // its coordinates, then its vector
    T S[4] = {0, 0, 0, 0};  // sum of c (v_a + v_b)
    T up = 0;  // the event's upstreams: g_total in lanes 0-3, g_m in 4, the given totals in 5-8
    double acc[4] = {0, 0, 0, 0};
    // Tile t0: partners [t0, t0 + 64), split evenly between the halves in
    // whole batches; batch c of a tile: partners b = t0 + hw half + kC c, ...
    T gv[kC];  // the upstreams on their way
    T nx[4];   // the partner on its way
    auto half_width = [&](int t0) { return min(32, ((n - t0 + 2 * kC - 1) / (2 * kC)) * kC); };
    int t0 = 0, c = 0, hw = half_width(0);    // the batch to load next
    int pt0 = 0, pc = 0, phw = 0;             // the batch loaded before
    bool last = false;
#pragma unroll 1
    for (bool loaded = false; !last; loaded = true) {
      last = t0 >= n;  // nothing left to load
      const int pb = pt0 + phw * half + pc * kC;
      if (loaded) {  // the last batch (and its partners) into LDS
        const bool before = pb < a0;
        wave_sync();  // what is overwritten has been read
        if (pc == 0) {
          T x[4];
          to_cart<COORDS, T, true>(nx[0], nx[1], nx[2], nx[3], x);
          cart[lane] = R4{x[0], x[1], x[2], x[3]};
          if (sum_v && pt0 + lane < n) {
#pragma unroll
            for (int d = 0; d < 4; ++d) acc[d] += (double)x[d];
          }
        }
        T* w = tile + (half * 32 + (before ? al : al / kC)) * kPitch + (before ? 0 : al % kC);
        const int ws = before ? 1 : kRows * kPitch;
#pragma unroll
        for (int u = 0; u < kC; ++u) w[u * ws] = gv[u];
        wave_sync();
      }
      if (!last) {  // the next batch on its way
        if (c == 0) {
          const int64_t i = lo + min(t0 + lane, n - 1);
#pragma unroll
          for (int d = 0; d < 4; ++d) nx[d] = A.p.c[d][i];
        }
        const int bk0 = t0 + c * kC, bk = bk0 + hw * half;
        const bool before = bk < a0;
        const int r0 = a0 + al / kC, col = bk + al % kC;
        // rows are addressed from row ub (its last pair is there: `spare`)
        const int ub = min(bk0, a0);
        const unsigned left = (unsigned)(n - ub), spare = (unsigned)(n - 1) * sizeof(T);
        const char* const base = reinterpret_cast<const char*>(g + row_at(ub, n));
        if (__ballot(bk >= a0 && bk < a0 + 32)) {  // a half inside the block: either order of the pair
#pragma unroll
          for (int u = 0; u < kC; ++u) {
            const int r = r0 + u * kRows, i = before ? bk + u : min(r, col), j = before ? a : max(r, col);
            const unsigned at = (rows_on((unsigned)(i - ub), left) + (unsigned)j) * sizeof(T);
            gv[u] = *reinterpret_cast<const T*>(base + (i != j && j < n ? at : spare));
          }
        } else {
          // before: rows bk + u at column a; after: rows r0 + kRows u at column col
          const int row = before ? bk : r0, by = before ? 1 : kRows;
          const int rows = before ? kC : col < n ? (n - r0 + kRows - 1) / kRows : 0;  // of them in the event
          unsigned at = (rows_on((unsigned)(row - ub), left) + (unsigned)(before ? a : col)) * sizeof(T);
          unsigned step = ((unsigned)(n - 1 - row) * by - (before ? 1u : kRows * (kRows + 1) / 2)) * sizeof(T);
          const unsigned dec = (before ? 1 : kRows * kRows) * sizeof(T);
          if (__ballot(rows < kC)) {
#pragma unroll
            for (int u = 0; u < kC; ++u) {
              gv[u] = *reinterpret_cast<const T*>(base + (u < rows ? at : spare));
              at += step;
              step -= dec;
            }
          } else {
#pragma unroll
            for (int u = 0; u < kC; ++u) {
              gv[u] = *reinterpret_cast<const T*>(base + at);
              at += step;
              step -= dec;
            }
          }
        }
      } else {  // the event's upstreams on their way during the last batch
        const T* at = nullptr;
        if (want_v) at = lane == 4 ? A.gem : at;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          at = lane == d ? A.gt[d] : at;
          if (want_v && !sum_v) at = lane == 5 + d ? A.tot[d] : at;
        }
        if (at) up = at[ev];
      }
      if (!loaded) {
        const LegJ<T> J = to_cart_j<COORDS, T, true>(v[0], v[1], v[2], v[3]);
        if (half == 0) {
          own[0] = R4{J.cp, J.sp, J.sh, J.ch};
          own[1] = R4{v[0], v[3], 0, 0};
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = J.v[d];
      }
      if (loaded) {  // the batch in LDS
        const T* const mine = tile + lane * kPitch;
        const R4* const vb = cart + (pb - pt0);
        // partners this lane has here: none past the event, not itself
        const int have = min(kC, n - pb), self = a0 + al - pb;
        if (__ballot(have < kC || (self >= 0 && self < kC))) {
#pragma unroll 2
          for (int u = 0; u < kC; ++u) {
            const R4 q = vb[u];
            T w[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d] = v[d] + q[d];
            T cf = pair_coef<T>(w, mine[u]);
            cf = (u < have && u != self) ? cf : T(0);
#pragma unroll
            for (int d = 0; d < 4; ++d) S[d] += cf * w[d];
          }
        } else {
#pragma unroll (sizeof(T) == 4 ? 4 : 2)
          for (int u = 0; u < kC; ++u) {
            const R4 q = vb[u];
            T w[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d] = v[d] + q[d];
            const T cf = pair_coef<T>(w, mine[u]);
#pragma unroll
            for (int d = 0; d < 4; ++d) S[d] += cf * w[d];
          }
        }
      }
      pt0 = t0;
      pc = c;
      phw = hw;
      c += 1;
      if (c * kC >= hw) {
        t0 += 64;
        c = 0;
        hw = half_width(t0);
      }
    }
    // the halves' sums, then the event's upstream
#pragma unroll
    for (int k = 0; k < 4; ++k) S[k] += __shfl_xor(S[k], 32);
    T ut[4] = {0, 0, 0, 0};
    if (want_v) {
      T tot[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) tot[k] = sum_v ? (T)wave_total(acc[k]) : lane_value(up, 5 + k);
      dmass<T>(tot, lane_value(up, 4), ut);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) ut[k] += lane_value(up, k);
    if (half == 0 && a0 + al < n) {
      T u[4], gr[4];
#pragma unroll
      for (int k = 0; k < 3; ++k) u[k] = ut[k] - S[k];
      u[3] = ut[3] + S[3];
      const R4 o0 = own[0], o1 = own[1];
      const LegJ<T> J{{v[0], v[1], v[2], v[3]}, o0[0], o0[1], o0[2], o0[3]};
      chain_coords<COORDS, T>(J, o1[0], o1[1], u, gr);
#pragma unroll
      for (int k = 0; k < 4; ++k) store_out(A.gp[k], ai, gr[k]);
    }
  };

  Share sh;
  int turn = 0;  // the workgroup's blocks so far: its wavefronts take them in turn
  const int64_t cap_pairs = npairs(A.cap);
  scan_share<B, bwd_dense_grid<T>(), 12>(
      A.off, A.poff, A.ne, L, &sh,
      [](int64_t) { return Nothing{}; },
      [&](Nothing, int64_t po, int64_t d) { return po + d > sh.q0 && (d > A.qcap || d > cap_pairs); },
      [](int64_t) { return false; },
      [&](int64_t win, int listed) {
        for (int li = 0; li < listed; ++li) {
          const int64_t lo = readlane64(L.lo[li], 0), po = readlane64(L.po[li], 0);
          const int n = __builtin_amdgcn_readfirstlane(L.n[li]);
          const int64_t ev = win + (__builtin_amdgcn_readfirstlane(L.e[li]) >> 1);
          const BlockRange r = share_blocks(sh, po, npairs(n), n);
          for (int64_t k = r.k0; k < r.k1; ++k, ++turn)
            if (turn % NW == wid) block(ev, lo, n, A.gpair + po, (int)(32 * k));
        }
      });
}

int big_grid(int64_t ne) {
  constexpr int64_t per = (int64_t)kBigBlock * kBigScan;
  return (int)std::min<int64_t>(std::max<int64_t>(1, (ne + per - 1) / per), 2048);
}


int grid_for(int64_t ne, int epb) {
  int64_t tiles = (ne + epb - 1) / epb;
  if (tiles < 1) tiles = 1;
  if (tiles > 0x7fffffff) tiles = 0x7fffffff;
  return (int)tiles;
}

// Pairs of one round that a tiling's wavefront stages and the particles beside
// them.  FP32 plain: the tiling's own limit on LDS leaves the staged pairs out
// (any pairs_per_round fits), so they get at most a quarter of the 64 KiB of a
// workgroup, and the particles at most the rest.
template <typename T, int MODE>
void fwd_caps(const Tiling& t, bool best, bool pairs, int* cap, int* qcap) {
  *cap = t.lds_particles;
  *qcap = t.pairs_per_round;
  if (sizeof(T) == 8 || MODE != GLV_PLAIN || best) return;
  const int room = 64 * 1024 / (t.block / 64);
  *qcap = pairs ? std::min(t.pairs_per_round, room / 4 / (int)sizeof(T)) : 0;
  if (!pairs) return;
  const int rest = room - (int)wave_lds_bytes<T, MODE, false>(0, *qcap, t.events_per_tile);
  *cap = std::min(t.lds_particles, rest / (4 * (int)sizeof(T)));
}

template <typename T, int COORDS, int MODE>
hipError_t fwd_typed(int64_t ne, const int64_t* off, const int64_t* poff, const void* const p[4],
                     void* const total[4], void* em, void* pm, const BestOut* best, unsigned long long* fb,
                     const Tiling& t, hipStream_t s) {
  FwdArgs<T, COORDS, MODE> A;
  A.best_rank = best ? best->rank : nullptr;
  A.best_m = best ? (T*)best->mass : nullptr;
  A.target = best ? best->target : 0.0;
  for (int k = 0; k < 4; ++k) {
    A.p.c[k] = (const T*)p[k];
    A.total[k] = total ? (T*)total[k] : nullptr;
  }
  A.off = off;
  A.poff = poff;
  A.event_m = (T*)em;
  A.pair_m = (T*)pm;
  A.fallback = fb;
  A.ne = ne;
  A.epb = t.events_per_tile;
  const bool pairs = best || pm || (MODE == GLV_COMPENSATED && em);  // evaluated: pair offsets are given
  fwd_caps<T, MODE>(t, best != nullptr, pairs, &A.cap, &A.qcap);
  A.small = pairs ? std::min(A.cap, kDenseFrom) : A.cap;
  const int waves = t.block / 64;
  const int64_t tiles = (ne + t.events_per_tile - 1) / t.events_per_tile;
  if (best) {
    A.wave_bytes = (int)wave_lds_bytes<T, MODE, true>(A.cap, A.qcap, A.epb);
    hipLaunchKernelGGL((k_event_reduce<T, COORDS, MODE, true>), dim3(grid_for(tiles, waves)), dim3(t.block),
                       (size_t)waves * A.wave_bytes, s, A);
  } else {
    A.wave_bytes = (int)wave_lds_bytes<T, MODE, false>(A.cap, A.qcap, A.epb);
    hipLaunchKernelGGL((k_event_reduce<T, COORDS, MODE, false>), dim3(grid_for(tiles, waves)), dim3(t.block),
                       (size_t)waves * A.wave_bytes, s, A);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (!pairs)
    hipLaunchKernelGGL((k_event_totals_big<T, COORDS, MODE>), dim3(big_grid(ne)), dim3(kBigBlock), 0, s, A);
  else if (best)
    hipLaunchKernelGGL((k_event_dense<T, COORDS, MODE, true>), dim3(dense_grid<MODE, true>()),
                       dim3(dense_block<MODE, true>()), 0, s, A);
  else
    hipLaunchKernelGGL((k_event_dense<T, COORDS, MODE, false>), dim3(dense_grid<MODE, false>()),
                       dim3(dense_block<MODE, false>()), 0, s, A);
  return hipGetLastError();
}

// The backward stages at most one particle per thread.
int bwd_cap(const Tiling& t) { return std::min(t.lds_particles, t.block); }

template <typename T, int COORDS>
hipError_t bwd_typed(int64_t ne, const int64_t* off, const int64_t* poff, const void* const p[4],
                     const void* const gt[4], const void* gem, const void* gpair, void* const gp[4],
                     const void* const tot[4], const Tiling& t, size_t lds, hipStream_t s) {
  BwdArgs<T, COORDS> A;
  for (int k = 0; k < 4; ++k) {
    A.p.c[k] = (const T*)p[k];
    A.gt[k] = gt ? (const T*)gt[k] : nullptr;
    A.tot[k] = tot ? (const T*)tot[k] : nullptr;
    A.gp[k] = (T*)gp[k];
  }
  A.off = off;
  A.poff = poff;
  A.gem = (const T*)gem;
  A.gpair = (const T*)gpair;
  A.ne = ne;
  A.epb = t.events_per_tile;
  A.cap = bwd_cap(t);
  A.qcap = t.pairs_per_round;
  hipLaunchKernelGGL((k_event_reduce_bwd<T, COORDS>), dim3(grid_for(ne, t.events_per_tile)), dim3(t.block), lds,
                     s, A);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (gpair)
    hipLaunchKernelGGL((k_event_bwd_dense<T, COORDS>), dim3(bwd_dense_grid<T>()), dim3(256), 0, s, A);
  else
    hipLaunchKernelGGL((k_event_reduce_bwd_big<T, COORDS>), dim3(big_grid(ne)), dim3(kBigBlock), 0, s, A);
  return hipGetLastError();
}

template <typename T>
hipError_t fwd_dt(glv_coords co, glv_mode mode, int64_t ne, const int64_t* off, const int64_t* poff,
                  const void* const p[4], void* const total[4], void* em, void* pm, const BestOut* b,
                  unsigned long long* fb, const Tiling& t, hipStream_t s) {
  if (mode == GLV_COMPENSATED)
    return fwd_typed<T, GLV_PTETAPHIM, GLV_COMPENSATED>(ne, off, poff, p, total, em, pm, b, fb, t, s);
  switch (co) {
    case GLV_PXPYPZE:
      return fwd_typed<T, GLV_PXPYPZE, GLV_PLAIN>(ne, off, poff, p, total, em, pm, b, nullptr, t, s);
    case GLV_PTETAPHIM:
      return fwd_typed<T, GLV_PTETAPHIM, GLV_PLAIN>(ne, off, poff, p, total, em, pm, b, nullptr, t, s);
    case GLV_PXPYPZM:
      return fwd_typed<T, GLV_PXPYPZM, GLV_PLAIN>(ne, off, poff, p, total, em, pm, b, nullptr, t, s);
    default:
      return fwd_typed<T, GLV_PTETAPHIE, GLV_PLAIN>(ne, off, poff, p, total, em, pm, b, nullptr, t, s);
  }
}

template <typename T>
hipError_t bwd_dt(glv_coords co, int64_t ne, const int64_t* off, const int64_t* poff, const void* const p[4],
                  const void* const gt[4], const void* gem, const void* gpair, void* const gp[4],
                  const void* const tot[4], const Tiling& t, size_t lds, hipStream_t s) {
  switch (co) {
    case GLV_PXPYPZE:
      return bwd_typed<T, GLV_PXPYPZE>(ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
    case GLV_PTETAPHIM:
      return bwd_typed<T, GLV_PTETAPHIM>(ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
    case GLV_PXPYPZM:
      return bwd_typed<T, GLV_PXPYPZM>(ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
    default:
      return bwd_typed<T, GLV_PTETAPHIE>(ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
  }
}

template <bool BEST>
size_t fwd_wave_bytes(glv_dtype dt, glv_mode mode, int cap, int qcap, int epb) {
  if (dt == GLV_F64)
    return mode == GLV_COMPENSATED ? wave_lds_bytes<double, GLV_COMPENSATED, BEST>(cap, qcap, epb)
                                   : wave_lds_bytes<double, GLV_PLAIN, BEST>(cap, qcap, epb);
  return mode == GLV_COMPENSATED ? wave_lds_bytes<float, GLV_COMPENSATED, BEST>(cap, qcap, epb)
                                 : wave_lds_bytes<float, GLV_PLAIN, BEST>(cap, qcap, epb);
}

}  // namespace

size_t event_reduce_lds_bytes(glv_dtype dt, glv_mode mode, const Tiling& t, bool best) {
  const size_t waves = (size_t)t.block / 64;
  const int cap = t.lds_particles, qcap = t.pairs_per_round, epb = t.events_per_tile;
  if (best) return waves * fwd_wave_bytes<true>(dt, mode, cap, qcap, epb);
  // staged FP32 plain masses do not count: fwd_caps fits them in
  return waves * fwd_wave_bytes<false>(dt, mode, cap, dt == GLV_F32 && mode == GLV_PLAIN ? 0 : qcap, epb);
}

size_t event_reduce_bwd_lds_bytes(glv_dtype dt, const Tiling& t) {
  const size_t tsz = (dt == GLV_F64) ? 8 : 4;
  const size_t cap = (size_t)bwd_cap(t), epb = (size_t)t.events_per_tile, qcap = (size_t)t.pairs_per_round;
  return 4 * (cap + epb) * tsz + (qcap + 2) * tsz + ((epb + 1) & ~(size_t)1) * tsz + 2 * (epb + 1) * 8 +
         (epb + 1) * sizeof(EvRec) + cap * sizeof(unsigned short);
}

hipError_t launch_pair_offsets(int64_t ne, const int64_t* off, int64_t* po, hipStream_t s) {
  const int64_t ntiles = (ne + kScanTile - 1) / kScanTile;
  if (ne <= kScanOnce) {  // also no events: pair_offsets = {0}
    hipLaunchKernelGGL(k_po_once, dim3((unsigned)std::max<int64_t>(ntiles, 1)), dim3(kScanThreads), 0, s, off, po, ne);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_po_tile_totals, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, off, po, ne);
  hipLaunchKernelGGL(k_po_scan_totals, dim3(1), dim3(1024), 0, s, po, ne, ntiles);
  hipLaunchKernelGGL(k_po_tile_scan, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, off, po, ne);
  return hipGetLastError();
}

hipError_t launch_validate_offsets(int64_t ne, const int64_t* off, int64_t np, long long* bad, hipStream_t s) {
  int64_t blocks = (ne + 1 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_validate_offsets, dim3((unsigned)blocks), dim3(256), 0, s, off, ne, np, bad);
  return hipGetLastError();
}

hipError_t launch_event_reduce(glv_dtype dt, glv_coords co, glv_mode mode, int64_t ne, const int64_t* off,
                               const int64_t* poff, const void* const p[4], void* const total[4], void* em,
                               void* pm, unsigned long long* fb, const Tiling& t, hipStream_t s,
                               const BestOut* best) {
  if (dt == GLV_F64) return fwd_dt<double>(co, mode, ne, off, poff, p, total, em, pm, best, nullptr, t, s);
  return fwd_dt<float>(co, mode, ne, off, poff, p, total, em, pm, best, fb, t, s);
}

hipError_t launch_event_reduce_bwd(glv_dtype dt, glv_coords co, int64_t ne, const int64_t* off,
                                   const int64_t* poff, const void* const p[4], const void* const gt[4],
                                   const void* gem, const void* gpair, void* const gp[4], const Tiling& t,
                                   hipStream_t s, const void* const tot[4]) {
  size_t lds = event_reduce_bwd_lds_bytes(dt, t);
  if (dt == GLV_F64) return bwd_dt<double>(co, ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
  return bwd_dt<float>(co, ne, off, poff, p, gt, gem, gpair, gp, tot, t, lds, s);
}

}  // namespace glv
