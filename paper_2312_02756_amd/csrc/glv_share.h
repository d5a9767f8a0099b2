// Which pairs, events and blocks of events fall to a workgroup of the
// large-event launches.  Plain integer arithmetic without any include but the
// integer types, so that it runs on the host as well.
#pragma once

#include <stdint.h>

namespace glv {

// A run [q0, q1) of the pairs of all events.
struct Share {
  int64_t q0, q1;
};

// Share `index` of nq pairs cut into `grid` equal runs of at least min_pairs.
__host__ __device__ __forceinline__ Share pair_share(int64_t nq, int64_t min_pairs, int64_t grid, int64_t index) {
  const int64_t even = (nq + grid - 1) / grid;
  const int64_t per = even > min_pairs ? even : min_pairs;
  const int64_t q0 = index * per, q1 = q0 + per;
  return {q0 < nq ? q0 : nq, q1 < nq ? q1 : nq};
}

// The share of a workgroup whose events are given to it by their index: all
// pairs there are.  (Not a bound beyond them: the ends of shares are added to
// below.)
__host__ __device__ __forceinline__ Share whole_share(int64_t nq) { return {0, nq}; }

// Where the events themselves are dealt out: the first event that thread tid of
// workgroup `index` of `grid` looks at.  kDealt neighbours (one cache line of
// their offsets) go to one workgroup, the next kDealt to the next; a workgroup
// of B threads takes B / kDealt such rows of the grid at a time, at another
// place in each (B / kDealt is a power of two that divides the grid), so that
// sizes that repeat with the row do not meet the same workgroup again.  Its next
// events are B grid further on.
constexpr int kDealt = 16;
template <int B>
__host__ __device__ __forceinline__ int dealt_event(int tid, int index, int grid) {
  constexpr int kRows = B / kDealt;
  const int row = tid / kDealt;
  const int place = index + (row * 5 & (kRows - 1)) * (grid / kRows);  // below 2 grid
  return (row * grid + (place < grid ? place : place - grid)) * kDealt + tid % kDealt;
}

// The reverse mode's blocks of 32 particles [k0, k1) of an event of n > 1
// particles, first pair po and `pairs` pairs that stand in a share: block k
// stands at pair po + k unit.
struct BlockRange {
  int64_t k0, k1;
};
__host__ __device__ __forceinline__ BlockRange share_blocks(Share s, int64_t po, int64_t pairs, int n) {
  const int64_t nblk = ((int64_t)n + 31) / 32, unit = pairs / nblk;
  const int64_t k1 = (s.q1 - po + unit - 1) / unit;
  return {s.q0 > po ? (s.q0 - po + unit - 1) / unit : 0, k1 < nblk ? k1 : nblk};
}

}  // namespace glv
