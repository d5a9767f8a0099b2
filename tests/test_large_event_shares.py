"""The shares of the large-event launches (csrc/glv_share.h), compiled for the
host with the undefined-behaviour sanitizer: over all workgroups of a launch
every block of every event is done exactly once, whether the workgroups share
the pairs or are given whole events; events that are dealt out are looked at
once each, and neighbours go to many workgroups."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include "glv_share.h"
#include <cstdio>
#include <vector>

static int64_t npairs(int64_t n) { return n * (n - 1) / 2; }

static int check(const std::vector<int64_t>& n, int64_t limit, int64_t grid, int64_t min_pairs, bool by_events) {
  std::vector<int64_t> po{0};
  for (int64_t c : n) po.push_back(po.back() + npairs(c));
  const int64_t nq = po.back();
  for (size_t e = 0; e < n.size(); ++e) {
    const int64_t d = npairs(n[e]);
    if (d <= limit) continue;
    std::vector<int> done((n[e] + 31) / 32, 0);
    for (int64_t b = 0; b < (by_events ? 1 : grid); ++b) {
      const glv::Share s = by_events ? glv::whole_share(nq) : glv::pair_share(nq, min_pairs, grid, b);
      if (s.q0 >= s.q1 || po[e] >= s.q1 || po[e] + d <= s.q0) continue;
      const glv::BlockRange r = glv::share_blocks(s, po[e], d, (int)n[e]);
      for (int64_t k = r.k0; k < r.k1; ++k)
        if (k < 0 || k >= (int64_t)done.size() || done[k]++) return 1;
    }
    for (int c : done)
      if (c != 1) {
        std::printf("event %zu of %lld particles, first pair %lld\n", e, (long long)n[e], (long long)po[e]);
        return 1;
      }
  }
  return 0;
}

// Events by workgroup, as a launch deals them out: window, slice, thread.
template <int B>
static int deal(int64_t ne, int grid, int slices) {
  std::vector<int> owner(ne, -1);
  const int64_t step = (int64_t)B * grid;
  for (int b = 0; b < grid; ++b)
    for (int tid = 0; tid < B; ++tid)
      for (int64_t win = 0; win < ne; win += slices * step)
        for (int sl = 0; sl < slices; ++sl) {
          const int64_t e = win + glv::dealt_event<B>(tid, b, grid) + sl * step;
          if (e >= ne) continue;
          if (owner[e] != -1) return 1;
          owner[e] = b;
        }
  for (int o : owner)
    if (o < 0) return 1;
  // a run of a thousand events, or the first hundred of every row of the grid
  for (int64_t from = 0; from + 1000 <= ne; from += 50021) {
    std::vector<int> mine(grid, 0);
    for (int64_t e = from; e < from + 1000; ++e)
      if (++mine[owner[e]] > 2 * glv::kDealt) return 1;
  }
  std::vector<int> mine(grid, 0);
  const int64_t row = (int64_t)grid * glv::kDealt;
  int64_t rows = 0;
  for (int64_t r = 0; r + 100 <= ne; r += row, ++rows)
    for (int64_t e = r; e < r + 100; ++e) ++mine[owner[e]];
  for (int c : mine)
    if (c > glv::kDealt * ((rows + 7) / 8 + 1)) return 1;
  return 0;
}

int main() {
  int bad = 0;
  for (int64_t ne : {1 << 18, (1 << 18) + 1, 700001, 1 << 21}) {
    bad += deal<256>(ne, 1024, 12) + deal<256>(ne, 768, 12) + deal<512>(ne, 512, 8);
  }
  for (bool by_events : {true, false})
    for (int64_t grid : {8, 1024})
      for (int64_t min_pairs : {64, 2048}) {
        for (int64_t n = 12; n < 200; ++n) {  // first, in the middle and last
          bad += check({n}, 60, grid, min_pairs, by_events);
          bad += check({n, 3, 0, 1, n, 2, 7, n + 1, 2}, 60, grid, min_pairs, by_events);
          bad += check({2, 5, n, 600, n}, 60, grid, min_pairs, by_events);
        }
        for (int64_t n : {1024, 1025, 5000, 380000}) bad += check({n, 40, n}, 60, grid, min_pairs, by_events);
      }
  return bad != 0;
}
"""


def test_every_block_is_done_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2312_02756_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
