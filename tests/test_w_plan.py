"""Host-only: the token ranges of the W-stationary kernel.  The planned time equals
a simulation of the workgroups on 256 CUs, and a call leaves 4096 tokens a
workgroup only for a plan that is a tenth shorter."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2608_03893_amd", "csrc")

PROGRAM = r"""
#include "kvx_wplan.h"
#include <algorithm>
#include <cstdio>
#include <functional>
#include <queue>
#include <random>
#include <vector>

static int64_t simulate(int64_t tasks, int64_t tiles, int64_t n) {
  std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> cu;
  for (int i = 0; i < 256; ++i) cu.push(0);
  int64_t last = 0;
  for (int64_t first = 0; first < tiles; first += n)
    for (int64_t t = 0; t < tasks; ++t) {
      const int64_t end = cu.top() + std::min(n, tiles - first) + 1;
      cu.pop();
      cu.push(end);
      last = std::max(last, end);
    }
  return last;
}

int main() {
  std::mt19937 rng(3);
  auto below = [&](int n) { return (int)(rng() % n); };
  for (int i = 0; i < 2000; ++i) {
    const int64_t tasks = 2 * (1 + below(600)), tiles = 1 + below(70), n = 1 + below(16);
    if (kvx::w_span(tasks, tiles, n) != simulate(tasks, tiles, n))
      return std::printf("%ld tasks, %ld tiles, ranges of %ld\n", (long)tasks, (long)tiles, (long)n), 1;
    const int64_t pick = kvx::w_tokens_per_wg(tasks, 256 * tiles) / 256;
    if (pick < 1 || pick > 16 || (pick < 16 && 10 * simulate(tasks, tiles, pick) > 9 * simulate(tasks, tiles, 16)))
      return std::printf("%ld tasks, %ld tiles: picks %ld\n", (long)tasks, (long)tiles, (long)pick), 1;
  }
  // one layer of 4096 tokens fills the chip; uneven last rounds that lose nothing stay
  const struct { int64_t tasks, T, want; } fixed[] = {
      {16, 4096, 256}, {126, 15015, 4096}, {1024, 8192, 4096}, {65534, 2147483647, 4096}, {2, 1, 4096}};
  for (const auto& f : fixed)
    if (const int got = kvx::w_tokens_per_wg(f.tasks, f.T); got != f.want)
      return std::printf("%ld tasks, %ld tokens: %d\n", (long)f.tasks, (long)f.T, got), 1;
  // 20 layers, 5 heads, 6646 tokens: ranges of 13 + 13 tiles take as long as 16 + 10
  return kvx::w_span(200, 26, 13) == kvx::w_span(200, 26, 16) ? 0 : 1;
}
"""


def test_planned_time_and_ranges(tmp_path):
    (tmp_path / "w.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(tmp_path / "w.cpp"), "-o", str(tmp_path / "w")],
                   check=True)
    r = subprocess.run([str(tmp_path / "w")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
