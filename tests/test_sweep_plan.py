"""Host-only: the plan of the layer-sweep kernels and their decoding of a unit of
work (the code that the kernels run, compiled for the host).  For all layer and
head counts and ragged token counts, with and without token segments, every
(layer, head, K|V, token) is computed once, token parts start on whole tiles and
stay inside the cache, and each layer's packed map has one writer."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_03893_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include "kvx_internal.h"
#include <cstdio>
#include <vector>

static int check(int nl, int H, int T) {
  const kvx::SweepPlan p = kvx::plan_sweep(nl, H, T);
  const size_t rows = (size_t)nl * H * 2;
  std::vector<unsigned char> seen(rows * T);
  std::vector<int> writers(rows);
  for (int unit = 0; unit < p.n_units; ++unit)
    for (int slot = 0; slot < 32; ++slot) {
      const kvx::SweepUnit u = kvx::sweep_unit_of(p, unit, slot, H, T, 16);
      if (u.t_end <= u.t_begin) continue;
      if (u.h < 0 || u.h >= H || u.kv < 0 || u.kv > 1 || u.t_begin % 16 != 0 || u.t_begin < 0 || u.t_end > T) return 1;
      for (int e = 0; e < 2; ++e) {
        const int r = 2 * u.pair + e;
        if (r >= u.g_n) continue;
        const int l = u.g0 + r;
        if (l >= nl) return 2;
        const size_t at = ((size_t)l * H + u.h) * 2 + u.kv;
        writers[at] += u.first;
        for (int64_t t = u.t_begin; t < u.t_end; ++t) ++seen[at * T + t];
      }
    }
  for (unsigned char n : seen)
    if (n != 1) return 3;
  for (int n : writers)
    if (n != 1) return 4;
  return 0;
}

int main() {
  int segmented = 0;
  for (int nl : {1, 2, 15, 16, 17, 22, 32, 33, 40, 63, 64, 65, 80, 130})
    for (int H = 1; H <= 24; ++H)
      for (int T : {1, 15, 16, 17, 100, 511, 1300, 2561, 5121, 8199}) {
        if ((long)nl * H * T > 4000000L) continue;
        segmented += kvx::plan_sweep(nl, H, T).segs > 1;
        if (const int e = check(nl, H, T)) return std::printf("error %d: %d layers, %d heads, %d tokens\n", e, nl, H, T), 1;
      }
  for (int nl : {64, 128, 256}) {   // the most layers, few tokens
    if (const int e = check(nl, 3, 70)) return std::printf("error %d: %d layers\n", e, nl), 1;
  }
  // the longest caches: positions alone (a plane of 2^31 - 1 tokens)
  const kvx::SweepPlan p = kvx::plan_sweep(16, 1, 2147483647);
  int64_t sum = 0;
  for (int unit = 0; unit < p.n_units; ++unit)
    for (int slot = 0; slot < 32; ++slot) {
      const kvx::SweepUnit u = kvx::sweep_unit_of(p, unit, slot, 1, 2147483647, 16);
      if (u.t_end > u.t_begin) sum += u.t_end - u.t_begin;
    }
  if (sum != 2147483647LL * 2 * 8) return std::printf("long caches: %lld\n", (long long)sum), 1;
  std::printf("%d segmented plans\n", segmented);
  return segmented > 30 ? 0 : 1;
}
"""


@pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")), reason="no HIP headers")
def test_every_token_once_and_one_writer_per_map(tmp_path):
    (tmp_path / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(tmp_path / "plan.cpp"),
                    "-o", str(tmp_path / "plan")], check=True)
    r = subprocess.run([str(tmp_path / "plan")], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
