"""Host side of the launches of several steps, on the CPU: the cut of a call into
launches, the order of the tiles and the division by the tiles in a row."""
import os
import subprocess

from paper_1501_04741_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "context.hpp"
#include "tiles.hpp"
#define CHECK(c) do { if (!(c)) { std::printf("%s\n", #c); std::exit(1); } } while (0)
using namespace lbmh;
int main() {
  for (int most = 1; most <= 8; ++most)
    for (int64_t steps = 0; steps <= 100; ++steps) {
      int64_t sum = 0, launches = 0;
      for (Split sp(steps, most); sp.next(); ++launches) {
        CHECK(sp.ns >= 1 && sp.ns <= most);
        sum += sp.ns;
      }
      CHECK(sum == steps && (launches - steps) % 2 == 0);  // the buffer one-step launches would end in
      for (int64_t done = 0; done < 4; ++done) {
        const int e = steps_there_and_back(done, steps, most);
        CHECK(e >= 0 && e % 2 == 0 && e <= most && 2 * e <= steps && (e == 0 || done % 2 == 0));
      }
    }
  for (int n = 1; n <= 200; ++n) {
    std::vector<int> seen(n);
    for (int i = 0; i < n; ++i) {
      const int t = lbmk::tile_index(i, n);
      CHECK(t >= 0 && t < n && !seen[t]++);
    }
  }
  const int big = 0x7fffffff;
  for (int n : {1, 2, 3, 5, 7, 8, 63, 64, 65, 1000, 46341, 1 << 20, big - 1, big})
    for (int64_t q : {0, 1, 2, 3, 1000, 46340, 1 << 20, big})
      for (int64_t i : {q * n - 1, q * n, q * n + 1, (int64_t)big - q})
        if (i >= 0 && i <= big) CHECK(lbmk::TileRow::of(n).divide((int)i) == (int)(i / n));
  return 0;
}
"""


def test_launch_cut_tile_order_and_division(tmp_path):
    src, exe = str(tmp_path / "t.hip"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-result", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), src, "-o", exe, "-L", build.ROCM_LIB,
                    "-Wl,-rpath," + build.ROCM_LIB, "-lrocprofiler-sdk-roctx"], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
