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


RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "context.hpp"
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
using namespace lbmh;
TileRule rule(int kind, int scalar, bool fp64, bool inplace, bool blended, uint64_t state, int members = 1) {
  lbm_ctx c[8];
  lbm_ctx* p[8];
  for (int k = 0; k < members; ++k) {
    c[k].cfg = lbm_config{};
    c[k].cfg.flow = LBM_D2Q9;
    c[k].cfg.scalar = (decltype(c[k].cfg.scalar))scalar;
    c[k].cfg.precision = fp64 ? LBM_FP64 : LBM_FP32;
    c[k].cfg.tau_s = 0.6;
    c[k].cfg.tau_s_solid = blended ? 2.0 : 0.0;
    c[k].plan.inplace = inplace;
    c[k].plan.state_bytes = state / members;
    p[k] = &c[k];
  }
  return tile_rule(p, members, (LaunchKind)kind);
}
int main() {
  const uint64_t MB = 1 << 20;
  for (int members : {1, 8})
    for (int kind : {STEPS, RECORDED, ADJOINT})
      for (bool fp64 : {false, true})
        for (uint64_t state : {1 * MB, 24 * MB, 48 * MB, 100 * MB, 160 * MB, 256 * MB, 300 * MB, 400 * MB, 2000 * MB}) {
          for (bool inplace : {false, true})  // D2Q9 alone: always, any rows
            CHECK(rule(kind, 0, fp64, inplace, false, state, members).tiles &&
                  !rule(kind, 0, fp64, inplace, false, state, members).whole_rows);
          CHECK(rule(kind, 5, fp64, false, false, state, members).tiles);  // ping-pong D2Q5
          const bool most = state > 128 * MB && state <= (kind == RECORDED ? 320 : 256) * MB;
          const TileRule r = rule(kind, 5, fp64, true, false, state, members);
          CHECK(r.tiles == !(most && (kind == RECORDED || (kind == STEPS && fp64))) && r.whole_rows == fp64);
          const TileRule pp = rule(kind, 5, fp64, false, true, state, members);
          CHECK(pp.tiles == (kind != ADJOINT || state <= (fp64 ? 36 : 56) * MB) && pp.whole_rows == (kind == RECORDED));
          const TileRule ip = rule(kind, 5, fp64, true, true, state, members);
          if (kind == ADJOINT) CHECK(ip.tiles == (fp64 ? !most : state <= 20 * MB));
          else CHECK(ip.tiles == r.tiles);
          CHECK(ip.whole_rows == (fp64 || kind == RECORDED));
        }
  return 0;
}
"""


def test_which_launches_take_tiles(tmp_path):
    src, exe = str(tmp_path / "r.hip"), str(tmp_path / "r")
    with open(src, "w") as f:
        f.write(RULE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-result", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), src, "-o", exe, "-L", build.ROCM_LIB,
                    "-Wl,-rpath," + build.ROCM_LIB, "-lrocprofiler-sdk-roctx"], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
