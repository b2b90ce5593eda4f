"""Launches of batched calls, on the CPU: the batched bodies over operations that
record their launches instead of making them."""
import os
import subprocess

from paper_1501_04741_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "ops.hpp"
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
using namespace lbmh;
struct Recorder {
  using RealT = float;
  static constexpr bool kTiled = true;
  static inline std::vector<int> primal_steps, adjoint_steps;  // per launch
  static inline int choices = 0;
  static TileChoice choose_tile(lbm_ctx* const*, int, LaunchKind) { ++choices; return TileChoice{8, 8, 5}; }
  static TileRow tile_row(lbm_ctx*, const TileChoice&) { return TileRow::of(1); }
  static int tiles(lbm_ctx*, const TileChoice&) { return 1; }
  static int batch_blocks(lbm_ctx*, int, int) { return 1; }
  static void objective(lbm_ctx*, const void*, double*) {}
  static void seed(lbm_ctx*, const void*, void*) {}
  static void fill(lbm_ctx*, void*, size_t) {}
  static void primal_many(lbm_ctx*, const void*, void*, void*, int, bool) {}
  static void primal_inplace(lbm_ctx*, void*, int64_t, void*) {}
  static void copy(lbm_ctx*, const void*, void*, size_t) {}
  static void primal_batch(hipStream_t, const BatchArgs<float>&, int, int = 0) { primal_steps.push_back(1); }
  static void adjoint_batch(hipStream_t, const BatchArgs<float>&, int, int = 0) { adjoint_steps.push_back(1); }
  static void primal_many_batch(hipStream_t, const BatchArgs<float>&, const TileChoice&, int ns, bool) {
    primal_steps.push_back(ns);
  }
  static void adjoint_many_batch(hipStream_t, const BatchArgs<float>&, const TileChoice&, int ns, bool) {
    adjoint_steps.push_back(ns);
  }
};
char memory[1 << 20];
int main() {
  lbm_ctx c[2];
  lbm_ctx* p[2] = {&c[0], &c[1]};
  for (lbm_ctx& k : c) {
    k.cfg = lbm_config{};
    k.cfg.nx = k.cfg.ny = 8;
    k.cfg.nsteps = 40;
    k.plan.C = 20;
    k.plan.S = 2;
    k.plan.state_bytes = 4096;
    k.plan.mom_bytes = 256;
    k.ckpt = k.mom = memory;
    for (int i = 0; i < 2; ++i) k.pp[i] = memory + 65536 * (i + 1), k.lam[i] = memory + 65536 * (i + 3);
    k.adj_started = true;
    k.rec_len = 40;
    k.t_adj = 20;   // the next reverse step is the first of segment 0 ...
    k.mom_seg = 1;  // ... whose moments are not held
  }
  RunAdjointBatch<Recorder>::run(p[0], p, 2, 1);  // one reverse step: the segment's 20 steps are recomputed
  int sum = 0;
  for (int ns : Recorder::primal_steps) sum += ns;
  CHECK(sum == 20 && Recorder::primal_steps.size() == 4);  // in launches of 5
  CHECK(Recorder::adjoint_steps == std::vector<int>({1}) && c[0].mom_seg == 0 && c[1].t_adj == 19);
  Recorder::choices = 0;
  RunAdjointBatch<Recorder>::run(p[0], p, 2, 2);  // too short for a launch of several
  CHECK(Recorder::choices == 0 && Recorder::adjoint_steps == std::vector<int>({1, 1, 1}));
  RunAdjointBatch<Recorder>::run(p[0], p, 2, 3);
  CHECK(Recorder::choices == 1 && Recorder::adjoint_steps == std::vector<int>({1, 1, 1, 3}) && c[0].t_adj == 14);
  return 0;
}
"""


def test_recompute_takes_its_own_launches_and_short_calls_choose_no_tile(tmp_path):
    src, exe = str(tmp_path / "t.hip"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-result", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), src, "-o", exe, "-L", build.ROCM_LIB,
                    "-Wl,-rpath," + build.ROCM_LIB, "-lrocprofiler-sdk-roctx"], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
