// Context, checkpoint plan and launch geometry of the adjoint lattice-Boltzmann
// library, and the dispatch from a context to the code of its lattice,
// precision and variant (ops.hpp).
//
// The library never allocates device memory: every buffer below is a slice of
// the caller's workspace.  Workspace layout (each slice 256-byte aligned):
//   w        N x Real      design field (copied in by lbm_set_design)
//   grad     N x Real      dJ/dw accumulator (one-shot: last estimate)
//   glob     boundary sums + J of the last objective evaluation, objective partials
//   desc     this context's batch descriptor (constants for batched launches)
//   lam[2]   2 states      adjoint ping-pong (in place: one state)
//   pp[2]    2 states      primal ping-pong
//   ckpt[S]  S states      checkpoints h^{sC-1}, s = 0..S-1 (ckpt[0] = h^{-1})
//   mom[C]   C moment sets the moments of f^k for the C steps k of one segment
// A "state" is Qt x N values of the context precision; a "moment set" is
// Mom::N x N values (rho, u and the scalar value: what the transposed
// Jacobians read), so the trajectory the adjoint needs costs 4-5 values per
// node and step instead of Qt.
//
// Trajectory bookkeeping (step k computes h^k from h^{k-1}, k = 0..N-1): a
// recorded step writes the moments of f^k to mom[k % C] and h^k to
// ckpt[(k+1)/C] when (k+1) % C == 0 (while slots are left), else to a primal
// ping-pong buffer.  The adjoint step n reads mom[n % C]; when segment
// s = n / C is not the one held in mom, it is recomputed from ckpt[s] (C
// primal steps through the ping-pong buffers).  With C = N (store-all) no
// step is ever recomputed.
//
// In-place plan (one primal working buffer and one adjoint buffer, each read
// and rewritten by every step in the alternating even/odd access patterns):
// store-all keeps the state in ckpt[0] and never recomputes.  With C < N the
// working buffer is a slot of its own; before recorded step k with k % C == 0
// it is copied to ckpt[k / C] (in the buffer layout of phase k), and segment s
// is recomputed in place inside ckpt[s] itself, which the backward sweep needs
// no more once the segment's moments are rebuilt (segments are reversed in
// decreasing order, each once).  Launches of several steps (2D lattices) cannot
// read and rewrite one buffer: they go through another and back, the primal's
// through the adjoint buffer, free until an adjoint or one-shot iteration starts,
// the adjoint's and a recomputed segment's through the working buffer, whose state
// the started adjoint has consumed (calls that read it are refused from then on).
// Captured calls take one step per launch (see most_in_place).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "../../include/lbm_adj.h"
#include "kernels.hpp"

namespace lbmh {

using namespace lbmk;

constexpr uint64_t kAlign = 256;
constexpr uint64_t kDescBytes = 1024;  // >= sizeof(BatchStatic<double>)
// Streaming stores bypass the caches when two primal states (what one step
// reads and writes) exceed the 256 MB last-level cache; below that, plain
// stores let the next step re-read the state from that cache.
constexpr uint64_t kLastLevelCacheBytes = 256ull << 20;
// glob region: kGlobSlots doubles of results, then the objective partial sums.
constexpr int kGlobSlots = 16;
constexpr uint64_t kGlobBytes = (kGlobSlots + kObjBlocks * kNG) * sizeof(double);

inline uint64_t align_up(uint64_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Row length of the workspace arrays: nx rounded up to whole 128-byte lines.
inline int64_t row_pitch(int32_t nx, int32_t precision) {
  const int64_t per_line = 128 / (precision == LBM_FP32 ? 4 : 8);
  return ((int64_t)nx + per_line - 1) / per_line * per_line;
}

constexpr int kCus = 256;                     // compute units of the GPU
constexpr uint64_t kL2Bytes = 8 * (4ull << 20);  // the L2s of its XCDs together

// What a launch of several steps does: unrecorded primal steps, recorded ones (a
// forward or a recomputed segment), adjoint steps.
enum LaunchKind : int { STEPS = 0, RECORDED = 1, ADJOINT = 2, LAUNCH_KINDS = 3 };

// Launches of several steps: the tile of a block and the steps per launch (1:
// one-step launches only).
struct TileChoice {
  int tx = 0, ty = 0;
  int ns = 1;
};

struct Plan {
  int Q = 0, QS = 0, QT = 0;
  int64_t N = 0;             // nodes
  int64_t pitch = 0, Np = 0; // padded row length, pitch*ny*nz
  uint64_t rs = 0;           // bytes per value
  uint64_t state_bytes = 0;  // aligned
  uint64_t mom_bytes = 0;    // aligned, one moment set
  uint64_t node_bytes = 0;   // aligned Np x Real
  int64_t C = 1, S = 1;      // checkpoint interval and slots
  bool inplace = false;      // one primal working buffer and one adjoint buffer, streamed in place
  int64_t W = 1;             // states averaged by the objective (the last W of the horizon)
  uint64_t cols_bytes = 0;   // inlet + outlet columns of one state (aligned)
  uint64_t win_bytes = 0;    // W > 1: W x (sums + J), then W x columns
  uint64_t total = 0;
};

}  // namespace lbmh

struct lbm_ctx {
  lbm_config cfg;
  lbmh::Plan plan;
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  uint64_t ws_bytes = 0;
  // carved buffers
  void* w = nullptr;
  void* grad = nullptr;
  double* glob = nullptr;
  void* desc = nullptr;
  void* lam[2] = {nullptr, nullptr};
  void* pp[2] = {nullptr, nullptr};
  char* ckpt = nullptr;
  char* mom = nullptr;
  void* work = nullptr;   // in place: the primal working buffer (ckpt[0] when store-all)
  char* win = nullptr;    // W > 1: window slots (sums + J, then inlet/outlet columns), W of them
  int64_t win_count = 0;  // window states captured since the run started at t = 0
  // time bookkeeping
  int64_t t = 0;          // primal time: current state is h^{t-1}
  int64_t rec_len = 0;    // recorded steps (trajectory h^{-1}..h^{rec_len-1})
  bool rec_open = true;   // recording can be continued
  void* cur = nullptr;    // buffer holding h^{t-1}
  bool design_set = false;
  bool adj_started = false;
  int64_t t_adj = -1;     // adjoint time (lambda^{t_adj} in lam[lam_cur])
  int lam_cur = 0;
  int64_t mom_seg = -1;   // trajectory segment whose moments mom holds
  bool os_active = false; // one-shot iteration running (adjoint state in lam[lam_cur])
  bool state_lost = false; // a new design arrived after an adjoint had started: the primal
                           // buffers may hold recomputed states, so c->cur is not h^{t-1}
  lbmh::TileChoice tile[lbmh::LAUNCH_KINDS];  // several steps per launch
  int static_dev = -1;     // device whose static workspace this context uses (-1: caller's)
  std::string err;
};

namespace lbmh {

// Named range on the profiler's marker timeline (rocprofv3 --marker-trace):
// forward segments, recomputed segments, adjoint segments and one-shot runs
// show up as spans around their kernel launches (host-side enqueue time).
struct Range {
  explicit Range(const char* name) { roctxRangePushA(name); }
  ~Range() { roctxRangePop(); }
  Range(const Range&) = delete;
  Range& operator=(const Range&) = delete;
};

inline lbm_status fail(lbm_ctx* c, lbm_status s, const char* fmt, ...) __attribute__((format(printf, 3, 4)));
inline lbm_status fail(lbm_ctx* c, lbm_status s, const char* fmt, ...) {
  if (c) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    c->err = buf;
  }
  return s;
}

inline lbm_status check_config(const lbm_config* c, std::string* why) {
  auto bad = [&](const char* m) {
    if (why) *why = m;
    return LBM_EINVAL;
  };
  if (!c) return bad("config is NULL");
  if (c->struct_size != sizeof(lbm_config)) return bad("struct_size does not match sizeof(lbm_config)");
  if (c->flow != LBM_D2Q9 && c->flow != LBM_D3Q19) return bad("flow must be LBM_D2Q9 or LBM_D3Q19");
  if (c->scalar != LBM_SCALAR_NONE && !((c->flow == LBM_D2Q9 && c->scalar == LBM_D2Q5) ||
                                        (c->flow == LBM_D3Q19 && c->scalar == LBM_D3Q7)))
    return bad("scalar lattice must be none, D2Q5 with D2Q9, or D3Q7 with D3Q19");
  if (c->precision != LBM_FP32 && c->precision != LBM_FP64) return bad("precision must be LBM_FP32 or LBM_FP64");
  if (c->nx < 3 || c->ny < 3 || c->nz < 1) return bad("nx, ny must be >= 3 and nz >= 1");
  if (c->flow == LBM_D2Q9 && c->nz != 1) return bad("D2Q9 needs nz = 1");
  if (c->flow == LBM_D3Q19 && c->nz < 3) return bad("D3Q19 needs nz >= 3");
  if (c->ny > 65535 || c->nz > 65535) return bad("ny and nz must be <= 65535");
  if (!(c->tau > 0.5) || (c->scalar && !(c->tau_s > 0.5))) return bad("relaxation times must exceed 1/2");
  if (!(std::fabs(c->u_in) < 1.0) || !(c->rho_out > 0.0)) return bad("need |u_in| < 1 and rho_out > 0");
  if (c->scalar_wall != LBM_WALL_ADIABATIC && c->scalar_wall != LBM_WALL_DIRICHLET) return bad("bad scalar_wall");
  if (c->s_split_axis < 0 || c->s_split_axis > 2) return bad("bad s_split_axis");
  if (c->switch_fn != LBM_G_POWER && c->switch_fn != LBM_G_RAMP) return bad("bad switch_fn");
  if (c->switch_fn == LBM_G_RAMP && !(c->switch_param > 0.0)) return bad("RAMP needs q > 0");
  if (c->switch_fn == LBM_G_POWER && !(c->switch_param >= 0.0)) return bad("POWER needs theta >= 0");
  if (c->reserved0 != 0) return bad("reserved0 must be 0");
  if (c->n_avg < 0) return bad("n_avg must be >= 0");
  if (c->n_avg > 1 && c->n_avg > c->nsteps)
    return bad("n_avg > 1 averages the last n_avg states of the horizon: needs nsteps >= n_avg");
  if (c->inlet != LBM_INLET_VELOCITY && c->inlet != LBM_INLET_PRESSURE) return bad("bad inlet");
  if (c->collision != LBM_COLL_BGK && c->collision != LBM_COLL_MRT) return bad("bad collision");
  if (c->collision == LBM_COLL_MRT) {
    if (c->flow != LBM_D3Q19) return bad("MRT collision is D3Q19 only");
    for (int k = 0; k < 5; ++k)
      if (!(c->mrt_rates[k] > 0.0 && c->mrt_rates[k] < 2.0)) return bad("MRT rates must lie in (0, 2)");
  }
  if (c->reserved2 != 0) return bad("reserved2 must be 0");
  if (c->tau_s_solid != 0.0 && !(c->tau_s_solid > 0.5)) return bad("tau_s_solid must be 0 or exceed 1/2");
  if (c->inplace != 0 && c->inplace != 1) return bad("inplace must be 0 or 1");
  if (c->reserved3 != 0) return bad("reserved3 must be 0");
  if (c->plate_x0 < 0 || c->plate_x1 < c->plate_x0 || c->plate_x1 > c->nx)
    return bad("heating plate needs 0 <= plate_x0 <= plate_x1 <= nx");
  if (c->inlet == LBM_INLET_PRESSURE && !(c->rho_in > 0.0 && c->u_cap >= 0.0 && c->u_cap < 1.0))
    return bad("pressure inlet needs rho_in > 0 and 0 <= u_cap < 1");
  if (c->nsteps < 0 || c->checkpoint_interval < 0) return bad("nsteps and checkpoint_interval must be >= 0");
  const int64_t Np = row_pitch(c->nx, c->precision) * c->ny * c->nz;
  const int QT = c->flow + c->scalar;
  if ((int64_t)QT * Np >= (int64_t(1) << 31)) return bad("lattice too large: Qt*N (rows padded) must be < 2^31");
  return LBM_OK;
}

// Workspace of a plan with checkpoint interval C and S checkpoint slots (N steps).
// Ping-pong: 2 adjoint + 2 primal states besides the checkpoints.  In place: one
// adjoint state, plus the working buffer unless C >= N (store-all: the state stays
// in ckpt[0]).
inline uint64_t plan_total(const Plan& p, int64_t C, int64_t S, int64_t N) {
  uint64_t t = 2 * p.node_bytes + align_up(kGlobBytes) + align_up(kDescBytes) + p.win_bytes;
  const uint64_t extra = p.inplace ? (C >= N ? 1 : 2) : 4;
  t += (uint64_t)(extra + S) * p.state_bytes + (uint64_t)C * p.mom_bytes;
  return t;
}

// Values per node in one moment set (must equal Mom<Q,QS>::N of the kernels).
// Blended (design-dependent) scalar diffusivity in use.
inline bool blended_diffusivity(const lbm_config* c) {
  return c->scalar != 0 && c->tau_s_solid != 0.0 && c->tau_s_solid != c->tau_s;
}

inline int mom_values(const lbm_config* c) {
  return (c->flow == LBM_D3Q19 ? 3 : 2) + 1 + (c->scalar ? (blended_diffusivity(c) ? c->scalar : 1) : 0);
}

inline lbm_status make_plan(const lbm_config* c, Plan* p, std::string* why) {
  lbm_status s = check_config(c, why);
  if (s != LBM_OK) return s;
  p->Q = c->flow;
  p->QS = c->scalar;
  p->QT = p->Q + p->QS;
  p->N = (int64_t)c->nx * c->ny * c->nz;
  p->pitch = row_pitch(c->nx, c->precision);
  p->Np = p->pitch * c->ny * c->nz;
  p->rs = (c->precision == LBM_FP32) ? 4 : 8;
  p->state_bytes = align_up((uint64_t)p->QT * p->Np * p->rs);
  p->mom_bytes = align_up((uint64_t)mom_values(c) * p->Np * p->rs);
  p->node_bytes = align_up((uint64_t)p->Np * p->rs);
  p->inplace = c->inplace != 0;
  p->W = c->n_avg > 1 ? c->n_avg : 1;
  p->win_bytes = 0;
  p->cols_bytes = align_up((uint64_t)2 * p->QT * c->ny * c->nz * p->rs);  // inlet + outlet columns
  if (p->W > 1) p->win_bytes = align_up((uint64_t)p->W * (kNG + 1) * sizeof(double)) + (uint64_t)p->W * p->cols_bytes;
  const int64_t Nst = std::max<int64_t>(c->nsteps, 1);
  if (p->inplace && c->nsteps == 0) {
    // unrecorded runs and the one-shot iteration only: the state and one adjoint buffer
    p->C = 0;
    p->S = 1;
    p->total = 2 * p->node_bytes + align_up(kGlobBytes) + align_up(kDescBytes) + 2 * p->state_bytes + p->win_bytes;
    return LBM_OK;
  }
  int64_t C;
  if (c->checkpoint_interval > 0) {
    C = std::min<int64_t>(c->checkpoint_interval, Nst);
  } else if (c->hbm_budget_bytes == 0 && p->inplace) {
    C = Nst;  // in place without a budget: every step's moments (no recompute)
  } else if (c->hbm_budget_bytes == 0) {
    // smallest workspace: minimise S*state + C*moments
    C = 1;
    uint64_t best = plan_total(*p, 1, Nst, Nst);
    for (int64_t cc = 2; cc <= Nst; ++cc) {
      const uint64_t t = plan_total(*p, cc, (Nst + cc - 1) / cc, Nst);
      if (t < best) {
        best = t;
        C = cc;
      }
    }
  } else {
    // largest C (fewest recomputed steps) whose workspace fits the budget
    C = 0;
    for (int64_t cc = Nst; cc >= 1; --cc) {
      const int64_t S = (Nst + cc - 1) / cc;
      if (plan_total(*p, cc, S, Nst) <= c->hbm_budget_bytes) {
        C = cc;
        break;
      }
    }
    if (C == 0) {
      if (why) *why = "no checkpoint interval fits hbm_budget_bytes";
      return LBM_ENOMEM;
    }
  }
  p->C = C;
  p->S = (Nst + C - 1) / C;
  p->total = plan_total(*p, p->C, p->S, Nst);
  return LBM_OK;
}

// ---------------------------------------------------------------- launches
template <typename Real>
Params<Real> make_params(const lbm_config& c, int64_t N) {
  Params<Real> p;
  p.nx = c.nx;
  p.ny = c.ny;
  p.nz = c.nz;
  p.periodic = c.periodic ? 1 : 0;
  p.N = (int)N;
  p.pitch = (int)row_pitch(c.nx, c.precision);
  p.Np = p.pitch * c.ny * c.nz;
  p.scalar_wall = c.scalar_wall;
  p.split_axis = c.s_split_axis;
  p.switch_fn = c.switch_fn;
  const double th = c.switch_param;
  p.theta_int = (c.switch_fn == LBM_G_POWER && th == std::floor(th) && th <= 16) ? (int)th : -1;
  p.om = (Real)(1.0 / c.tau);
  p.oms = (Real)(c.scalar ? 1.0 / c.tau_s : 0.0);
  p.u_in = (Real)c.u_in;
  p.rho_out = (Real)c.rho_out;
  p.s_wall = (Real)c.s_wall;
  p.s_in_lo = (Real)c.s_in_lo;
  p.s_in_hi = (Real)c.s_in_hi;
  p.sw_param = (Real)c.switch_param;
  p.inlet_mode = (c.inlet == LBM_INLET_PRESSURE) ? IN_PRESSURE : IN_VELOCITY;
  p.drho_in = (Real)(c.rho_in - 1.0);
  p.u_cap = (Real)c.u_cap;
  p.rho_in = c.rho_in;
  p.c_dp = c.c_dp;
  p.c_hf = c.c_hf;
  p.c_var = c.c_var;
  p.c_mix = c.c_mix;
  p.taus_f = (Real)c.tau_s;
  p.taus_s = (Real)(c.tau_s_solid != 0.0 ? c.tau_s_solid : c.tau_s);
  p.plate_x0 = c.periodic ? 0 : c.plate_x0;
  p.plate_x1 = c.periodic ? 0 : c.plate_x1;
  p.s_plate = (Real)c.s_plate;
  // MRT row scales (1 - rate) / |row|^2; rows of group 0 relax at 1/tau
  for (int k = 0; k < 19; ++k) {
    const int gr = Mrt19::group(k);
    const double rate = (gr == 0) ? 1.0 / c.tau : c.mrt_rates[gr - 1];
    p.mrt_k[k] = (Real)((1.0 - rate) / Mrt19::norm2(k));
  }
  return p;
}

struct Geo {
  dim3 grid, block;
};

// One thread per node of an x row, rows padded to whole waves; the block is the
// widest run of at most four waves that divides the row's waves, so no block
// holds more idle lanes than that padding (nx = 384: 2 x 192 threads instead of
// 2 x 256, where a quarter of the lanes idled).
inline Geo node_geometry(const lbm_config& c) {
  const int waves = (c.nx + 63) / 64;
  int k = 4;
  while (waves % k) --k;
  Geo g;
  g.block = dim3(64 * k, 1, 1);
  g.grid = dim3(waves / k, c.ny, c.nz);
  return g;
}

// Waves per block the hot kernels (primal, adjoint, one-shot) and batched
// launches aim for when a row is narrower (their kernels are bounded to 256
// threads).  Measured on D3Q19 FP32: 96x48x48 recorded in place 0.43 -> 0.48 of
// HBM peak (one 128-thread row per block against two rows per block); no change
// at 128x192x192, 192x96x96 or 256x128x128.
constexpr int kHotWaves = 4;

// x-shifted populations through LDS (kernels' LX variants): when one block
// part spans a whole row, i.e. nx <= 256.  Measured on the 256x128x128 D3Q19
// FP32 channel (fraction of HBM peak): recorded in-place primal 0.839 -> 0.892,
// in-place adjoint 0.846 -> 0.903, ping-pong primal 0.732 -> 0.752, ping-pong
// adjoint 0.798 -> 0.807; FP64 and the one-shot unchanged.  MRT lengthens the chain that
// a block's barriers hold together, and loses with staging although its primal would have
// more waves (FP32 57 VGPRs against 74; us a recorded step, plain / staged: 96x48x48 10.1 /
// 11.0, 131x67x45 15.2 / 16.1, with D3Q7 18.4 / 24.6, 256x128x128 116.5 / 119.2; the adjoint,
// 89 VGPRs either way, 0.80 -> 0.75 of peak at 256x128x128): it keeps the plain access.
inline bool lx_rows(const lbm_config& c) { return c.nx <= kHotThreads && c.collision != LBM_COLL_MRT; }

// Launch geometry of the hot kernels: a row of up to kHotThreads / 64 waves
// (nx <= 256) is one block (its x-shifts are then staged in LDS), and when a
// row is narrower than kHotWaves waves, R consecutive rows share a block
// (blockDim.y = R) so that it holds about that many; wider rows as
// node_geometry.
inline Geo hot_geometry(const lbm_config& c) {
  Geo g = node_geometry(c);
  const int waves = (c.nx + 63) / 64;
  if (waves * 64 <= kHotThreads) {
    const int R = std::max(1, kHotWaves / waves);
    g.block = dim3(64 * waves, R, 1);
    g.grid = dim3(1, (c.ny + R - 1) / R, c.nz);
  }
  return g;
}

inline dim3 flat_grid(size_t n) {
  size_t b = (n + 255) / 256;
  return dim3((unsigned)std::min<size_t>(std::max<size_t>(b, 1), 65536), 1, 1);
}

inline lbm_status launch_check(lbm_ctx* c, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, LBM_EHIP, "%s: %s", what, hipGetErrorString(e));
  return LBM_OK;
}

// Waves per x row of a context (rows padded to whole waves).
inline int batch_waves(const lbm_ctx* c) { return (c->cfg.nx + 63) / 64; }

// Waves per block of a batched launch: the widest of 4, 3, 2, 1 that divides
// every member's waves per row (as in the single-context launch geometry, which
// measured 0.737 of HBM peak with one-wave blocks against 0.835 with four).
inline int batch_block_waves(lbm_ctx* const* cs, int n) {
  for (int kw = 4; kw > 1; --kw) {
    bool all = true;
    for (int k = 0; k < n && all; ++k) all = batch_waves(cs[k]) % kw == 0;
    if (all) return kw;
  }
  return 1;
}

// Row parts per block of a batched launch: several rows per block only when
// every member's row is a single part of kw waves.
inline int batch_rows_per_block(lbm_ctx* const* cs, int n, int kw) {
  for (int k = 0; k < n; ++k)
    if (batch_waves(cs[k]) != kw) return 1;
  return std::max(1, kHotWaves / kw);
}

// x-shifted populations through LDS in a batched launch: when every member's
// row is a single row part (as lx_rows for one context).
inline int batch_lx(lbm_ctx* const* cs, int n, int kw) {
  for (int k = 0; k < n; ++k)
    if (batch_waves(cs[k]) != kw) return 0;
  return 1;
}

// Whether the 2D lattices `cs` advance several steps per launch, in tiles, and whether the
// tiles' rows are whole 64-byte pieces.  D2Q9 always gains (0.5-0.95 of the time of one-step
// launches from 512x256 to 4096x2048); with D2Q5 there are three exceptions (times per step,
// tiles against one-step launches; S: bytes of the states together).
//  - In place, S between half the cache and about its size: one state stays in the cache,
//    the two that the tiles go through do not.  Recorded 2400x1200 FP32 59.4 against 49.2 us,
//    2048x1024 FP64 97.9 / 67.6 (S = 1.2 caches still 1.02); unrecorded FP64 1700x850 46.3 / 43.7.
//  - Blended diffusivity records and reads 8 moment planes.  The adjoint reads them over the
//    whole region of a tile.  Ping-pong, FP32 1100x560 16.8 / 19.1, 1400x700 26.0 / 27.0,
//    1536x768 33.1 / 32.2, 2048x1024 59.5 / 53.6; FP64 600x300 11.9 / 12.9, 760x380 18.0 / 18.6,
//    900x450 24.3 / 23.6, 2048x1024 117.6 / 103.3.  In place, FP32 800x400 10.6 / 11.8,
//    1000x500 13.8 / 14.4, 1024x512 16.2 / 14.5, 1152x576 19.1 / 18.1, 2048x1024 59.4 / 47.8;
//    FP64 gains (1024x512 0.83).
//  - Rows that end inside a 64-byte piece store moments as parts of one: blended recorded
//    1400x700 FP32 30.8 with 20-wide tiles, 17.4 with 16-wide ones (one-step 20.4); FP64 in
//    place takes 16x12 for 12x16 (3000x2000 recorded 281 -> 213, adjoint 238 -> 211).
struct TileRule {
  bool tiles, whole_rows;
};
inline TileRule tile_rule(lbm_ctx* const* cs, int n, LaunchKind kind) {
  const lbm_config& k = cs[0]->cfg;
  if (k.scalar == 0) return {true, false};
  uint64_t s = 0;
  for (int q = 0; q < n; ++q) s += cs[q]->plan.state_bytes;
  const bool fp64 = k.precision == LBM_FP64, inplace = cs[0]->plan.inplace, blended = blended_diffusivity(&k);
  const uint64_t most = kind == RECORDED ? kLastLevelCacheBytes / 4 * 5 : kLastLevelCacheBytes;
  const bool resident = inplace && 2 * s > kLastLevelCacheBytes && s <= most;  // one state is, two are not
  const bool rows = (blended && kind == RECORDED) || (fp64 && inplace);
  if (kind == RECORDED || (kind == STEPS && fp64)) return {!resident, rows};
  if (kind == ADJOINT && blended)
    return {inplace && fp64 ? !resident : s <= uint64_t(inplace ? 20 : fp64 ? 36 : 56) << 20, rows};
  return {true, rows};
}

// Streaming stores and hints in a batched ping-pong launch: decided on the
// states the launch touches together (a source and a destination per member),
// not per member: eight 90 MB states are far beyond the cache although each
// member's pair alone fits.
inline int batch_nt(lbm_ctx* const* cs, int n) {
  uint64_t bytes = 0;
  for (int k = 0; k < n; ++k) bytes += 2 * cs[k]->plan.state_bytes;
  return bytes > kLastLevelCacheBytes ? 1 : 0;
}

// The same for an in-place launch (one buffer per member, read and rewritten),
// with the single-context rule: recorded and adjoint steps stream once the
// buffers exceed the cache; unrecorded steps stream in the odd phase only
// between one and two caches (4 x 128x96x96 D3Q19 FP32, 0.36 GB together: 0.69 ->
// 0.80 of HBM peak; 5 x: 0.67 -> 0.74) and in both phases beyond; the even
// phase's loads take the hint too beyond twice the cache (8 x 128x96x96 recorded,
// 0.72 GB together: primal 0.64, adjoint 0.66 of HBM peak without it).
inline void batch_nt_inplace(lbm_ctx* const* cs, int n, bool unrecorded, bool odd, int* nt, int* nte) {
  uint64_t bytes = 0;
  for (int k = 0; k < n; ++k) bytes += cs[k]->plan.state_bytes;
  const bool far = bytes > 2 * kLastLevelCacheBytes;
  const bool over = bytes > kLastLevelCacheBytes;
  *nt = (unrecorded ? far || (odd && over) : over) ? 1 : 0;
  *nte = far ? 1 : 0;
}

// Window of the time-averaged objective: slot s holds state f^{N-W+1+s}.
inline double* win_glob(lbm_ctx* c, int64_t s) { return (double*)c->win + s * (kNG + 1); }
inline void* win_cols(lbm_ctx* c, int64_t s) {
  return c->win + align_up((uint64_t)c->plan.W * (kNG + 1) * sizeof(double)) + (uint64_t)s * c->plan.cols_bytes;
}

// Launches of one lattice, precision and variant (ops.hpp).
template <int Q, int QS, typename Real, int V = 0>
struct Ops;

// Bodies of the C ABI calls (ops.hpp), instantiated in variants.hip.
template <class O>
struct RunPrimal {
  static lbm_status run(lbm_ctx* c, int64_t nsteps, int record);
};

template <class O>
struct RunObjective {
  static lbm_status run(lbm_ctx* c, double* J_dev);
};

template <class O>
struct RunAdjoint {
  static lbm_status run(lbm_ctx* c, int64_t nsteps);
};

template <class O>
struct RunReset {
  static lbm_status run(lbm_ctx* c);
};

template <class O>
struct RunSetState {
  static lbm_status run(lbm_ctx* c, const double* f, const double* g);
};

template <class O>
struct RunGradient {
  static lbm_status run(lbm_ctx* c, void* out);
};

template <class O>
struct RunGradientPenalty {
  static lbm_status run(lbm_ctx* c, double pen, void* out);
};

template <class O>
struct RunFields {
  static lbm_status run(lbm_ctx* c, double* rho, double* u, double* s);
};

template <class O>
struct RunGetState {
  static lbm_status run(lbm_ctx* c, double* f, double* g);
};

template <class O>
struct RunGetAdjoint {
  static lbm_status run(lbm_ctx* c, double* lf, double* lg);
};

template <class O>
struct RunMaps {
  static lbm_status run(lbm_ctx* c, uint8_t* mask, int64_t* src);
};

template <class O>
struct RunSetDesign {
  static lbm_status run(lbm_ctx* c, const void* w);
};

template <class O>
struct RunOneshot {
  static lbm_status run(lbm_ctx* c, int64_t nsteps, double zeta, double pen);
};

template <class O>
struct RunGetDesign {
  static lbm_status run(lbm_ctx* c, void* out);
};

template <class O>
struct RunWriteStatic {
  static lbm_status run(lbm_ctx* c);
};

template <class O>
struct RunPrimalBatch {
  static lbm_status run(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps, int record);
};

template <class O>
struct RunAdjointBatch {
  static lbm_status run(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps);
};

// Calls F::template run<Ops<...>>(args) for the context's lattice/precision.
template <template <class> class F, class... A>
lbm_status dispatch(lbm_ctx* c, A&&... a) {
  const lbm_config& k = c->cfg;
  const bool f32 = k.precision == LBM_FP32;
  const bool mrt = k.collision == LBM_COLL_MRT;
  const bool vd = blended_diffusivity(&k);
  if (k.flow == 9 && k.scalar == 0) return f32 ? F<Ops<9, 0, float>>::run(c, a...) : F<Ops<9, 0, double>>::run(c, a...);
  if (k.flow == 9 && k.scalar == 5) {
    if (vd) return f32 ? F<Ops<9, 5, float, kVarVD>>::run(c, a...) : F<Ops<9, 5, double, kVarVD>>::run(c, a...);
    return f32 ? F<Ops<9, 5, float>>::run(c, a...) : F<Ops<9, 5, double>>::run(c, a...);
  }
  if (k.flow == 19 && k.scalar == 0) {
    if (mrt)
      return f32 ? F<Ops<19, 0, float, kVarMRT>>::run(c, a...) : F<Ops<19, 0, double, kVarMRT>>::run(c, a...);
    return f32 ? F<Ops<19, 0, float>>::run(c, a...) : F<Ops<19, 0, double>>::run(c, a...);
  }
  if (mrt && vd) {
    constexpr int V = kVarMRT | kVarVD;
    return f32 ? F<Ops<19, 7, float, V>>::run(c, a...) : F<Ops<19, 7, double, V>>::run(c, a...);
  }
  if (mrt) return f32 ? F<Ops<19, 7, float, kVarMRT>>::run(c, a...) : F<Ops<19, 7, double, kVarMRT>>::run(c, a...);
  if (vd) return f32 ? F<Ops<19, 7, float, kVarVD>>::run(c, a...) : F<Ops<19, 7, double, kVarVD>>::run(c, a...);
  return f32 ? F<Ops<19, 7, float>>::run(c, a...) : F<Ops<19, 7, double>>::run(c, a...);
}

inline void* ckpt_slot(lbm_ctx* c, int64_t s) { return c->ckpt + (uint64_t)s * c->plan.state_bytes; }
// Moment set of step k (slot k mod C).
inline void* mom_slot(lbm_ctx* c, int64_t k) { return c->mom + (uint64_t)(k % c->plan.C) * c->plan.mom_bytes; }
// Trajectory segment holding the horizon's last step (0 in a store-all plan).
inline int64_t last_segment(lbm_ctx* c) { return c->cfg.nsteps > 0 ? (c->cfg.nsteps - 1) / c->plan.C : 0; }
inline void* other_pp(lbm_ctx* c, const void* cur) { return (cur == c->pp[0]) ? c->pp[1] : c->pp[0]; }

// In-place plan with checkpoints (C < N): the working buffer is a slot of its own.
inline bool checkpointed(const lbm_ctx* c) { return c->plan.inplace && c->plan.C < c->cfg.nsteps; }

// Ping-pong steps cut into launches of at most `most` steps, about equally long,
// as many of them as keep the number of launches odd or even with the number of
// steps: a call leaves its result in the buffer that one-step launches would
// have (a captured call of an even number of steps can be replayed).
struct Split {
  int64_t left, launches;
  int ns = 0;  // steps of the current launch
  Split(int64_t steps, int most) : left(steps), launches((steps + most - 1) / most) {
    if ((launches ^ steps) & 1) ++launches;
  }
  bool next() {
    if (left == 0) return false;
    ns = (int)((left + launches - 1) / launches);
    left -= ns;
    --launches;
    return true;
  }
};

// In place, several steps per launch go to another buffer and the next launch
// brings the state back: e steps there and e back (0: run single steps).  Both
// buffers hold the layout of an even phase, so `done` (steps so far) and e are even.
inline int steps_there_and_back(int64_t done, int64_t room, int most) {
  if (done % 2 != 0) return 0;
  const int64_t e = std::min<int64_t>(most, room / 2) & ~(int64_t)1;
  return (int)e;
}

// Most steps per launch of an in-place call.  The buffer that several steps go through
// is free when the call is made: the adjoint buffer before an adjoint or one-shot
// iteration, the working buffer once the adjoint has consumed its state.  A captured
// call runs when its graph is replayed, and the buffer may be in use by then, so such a
// call streams in its own buffer, one step per launch.
inline int most_in_place(lbm_ctx* c, int most) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &s) != hipSuccess) {
    (void)hipGetLastError();
    return 1;
  }
  return s == hipStreamCaptureStatusNone ? most : 1;
}

// Destination of h^k while recording: a checkpoint slot or a ping-pong buffer.
inline void* rec_dst(lbm_ctx* c, int64_t k) {
  const int64_t C = c->plan.C;
  const int64_t s = (k + 1) / C, i = (k + 1) % C;
  if (i == 0 && s < c->plan.S) return ckpt_slot(c, s);
  return other_pp(c, c->cur);
}

// Whole window captured and the run at its end: the objective is the window mean.
inline bool window_complete(const lbm_ctx* c) {
  return c->plan.W > 1 && c->win_count == c->plan.W && c->t == c->cfg.nsteps;
}

// The buffer that holds the state at t = 0: the in-place working buffer, or
// checkpoint slot 0 (ping-pong: the first checkpoint itself).
inline void* initial_buffer(lbm_ctx* c) { return c->plan.inplace ? c->work : ckpt_slot(c, 0); }

// Checks shared by every batched call: same lattice/precision/stream, distinct.
inline lbm_status check_batch(lbm_ctx* const* cs, int32_t n) {
  if (!cs || n < 1 || n > kBatchMax) return LBM_EINVAL;
  for (int k = 0; k < n; ++k) {
    if (!cs[k]) return LBM_EINVAL;
    for (int q = 0; q < k; ++q)
      if (cs[q] == cs[k]) return fail(cs[0], LBM_EINVAL, "batch: context %d appears twice", k);
    if (cs[k]->plan.inplace != cs[0]->plan.inplace)
      return fail(cs[0], LBM_EINVAL, "batch: context %d %s in place, context 0 %s", k,
                  cs[k]->plan.inplace ? "streams" : "does not stream", cs[0]->plan.inplace ? "does" : "does not");
    if (cs[k]->plan.W > 1) return fail(cs[0], LBM_EINVAL, "batch: context %d averages its objective", k);
    const lbm_config &a = cs[0]->cfg, &b = cs[k]->cfg;
    if (a.flow != b.flow || a.scalar != b.scalar || a.precision != b.precision)
      return fail(cs[0], LBM_EINVAL, "batch: context %d has another lattice or precision", k);
    if (cs[k]->stream != cs[0]->stream) return fail(cs[0], LBM_EINVAL, "batch: context %d uses another stream", k);
  }
  return LBM_OK;
}

// Kernel variant of a context (the V of its Ops).  A launch runs one variant, and the
// variants record different moments: the members of a batch that differ in it are
// launched apart.
inline int kernel_variant(const lbm_ctx* c) {
  return (c->cfg.collision == LBM_COLL_MRT ? kVarMRT : 0) | (blended_diffusivity(&c->cfg) ? kVarVD : 0);
}

// The members of a batch whose kernel variant is that of cs[first], from cs[first] on, when
// no member before it has this variant (else none: they went with that one).
inline int batch_part(lbm_ctx* const* cs, int n, int first, lbm_ctx** part) {
  const int v = kernel_variant(cs[first]);
  for (int k = 0; k < first; ++k)
    if (kernel_variant(cs[k]) == v) return 0;
  int m = 0;
  for (int k = first; k < n; ++k)
    if (kernel_variant(cs[k]) == v) part[m++] = cs[k];
  return m;
}

inline void reset_times(lbm_ctx* c) {
  c->t = 0;
  c->rec_len = 0;
  c->rec_open = true;
  c->cur = initial_buffer(c);
  c->adj_started = false;
  c->t_adj = -1;
  c->lam_cur = 0;
  c->mom_seg = -1;
  c->os_active = false;
  c->state_lost = false;
  c->win_count = 0;
}

inline lbm_status sync_check(lbm_ctx* c, const char* what) {
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return fail(c, LBM_EHIP, "%s: %s", what, hipGetErrorString(e));
  return LBM_OK;
}

}  // namespace lbmh
