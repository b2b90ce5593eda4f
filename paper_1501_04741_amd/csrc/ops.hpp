// Typed operations of one lattice, precision and variant: Ops<Q, QS, Real, V>
// launches the kernels, the Run* templates are the bodies of the C ABI calls
// (declared in context.hpp).  Only variants.hip includes this file: each
// instantiation is a translation unit of its own.
#pragma once

#include "context.hpp"
#include "tiles.hpp"

namespace lbmh {

// Typed operations on one context.
template <int Q, int QS, typename Real, int V>
struct Ops {
  using RealT = Real;
  static constexpr int kQ = Q, kQS = QS;
  static constexpr bool kLx = !(V & kVarMRT);  // staged kernels; MRT keeps the plain access (see lx_rows)
  static Params<Real> P(lbm_ctx* c) { return make_params<Real>(c->cfg, c->plan.N); }
  static int batch_blocks(lbm_ctx* c, int kw, int rpb) {
    const int rows = c->cfg.ny * c->cfg.nz;
    return rpb == 1 ? batch_waves(c) / kw * rows : (rows + rpb - 1) / rpb;
  }
  // batched steps in access pattern acc (ping-pong, or one in-place phase)
  template <bool NTV, bool MOMV>
  static void primal_batch_acc(hipStream_t st, const BatchArgs<Real>& A, dim3 g, dim3 b, int acc) {
    if (acc == ACC_EVEN && NTV && A.nte)
      hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_EVEN, true>), g, b, 0, st, A);
    else if (acc == ACC_EVEN) hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_EVEN>), g, b, 0, st, A);
    else if (acc == ACC_ODD && A.lx)
      hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_ODD, false, kLx>), g, b, 0, st, A);
    else if (acc == ACC_ODD) hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_ODD>), g, b, 0, st, A);
    else if (A.lx) hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_PP, false, kLx>), g, b, 0, st, A);
    else hipLaunchKernelGGL((k_primal_batch<Q, QS, Real, V, NTV, MOMV, ACC_PP>), g, b, 0, st, A);
  }
  static void primal_batch(hipStream_t st, const BatchArgs<Real>& A, int blocks, int acc = ACC_PP) {
    const dim3 g(blocks), b(kWave * A.kw * A.rpb);
    const bool mom = A.m[0] != nullptr;  // every member records, or none
    if (A.nt) {
      if (mom) primal_batch_acc<true, true>(st, A, g, b, acc);
      else primal_batch_acc<true, false>(st, A, g, b, acc);
    } else {
      if (mom) primal_batch_acc<false, true>(st, A, g, b, acc);
      else primal_batch_acc<false, false>(st, A, g, b, acc);
    }
  }
  // streaming stores and hints whatever the state size (see adjoint_inplace)
  static void adjoint_batch(hipStream_t st, const BatchArgs<Real>& A, int blocks, int acc = ACC_PP) {
    const dim3 g(blocks), b(kWave * A.kw * A.rpb);
    if (acc == ACC_EVEN && A.nte)
      hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_EVEN, true>), g, b, 0, st, A);
    else if (acc == ACC_EVEN) hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_EVEN>), g, b, 0, st, A);
    else if (acc == ACC_ODD && A.lx && A.nte)
      hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_ODD, true, kLx>), g, b, 0, st, A);
    else if (acc == ACC_ODD && A.lx)
      hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_ODD, false, kLx>), g, b, 0, st, A);
    else if (acc == ACC_ODD) hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_ODD>), g, b, 0, st, A);
    else if (A.lx) hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_PP, false, kLx>), g, b, 0, st, A);
    else hipLaunchKernelGGL((k_adjoint_batch<Q, QS, Real, V, true, ACC_PP>), g, b, 0, st, A);
  }

  // ---- several steps per launch (2D tiles, tiles.hpp)
  static constexpr bool kTiled = Q == 9;
  // Tile and steps per launch of the 2D lattices `cs` advance together: the least time per
  // step by what tile launches were measured to take (us).  A launch: 3.75 (its gap, the
  // first loads, the last stores) and the states read and written once at 5 TB/s; a step:
  // 0.75 + k W, W the wavefronts of valid region nodes per SIMD, k = 0.37 (FP32 D2Q9), 0.62
  // (with D2Q5), 0.9 and 2.5 in FP64.  In place only an even number of steps (see
  // steps_there_and_back).  Measured, whole evaluations, per step (one-step launches): 256x128
  // in FP32, 7 steps of 8x16 tiles 1.7 us (4.2); 1024x512, 5 steps of 16x32 tiles 6.6 (10.0);
  // 512x256 with D2Q5, 5 steps of 16x16 tiles 3.6 (6.0); 64x32 in FP64, 7 steps of 4x4 tiles
  // 1.6 (4.5); in place, 1100x560 with D2Q5 in FP64, 2 steps 21.0 (26.5), 4 steps 24.5.  The
  // model compares tiles with each other only; where one-step launches are the faster
  // ones is tile_rule's.  Whole rows cost no time where the states fit the L2s.
  static TileChoice choose_tile(lbm_ctx* const* cs, int n, LaunchKind kind) {
    constexpr int kSizes[] = {4, 8, 12, 16, 20, 24, 28, 32, 48, 56};
    constexpr int kMostThreads =
        std::min<int>(tile_threads_max<Real>(), 65536 / (2 * tile_values<Q, QS>() * (int)sizeof(Real)));
    constexpr double k = sizeof(Real) == 8 ? (QS > 0 ? 2.5 : 0.9) : (QS > 0 ? 0.62 : 0.37);
    const int by = cs[0]->plan.inplace ? 2 : 1;
    const TileRule rule = tile_rule(cs, n, kind);
    TileChoice best;
    if (!rule.tiles) return best;
    double least = 0, bytes = 0;
    int64_t tiles[std::size(kSizes)][std::size(kSizes)] = {};
    for (int q = 0; q < n; ++q) {
      bytes += 2.0 * cs[q]->plan.state_bytes;
      int gx[std::size(kSizes)];
      for (size_t i = 0; i < std::size(kSizes); ++i) gx[i] = (cs[q]->cfg.nx + kSizes[i] - 1) / kSizes[i];
      for (size_t j = 0; j < std::size(kSizes); ++j) {
        const int64_t gy = (cs[q]->cfg.ny + kSizes[j] - 1) / kSizes[j];
        for (size_t i = 0; i < std::size(kSizes); ++i) tiles[j][i] += gx[i] * gy;
      }
    }
    for (int ns = 2; ns <= 8; ns += by)
      for (size_t j = 0; j < std::size(kSizes); ++j)
        for (size_t i = 0; i < std::size(kSizes); ++i) {
          const int tx = kSizes[i], ty = kSizes[j];
          if (rule.whole_rows && bytes > kL2Bytes && tx * sizeof(Real) % 64 != 0) continue;
          const int threads = (tx + 2 * (ns - 1)) * (ty + 2 * (ns - 1));
          if (threads > kMostThreads) break;
          const int64_t blocks = tiles[j][i];
          int64_t valid = 0;
          for (int s = 0; s < ns; ++s) valid += (tx + 2 * s) * (ty + 2 * s);
          const double per_cu = blocks <= 2 * kCus ? (double)((blocks + kCus - 1) / kCus) : (double)blocks / kCus;
          const double waves = per_cu * ((threads + 63) / 64) / 4.0 * (double)valid / (ns * threads);
          const double cost = (3.75 + bytes / 5e6) / ns + 0.75 + k * waves;
          if (best.ns == 1 || cost < least) {
            least = cost;
            best = TileChoice{tx, ty, ns};
          }
        }
    return best;
  }
  // called once, when the context is created
  static void choose(lbm_ctx* c) {
    if constexpr (kTiled)
      for (const LaunchKind k : {STEPS, RECORDED, ADJOINT}) c->tile[k] = choose_tile(&c, 1, k);
  }
  static dim3 tile_block(const TileChoice& t, int ns) { return dim3(t.tx + 2 * (ns - 1), t.ty + 2 * (ns - 1), 1); }
  static size_t tile_bytes(const TileChoice& t, int ns) {
    const dim3 b = tile_block(t, ns);
    return ns > 1 ? (size_t)2 * tile_values<Q, QS>() * b.x * b.y * sizeof(Real) : 0;
  }
  static TileRow tile_row(lbm_ctx* c, const TileChoice& t) { return TileRow::of((c->cfg.nx + t.tx - 1) / t.tx); }
  static int tiles(lbm_ctx* c, const TileChoice& t) {
    return ((c->cfg.nx + t.tx - 1) / t.tx) * ((c->cfg.ny + t.ty - 1) / t.ty);
  }
  static size_t mom_stride(lbm_ctx* c) { return c->plan.mom_bytes / sizeof(Real); }
  // ns primal steps from src to dst (different buffers), recording from moment set mom when
  // it is set.  inplace: both in the in-place layout of an even time, ns even.
  static void primal_many(lbm_ctx* c, const void* src, void* dst, void* mom, int ns, bool inplace) {
    if constexpr (kTiled) {
      const TileChoice& t = c->tile[mom ? RECORDED : STEPS];
#define LBM_TILE(MOMV, ACCV)                                                                                        \
  hipLaunchKernelGGL((k_primal_tile<Q, QS, Real, MOMV, V, ACCV>), dim3(tiles(c, t)), tile_block(t, ns),             \
                     tile_bytes(t, ns), c->stream, P(c), (const Real*)src, (Real*)dst, (const Real*)c->w, (Real*)mom, \
                     mom_stride(c), ns, tile_row(c, t))
      if (inplace) {
        if (mom) LBM_TILE(true, ACC_EVEN);
        else LBM_TILE(false, ACC_EVEN);
      } else {
        if (mom) LBM_TILE(true, ACC_PP);
        else LBM_TILE(false, ACC_PP);
      }
#undef LBM_TILE
    }
  }
  // ns adjoint steps from lin to lout (different buffers), the first of them with moment set
  // mom.  inplace: both in the layout after an even number of adjoint steps, ns even.
  static void adjoint_many(lbm_ctx* c, const void* mom, const void* lin, void* lout, int ns, bool inplace) {
    if constexpr (kTiled) {
      const TileChoice& t = c->tile[ADJOINT];
#define LBM_TILE(ACCV)                                                                                              \
  hipLaunchKernelGGL((k_adjoint_tile<Q, QS, Real, V, ACCV>), dim3(tiles(c, t)), tile_block(t, ns),                  \
                     tile_bytes(t, ns), c->stream, P(c), (const Real*)mom, (const Real*)lin, (Real*)lout,           \
                     (const Real*)c->w, (Real*)c->grad, mom_stride(c), ns, tile_row(c, t))
      if (inplace) LBM_TILE(ACC_ODD);
      else LBM_TILE(ACC_PP);
#undef LBM_TILE
    }
  }

  // The same over the members of a batch: A's buffers, one tile t for all of them.
  static void primal_many_batch(hipStream_t st, const BatchArgs<Real>& A, const TileChoice& t, int ns, bool inplace) {
    if constexpr (kTiled) {
      const dim3 g(A.start[A.n]);
#define LBM_TILE(MOMV, ACCV)                                                                               \
  hipLaunchKernelGGL((k_primal_tile_batch<Q, QS, Real, MOMV, V, ACCV>), g, tile_block(t, ns), tile_bytes(t, ns), st, \
                     A, ns)
      const bool mom = A.m[0] != nullptr;  // every member records, or none
      if (inplace) {
        if (mom) LBM_TILE(true, ACC_EVEN);
        else LBM_TILE(false, ACC_EVEN);
      } else {
        if (mom) LBM_TILE(true, ACC_PP);
        else LBM_TILE(false, ACC_PP);
      }
#undef LBM_TILE
    }
  }
  static void adjoint_many_batch(hipStream_t st, const BatchArgs<Real>& A, const TileChoice& t, int ns, bool inplace) {
    if constexpr (kTiled) {
      const dim3 g(A.start[A.n]);
#define LBM_TILE(ACCV)                                                                                   \
  hipLaunchKernelGGL((k_adjoint_tile_batch<Q, QS, Real, V, ACCV>), g, tile_block(t, ns), tile_bytes(t, ns), st, A, ns)
      if (inplace) LBM_TILE(ACC_ODD);
      else LBM_TILE(ACC_PP);
#undef LBM_TILE
    }
  }

  // streaming stores (and cotangent loads) when the state buffers a launch touches exceed the
  // last-level cache: ping-pong primal and adjoint 2, in-place primal 1, one-shot 4 (2 in place)
  static bool nt(lbm_ctx* c, int buffers) { return buffers * c->plan.state_bytes > kLastLevelCacheBytes; }
  // dynamic LDS of an LX launch: the staging runs of `states` states, one value per thread each
  static size_t lx_bytes(const Geo& g, int states) {
    return (size_t)states * Shifted<Q, QS>::count() * g.block.x * g.block.y * sizeof(Real);
  }
  // LX variant for this context and launch: rows that fit a block, and staging
  // within 64 KB of LDS per block (the FP64 one-shot of D3Q19 + D3Q7 on 512-wide
  // blocks would need 96 KB and keeps the plain access)
  static bool lx(lbm_ctx* c, const Geo& g, int states) {
    return lx_rows(c->cfg) && lx_bytes(g, states) <= 65536;
  }
  // access pattern of the current state buffer: ping-pong, or the in-place phase of step t
  static int acc(lbm_ctx* c) { return c->plan.inplace ? ((c->t % 2 == 0) ? ACC_EVEN : ACC_ODD) : ACC_PP; }
  // One in-place step from the current phase; records the moments when mom != null.
  // Streaming stores and hints: a recorded step takes them once its state exceeds
  // the last-level cache (plain stores: 0.819 -> 0.748 of peak, D3Q19 FP32
  // 256x128x128), its even phase's loads only beyond twice the cache.  An
  // unrecorded step stores plainly up to the cache size (NT stores in the odd
  // phase cost 0.76 -> 0.73 at 128x96x96 and 0.88 -> 0.86 at 192x128x128); between
  // one and two caches its odd (staged) phase takes NT stores and the even phase
  // stays plain (0.787 -> 0.860 at 256x128x128; NT stores in both phases 0.741,
  // with the even-phase load hint 0.839); beyond twice the cache it takes NT
  // stores and hinted loads in both phases (0.662 -> 0.750 at 512x256x128, 0.668 ->
  // 0.815 at 512x128x128; a plain even phase there 0.66 and 0.67).
  static void primal_inplace(lbm_ctx* c, void* buf, int64_t t, void* mom) {
    Geo g = hot_geometry(c->cfg);
    Real* a = (Real*)buf;
    const Real* w = (const Real*)c->w;
    Real* m = (Real*)mom;
    const bool even = (t % 2 == 0);
    const bool lx = Ops::lx(c, g, 1);
#define LBM_PI(NTV, MOMV, ACCV)                                                                                    \
  do {                                                                                                             \
    if (ACCV == ACC_ODD && lx)                                                                                     \
      hipLaunchKernelGGL((k_primal_inplace<Q, QS, Real, NTV, MOMV, V, ACC_ODD, false, kLx>), g.grid, g.block,     \
                         lx_bytes(g, 1), c->stream, P(c), a, w, m);                                                \
    else                                                                                                           \
      hipLaunchKernelGGL((k_primal_inplace<Q, QS, Real, NTV, MOMV, V, ACCV>), g.grid, g.block, 0, c->stream, P(c), \
                         a, w, m);                                                                                 \
  } while (0)
    if (m && nt(c, 1)) {
      // the even phase's loads take the streaming hint too once the state is far beyond the cache
      if (even && c->plan.state_bytes > 2 * kLastLevelCacheBytes)
        hipLaunchKernelGGL((k_primal_inplace<Q, QS, Real, true, true, V, ACC_EVEN, true>), g.grid, g.block, 0,
                           c->stream, P(c), a, w, m);
      else if (even) LBM_PI(true, true, ACC_EVEN);
      else LBM_PI(true, true, ACC_ODD);
    } else if (m) {
      if (even) LBM_PI(false, true, ACC_EVEN);
      else LBM_PI(false, true, ACC_ODD);
    } else if (c->plan.state_bytes > 2 * kLastLevelCacheBytes) {
      // unrecorded, state far beyond the cache: streaming stores and hinted loads in both phases
      if (even)
        hipLaunchKernelGGL((k_primal_inplace<Q, QS, Real, true, false, V, ACC_EVEN, true>), g.grid, g.block, 0,
                           c->stream, P(c), a, w, m);
      else LBM_PI(true, false, ACC_ODD);
    } else if (nt(c, 1)) {
      // unrecorded, state between one and two caches: streaming stores in the odd phase only
      if (even) LBM_PI(false, false, ACC_EVEN);
      else LBM_PI(true, false, ACC_ODD);
    } else {
      if (even) LBM_PI(false, false, ACC_EVEN);
      else LBM_PI(false, false, ACC_ODD);
    }
#undef LBM_PI
  }
  static void oneshot_inplace(lbm_ctx* c, double zeta, double pen) {
    Geo g = hot_geometry(c->cfg);
    Real* a = (Real*)c->cur;
    Real* l = (Real*)c->lam[0];
    Real* w = (Real*)c->w;
    Real* gr = (Real*)c->grad;
    const double* gl = (const double*)c->glob;
    const bool even = (c->t % 2 == 0);
    const bool lx = Ops::lx(c, g, 2);
#define LBM_OS_INPLACE(NTV, ACCV)                                                                                 \
  do {                                                                                                            \
    if (ACCV == ACC_ODD && lx)                                                                                    \
      hipLaunchKernelGGL((k_oneshot_inplace<Q, QS, Real, NTV, V, ACC_ODD, kLx>), g.grid, g.block, lx_bytes(g, 2),  \
                         c->stream, P(c), a, l, w, gr, gl, (Real)zeta, (Real)pen);                                \
    else                                                                                                          \
      hipLaunchKernelGGL((k_oneshot_inplace<Q, QS, Real, NTV, V, ACCV>), g.grid, g.block, 0, c->stream, P(c), a, l, \
                         w, gr, gl, (Real)zeta, (Real)pen);                                                       \
  } while (0)
    if (nt(c, 2)) {
      if (even) LBM_OS_INPLACE(true, ACC_EVEN);
      else LBM_OS_INPLACE(true, ACC_ODD);
    } else {
      if (even) LBM_OS_INPLACE(false, ACC_EVEN);
      else LBM_OS_INPLACE(false, ACC_ODD);
    }
#undef LBM_OS_INPLACE
  }
  static lbm_status write_static(lbm_ctx* c) {
    static_assert(sizeof(BatchStatic<Real>) <= kDescBytes, "descriptor region too small");
    BatchStatic<Real> h;
    h.p = P(c);
    h.waves = batch_waves(c);
    h.mom_stride = mom_stride(c);
    hipLaunchKernelGGL((k_write_desc<Real>), dim3(1), dim3(64), 0, c->stream, h, (BatchStatic<Real>*)c->desc);
    return launch_check(c, "descriptor upload");
  }
  static_assert(Mom<Q, QS, V>::N == (Q == 19 ? 3 : 2) + 1 + (QS > 0 ? ((V & kVarVD) ? QS : 1) : 0),
                "moment count mismatch");
  // One primal step; records the moments of the pulled state when mom != null.
  static void primal(lbm_ctx* c, const void* src, void* dst, void* mom = nullptr) {
    Geo g = hot_geometry(c->cfg);
    const Real* s = (const Real*)src;
    Real* d = (Real*)dst;
    const Real* w = (const Real*)c->w;
    Real* m = (Real*)mom;
#define LBM_PP(NTV, MOMV)                                                                                     \
  do {                                                                                                        \
    if (Ops::lx(c, g, 1))                                                                                     \
      hipLaunchKernelGGL((k_primal<Q, QS, Real, NTV, MOMV, V, kLx>), g.grid, g.block, lx_bytes(g, 1), c->stream,  \
                         P(c), s, d, w, m);                                                                   \
    else                                                                                                      \
      hipLaunchKernelGGL((k_primal<Q, QS, Real, NTV, MOMV, V>), g.grid, g.block, 0, c->stream, P(c), s, d, w, m); \
  } while (0)
    if (nt(c, 2)) {
      if (m) LBM_PP(true, true);
      else LBM_PP(true, false);
    } else {
      if (m) LBM_PP(false, true);
      else LBM_PP(false, false);
    }
#undef LBM_PP
  }
  static void objective(lbm_ctx* c, const void* src, double* out) {
    double* part = c->glob + kGlobSlots;
    hipLaunchKernelGGL((k_objective_partial<Q, QS, Real>), dim3(kObjBlocks), dim3(kObjThreads), 0, c->stream, P(c),
                       (const Real*)src, part, acc(c));
    hipLaunchKernelGGL((k_objective_final<Q, QS, Real>), dim3(1), dim3(64), 0, c->stream, P(c),
                       (const double*)part, out);
  }
  static void seed(lbm_ctx* c, const void* src, void* lam) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_seed<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)src,
                       (const double*)c->glob, (Real*)lam, acc(c), c->plan.inplace ? 1 : 0,
                       1.0 / (double)c->plan.W);
  }
  // Window state s: its boundary sums and objective, and its inlet/outlet columns.
  static void capture(lbm_ctx* c, const void* src, int64_t s) {
    objective(c, src, win_glob(c, s));
    const int n = 2 * c->cfg.ny * c->cfg.nz;
    hipLaunchKernelGGL((k_capture_columns<Q, QS, Real>), dim3((n + 255) / 256), dim3(256), 0, c->stream, P(c),
                       (const Real*)src, acc(c), (Real*)win_cols(c, s));
  }
  // lambda^n += (1/W) dJ/df^n of window state s, lambda^n in layout pattern.
  static void window_seed(lbm_ctx* c, int64_t s, void* lam, int pattern) {
    const int n = 2 * c->cfg.ny * c->cfg.nz;
    hipLaunchKernelGGL((k_window_seed<Q, QS, Real>), dim3((n + 255) / 256), dim3(256), 0, c->stream, P(c),
                       (const Real*)win_cols(c, s), (const double*)win_glob(c, s), (Real*)lam, pattern,
                       1.0 / (double)c->plan.W);
  }
  // One in-place adjoint step: the cotangent buffer is in the odd-pattern layout
  // after an even number of adjoint steps (the seed writes that layout).
  static void adjoint_inplace(lbm_ctx* c, const void* mom, int64_t steps_done) {
    Geo g = hot_geometry(c->cfg);
    const Real* m = (const Real*)mom;
    Real* l = (Real*)c->lam[0];
    const Real* w = (const Real*)c->w;
    Real* gr = (Real*)c->grad;
    const bool odd = (steps_done % 2 == 0);
    const bool lx = Ops::lx(c, g, 1);
    const bool far = c->plan.state_bytes > 2 * kLastLevelCacheBytes;  // streaming hints on the staged accesses
#define LBM_AI(NTV, ACCV)                                                                                         \
  do {                                                                                                            \
    if (ACCV == ACC_ODD && lx && far)                                                                             \
      hipLaunchKernelGGL((k_adjoint_inplace<Q, QS, Real, NTV, V, ACC_ODD, true, kLx>), g.grid, g.block,          \
                         lx_bytes(g, 1), c->stream, P(c), m, l, w, gr);                                           \
    else if (ACCV == ACC_ODD && lx)                                                                               \
      hipLaunchKernelGGL((k_adjoint_inplace<Q, QS, Real, NTV, V, ACC_ODD, false, kLx>), g.grid, g.block,         \
                         lx_bytes(g, 1), c->stream, P(c), m, l, w, gr);                                           \
    else                                                                                                          \
      hipLaunchKernelGGL((k_adjoint_inplace<Q, QS, Real, NTV, V, ACCV>), g.grid, g.block, 0, c->stream, P(c), m, l, \
                         w, gr);                                                                                  \
  } while (0)
    // streaming stores and hints whatever the state size: the adjoint also streams a moment set per
    // step, and a cotangent state that fits the last-level cache gains nothing from staying there
    // (192x96x96 D3Q19 FP32, 134 MB: 0.769 -> 0.836 of HBM peak; 128x96x96: 0.738 -> 0.771)
    if (odd) LBM_AI(true, ACC_ODD);
    else if (c->plan.state_bytes > 2 * kLastLevelCacheBytes)  // even-phase hint far beyond the cache
      hipLaunchKernelGGL((k_adjoint_inplace<Q, QS, Real, true, V, ACC_EVEN, true>), g.grid, g.block, 0, c->stream,
                         P(c), m, l, w, gr);
    else LBM_AI(true, ACC_EVEN);
#undef LBM_AI
  }
  static void adjoint(lbm_ctx* c, const void* mom, const void* lin, void* lout) {
    Geo g = hot_geometry(c->cfg);
    const Real *m = (const Real*)mom, *li = (const Real*)lin, *w = (const Real*)c->w;
    Real *lo = (Real*)lout, *gr = (Real*)c->grad;
    const bool lx = Ops::lx(c, g, 1);
    // streaming whatever the state size, as the in-place adjoint
    if (lx)
      hipLaunchKernelGGL((k_adjoint<Q, QS, Real, true, V, kLx>), g.grid, g.block, lx_bytes(g, 1), c->stream, P(c), m,
                         li, lo, w, gr);
    else
      hipLaunchKernelGGL((k_adjoint<Q, QS, Real, true, V>), g.grid, g.block, 0, c->stream, P(c), m, li, lo, w, gr);
  }
  static void oneshot(lbm_ctx* c, const void* src, void* dst, const void* lin, void* lout, double zeta,
                      double pen) {
    Geo g = hot_geometry(c->cfg);
    const Real *s = (const Real*)src, *li = (const Real*)lin;
    Real *d = (Real*)dst, *lo = (Real*)lout, *w = (Real*)c->w, *gr = (Real*)c->grad;
    const double* gl = (const double*)c->glob;
    const bool lx = Ops::lx(c, g, 2);
#define LBM_OS(NTV, LXV)                                                                                   \
  hipLaunchKernelGGL((k_oneshot<Q, QS, Real, NTV, V, LXV && kLx>), g.grid, g.block, LXV ? lx_bytes(g, 2) : 0, c->stream, \
                     P(c), s, d, li, lo, w, gr, gl, (Real)zeta, (Real)pen)
    if (nt(c, 4)) {
      if (lx) LBM_OS(true, true);
      else LBM_OS(true, false);
    } else {
      if (lx) LBM_OS(false, true);
      else LBM_OS(false, false);
    }
#undef LBM_OS
  }
  static void get_adjoint(lbm_ctx* c, const void* lam, double* lf, double* lg, int pattern) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_get_adjoint<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)lam, lf, lg,
                       pattern);
  }
  static void fields(lbm_ctx* c, const void* src, double* rho, double* u, double* s) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_fields<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)src, rho, u, s,
                       acc(c));
  }
  static void get_state(lbm_ctx* c, const void* src, double* f, double* gg) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_get_state<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)src, f, gg,
                       acc(c));
  }
  static void set_state(lbm_ctx* c, const double* f, const double* gg, void* dst) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_set_state<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), f, gg, (Real*)dst,
                       c->plan.inplace ? ACC_EVEN : ACC_PP);
  }
  static void maps(lbm_ctx* c, uint8_t* mask, int64_t* src) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_maps<Q, QS, Real>), g.grid, g.block, 0, c->stream, P(c), mask, src);
  }
  static void fill(lbm_ctx* c, void* a, size_t n) {
    hipLaunchKernelGGL((k_fill<Real>), flat_grid(n), dim3(256), 0, c->stream, (Real*)a, n, Real(0));
  }
  static void copy(lbm_ctx* c, const void* a, void* b, size_t n) {
    hipLaunchKernelGGL((k_copy<Real>), flat_grid(n), dim3(256), 0, c->stream, (const Real*)a, (Real*)b, n);
  }
  // node array: compact ABI layout -> padded workspace layout, and back
  static void node_in(lbm_ctx* c, const void* a, void* b) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_node_in<Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)a, (Real*)b);
  }
  static void grad_penalty(lbm_ctx* c, double pen, void* b) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_grad_penalty<Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)c->grad,
                       (const Real*)c->w, (Real)pen, (Real*)b);
  }
  static void node_out(lbm_ctx* c, const void* a, void* b) {
    Geo g = node_geometry(c->cfg);
    hipLaunchKernelGGL((k_node_out<Real>), g.grid, g.block, 0, c->stream, P(c), (const Real*)a, (Real*)b);
  }
};

// Time-averaged objective: capture the state just produced (time t) when it is
// the next state of the window [N - W + 1, N] of a run that started at t = 0.
template <class O>
void capture_window(lbm_ctx* c) {
  const int64_t W = c->plan.W, first = c->cfg.nsteps - W + 1;
  if (W > 1 && c->t >= first && c->t - first == c->win_count) {
    O::capture(c, c->cur, c->win_count);
    ++c->win_count;
  }
}

// Steps from time t that may share launches: up to `left`, within the segment
// of t when segments matter (recorded: their ends are checkpoints and the moment
// sets of one are contiguous), and before the window of a time-averaged objective,
// whose states are captured one by one.
inline int64_t steps_together(lbm_ctx* c, int64_t t, int64_t left, bool segments) {
  if (segments) left = std::min<int64_t>(left, c->plan.C - t % c->plan.C);
  if (c->plan.W > 1) left = std::min<int64_t>(left, c->cfg.nsteps - c->plan.W - t);
  return std::max<int64_t>(left, 1);
}

template <class O>
lbm_status RunPrimal<O>::run(lbm_ctx* c, int64_t nsteps, int record) {
  // A recorded run keeps the moments of the horizon's last segment only (all of
  // them in a store-all plan): the backward recomputes every earlier segment
  // from its checkpoint before it reads that segment's moments.
  const int64_t keep_from = last_segment(c) * c->plan.C;
  const auto mom = [&](int64_t t) { return record && t >= keep_from ? mom_slot(c, t) : nullptr; };
  const auto most = [&](int64_t t) {
    const int ns = c->tile[mom(t) ? RECORDED : STEPS].ns;
    return c->plan.inplace ? most_in_place(c, ns) : ns;
  };
  if (c->plan.inplace) {
    const bool ckpts = record && checkpointed(c);
    for (int64_t i = 0; i < nsteps;) {
      if (ckpts && c->t % c->plan.C == 0)  // the state at t = sC, in its phase's layout
        O::copy(c, c->work, ckpt_slot(c, c->t / c->plan.C), (size_t)c->plan.QT * c->plan.Np);
      const int64_t room = steps_together(c, c->t, nsteps - i, record != 0);
      const int e = c->os_active ? 0 : steps_there_and_back(c->t, room, most(c->t));
      if (e) {  // through the adjoint buffer, free until the adjoint starts, and back
        O::primal_many(c, c->work, c->lam[0], mom(c->t), e, true);
        O::primal_many(c, c->lam[0], c->work, mom(c->t + e), e, true);
        c->t += 2 * e;
        i += 2 * e;
        continue;
      }
      O::primal_inplace(c, c->work, c->t, mom(c->t));
      ++c->t;
      ++i;
      capture_window<O>(c);
    }
    return launch_check(c, "in-place primal step");
  }
  for (int64_t i = 0; i < nsteps;) {
    const int64_t room = steps_together(c, c->t, nsteps - i, record != 0);
    for (Split sp(room, most(c->t)); sp.next();) {
      void* src = c->cur;
      void* dst = record ? rec_dst(c, c->t + sp.ns - 1) : other_pp(c, c->cur);
      if (sp.ns > 1) O::primal_many(c, src, dst, mom(c->t), sp.ns, false);
      else O::primal(c, src, dst, mom(c->t));
      c->cur = dst;
      c->t += sp.ns;
      i += sp.ns;
    }
    capture_window<O>(c);
  }
  return launch_check(c, "primal step");
}

template <class O>
lbm_status RunObjective<O>::run(lbm_ctx* c, double* J_dev) {
  O::objective(c, c->cur, c->glob);
  if (window_complete(c))
    hipLaunchKernelGGL((k_window_mean<double>), dim3(1), dim3(64), 0, c->stream, (const double*)c->win, (int)c->plan.W,
                       c->glob);
  if (J_dev) {
    hipError_t e = hipMemcpyAsync(J_dev, c->glob + kNG, sizeof(double), hipMemcpyDeviceToDevice, c->stream);
    if (e != hipSuccess) return fail(c, LBM_EHIP, "objective copy: %s", hipGetErrorString(e));
  }
  return launch_check(c, "objective");
}

// Recompute segment s from its checkpoint: steps k = sC .. min(sC + C, N) - 1,
// recording their moments (the states themselves go through the ping-pong).
template <class O>
void recompute_segment(lbm_ctx* c, int64_t s) {
  Range r("lbm recompute segment");
  const int64_t C = c->plan.C;
  const int64_t end = std::min<int64_t>(s * C + C, c->rec_len);
  const void* src = ckpt_slot(c, s);
  int64_t k = s * C;
  for (Split sp(end - k, c->tile[RECORDED].ns); sp.next();) {
    void* dst = other_pp(c, src);
    if (sp.ns > 1) O::primal_many(c, src, dst, mom_slot(c, k), sp.ns, false);
    else O::primal(c, src, dst, mom_slot(c, k));
    src = dst;
    k += sp.ns;
  }
  c->mom_seg = s;
}

// In-place plan: recompute segment s inside its own checkpoint slot (its last
// use), recording the moments of steps sC .. min(sC + C, N) - 1; step k runs in
// the access pattern of its phase k mod 2, the layout the slot was saved in.
// Several steps per launch go through the working buffer, whose state the
// adjoint has consumed.
template <class O>
void recompute_segment_inplace(lbm_ctx* c, int64_t s) {
  const int most = most_in_place(c, c->tile[RECORDED].ns);
  Range r("lbm recompute segment (in place)");
  const int64_t C = c->plan.C;
  const int64_t end = std::min<int64_t>(s * C + C, c->rec_len);
  void* buf = ckpt_slot(c, s);
  for (int64_t k = s * C; k < end;) {
    if (const int e = steps_there_and_back(k, end - k, most)) {
      O::primal_many(c, buf, c->work, mom_slot(c, k), e, true);
      O::primal_many(c, c->work, buf, mom_slot(c, k + e), e, true);
      k += 2 * e;
      continue;
    }
    O::primal_inplace(c, buf, k, mom_slot(c, k));
    ++k;
  }
  c->mom_seg = s;
}

// Seeds lambda^N = dJ/df^N and zeroes the gradient (first adjoint call).
template <class O>
void start_adjoint(lbm_ctx* c) {
  const int64_t C = c->plan.C;
  O::objective(c, c->cur, c->glob);
  O::seed(c, c->cur, c->lam[0]);
  O::fill(c, c->grad, (size_t)c->plan.Np);
  c->lam_cur = 0;
  c->t_adj = c->rec_len;
  // the recorded run's moments are held when it ended in the horizon's last segment
  // (a batched run records every step, so this can miss a segment it holds: that
  // segment is then recomputed, with the same result)
  const int64_t s = c->rec_len > 0 ? (c->rec_len - 1) / C : -1;
  c->mom_seg = s == last_segment(c) ? s : -1;
  c->adj_started = true;
}

template <class O>
lbm_status RunAdjoint<O>::run(lbm_ctx* c, int64_t nsteps) {
  const int64_t C = c->plan.C;
  const int most = c->plan.inplace ? most_in_place(c, c->tile[ADJOINT].ns) : c->tile[ADJOINT].ns;
  // window states n < N whose objective terms enter lambda^n (none unless W > 1)
  const int64_t first = c->plan.W > 1 ? c->cfg.nsteps - c->plan.W + 1 : INT64_MAX;
  if (!c->adj_started) start_adjoint<O>(c);
  if (c->plan.inplace) {  // store-all never recomputes; C < N recomputes each segment in place
    for (int64_t i = 0; i < nsteps;) {
      const int64_t n = c->t_adj - 1;
      const int64_t s = n / C;
      if (s != c->mom_seg) recompute_segment_inplace<O>(c, s);
      const int64_t done = c->rec_len - c->t_adj;
      const int64_t room = n >= first ? 1 : std::min<int64_t>(nsteps - i, n % C + 1);
      if (const int e = steps_there_and_back(done, room, most)) {
        // through the working buffer, whose state the adjoint has consumed, and back
        O::adjoint_many(c, mom_slot(c, n), c->lam[0], c->work, e, true);
        O::adjoint_many(c, mom_slot(c, n - e), c->work, c->lam[0], e, true);
        c->t_adj -= 2 * e;
        i += 2 * e;
        continue;
      }
      O::adjoint_inplace(c, mom_slot(c, n), done);
      --c->t_adj;
      ++i;
      if (n >= first)  // lambda^n now in the layout of its step count
        O::window_seed(c, n - first, c->lam[0], ((c->rec_len - c->t_adj) % 2 == 0) ? ACC_ODD : ACC_EVEN);
    }
    return launch_check(c, "in-place adjoint step");
  }
  for (int64_t i = 0; i < nsteps;) {
    const int64_t n0 = c->t_adj - 1;
    const int64_t s = n0 / C;
    if (s != c->mom_seg) recompute_segment<O>(c, s);
    for (Split sp(n0 >= first ? 1 : std::min<int64_t>(nsteps - i, n0 % C + 1), most); sp.next();) {
      const void* mom = mom_slot(c, c->t_adj - 1);
      if (sp.ns > 1) O::adjoint_many(c, mom, c->lam[c->lam_cur], c->lam[1 - c->lam_cur], sp.ns, false);
      else O::adjoint(c, mom, c->lam[c->lam_cur], c->lam[1 - c->lam_cur]);
      c->lam_cur ^= 1;
      c->t_adj -= sp.ns;
      i += sp.ns;
    }
    if (n0 >= first) O::window_seed(c, n0 - first, c->lam[c->lam_cur], ACC_PP);
  }
  return launch_check(c, "adjoint step");
}

template <class O>
lbm_status RunReset<O>::run(lbm_ctx* c) {
  O::fill(c, initial_buffer(c), (size_t)c->plan.QT * c->plan.Np);
  return launch_check(c, "reset");
}

template <class O>
lbm_status RunSetState<O>::run(lbm_ctx* c, const double* f, const double* g) {
  O::set_state(c, f, g, initial_buffer(c));
  return launch_check(c, "set_state");
}

template <class O>
lbm_status RunGradient<O>::run(lbm_ctx* c, void* out) {
  O::node_out(c, c->grad, out);
  return launch_check(c, "gradient");
}

template <class O>
lbm_status RunGradientPenalty<O>::run(lbm_ctx* c, double pen, void* out) {
  O::grad_penalty(c, pen, out);
  return launch_check(c, "gradient_penalty");
}

template <class O>
lbm_status RunFields<O>::run(lbm_ctx* c, double* rho, double* u, double* s) {
  O::fields(c, c->cur, rho, u, s);
  return launch_check(c, "fields");
}

template <class O>
lbm_status RunGetState<O>::run(lbm_ctx* c, double* f, double* g) {
  O::get_state(c, c->cur, f, g);
  return launch_check(c, "get_state");
}

template <class O>
lbm_status RunGetAdjoint<O>::run(lbm_ctx* c, double* lf, double* lg) {
  // the one-shot's in-place buffer follows the primal's phase; the unsteady adjoint's
  // alternates from the seed's layout (odd pattern after an even number of steps)
  int pattern = c->adj_started ? ACC_PP : O::acc(c);
  if (c->plan.inplace && c->adj_started) pattern = ((c->rec_len - c->t_adj) % 2 == 0) ? ACC_ODD : ACC_EVEN;
  O::get_adjoint(c, c->lam[c->lam_cur], lf, c->plan.QS ? lg : nullptr, pattern);
  return launch_check(c, "get_adjoint");
}

template <class O>
lbm_status RunMaps<O>::run(lbm_ctx* c, uint8_t* mask, int64_t* src) {
  O::maps(c, mask, src);
  return launch_check(c, "export_maps");
}

template <class O>
lbm_status RunSetDesign<O>::run(lbm_ctx* c, const void* w) {
  O::node_in(c, w, c->w);
  return launch_check(c, "set_design");
}

// One-shot iterations: each is [objective sums of f^n when the seed depends
// on them] + one fused k_oneshot launch.  The first call zeroes lambda.
template <class O>
lbm_status RunOneshot<O>::run(lbm_ctx* c, int64_t nsteps, double zeta, double pen) {
  if (!c->os_active) {
    O::fill(c, c->lam[0], (size_t)c->plan.QT * c->plan.Np);
    c->lam_cur = 0;
    O::objective(c, c->cur, c->glob);
    c->os_active = true;
    c->rec_open = false;
  }
  // the variance term's source depends on the current outlet mean: refresh the sums every iteration
  const bool state_dependent_seed = (c->cfg.c_var != 0.0);
  for (int64_t i = 0; i < nsteps; ++i) {
    if (state_dependent_seed) O::objective(c, c->cur, c->glob);
    if (c->plan.inplace) {
      O::oneshot_inplace(c, zeta, pen);
      ++c->t;
      continue;
    }
    void* dst = (c->cur == c->pp[0]) ? c->pp[1] : c->pp[0];
    O::oneshot(c, c->cur, dst, c->lam[c->lam_cur], c->lam[1 - c->lam_cur], zeta, pen);
    c->cur = dst;
    c->lam_cur ^= 1;
    ++c->t;
  }
  return launch_check(c, "one-shot step");
}

template <class O>
lbm_status RunGetDesign<O>::run(lbm_ctx* c, void* out) {
  O::node_out(c, c->w, out);
  return launch_check(c, "get_design");
}

template <class O>
lbm_status RunWriteStatic<O>::run(lbm_ctx* c) {
  O::choose(c);
  return O::write_static(c);
}

// Member k of a launch over tiles or row parts.
template <class O>
void batch_member(BatchArgs<typename O::RealT>& A, int k, lbm_ctx* c, const void* a, const void* b, void* to, void* m) {
  using Real = typename O::RealT;
  A.st[k] = (const BatchStatic<Real>*)c->desc;
  A.w[k] = (const Real*)c->w;
  A.g[k] = (Real*)c->grad;
  A.a[k] = (const Real*)a;
  A.b[k] = (const Real*)b;
  A.c[k] = (Real*)to;
  A.m[k] = (Real*)m;
}

// Launch geometry of a batch of members `mem`: one-step launches (tile.ns or ns 1) in
// row parts, several steps in tiles.
template <class O>
int batch_geometry(BatchArgs<typename O::RealT>& A, lbm_ctx* const* mem, int nm, const TileChoice& tile, int ns) {
  A.n = nm;
  int total = 0;
  if (ns == 1) {
    A.kw = batch_block_waves(mem, nm);
    A.rpb = batch_rows_per_block(mem, nm, A.kw);
    A.lx = batch_lx(mem, nm, A.kw);
  }
  for (int k = 0; k < nm; ++k) {
    A.start[k] = total;
    if (ns > 1) A.row[k] = O::tile_row(mem[k], tile);
    total += ns > 1 ? O::tiles(mem[k], tile) : O::batch_blocks(mem[k], A.kw, A.rpb);
  }
  A.start[nm] = total;
  return total;
}

// The tile of the batched steps to come: chosen for the members together, whose tiles
// share the CUs (a batch of 8 fills them with larger tiles and fewer steps than one
// lattice).  Fewer steps than a launch of several needs (see Split and
// steps_there_and_back) are not worth the choice: two steps of 32 lattices of 64x32
// take 13.0 us, 13.6 with it.
template <class O>
TileChoice batch_tile_choice(lbm_ctx* const* cs, int n, int64_t nsteps, LaunchKind kind) {
  if constexpr (O::kTiled)
    if (nsteps >= (cs[0]->plan.inplace ? 4 : 3)) return O::choose_tile(cs, n, kind);
  return TileChoice();
}

// Batched primal steps: one launch per step, or per several steps of a 2D
// lattice, covers every context.
// In place: per step, the checkpoint copies of members at t = sC (checkpointed
// plans), then one launch per phase among the members (two when their
// parities differ), each member's buffer read and rewritten in place; several
// steps per launch when every member is at an even time.
template <class O>
lbm_status primal_batch_inplace(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps, int record) {
  using Real = typename O::RealT;
  BatchArgs<Real> A;
  std::memset(&A, 0, sizeof A);
  TileChoice tile = batch_tile_choice<O>(cs, n, nsteps, record ? RECORDED : STEPS);
  tile.ns = most_in_place(c0, tile.ns);
  for (int64_t i = 0; i < nsteps;) {
    int e = tile.ns;
    for (int k = 0; k < n; ++k) {
      lbm_ctx* c = cs[k];
      const bool ckpts = record && checkpointed(c);
      if (ckpts && c->t % c->plan.C == 0)
        O::copy(c, c->work, ckpt_slot(c, c->t / c->plan.C), (size_t)c->plan.QT * c->plan.Np);
      const int64_t room = steps_together(c, c->t, nsteps - i, record != 0);
      e = std::min(e, c->os_active ? 0 : steps_there_and_back(c->t, room, tile.ns));
    }
    if (e > 1) {  // through the adjoint buffers and back
      batch_geometry<O>(A, cs, n, tile, e);
      for (int back = 0; back < 2; ++back) {
        for (int k = 0; k < n; ++k) {
          lbm_ctx* c = cs[k];
          batch_member<O>(A, k, c, back ? c->lam[0] : c->work, nullptr, back ? c->work : c->lam[0],
                          record ? mom_slot(c, c->t) : nullptr);
          c->t += e;
        }
        O::primal_many_batch(c0->stream, A, tile, e, true);
      }
      i += 2 * e;
      continue;
    }
    for (int phase = 0; phase < 2; ++phase) {
      lbm_ctx* mem[kBatchMax];
      int nm = 0;
      for (int k = 0; k < n; ++k)
        if (cs[k]->t % 2 == phase) mem[nm++] = cs[k];
      if (nm == 0) continue;
      const int total = batch_geometry<O>(A, mem, nm, tile, 1);
      batch_nt_inplace(mem, nm, !record, phase == 1, &A.nt, &A.nte);
      for (int k = 0; k < nm; ++k)
        batch_member<O>(A, k, mem[k], mem[k]->work, nullptr, mem[k]->work, record ? mom_slot(mem[k], mem[k]->t) : nullptr);
      O::primal_batch(c0->stream, A, total, phase == 0 ? ACC_EVEN : ACC_ODD);
    }
    for (int k = 0; k < n; ++k) ++cs[k]->t;
    ++i;
  }
  return launch_check(c0, "batched in-place primal step");
}

template <class O>
lbm_status RunPrimalBatch<O>::run(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps, int record) {
  using Real = typename O::RealT;
  if (c0->plan.inplace) return primal_batch_inplace<O>(c0, cs, n, nsteps, record);
  BatchArgs<Real> A;
  std::memset(&A, 0, sizeof A);
  const TileChoice tile = batch_tile_choice<O>(cs, n, nsteps, record ? RECORDED : STEPS);
  A.nt = batch_nt(cs, n);
  int geometry = 0, total = 0;  // steps per launch that A's geometry is for
  for (int64_t i = 0; i < nsteps;) {
    int64_t room = nsteps - i;
    for (int k = 0; k < n; ++k) room = std::min(room, steps_together(cs[k], cs[k]->t, room, record != 0));
    for (Split sp(room, tile.ns); sp.next();) {
      if (sp.ns != geometry) total = batch_geometry<O>(A, cs, n, tile, geometry = sp.ns);
      for (int k = 0; k < n; ++k) {
        lbm_ctx* c = cs[k];
        void* dst = record ? rec_dst(c, c->t + sp.ns - 1) : other_pp(c, c->cur);
        batch_member<O>(A, k, c, c->cur, nullptr, dst, record ? mom_slot(c, c->t) : nullptr);
        c->cur = dst;
        c->t += sp.ns;
      }
      if (sp.ns > 1) O::primal_many_batch(c0->stream, A, tile, sp.ns, false);
      else O::primal_batch(c0->stream, A, total);
      i += sp.ns;
    }
  }
  return launch_check(c0, "batched primal step");
}

// Batched adjoint steps.  Contexts that still have to be seeded are seeded
// first; before each reverse step, the contexts whose next step lies in a
// segment whose moments are not held recompute it, batched together.
// In place: members whose next step lies in a segment whose moments are not
// held recompute it inside its checkpoint (single-context launches); then one
// launch per cotangent pattern among the members, or several steps per launch
// when every member is in the seed's layout.
template <class O>
lbm_status adjoint_batch_inplace(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps) {
  using Real = typename O::RealT;
  BatchArgs<Real> A;
  std::memset(&A, 0, sizeof A);
  TileChoice tile = batch_tile_choice<O>(cs, n, nsteps, ADJOINT);
  tile.ns = most_in_place(c0, tile.ns);
  for (int64_t i = 0; i < nsteps;) {
    int e = tile.ns;
    for (int k = 0; k < n; ++k) {
      lbm_ctx* c = cs[k];
      const int64_t last = c->t_adj - 1, s = last / c->plan.C;
      if (s != c->mom_seg) recompute_segment_inplace<O>(c, s);
      const int64_t room = std::min<int64_t>(nsteps - i, last % c->plan.C + 1);
      e = std::min(e, steps_there_and_back(c->rec_len - c->t_adj, room, tile.ns));
    }
    if (e > 1) {  // through the working buffers and back
      batch_geometry<O>(A, cs, n, tile, e);
      for (int back = 0; back < 2; ++back) {
        for (int k = 0; k < n; ++k) {
          lbm_ctx* c = cs[k];
          batch_member<O>(A, k, c, mom_slot(c, c->t_adj - 1), back ? c->work : c->lam[0], back ? c->lam[0] : c->work,
                          nullptr);
          c->t_adj -= e;
        }
        O::adjoint_many_batch(c0->stream, A, tile, e, true);
      }
      i += 2 * e;
      continue;
    }
    for (int odd = 0; odd < 2; ++odd) {
      lbm_ctx* mem[kBatchMax];
      int nm = 0;
      for (int k = 0; k < n; ++k)  // the cotangent is in the odd-pattern layout after an even step count
        if (((cs[k]->rec_len - cs[k]->t_adj) % 2 == 0) == (odd == 1)) mem[nm++] = cs[k];
      if (nm == 0) continue;
      const int total = batch_geometry<O>(A, mem, nm, tile, 1);
      batch_nt_inplace(mem, nm, false, false, &A.nt, &A.nte);
      for (int k = 0; k < nm; ++k)
        batch_member<O>(A, k, mem[k], mom_slot(mem[k], mem[k]->t_adj - 1), mem[k]->lam[0], mem[k]->lam[0], nullptr);
      O::adjoint_batch(c0->stream, A, total, odd ? ACC_ODD : ACC_EVEN);
    }
    for (int k = 0; k < n; ++k) --cs[k]->t_adj;
    ++i;
  }
  return launch_check(c0, "batched in-place adjoint step");
}

// Ping-pong: recomputes the segments of the next reverse steps that are not held, in
// launches of its own length, however many reverse steps the call asks for.
template <class O>
void recompute_batch(lbm_ctx* c0, lbm_ctx* const* cs, int n) {
  BatchArgs<typename O::RealT> A;
  std::memset(&A, 0, sizeof A);
  lbm_ctx* need[kBatchMax];
  int64_t next[kBatchMax], end[kBatchMax];
  const void* src[kBatchMax];
  int nn = 0;
  for (int k = 0; k < n; ++k) {
    lbm_ctx* c = cs[k];
    const int64_t s = (c->t_adj - 1) / c->plan.C;
    if (s == c->mom_seg) continue;
    need[nn] = c;
    next[nn] = s * c->plan.C;
    end[nn] = std::min<int64_t>(next[nn] + c->plan.C, c->rec_len);
    src[nn++] = ckpt_slot(c, s);
    c->mom_seg = s;
  }
  for (;;) {
    lbm_ctx* mem[kBatchMax];  // the contexts with recompute steps left
    int at[kBatchMax], nm = 0;
    int64_t room = INT64_MAX;
    for (int q = 0; q < nn; ++q)
      if (next[q] < end[q]) {
        room = std::min(room, end[q] - next[q]);
        at[nm] = q;
        mem[nm++] = need[q];
      }
    if (nm == 0) return;
    const TileChoice tile = batch_tile_choice<O>(mem, nm, room, RECORDED);
    A.nt = batch_nt(mem, nm);
    int geometry = 0, total = 0;
    for (Split sp(room, tile.ns); sp.next();) {
      if (sp.ns != geometry) total = batch_geometry<O>(A, mem, nm, tile, geometry = sp.ns);
      for (int k = 0; k < nm; ++k) {
        const int q = at[k];
        void* dst = other_pp(mem[k], src[q]);
        batch_member<O>(A, k, mem[k], src[q], nullptr, dst, mom_slot(mem[k], next[q]));
        src[q] = dst;
        next[q] += sp.ns;
      }
      if (sp.ns > 1) O::primal_many_batch(c0->stream, A, tile, sp.ns, false);
      else O::primal_batch(c0->stream, A, total);
    }
  }
}

template <class O>
lbm_status RunAdjointBatch<O>::run(lbm_ctx* c0, lbm_ctx* const* cs, int n, int64_t nsteps) {
  using Real = typename O::RealT;
  for (int k = 0; k < n; ++k)
    if (!cs[k]->adj_started) start_adjoint<O>(cs[k]);
  if (c0->plan.inplace) return adjoint_batch_inplace<O>(c0, cs, n, nsteps);
  BatchArgs<Real> A;
  std::memset(&A, 0, sizeof A);
  const TileChoice tile = batch_tile_choice<O>(cs, n, nsteps, ADJOINT);
  int geometry = 0, total = 0;
  for (int64_t i = 0; i < nsteps;) {
    recompute_batch<O>(c0, cs, n);
    int64_t room = nsteps - i;
    for (int k = 0; k < n; ++k) room = std::min(room, (cs[k]->t_adj - 1) % cs[k]->plan.C + 1);
    for (Split sp(room, tile.ns); sp.next();) {
      if (sp.ns != geometry) total = batch_geometry<O>(A, cs, n, tile, geometry = sp.ns);
      for (int k = 0; k < n; ++k) {
        lbm_ctx* c = cs[k];
        batch_member<O>(A, k, c, mom_slot(c, c->t_adj - 1), c->lam[c->lam_cur], c->lam[1 - c->lam_cur], nullptr);
        c->lam_cur ^= 1;
        c->t_adj -= sp.ns;
      }
      if (sp.ns > 1) O::adjoint_many_batch(c0->stream, A, tile, sp.ns, false);
      else O::adjoint_batch(c0->stream, A, total);
      i += sp.ns;
    }
  }
  return launch_check(c0, "batched adjoint step");
}

}  // namespace lbmh
