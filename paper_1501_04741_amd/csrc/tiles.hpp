// Several time steps of a 2D lattice in one launch (D2Q9, with or without D2Q5).
//
// A 2D state of the sizes in use (up to about a million nodes) lives in the caches,
// and a one-step launch is bound by latency: the launch itself, the loads at its
// start, one wave's chain of instructions, the stores at its end.  Here a block
// loads a region of nodes once, advances it ns steps with the populations in
// registers, exchanging them through LDS between steps, and stores the tile in
// its middle: of a region of RX x RY nodes the nodes at least s away from its edge
// are valid at step s, so the tile is (RX - 2 ns + 2) x (RY - 2 ns + 2) and the rest
// is computed by the neighbouring blocks as well.  Source and destination are
// different buffers, since neighbours read the nodes around their tiles.
//
// One thread per region node (blockDim = (RX, RY)).  LDS holds the post-collision
// populations but the rest ones (which do not move) twice, alternating, so that one
// barrier per step suffices.  Each node update is the same device code as in the
// one-step kernels: results are bitwise theirs.
#pragma once

#include "kernels.hpp"

namespace lbmk {

// Populations of a node that move, i.e. LDS values per node and buffer.
template <int Q, int QS>
constexpr int tile_values() {
  return Q - 1 + (QS > 0 ? QS - 1 : 0);
}

// Widest block: FP64 nodes hold twice the registers.
template <typename Real>
constexpr int tile_threads_max() {
  return sizeof(Real) == 8 ? 512 : 1024;
}

// v into [0, n): one turn of a loop unless the lattice is smaller than a region, and
// cheaper than a remainder.
__device__ __forceinline__ int wrap(int v, int n) {
  while (v < 0) v += n;
  while (v >= n) v -= n;
  return v;
}

// The calling thread's place in its tile.
struct TilePos {
  int x, y;     // node (wrapped into the lattice)
  int tid, rx;  // position in the region's LDS runs, row length
  int edge;     // distance to the region's edge
  bool mine;    // the node belongs to this block's tile
};

template <typename P>
__device__ __forceinline__ TilePos tile_pos(const P& p, int ns, int bx, int by) {
  const int RX = blockDim.x, RY = blockDim.y, h = ns - 1;  // blockDim = tile + 2 h
  const int i = threadIdx.x, j = threadIdx.y;
  const int gx = bx * (RX - 2 * h) - h + i, gy = by * (RY - 2 * h) - h + j;
  TilePos t;
  t.x = wrap(gx, p.nx);
  t.y = wrap(gy, p.ny);
  t.tid = j * RX + i;
  t.rx = RX;
  t.edge = min(min(i, RX - 1 - i), min(j, RY - 1 - j));
  t.mine = t.edge >= h && gx < p.nx && gy < p.ny;
  return t;
}

// ns primal steps.  ACC_PP: pull from src, store as ping-pong.  ACC_EVEN: src in
// the in-place layout of an even time, ns even, dst in the same layout (the last
// step stores in the odd pattern).  mom: the moment set of the first step; the
// next steps' follow at mom_stride values (MOM).
template <int Q, int QS, typename Real, bool MOM, int V, int ACC>
__device__ __forceinline__ void tile_primal(const Params<Real>& p, const Real* __restrict__ src,
                                            Real* __restrict__ dst, const Real* __restrict__ w,
                                            Real* __restrict__ mom, size_t mom_stride, int ns, int bx, int by,
                                            Real* lds) {
  using L = Lat<Q>;
  using S = SLat<QS>;
  constexpr int QT = Q + QS, NV = tile_values<Q, QS>();
  static_assert(Q == 9 && ACC != ACC_ODD, "2D tiles start at an even phase");
  const TilePos t = tile_pos(p, ns, bx, by);
  const int T = blockDim.x * blockDim.y;
  const Nbr b = make_nbr(p, t.x, t.y, 0);
  const int n = own_inode(b);
  const int cls = node_class(p, t.x, t.y, 0, false);
  const Real wn = w[n];
  const SwitchValues<Real> sw = switch_values(p, wn);
  Real f[Q], g[QS > 0 ? QS : 1];
#pragma unroll
  for (int j = 0; j < Q; ++j)
    f[j] = src[ACC == ACC_EVEN ? own_addr<QT>(b, j) : pull_addr<QT>(b, j, L::ex(j), L::ey(j), 0)];
#pragma unroll
  for (int i = 0; i < QS; ++i)
    g[i] = src[ACC == ACC_EVEN ? own_addr<QT>(b, Q + i) : pull_addr<QT>(b, Q + i, S::ex(i), S::ey(i), 0)];
  for (int s = 0;; ++s) {
    if (t.edge >= s) {
      if (cls == WALL) {
        collide_wall<Q, QS, Real>(p, t.x, t.y, f, g);
      } else {
        Real m[Mom<Q, QS, V>::N];
        primal_open<Q, QS, Real, MOM, V>(p, cls, wn, sw, t.y, 0, f, g, m);
        if constexpr (MOM) {
          if (t.mine && has_moments(p, cls)) {
#pragma unroll
            for (int k = 0; k < Mom<Q, QS, V>::N; ++k)
              __builtin_nontemporal_store(m[k], mom + s * mom_stride + (size_t)k * p.Np + n);
          }
        }
      }
    }
    if (s + 1 == ns) break;
    Real* buf = lds + (s & 1) * NV * T + t.tid;
#pragma unroll
    for (int j = 1; j < Q; ++j) buf[(j - 1) * T] = f[j];
#pragma unroll
    for (int i = 1; i < QS; ++i) buf[(Q + i - 2) * T] = g[i];
    __syncthreads();
    if (t.edge >= s + 1) {
#pragma unroll
      for (int j = 1; j < Q; ++j) f[j] = buf[(j - 1) * T - L::ex(j) - L::ey(j) * t.rx];
#pragma unroll
      for (int i = 1; i < QS; ++i) g[i] = buf[(Q + i - 2) * T - S::ex(i) - S::ey(i) * t.rx];
    }
  }
  if (!t.mine) return;
#pragma unroll
  for (int j = 0; j < Q; ++j)
    dst[ACC == ACC_EVEN ? push_addr<QT>(b, j, L::ex(j), L::ey(j), 0) : own_addr<QT>(b, j)] = f[j];
#pragma unroll
  for (int i = 0; i < QS; ++i)
    dst[ACC == ACC_EVEN ? push_addr<QT>(b, Q + i, S::ex(i), S::ey(i), 0) : own_addr<QT>(b, Q + i)] = g[i];
}

// ns adjoint steps n, n - 1, ...  ACC_PP: ping-pong.  ACC_ODD: lin in the layout
// the seed writes (an even number of steps done), ns even, lout in the same layout
// (the last step stores in the even pattern).  mom: the moment set of step n; step
// n - s reads the set s * mom_stride values before it (loaded one step ahead).
template <int Q, int QS, typename Real, int V, int ACC>
__device__ __forceinline__ void tile_adjoint(const Params<Real>& p, const Real* __restrict__ mom,
                                             const Real* __restrict__ lin, Real* __restrict__ lout,
                                             const Real* __restrict__ w, Real* __restrict__ grad, size_t mom_stride,
                                             int ns, int bx, int by, Real* lds) {
  using L = Lat<Q>;
  using S = SLat<QS>;
  using M = Mom<Q, QS, V>;
  constexpr int QT = Q + QS, NV = tile_values<Q, QS>(), QSA = QS > 0 ? QS : 1;
  static_assert(Q == 9 && ACC != ACC_EVEN, "2D tiles start in the seed's layout");
  const TilePos t = tile_pos(p, ns, bx, by);
  const int T = blockDim.x * blockDim.y;
  const Nbr b = make_nbr(p, t.x, t.y, 0);
  const int n = own_inode(b);
  const int cls = node_class(p, t.x, t.y, 0, false);
  const Real wn = w[n];
  Real m[M::N], mu[Q], nu[QSA];
#pragma unroll
  for (int k = 0; k < M::N; ++k) m[k] = mom[(size_t)k * p.Np + n];
#pragma unroll
  for (int j = 0; j < Q; ++j) mu[j] = lin[push_addr<QT>(b, ACC == ACC_ODD ? L::opp(j) : j, L::ex(j), L::ey(j), 0)];
#pragma unroll
  for (int i = 0; i < QS; ++i)
    nu[i] = lin[push_addr<QT>(b, Q + (ACC == ACC_ODD ? S::opp(i) : i), S::ex(i), S::ey(i), 0)];
  const SwitchValues<Real> sw = switch_values(p, wn);
  Real gsum = t.mine && cls == INTERIOR ? grad[n] : Real(0);
  for (int s = 0;; ++s) {
    Real next[M::N];
#pragma unroll
    for (int k = 0; k < M::N; ++k) next[k] = Real(0);
    if (s + 1 < ns && t.edge >= s + 1) {
#pragma unroll
      for (int k = 0; k < M::N; ++k) next[k] = (mom - (s + 1) * mom_stride)[(size_t)k * p.Np + n];
    }
    if (t.edge >= s) {
      if (cls == WALL) {
        Real lf[Q], lg[QSA];
        adjoint_wall<Q, QS, Real>(p, t.x, t.y, mu, nu, lf, lg);
#pragma unroll
        for (int j = 0; j < Q; ++j) mu[j] = lf[j];
#pragma unroll
        for (int i = 0; i < QS; ++i) nu[i] = lg[i];
      } else {
        Real gw;
        // branches held apart: 87 VGPRs with D2Q5 blended (91 without), in FP64 126 (138)
        adjoint_open<Q, QS, Real, V, true>(p, cls, wn, sw, m, mu, nu, gw);
        gsum += gw;
      }
    }
    if (s + 1 == ns) break;
    Real* buf = lds + (s & 1) * NV * T + t.tid;
#pragma unroll
    for (int j = 1; j < Q; ++j) buf[(j - 1) * T] = mu[j];
#pragma unroll
    for (int i = 1; i < QS; ++i) buf[(Q + i - 2) * T] = nu[i];
    __syncthreads();
    if (t.edge >= s + 1) {
#pragma unroll
      for (int j = 1; j < Q; ++j) mu[j] = buf[(j - 1) * T + L::ex(j) + L::ey(j) * t.rx];
#pragma unroll
      for (int i = 1; i < QS; ++i) nu[i] = buf[(Q + i - 2) * T + S::ex(i) + S::ey(i) * t.rx];
    }
#pragma unroll
    for (int k = 0; k < M::N; ++k) m[k] = next[k];
  }
  if (!t.mine) return;
  if (cls == INTERIOR) grad[n] = gsum;
#pragma unroll
  for (int j = 0; j < Q; ++j) lout[own_addr<QT>(b, ACC == ACC_ODD ? L::opp(j) : j)] = mu[j];
#pragma unroll
  for (int i = 0; i < QS; ++i) lout[own_addr<QT>(b, Q + (ACC == ACC_ODD ? S::opp(i) : i))] = nu[i];
}

// LDS of a tile launch, in dynamic shared memory.
template <typename Real>
__device__ __forceinline__ Real* tile_lds() {
  return lx_lds<Real>();
}

// Tile of a block.  Consecutive blocks go to the 8 XCDs in turn; here each XCD gets a
// run of consecutive tiles instead, so that neighbouring tiles, which read each
// other's nodes and share the cache lines at their edges, meet in one L2.  Measured,
// per step of an evaluation: 1024x512 in FP32 7.2 -> 6.9 us, 512x256 with D2Q5 4.4 ->
// 4.0, 2048x1024 23.6 -> 19.7, 4096x2048 98.8 -> 84.7 (in place, 4 steps per launch,
// 130 -> 102).
__host__ __device__ inline int tile_index(int block, int blocks) {
  constexpr int kXcds = 8;
  const int xcd = block % kXcds, left = blocks % kXcds;
  return xcd * (blocks / kXcds) + (xcd < left ? xcd : left) + block / kXcds;
}

struct Tile {
  int k, bx, by;  // member of a batch, tile within its lattice
};

template <int Q, int QS, typename Real, bool MOM, int V, int ACC>
__global__ __launch_bounds__(tile_threads_max<Real>()) void k_primal_tile(Params<Real> p, const Real* __restrict__ src,
                                                      Real* __restrict__ dst, const Real* __restrict__ w,
                                                      Real* __restrict__ mom, size_t mom_stride, int ns, TileRow row) {
  const int i = tile_index(blockIdx.x, gridDim.x), by = row.divide(i), bx = i - by * row.n;
  tile_primal<Q, QS, Real, MOM, V, ACC>(p, src, dst, w, mom, mom_stride, ns, bx, by, tile_lds<Real>());
}

template <int Q, int QS, typename Real, int V, int ACC>
__global__ __launch_bounds__(tile_threads_max<Real>()) void k_adjoint_tile(Params<Real> p, const Real* __restrict__ mom,
                                                       const Real* __restrict__ lin, Real* __restrict__ lout,
                                                       const Real* __restrict__ w, Real* __restrict__ grad,
                                                       size_t mom_stride, int ns, TileRow row) {
  const int i = tile_index(blockIdx.x, gridDim.x), by = row.divide(i), bx = i - by * row.n;
  tile_adjoint<Q, QS, Real, V, ACC>(p, mom, lin, lout, w, grad, mom_stride, ns, bx, by, tile_lds<Real>());
}

// The batched form: members' tiles in turn (A.start), A.row[k] tiles in a row of member k.
template <typename Real>
__device__ __forceinline__ Tile batch_tile(const BatchArgs<Real>& A) {
  const int i = tile_index(blockIdx.x, gridDim.x), k = batch_find(A, i), by = A.row[k].divide(i - A.start[k]);
  return {k, i - A.start[k] - by * A.row[k].n, by};
}

template <int Q, int QS, typename Real, bool MOM, int V, int ACC>
__global__ __launch_bounds__(tile_threads_max<Real>()) void k_primal_tile_batch(BatchArgs<Real> A, int ns) {
  const Tile t = batch_tile(A);
  const Params<Real> p = A.st[t.k]->p;
  tile_primal<Q, QS, Real, MOM, V, ACC>(p, A.a[t.k], A.c[t.k], A.w[t.k], MOM ? A.m[t.k] : nullptr,
                                        A.st[t.k]->mom_stride, ns, t.bx, t.by, tile_lds<Real>());
}

template <int Q, int QS, typename Real, int V, int ACC>
__global__ __launch_bounds__(tile_threads_max<Real>()) void k_adjoint_tile_batch(BatchArgs<Real> A, int ns) {
  const Tile t = batch_tile(A);
  const Params<Real> p = A.st[t.k]->p;
  tile_adjoint<Q, QS, Real, V, ACC>(p, A.a[t.k], A.b[t.k], A.c[t.k], A.w[t.k], A.g[t.k], A.st[t.k]->mom_stride, ns,
                                    t.bx, t.by, tile_lds<Real>());
}

}  // namespace lbmk
