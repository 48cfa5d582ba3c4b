// Definitions of Engine<S> (see lbm_engine.h). Included once per storage type.
#pragma once

#include <algorithm>

#include "lbm_engine.h"
#include "lbm_march.h"
#include "lbm_pair.h"
#include "lbm_step.h"
#include "lbm_tile.h"

namespace lbm {

// --- geometry -----------------------------------------------------------------------------

__host__ __device__ __forceinline__ int row_pos(int x, int S) { return (x % S) * kLanes + x / S; }

inline Geo make_geo(const RunDesc& d, int npt, int block_threads = kBlock) {
  Geo g;
  g.nx = d.nx;
  g.ny = d.ny;
  g.S = d.pitch / kLanes;
  g.ps = d.pitch;
  g.rs = d.rs;
  const int groups_per_block = (block_threads / kLanes) * npt;
  g.nseg = (g.S + groups_per_block - 1) / groups_per_block;
  g.plast = row_pos(d.nx - 1, g.S);
  g.xcd = d.xcd;
  return g;
}

inline dim3 step_grid(const Geo& g) {
  return dim3(unsigned(g.nseg), unsigned(std::min(g.ny, kRowsY)), unsigned((g.ny + kRowsY - 1) / kRowsY));
}

// The auxiliary kernels run one thread per storage position (pitch * ny of them), so their
// nine population accesses are coalesced; the dense [ny][nx] fields are indexed by node.
inline int node_blocks(const RunDesc& d) { return int((int64_t(d.pitch) * d.ny + kBlock - 1) / kBlock); }

// Storage position t (row y, in-row position q) -> node x; false for padding and past the end.
__device__ __forceinline__ bool storage_node(int64_t t, const RunDesc& d, int& y, int& q, int& x) {
  if (t >= int64_t(d.pitch) * d.ny) return false;
  y = int(t / d.pitch);
  q = int(t - int64_t(y) * d.pitch);
  x = d.contig ? q : (q % kLanes) * (d.pitch / kLanes) + q / kLanes;
  return x < d.nx;
}

// Buffer index of population i of node (x, y) under a stored-state convention L (with contiguous
// rows, C, always A-B's).
template <bool C>
__device__ __forceinline__ int64_t layout_index(int i, int x, int y, const RunDesc& d, LayoutSel L) {
  const int slot = !C && L.swap ? opp(i) : i, shift = C ? 1 : L.shift;
  int xs = x - shift * cx(i);
  xs = xs < 0 ? xs + d.nx : (xs >= d.nx ? xs - d.nx : xs);
  int ys = y - shift * cy(i);
  ys = ys < 0 ? ys + d.ny : (ys >= d.ny ? ys - d.ny : ys);
  return int64_t(ys) * d.rs + slot * d.pitch + (C ? xs : row_pos(xs, d.pitch / kLanes));
}

// Buffer index of entry i of node (x, y) stored at in-row position q (no shift).
__device__ __forceinline__ int64_t local_index(int i, int q, int y, const RunDesc& d) {
  return int64_t(y) * d.rs + i * d.pitch + q;
}

// --- per-node auxiliary kernels --------------------------------------------------------------

// The per-node auxiliary kernels exchange the dense [ny][nx] fields with lane-strided rows
// through LDS: a block takes kTileGroups groups of one row (one wavefront per group, lane l
// holding node x = l S + s as in the storage layout), and the dense entries of those nodes --
// kTileGroups consecutive x per lane -- are read or written by consecutive threads. (Indexing
// the dense fields by each thread's own node strides a wavefront's accesses by S elements.) With
// contiguous rows a thread's storage node and its dense entry are the same node.
constexpr int kTileGroups = kBlock / kLanes;
inline dim3 tile_grid(const RunDesc& d) {
  const int S = d.pitch / kLanes;
  return dim3(unsigned((S + kTileGroups - 1) / kTileGroups), unsigned(std::min(d.ny, kRowsY)),
              unsigned((d.ny + kRowsY - 1) / kRowsY));
}
// A block's row y; the thread's wavefront w, lane, storage node x at in-row position q (-1
// outside the row or in the padding); its dense entry, node xt (-1: none), held by lane lt of
// wavefront jt.
struct Tile {
  int y, w, lane, x, q, lt, jt, xt;
};
template <bool C>
__device__ __forceinline__ Tile tile_of(const RunDesc& d) {
  Tile t;
  t.y = int(blockIdx.z) * kRowsY + int(blockIdx.y);
  t.w = int(threadIdx.x) / kLanes;
  t.lane = int(threadIdx.x) % kLanes;
  const int S = d.pitch / kLanes, s0 = int(blockIdx.x) * kTileGroups;
  const int s = s0 + t.w;
  t.q = s * kLanes + t.lane;
  if constexpr (C) {
    t.x = t.q < d.nx ? t.q : -1;
    t.jt = t.w;
    t.lt = t.lane;
    t.xt = t.x;
    return t;
  }
  t.x = t.lane * S + s;
  if (s >= S || t.x >= d.nx) t.x = -1;
  t.lt = int(threadIdx.x) / kTileGroups;
  t.jt = int(threadIdx.x) % kTileGroups;
  const int x = t.lt * S + s0 + t.jt;
  t.xt = (s0 + t.jt < S && x < d.nx) ? x : -1;
  return t;
}

// Values of the block's nodes between their dense entries and their storage nodes: through LDS
// with lane-strided rows, the thread's own with contiguous ones.
template <bool C, class T, int N>
struct Exchange {
  T v[N];
  __device__ __forceinline__ void swap(const Tile& t, T (*sh)[kTileGroups][kLanes], bool to_storage) {
    if constexpr (!C) {
      const int w0 = to_storage ? t.jt : t.w, l0 = to_storage ? t.lt : t.lane;
      const int w1 = to_storage ? t.w : t.jt, l1 = to_storage ? t.lane : t.lt;
#pragma unroll
      for (int c = 0; c < N; ++c) sh[c][w0][l0] = v[c];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < N; ++c) v[c] = sh[c][w1][l1];
    }
  }
};

// f^0 = f^eq(rho, u) of the guided equilibrium (eq:guidedEq), stored shifted, computed from
// the caller's FP64 fields in FP64 as drho Phi_x Phi_y + rho0 (d_x Phi_y + r_x d_y) (no
// cancellation against w_i rho0) and rounded once to the storage type. Here and in the export
// and import the fused products are written out: left to the compiler they changed with the code
// around them, and an unstable flow amplifies the last bit of its initial state.
template <class S, bool C>
__global__ void __launch_bounds__(kBlock)
k_init(S* buf, RunDesc d, LayoutSel L, const double* rho, const double* ux, const double* uy) {
#pragma clang fp contract(off)
  using Tr = StorageTraits<S>;
  __shared__ double sh[C ? 1 : 3][kTileGroups][kLanes];
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, double, 3> e{};
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
    e.v[0] = rho ? rho[n] : d.rho0;
    e.v[1] = ux[n];
    e.v[2] = uy[n];
  }
  e.swap(tl, sh, true);
  if (tl.x < 0) return;
  const double vx = e.v[1], vy = e.v[2], drho = e.v[0] - d.rho0;
  const double rr[3] = {0.5 * d.theta, 1.0 - d.theta, 0.5 * d.theta};
  const double tx[3] = {fmad(vx, vx, -vx), -(vx * vx), fmad(vx, vx, vx)};  // 2 d_x, d_x, 2 d_x
  const double ty[3] = {fmad(vy, vy, -vy), -(vy * vy), fmad(vy, vy, vy)};
  const double dx[3] = {0.5 * tx[0], tx[1], 0.5 * tx[2]}, dy[3] = {0.5 * ty[0], ty[1], 0.5 * ty[2]};
  const double hx[3] = {fmad(0.5, tx[0], rr[0]), fmad(-vx, vx, rr[1]), fmad(0.5, tx[2], rr[2])};
  const double hy[3] = {fmad(0.5, ty[0], rr[0]), fmad(-vy, vy, rr[1]), fmad(0.5, ty[2], rr[2])};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int a = cx(i) + 1, b = cy(i) + 1;
    const double t = cx(i) == 0 ? fmad(rr[a], dy[b], dx[a] * hy[b]) : fmad(dx[a], hy[b], rr[a] * dy[b]);
    buf[layout_index<C>(i, tl.x, tl.y, d, L)] = Tr::from_f64(fmad(drho * hx[a], hy[b], d.rho0 * t));
  }
}

// The rest weight w_i.
__device__ __forceinline__ double rest_weight(int i, double th) {
  return (cx(i) == 0 ? 1.0 - th : 0.5 * th) * (cy(i) == 0 ? 1.0 - th : 0.5 * th);
}

// Export to FP64 or FP32: f = g + w rho0 in FP64 (exact for every storage type's g before the
// addition), rounded once to the output type.
template <class S, class O, bool C>
__global__ void __launch_bounds__(kBlock)
k_get(const S* buf, RunDesc d, LayoutSel L, O* out) {
#pragma clang fp contract(off)
  using Tr = StorageTraits<S>;
  __shared__ O sh[C ? 1 : Q][kTileGroups][kLanes];
  const int64_t N = int64_t(d.nx) * d.ny;
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, O, Q> e{};
  if (tl.x >= 0) {
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const double g = double(Tr::load(buf[layout_index<C>(i, tl.x, tl.y, d, L)]));
      e.v[i] = O(fmad(rest_weight(i, d.theta), d.rho0, g));
    }
  }
  e.swap(tl, sh, false);
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
#pragma unroll
    for (int i = 0; i < Q; ++i) out[i * N + n] = e.v[i];
  }
}

// Import of the caller's FP64 populations: g = f - w rho0 in FP64, rounded once to the
// storage type.
template <class S, bool C>
__global__ void __launch_bounds__(kBlock)
k_set(S* buf, RunDesc d, LayoutSel L, const double* in) {
#pragma clang fp contract(off)
  using Tr = StorageTraits<S>;
  __shared__ double sh[C ? 1 : Q][kTileGroups][kLanes];
  const int64_t N = int64_t(d.nx) * d.ny;
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, double, Q> e{};
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
#pragma unroll
    for (int i = 0; i < Q; ++i) e.v[i] = in[i * N + n];
  }
  e.swap(tl, sh, true);
  if (tl.x < 0) return;
#pragma unroll
  for (int i = 0; i < Q; ++i)
    buf[layout_index<C>(i, tl.x, tl.y, d, L)] = Tr::from_f64(fmad(-d.rho0, rest_weight(i, d.theta), e.v[i]));
}

// rho - rho0 and j of one node from the stored state, accumulated in A: FP64 for the global
// totals, the compute type for everything else.
template <class A, bool C, class S>
__device__ __forceinline__ void node_moments(const S* buf, const RunDesc& d, LayoutSel L, int x, int y,
                                             A& drho, A& jx, A& jy, bool* bad = nullptr) {
  using Tr = StorageTraits<S>;
  drho = jx = jy = A(0);
  bool nf = false;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const A g = A(Tr::load(buf[layout_index<C>(i, x, y, d, L)]));
    nf |= !isfinite(g);
    drho += g;
    jx += A(cx(i)) * g;
    jy += A(cy(i)) * g;
  }
  if (bad) *bad = nf;
}

// rho and u = j / rho of every node, in the compute type, written as O.
template <class S, class O, bool C>
__global__ void __launch_bounds__(kBlock)
k_moments(const S* buf, RunDesc d, LayoutSel L, O* rho, O* ux, O* uy) {
  using T = typename StorageTraits<S>::T;
  __shared__ O sh[C ? 1 : 3][kTileGroups][kLanes];
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, O, 3> e{};
  if (tl.x >= 0) {
    T drho, jx, jy;
    node_moments<T, C>(buf, d, L, tl.x, tl.y, drho, jx, jy);
    const T r = T(d.rho0) + drho;
    e.v[0] = O(r);
    e.v[1] = O(jx / r);
    e.v[2] = O(jy / r);
  }
  e.swap(tl, sh, false);
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
    if (rho) rho[n] = e.v[0];
    if (ux) ux[n] = e.v[1];
    if (uy) uy[n] = e.v[2];
  }
}

// FP64 totals, first stage: fixed grid of kReduceBlocks blocks, deterministic order.
template <class S, bool C>
__global__ void __launch_bounds__(kBlock)
k_reduce_partial(const S* buf, RunDesc d, LayoutSel L, double* partial) {
  __shared__ double sh[4][kBlock];
  const int64_t T = int64_t(d.pitch) * d.ny;
  double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
  for (int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x; t < T; t += int64_t(gridDim.x) * kBlock) {
    int y, q, x;
    if (!storage_node(t, d, y, q, x)) continue;
    double drho, jx, jy;
    bool bad;
    node_moments<double, C>(buf, d, L, x, y, drho, jx, jy, &bad);
    s0 += drho;
    s1 += jx;
    s2 += jy;
    s3 += bad ? 1.0 : 0.0;
  }
  sh[0][threadIdx.x] = s0;
  sh[1][threadIdx.x] = s1;
  sh[2][threadIdx.x] = s2;
  sh[3][threadIdx.x] = s3;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w)
      for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) partial[blockIdx.x * 4 + threadIdx.x] = sh[threadIdx.x][0];
}

// Second stage: one block sums the partials; result = {sum rho, sum jx, sum jy, #non-finite}.
template <class S>
__global__ void __launch_bounds__(kBlock)
k_reduce_final(const double* partial, int nparts, double mass_offset, double* result) {
  __shared__ double sh[4][kBlock];
  double s[4] = {0, 0, 0, 0};
  for (int b = threadIdx.x; b < nparts; b += kBlock)
    for (int c = 0; c < 4; ++c) s[c] += partial[b * 4 + c];
  for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] = s[c];
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w)
      for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    result[0] = mass_offset + sh[0][0];
    result[1] = sh[1][0];
    result[2] = sh[2][0];
    result[3] = sh[3][0];
  }
}

// Seed of the reverse sweep: fbar^N_i = rho_bar + (u_bar . (c_i - u)) / rho, the adjoint of
// the moments (rho, u) at t = N with respect to the populations (derivative of rho and
// u = sum c f / rho with respect to f_i), written to fbar (population layout, compute type).
template <class S, class T, bool C>
__global__ void __launch_bounds__(kBlock)
k_seed(const S* buf, RunDesc d, LayoutSel L, const T* rhob, const T* uxb, const T* uyb, T* fbar) {
  __shared__ T sh[C ? 1 : 3][kTileGroups][kLanes];
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, T, 3> e{};
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
    e.v[0] = rhob ? rhob[n] : T(0);
    e.v[1] = uxb[n];
    e.v[2] = uyb[n];
  }
  e.swap(tl, sh, true);
  if (tl.x < 0) return;
  T drho, jx, jy;
  node_moments<T, C>(buf, d, L, tl.x, tl.y, drho, jx, jy);
  const T r = T(d.rho0) + drho;
  const T vx = jx / r, vy = jy / r;
  const T ax = e.v[1] / r, ay = e.v[2] / r;
#pragma unroll
  for (int i = 0; i < Q; ++i)
    fbar[local_index(i, tl.q, tl.y, d)] = e.v[0] + ax * (T(cx(i)) - vx) + ay * (T(cy(i)) - vy);
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_fbar_import(RunDesc d, const T* dense, T* fbar) {
  const int64_t N = int64_t(d.nx) * d.ny;
  int y, q, x;
  if (!storage_node(int64_t(blockIdx.x) * kBlock + threadIdx.x, d, y, q, x)) return;
  const int64_t n = int64_t(y) * d.nx + x;
#pragma unroll
  for (int i = 0; i < Q; ++i) fbar[local_index(i, q, y, d)] = dense[i * N + n];
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_fbar_export(RunDesc d, const T* fbar, T* dense) {
  const int64_t N = int64_t(d.nx) * d.ny;
  int y, q, x;
  if (!storage_node(int64_t(blockIdx.x) * kBlock + threadIdx.x, d, y, q, x)) return;
  const int64_t n = int64_t(y) * d.nx + x;
#pragma unroll
  for (int i = 0; i < Q; ++i) dense[i * N + n] = fbar[local_index(i, q, y, d)];
}

// Initial-condition adjoint: f^0 = f^eq(rho0_field, u0) with rho held fixed, so
// u0bar_a = sum_i fbar^0_i d f_i^eq / d u_a, with dPhi(0,u)/du = -2u, dPhi(+-1,u)/du = u +- 1/2.
// rho and u are the moments of the recorded state at t = 0.
template <class S, class T, bool C>
__global__ void __launch_bounds__(kBlock)
k_ic_adjoint(const S* buf0, RunDesc d, LayoutSel L, const T* fbar, T* uxb, T* uyb) {
  __shared__ T sh[C ? 1 : 2][kTileGroups][kLanes];
  const Tile tl = tile_of<C>(d);
  if (tl.y >= d.ny) return;  // whole block
  Exchange<C, T, 2> e{};
  if (tl.x >= 0) {
    T drho, jx, jy;
    node_moments<T, C>(buf0, d, L, tl.x, tl.y, drho, jx, jy);
    const T r = T(d.rho0) + drho;
    const T vx = jx / r, vy = jy / r;
    const T th = T(d.theta);
    const T hx[3] = {T(0.5) * (th + vx * vx - vx), T(1) - th - vx * vx, T(0.5) * (th + vx * vx + vx)};
    const T hy[3] = {T(0.5) * (th + vy * vy - vy), T(1) - th - vy * vy, T(0.5) * (th + vy * vy + vy)};
    const T gx[3] = {vx - T(0.5), T(-2) * vx, vx + T(0.5)};
    const T gy[3] = {vy - T(0.5), T(-2) * vy, vy + T(0.5)};
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int a = cx(i) + 1, b = cy(i) + 1;
      const T fb = fbar[local_index(i, tl.q, tl.y, d)];
      e.v[0] += fb * r * gx[a] * hy[b];
      e.v[1] += fb * r * hx[a] * gy[b];
    }
  }
  e.swap(tl, sh, false);
  if (tl.xt >= 0) {
    const int64_t n = int64_t(tl.y) * d.nx + tl.xt;
    uxb[n] = e.v[0];
    uyb[n] = e.v[1];
  }
}

// --- step dispatch ---------------------------------------------------------------------------

// Threads per block of the step kernel: of A-B, the largest block whose wavefronts idle no more
// groups at the end of a row than those of 256 threads (rows of up to four groups, 19 or 20 groups
// against 32).
template <class S>
int step_threads(const RunDesc& d, int phase, int npt) {
  const int s = d.pitch / kLanes;
  auto idle = [&](int threads) { const int g = threads / kLanes * npt; return (s + g - 1) / g * g - s; };
  int best = kBlock;
  if (phase == PH_AB)
    for (int t = 2 * kBlock; t <= kStepBlock<S>; t *= 2)
      if (idle(t) <= idle(best)) best = t;
  return best;
}

template <class S, int MODEL, int NPT, int STREAM>
hipError_t launch_step_w(const RunDesc& d, int phase, const void* src, void* dst, void* rec, hipStream_t st) {
  using T = typename StorageTraits<S>::T;
  const int threads = step_threads<S>(d, phase, NPT);
  const Geo g = make_geo(d, NPT, threads);
  const Coef<T> k = make_coef<T>(d);
  const S* s = static_cast<const S*>(src);
  S* o = static_cast<S*>(dst);
  T* r = static_cast<T*>(rec);
  const dim3 grid = step_grid(g), block{unsigned(threads)};
  if (d.walls) {
    hipLaunchKernelGGL((k_step<S, MODEL, PH_AB, false, NPT, STREAM, true>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
  } else if (rec) {
    if (phase == PH_AB) hipLaunchKernelGGL((k_step<S, MODEL, PH_AB, true, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
    else if (phase == PH_AA_EVEN) hipLaunchKernelGGL((k_step<S, MODEL, PH_AA_EVEN, true, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
    else hipLaunchKernelGGL((k_step<S, MODEL, PH_AA_ODD, true, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
  } else {
    if (phase == PH_AB) hipLaunchKernelGGL((k_step<S, MODEL, PH_AB, false, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
    else if (phase == PH_AA_EVEN) hipLaunchKernelGGL((k_step<S, MODEL, PH_AA_EVEN, false, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
    else hipLaunchKernelGGL((k_step<S, MODEL, PH_AA_ODD, false, NPT, STREAM>), grid, block, 0, st, s, o, g, k, r, d.rs_rec);
  }
  return hipGetLastError();
}

template <class S, int MODEL, int NPT>
hipError_t launch_step_n(const RunDesc& d, int phase, const void* src, void* dst, void* rec, hipStream_t st) {
  // STREAM_ALL differs for AA's 16-bit loads alone.
  if constexpr (sizeof(S) == 2)
    if (d.stream == STREAM_ALL && phase != PH_AB) return launch_step_w<S, MODEL, NPT, STREAM_ALL>(d, phase, src, dst, rec, st);
  return d.stream ? launch_step_w<S, MODEL, NPT, STREAM_ON>(d, phase, src, dst, rec, st)
                  : launch_step_w<S, MODEL, NPT, STREAM_OFF>(d, phase, src, dst, rec, st);
}

// Nodes per thread of the step kernel. Two or four nodes per thread put more loads in flight
// before the first collision, which pays where the collision is long relative to the bytes
// moved (16-bit storage); the FP32 and FP64 paths are bandwidth-bound and run fastest with one.
// Measured on MI355X, 8192^2, complete model (GLUPS, 1/2/4 nodes per thread): FP16
// 148/160/167, BF16 149/168/168, FP32 90.6/82.6/81.0; LBGK FP16 176/178/168.
template <class S> struct NodesPerThread { static constexpr int oreg = 1, bgk = 1; };
template <> struct NodesPerThread<_Float16> { static constexpr int oreg = 4, bgk = 2; };
template <> struct NodesPerThread<bf16_t> { static constexpr int oreg = 2, bgk = 2; };

template <class S, int MODEL>
hipError_t launch_step_m(const RunDesc& d, int phase, const void* src, void* dst, void* rec, hipStream_t st) {
  constexpr int npt = MODEL == M_BGK ? NodesPerThread<S>::bgk : NodesPerThread<S>::oreg;
  // A wavefront's NPT groups must all lie inside the row or all past it.
  if constexpr (npt > 1) {
    if ((d.pitch / kLanes) % (npt * kBlock / kLanes) == 0)
      return launch_step_n<S, MODEL, npt>(d, phase, src, dst, rec, st);
  }
  return launch_step_n<S, MODEL, 1>(d, phase, src, dst, rec, st);
}

// f(std::integral_constant<int, MODEL>) for the run's model.
template <class F>
hipError_t with_model(int model, F&& f) {
  switch (model) {
    case M_BGK: return f(std::integral_constant<int, M_BGK>{});
    case M_UC: return f(std::integral_constant<int, M_UC>{});
    case M_PARTIAL: return f(std::integral_constant<int, M_PARTIAL>{});
    default: return f(std::integral_constant<int, M_COMPLETE>{});
  }
}

template <class S>
hipError_t Engine<S>::step(const RunDesc& d, int phase, const void* src, void* dst, void* rec, hipStream_t st) {
  if (d.walls && (phase != PH_AB || rec)) return hipErrorInvalidValue;
  return with_model(d.model, [&](auto m) {
    constexpr int MODEL = decltype(m)::value;
    return launch_step_m<S, MODEL>(d, phase, src, dst, rec, st);
  });
}

// --- several steps per launch ------------------------------------------------------------------

inline MarchGeo march_geo(const RunDesc& d, const MarchPlan& p) {
  MarchGeo g;
  g.nx = d.nx;
  g.ny = d.ny;
  g.ps = d.pitch;
  g.rs = d.rs;
  g.rec_rs = d.rs_rec;
  g.ncol = p.ncol;
  g.w = p.w;
  g.xlast = p.xlast;
  g.halo = p.halo;
  g.nrb = p.nrb;
  return g;
}
inline dim3 march_grid(const MarchPlan& p) { return dim3(unsigned((p.ncol + p.waves - 1) / p.waves) * unsigned(p.nrb)); }

template <class S, int MODEL, bool REC>
hipError_t launch_march(const RunDesc& d, const MarchPlan& p, int ns, const S* src, S* dst,
                        const MarchRec<typename StorageTraits<S>::T>& rec, hipStream_t st) {
  using T = typename StorageTraits<S>::T;
  const MarchGeo g = march_geo(d, p);
  const Coef<T> k = make_coef<T>(d);
  const dim3 grid = march_grid(p), block(unsigned(p.waves * kLanes));
  switch (ns) {
    case 2: hipLaunchKernelGGL((k_march<S, MODEL, 2, REC>), grid, block, 0, st, src, dst, g, k, rec); break;
    case 3: hipLaunchKernelGGL((k_march<S, MODEL, 3, REC>), grid, block, 0, st, src, dst, g, k, rec); break;
    case 4: hipLaunchKernelGGL((k_march<S, MODEL, 4, REC>), grid, block, 0, st, src, dst, g, k, rec); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::adjoint_march(const RunDesc& d, int ns, const T* fbar_next, T* fbar, const T* rec,
                                    int64_t rec_slot, hipStream_t st) {
  if (!d.contig || ns > d.adj_march.steps) return hipErrorInvalidValue;
  const MarchGeo g = march_geo(d, d.adj_march);
  const Coef<T> k = make_coef<T>(d);
  const dim3 grid = march_grid(d.adj_march), block(unsigned(d.adj_march.waves * kLanes));
  MarchRec<const T> r{};
  for (int s = 0; s < ns; ++s) r.p[s] = rec - s * rec_slot;
  return with_model(d.model, [&](auto m) -> hipError_t {
    constexpr int MODEL = decltype(m)::value;
    switch (ns) {
      case 2: hipLaunchKernelGGL((k_march_adjoint<T, MODEL, 2>), grid, block, 0, st, fbar_next, fbar, g, k, r); break;
      case 3: hipLaunchKernelGGL((k_march_adjoint<T, MODEL, 3>), grid, block, 0, st, fbar_next, fbar, g, k, r); break;
      case 4: hipLaunchKernelGGL((k_march_adjoint<T, MODEL, 4>), grid, block, 0, st, fbar_next, fbar, g, k, r); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  });
}

// The tile plan's geometry for a launch of ns steps.
inline TileGeo tile_geo(const RunDesc& d, const TilePlan& p, int ns) {
  TileGeo g;
  g.nx = d.nx;
  g.ny = d.ny;
  g.ps = d.pitch;
  g.rs = int(d.rs);
  g.rec_rs = int(d.rs_rec);
  g.tw = p.tw;
  g.th = p.th;
  g.ntx = (d.nx + p.tw - 1) / p.tw;
  g.wrapx = p.wrapx;
  g.wrapy = p.wrapy;
  g.hx = p.wrapx ? 0 : ns - 1;
  g.hy = p.wrapy ? 0 : ns - 1;
  g.rw = p.tw + 2 * g.hx;
  g.rh = p.th + 2 * g.hy;
  g.ns = ns;
  return g;
}

template <class S, int MODEL, int KIND, class... Args>
hipError_t launch_tile(const RunDesc& d, const TilePlan& p, int ns, hipStream_t st, Args... args) {
  using T = typename StorageTraits<S>::T;
  const TileGeo g = tile_geo(d, p, ns);
  const TileConfig c = kTileConfigs[p.cfg];
  if (int64_t(g.rw) * g.rh > int64_t(c.threads) * c.nodes) return hipErrorInvalidValue;
  const dim3 grid(unsigned(g.ntx) * unsigned((d.ny + p.th - 1) / p.th)), block(unsigned(c.threads));
  const Coef<T> k = make_coef<T>(d);
  auto go = [&](auto kernel, const S* src, S* dst, T* rec, int64_t slot) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, src, dst, g, k, rec, slot);
  };
  switch (p.cfg) {
    case 0: go(k_tile<S, MODEL, 256, 1, KIND>, args...); break;
    case 1: go(k_tile<S, MODEL, 512, 1, KIND>, args...); break;
    case 2: go(k_tile<S, MODEL, 1024, 1, KIND>, args...); break;
    case 3:
      // Reverse FP64 tiles have no registers for two nodes per thread (CostModel::max_cells).
      if constexpr (KIND == TILE_ADJOINT && sizeof(S) == 8) return hipErrorInvalidValue;
      else go(k_tile<S, MODEL, 1024, 2, KIND>, args...);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::steps(const RunDesc& d, int ns, const void* src, void* dst, T* rec, int64_t rec_slot,
                            hipStream_t st) {
  const bool two = ns == 2 && (d.two.march.steps || d.two.tile.steps);
  const MarchPlan& mp = two ? d.two.march : d.march;
  const TilePlan& tp = two ? d.two.tile : d.tile;
  if (!d.contig || (d.walls && rec) || ns > std::max(mp.steps, tp.steps)) return hipErrorInvalidValue;
  const S* s = static_cast<const S*>(src);
  S* o = static_cast<S*>(dst);
  if constexpr (sizeof(S) >= 4) {
    if (ns == 2 && d.two_rb && !rec) {
      const Geo g = make_geo(d, 1);
      const dim3 grid(unsigned(d.nx / kPairNodes), unsigned(d.two_rb)), block(kPairNodes + kLanes);
      return with_model(d.model, [&](auto m) {
        constexpr int MODEL = decltype(m)::value;
        if (d.stream) hipLaunchKernelGGL((k_pair<S, MODEL, STREAM_ON>), grid, block, 0, st, s, o, g, make_coef<T>(d));
        else hipLaunchKernelGGL((k_pair<S, MODEL, STREAM_OFF>), grid, block, 0, st, s, o, g, make_coef<T>(d));
        return hipGetLastError();
      });
    }
  }
  return with_model(d.model, [&](auto m) {
    constexpr int MODEL = decltype(m)::value;
    if (tp.steps) {
      if (d.walls) return launch_tile<S, MODEL, TILE_WALLS>(d, tp, ns, st, s, o, rec, rec_slot);
      if (rec) return launch_tile<S, MODEL, TILE_REC>(d, tp, ns, st, s, o, rec, rec_slot);
      return launch_tile<S, MODEL, TILE_STEP>(d, tp, ns, st, s, o, rec, rec_slot);
    }
    if (d.walls) return hipErrorInvalidValue;
    MarchRec<T> r{};
    for (int k = 0; rec && k < ns; ++k) r.p[k] = rec + k * rec_slot;
    return rec ? launch_march<S, MODEL, true>(d, mp, ns, s, o, r, st) : launch_march<S, MODEL, false>(d, mp, ns, s, o, r, st);
  });
}

template <class S>
hipError_t Engine<S>::adjoint_tile(const RunDesc& d, int ns, const T* fbar_next, T* fbar, const T* rec,
                                   int64_t rec_slot, hipStream_t st) {
  if (!d.contig || ns > d.adj_tile.steps) return hipErrorInvalidValue;
  return with_model(d.model, [&](auto m) {
    constexpr int MODEL = decltype(m)::value;
    return launch_tile<T, MODEL, TILE_ADJOINT>(d, d.adj_tile, ns, st, fbar_next, fbar, const_cast<T*>(rec), rec_slot);
  });
}

// Row blocks of the two-step adjoint kernel, and the rule behind lbm_steps_per_launch. A block of
// h rows computes h + 2 rows of step 1 and h of step 2, and a compute unit works through its share
// of the blocks in turn, so a launch takes about ceil(blocks / CUs) (2 h + 2) row-steps of one
// block, h the tallest block. The planner takes the row-block count of least such cost with
// blocks of kFuseMinRows to max_rows rows (ties: the taller blocks; 0: none); for each count of
// blocks per compute unit only the largest row-block count that keeps it needs checking.
inline long plan_rows(long ny, long cols, long cus, long max_rows) {
  const long nb_lo = (ny + max_rows - 1) / max_rows;
  const long nb_hi = std::min(std::max(nb_lo, ny / kFuseMinRows), 65535L);
  if (nb_lo > nb_hi) return 0;
  long best = 0, best_cost = 0;
  const long w0 = std::max(1L, (cols * nb_lo + cus - 1) / cus);
  for (long w = w0; w < w0 + 4096; ++w) {
    const long nb = std::min(nb_hi, std::max(nb_lo, w * cus / cols));
    const long rows = (ny + nb - 1) / nb;
    const long cost = (cols * nb + cus - 1) / cus * (2 * rows + 2);
    if (best == 0 || cost < best_cost) best = nb, best_cost = cost;
    if (nb == nb_hi) break;
  }
  return best;
}

// mode 0 asks for a block on three quarters of the compute units. tall: also consider blocks of
// up to kFuseRowsTall rows, taken when the grid then gives every block a compute unit of its own
// (one round of blocks).
inline int plan_row_blocks(const RunDesc& d, int mode, bool tall, int cus) {
  if (d.nx % kLanes != 0 || (d.pitch / kLanes) % kFuseGroups != 0) return 0;
  const long cols = d.pitch / kLanes / kFuseGroups;
  long best = plan_rows(d.ny, cols, cus, kFuseRows);
  if (tall) {
    const long t = plan_rows(d.ny, cols, cus, kFuseRowsTall);
    if (t > 0 && cols * t <= cus) best = t;
  }
  if (best == 0 || (mode == 0 && 4 * cols * best < 3L * cus)) return 0;
  return int(best);
}

template <class S>
void plan_steps(RunDesc& d, int cus, bool force_march, bool no_single, int row_blocks, int64_t horizon) {
  using T = typename StorageTraits<S>::T;
  // The tile kernel addresses a whole buffer with 32-bit byte offsets.
  const bool tiles = d.rs * d.ny * int64_t(sizeof(T)) < (int64_t(1) << 31);
  auto choose = [&](MarchPlan& march, TilePlan& tile, double single) {
    const bool several = no_single && (march.steps || tile.steps);
    if (force_march && march.steps) tile.steps = 0;
    else if (march.us_per_step < tile.us_per_step) tile.steps = 0;
    else march.steps = 0;
    if (!force_march && !several && single < march.us_per_step && single < tile.us_per_step) march.steps = tile.steps = 0;
  };
  const CostModel cm = cost_model(int(sizeof(S)), d.model == M_BGK, false, std::is_same_v<S, bf16_t>);
  if (!d.walls) d.march = plan_march(d.nx, d.ny, MarchNodes<S>::value, kMarchHalo, kMarchMax, kMarchWaves, cus, horizon, cm);
  if (tiles) d.tile = plan_tile(d.nx, d.ny, cus, horizon, cm);
  choose(d.march, d.tile, single_step_us(d.nx, d.ny, cus, cm));
  // Launches of two steps: the pair kernel (see lbm_pair.h) or a plan of their own.
  const bool pair = row_blocks > 0 && d.nx % kPairNodes == 0 && (sizeof(S) == 4 || (sizeof(S) == 8 && (d.stream || d.tile.steps)));
  d.two_rb = pair ? row_blocks : 0;
  d.two = {};
  if ((d.march.steps || d.tile.steps) && !(d.tile.wrapx && d.tile.wrapy) && !force_march && !d.two_rb)
    d.two = plan_two(d.nx, d.ny, MarchNodes<S>::value, kMarchWaves, cus, !d.walls, d.tile, cm);
  if (horizon > 0) {
    const CostModel ca = cost_model(int(sizeof(T)), d.model == M_BGK, true);
    d.adj_march = plan_march(d.nx, d.ny, kMarchAdjointNodes, kMarchHalo, kMarchMax, kMarchWaves, cus, horizon, ca);
    if (tiles) d.adj_tile = plan_tile(d.nx, d.ny, cus, horizon, ca);
    choose(d.adj_march, d.adj_tile, single_step_us(d.nx, d.ny, cus, ca));
  }
}

template <class S>
void Engine<S>::plan(RunDesc& d, int mode, int64_t segment, bool captured) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return;
  const int row_blocks = mode >= 0 && !d.walls ? plan_row_blocks(d, mode, FuseTall<S>::value, cus) : 0;
  const bool pair = row_blocks > 0;
  d.pair = d.contig && pair;
  if (mode < 0) return;
  if (!d.contig) {
    if (segment > 0) d.adj_rb = plan_row_blocks(d, mode, FuseTall<T>::value, cus);
    return;
  }
  // mode 1 takes the marching kernel on every grid of whole pairs (the documented rule), mode 0
  // whatever the cost model finds fastest.
  const bool force = mode == 1 && d.nx % kLanes == 0 && (d.pitch / kLanes) % kFuseGroups == 0;
  plan_steps<S>(d, cus, force, captured && pair, row_blocks, segment);
}

// f(std::bool_constant<contiguous rows>).
template <class F>
hipError_t with_layout(const RunDesc& d, F&& f) {
  if (d.contig) f(std::true_type{});
  else f(std::false_type{});
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::init(const RunDesc& d, LayoutSel L, void* buf, const double* rho, const double* ux,
                           const double* uy, hipStream_t st) {
  return with_layout(d, [&](auto c) {
    hipLaunchKernelGGL((k_init<S, decltype(c)::value>), tile_grid(d), dim3(kBlock), 0, st, static_cast<S*>(buf), d, L,
                       rho, ux, uy);
  });
}

template <class S>
hipError_t Engine<S>::get(const RunDesc& d, LayoutSel L, const void* buf, bool out_f64, void* out, hipStream_t st) {
  return with_layout(d, [&](auto c) {
    constexpr bool C = decltype(c)::value;
    const S* b = static_cast<const S*>(buf);
    if (out_f64) hipLaunchKernelGGL((k_get<S, double, C>), tile_grid(d), dim3(kBlock), 0, st, b, d, L, static_cast<double*>(out));
    else hipLaunchKernelGGL((k_get<S, float, C>), tile_grid(d), dim3(kBlock), 0, st, b, d, L, static_cast<float*>(out));
  });
}

template <class S>
hipError_t Engine<S>::set(const RunDesc& d, LayoutSel L, void* buf, const double* in, hipStream_t st) {
  return with_layout(d, [&](auto c) {
    hipLaunchKernelGGL((k_set<S, decltype(c)::value>), tile_grid(d), dim3(kBlock), 0, st, static_cast<S*>(buf), d, L, in);
  });
}

template <class S>
hipError_t Engine<S>::moments(const RunDesc& d, LayoutSel L, const void* buf, bool out_f64, void* rho, void* ux,
                              void* uy, hipStream_t st) {
  return with_layout(d, [&](auto c) {
    constexpr bool C = decltype(c)::value;
    const S* b = static_cast<const S*>(buf);
    if (out_f64)
      hipLaunchKernelGGL((k_moments<S, double, C>), tile_grid(d), dim3(kBlock), 0, st, b, d, L, static_cast<double*>(rho),
                         static_cast<double*>(ux), static_cast<double*>(uy));
    else
      hipLaunchKernelGGL((k_moments<S, float, C>), tile_grid(d), dim3(kBlock), 0, st, b, d, L, static_cast<float*>(rho),
                         static_cast<float*>(ux), static_cast<float*>(uy));
  });
}

template <class S>
hipError_t Engine<S>::invariants(const RunDesc& d, LayoutSel L, const void* buf, double* partial, double* result,
                                 hipStream_t st) {
  const hipError_t e = with_layout(d, [&](auto c) {
    hipLaunchKernelGGL((k_reduce_partial<S, decltype(c)::value>), dim3(kReduceBlocks), dim3(kBlock), 0, st,
                       static_cast<const S*>(buf), d, L, partial);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_reduce_final<S>, dim3(1), dim3(kBlock), 0, st, partial, kReduceBlocks,
                     d.rho0 * double(d.nx) * double(d.ny), result);
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::seed(const RunDesc& d, LayoutSel L, const void* buf, const T* rhob, const T* uxb, const T* uyb,
                           T* fbar, hipStream_t st) {
  return with_layout(d, [&](auto c) {
    hipLaunchKernelGGL((k_seed<S, T, decltype(c)::value>), tile_grid(d), dim3(kBlock), 0, st,
                       static_cast<const S*>(buf), d, L, rhob, uxb, uyb, fbar);
  });
}

template <class S>
hipError_t Engine<S>::fbar_import(const RunDesc& d, const T* dense, T* fbar, hipStream_t st) {
  hipLaunchKernelGGL(k_fbar_import<T>, dim3(node_blocks(d)), dim3(kBlock), 0, st, d, dense, fbar);
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::fbar_export(const RunDesc& d, const T* fbar, T* dense, hipStream_t st) {
  hipLaunchKernelGGL(k_fbar_export<T>, dim3(node_blocks(d)), dim3(kBlock), 0, st, d, fbar, dense);
  return hipGetLastError();
}

template <class S>
hipError_t Engine<S>::adjoint_step2(const RunDesc& d, const T* fbar_next, T* fbar, const T* rec_hi, const T* rec_lo,
                                    hipStream_t st) {
  if (d.contig || d.adj_rb < 1 || d.adj_rb > d.ny) return hipErrorInvalidValue;
  const Geo g = make_geo(d, 1);
  const Coef<T> k = make_coef<T>(d);
  const dim3 grid(unsigned(g.S / kFuseGroups), unsigned(d.adj_rb)), block((kFuseGroups + 2) * kLanes);
  return with_model(d.model, [&](auto m) {
    hipLaunchKernelGGL((k_adjoint_step2<T, decltype(m)::value>), grid, block, 0, st, fbar_next, fbar, g, k, rec_hi, rec_lo, d.rs_rec);
    return hipGetLastError();
  });
}

template <class S>
hipError_t Engine<S>::adjoint_step(const RunDesc& d, const T* fbar_next, T* fbar, const T* rec, hipStream_t st) {
  const Geo g = make_geo(d, 1);
  const Coef<T> k = make_coef<T>(d);
  const dim3 grid = step_grid(g), block(kBlock);
  return with_model(d.model, [&](auto m) {
    constexpr int MODEL = decltype(m)::value;
    if (d.contig) hipLaunchKernelGGL((k_adjoint_step<T, MODEL, true>), grid, block, 0, st, fbar_next, fbar, g, k, rec, d.rs_rec);
    else hipLaunchKernelGGL((k_adjoint_step<T, MODEL, false>), grid, block, 0, st, fbar_next, fbar, g, k, rec, d.rs_rec);
    return hipGetLastError();
  });
}

template <class S>
hipError_t Engine<S>::ic_adjoint(const RunDesc& d, LayoutSel L, const void* buf0, const T* fbar, T* uxb, T* uyb,
                                 hipStream_t st) {
  return with_layout(d, [&](auto c) {
    hipLaunchKernelGGL((k_ic_adjoint<S, T, decltype(c)::value>), tile_grid(d), dim3(kBlock), 0, st,
                       static_cast<const S*>(buf0), d, L, fbar, uxb, uyb);
  });
}

}  // namespace lbm
