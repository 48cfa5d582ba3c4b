// Two A-B steps per launch, for calls of two steps and what longer ones leave over, FP32 and FP64.
//
// The marching kernel needs three or four steps per launch there: a strip's edges share cache lines
// with its neighbours, so its stores cannot bypass the caches, which costs a tenth of the memory
// rate as soon as the launch is bound by it. Here a block owns 512 adjacent nodes, whole lines, and
// the rows [y0, y1). Phase A runs step 1 of row r from global memory (eight interior wavefronts of
// 64 nodes; two lanes of a ninth take the columns at either side) into a ring of three rows in
// LDS, rounded as the buffer would hold it; phase B runs step 2 of row r - 1 from the ring and
// stores it, past the caches on streaming grids. The loads of row r + 1 are under way meanwhile. Bit-identical to two
// single steps. us per call of two, single steps / the march / this: FP32 512^2 9.2 / 9.1 / 8.4,
// 1024^2 23.8 / 18.3 / 17.2, 2048^2 93 / 65 / 60, 4096^2 366 / 239 / 197, 8192^2 1455 / 969 / 802;
// FP64 1024^2 45 / 26.6 / 27.1 (marches), 1536^2 108 / 76 / 68, 2048^2 191 / 124 / 107, 4096^2 754 /
// 466 / 405. 16-bit storage, bound by its instructions, marches (FP16 8192^2 677, BF16 694).
#pragma once

#include "lbm_step.h"

namespace lbm {

constexpr int kPairNodes = kFuseGroups * kLanes;  // of a block's row

// Block barrier and scheduling fence: without the fence the compiler moves phase A's collision,
// which reads registers only, above the barrier before it and waits for its loads there.
__device__ __forceinline__ void pair_sync() {
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
}

// Grid: (nx / kPairNodes, row blocks), nx a multiple of kPairNodes, at most ny row blocks.
template <class S, int MODEL, int STREAM>
__global__ void __launch_bounds__(kPairNodes + kLanes)
k_pair(const S* __restrict__ src, S* __restrict__ dst, Geo geo, Coef<typename StorageTraits<S>::T> k) {
  using T = typename StorageTraits<S>::T;
  using Tr = StorageTraits<S>;
  __shared__ S ring[3][Q][kPairNodes + 2];
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kLanes));
  const int lane = int(threadIdx.x % kLanes);
  int bx, by;
  xcd_tile(bx, by);
  const int y0 = int(int64_t(by) * geo.ny / gridDim.y);
  const int y1 = int(int64_t(by + 1) * geo.ny / gridDim.y);
  const bool interior = w < kFuseGroups, active = interior || lane < 2;
  // The thread's place in the ring's rows (1: the block's first node) and its node.
  const int p = interior ? int(threadIdx.x) + 1 : lane * (kPairNodes + 1);
  int x = bx * kPairNodes + p - 1;
  x = x < 0 ? geo.nx - 1 : x >= geo.nx ? x - geo.nx : x;
  RowPos ra;
  ra.p0 = x;
  ra.pm = x > 0 ? x - 1 : geo.nx - 1;
  ra.pp = x + 1 < geo.nx ? x + 1 : 0;
  const size_t rsb = size_t(geo.rs) * sizeof(S);
  const int psb = geo.ps * int(sizeof(S));

  S gs[Q];
  auto load = [&](const int r) {
    const int y = r < 0 ? r + geo.ny : (r >= geo.ny ? r - geo.ny : r);
    const int ym = (y == 0) ? geo.ny - 1 : y - 1, yp = (y == geo.ny - 1) ? 0 : y + 1;
    const RowRes sr[3] = {row_res(src, rsb, ym), row_res(src, rsb, y), row_res(src, rsb, yp)};
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      gs[i] = ldb<S, STREAM && cx(i) == 0 && sizeof(S) == 4>(sr[-cy(i) + 1], i * psb,
                                                   uint32_t(ra.template of<-cx(i)>()) * uint32_t(sizeof(S)));
    });
  };
  auto phase_a = [&](const int r) {
    const int slot = (r - y0 + 1) % 3;
    T g[Q], out[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = Tr::load(gs[i]);
    collide<T, MODEL, ConserveMode<S>::value>(g, out, k, nullptr);
#pragma unroll
    for (int i = 0; i < Q; ++i) ring[slot][i][p] = Tr::store(out[i]);
  };
  auto phase_b = [&](const int yr) {
    T g[Q], out[Q];
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      g[i] = Tr::load(ring[(yr - cy(i) - y0 + 1) % 3][i][p - cx(i)]);
    });
    collide<T, MODEL, ConserveMode<S>::value>(g, out, k, nullptr);
    const RowRes dr = row_res(dst, rsb, yr);
#pragma unroll
    for (int i = 0; i < Q; ++i)
      stb<S, kAuxStore<STREAM>>(dr, i * psb, uint32_t(x) * uint32_t(sizeof(S)), Tr::store(out[i]));
  };

  // Per row r = y0 - 1 .. y1 every wavefront runs phase A of r, issues the loads of r + 1 and passes
  // two barriers; between them the interior ones run phase B of r - 1 (from r = y0 + 1 on).
  if (!interior || sizeof(S) == 8) {
    if (active) load(y0 - 1);
    for (int r = y0 - 1; r <= y1; ++r) {
      if (active) {
        phase_a(r);
        if (r < y1) load(r + 1);
      }
      pair_sync();
      if (interior && r > y0) phase_b(r - 1);
      pair_sync();
    }
    return;
  }
  // FP32, interior: the same sequence, the loop entered right after the loads of the next row. On
  // every path into it those are the most recent memory operations, so that phase A waits for them
  // alone and not for phase B's stores.
  load(y0 - 1);
  phase_a(y0 - 1);
  load(y0);
  pair_sync();
  pair_sync();
  phase_a(y0);
  load(y0 + 1);
  pair_sync();
  pair_sync();
  phase_a(y0 + 1);
  if (y0 + 1 < y1) {
    load(y0 + 2);
    for (int r = y0 + 2; r < y1; ++r) {
      pair_sync();
      phase_b(r - 2);
      pair_sync();
      phase_a(r);
      load(r + 1);
    }
    pair_sync();
    phase_b(y1 - 2);
    pair_sync();
    phase_a(y1);
  }
  pair_sync();
  phase_b(y1 - 1);
  pair_sync();
}

}  // namespace lbm
