// Several A-B time steps (or reverse steps) per launch on grids too small to fill the chip with
// one step: a block takes a tile of the box, keeps it in LDS and runs up to 64 steps on
// it (4096 where one block holds the whole box), recomputing the tile's surroundings instead of
// exchanging them.
//
// A launch of one dependent step costs 2.5-3.5 us on MI355X however little it computes, a step of
// at most 256 nodes inside a block about 0.4 us, so the launches are what small grids pay for.
// The tile of tw x th stored nodes is computed on a region of rw x rh nodes, ns - 1 nodes larger
// on each side that is not the whole box (a side that is wraps inside the block instead); one
// node of the region per thread (M at most), in row order. Step 1 pulls from global memory; the
// steps between go through one LDS copy of the region in the AA scheme: an even step reads and
// writes a node's own nine cells (populations swapped), an odd one pulls from the neighbours'
// cells and pushes back into the same ones, so every cell has one reader and one writer per step,
// which are the same thread, and one barrier per step suffices. Step s computes the region less
// s rows at its lower and upper edges; columns past the valid ones keep being computed from
// whatever their cells hold (a row's end continues in the next row: still one reader and writer
// per cell) and reach no stored node. The last step stores to global memory. Cells hold the
// storage type, so the result is bit-identical to single steps.
//
// Measured, us per step, replayed graphs or single or paired launches before -> this: 1 x 200
// FP64 2.8 -> 0.55 (one block: the chain of one collision per step); 64^2 FP64 2.6 -> 0.92; 200^2
// FP64 4.0 -> 1.6; 512^2 FP32 3.95 -> 2.6; 1024^2 FP32 9.1 -> 8.2, where vector issue binds: the
// surroundings make it 1.8 node slots per stored node. Larger grids march.
#pragma once

#include "lbm_march.h"

namespace lbm {

enum { TILE_STEP = 0, TILE_REC = 1, TILE_WALLS = 2, TILE_ADJOINT = 3 };

struct TileGeo {
  int nx, ny, ps, rs, rec_rs;  // buffers below 2^31 bytes: 32-bit indices
  int tw, th, ntx;             // stored nodes of a tile, tiles per row of tiles
  int hx, hy;                  // region = tile + hx, hy nodes on each side; 0 where it wraps
  int rw, rh;
  int wrapx, wrapy;
  int ns;
};

// A region's cells: one population after the other, one spare cell at either end (the odd steps'
// neighbours of the first and last cell). own: see kTileWaves.
template <class S, int CELLS, bool PARK>
struct TileCells {
  S c[Q][CELLS + 2];
  int own[PARK ? CELLS + 2 : 1];
};

// Least wavefronts per SIMD that the registers have to allow. FP32 reverse tiles of one node per
// thread want 70 registers, which leaves a compute unit one block of 1024 threads; held to 64 it
// takes two: 8 reverse steps of 1024^2 in one segment 155.8 -> 140.6 us. They then keep what the
// last step alone needs (own) in LDS. Spilled to scratch memory instead, the one register costs
// each launch 0.7 us (142.6). Smaller blocks need no bound.
template <class S, int NT, int M, int KIND>
constexpr int kTileWaves = KIND == TILE_ADJOINT && sizeof(S) == 4 && M == 1 && NT == 1024 ? 8 : 1;

// KIND TILE_STEP / TILE_WALLS: ns forward steps (with the bounce-back columns of k_step);
// TILE_REC: step s also writes its moments to rec + s rec_slot; TILE_ADJOINT: ns reverse steps
// on fbar (S is the compute type), reverse step s with the moments at rec - s rec_slot.
template <class S, int MODEL, int NT, int M, int KIND>
__global__ void __launch_bounds__(NT, (kTileWaves<S, NT, M, KIND>))
k_tile(const S* __restrict__ src, S* __restrict__ dst, TileGeo g, Coef<typename StorageTraits<S>::T> k,
       typename StorageTraits<S>::T* rec, int64_t rec_slot) {
  using T = typename StorageTraits<S>::T;
  using Tr = StorageTraits<S>;
  constexpr bool ADJ = KIND == TILE_ADJOINT;
  constexpr int D = ADJ ? -1 : 1;  // inputs come from x - D c
  constexpr bool PARK = kTileWaves<S, NT, M, KIND> > 1;  // own waits in LDS for the last step
  __shared__ TileCells<S, NT * M, PARK> lds;
  const int n_cells = g.rw * g.rh;
  const int tx0 = (int(blockIdx.x) % g.ntx) * g.tw, ty0 = (int(blockIdx.x) / g.ntx) * g.th;
  const size_t srcb = size_t(g.rs) * g.ny * sizeof(S), recb = size_t(g.rec_rs) * g.ny * sizeof(T);
  const RowRes rs_src = row_res(src, srcb, 0), rs_dst = row_res(dst, srcb, 0);

  int dl[M], dr[M], dd[M], du[M];  // cells of the neighbours at x - 1, x + 1, y - 1, y + 1
  int own[M];                      // index of the node in a population plane; -1: not stored
  int rpos[M];                     // its index in a record entry
  bool wall[M];
  T g9[M][Q], rv[M][NREC];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int n = int(threadIdx.x) + m * NT;
    const int ly = n / g.rw, lx = n - ly * g.rw;
    dl[m] = g.wrapx && lx == 0 ? g.rw - 1 : -1;
    dr[m] = g.wrapx && lx == g.rw - 1 ? 1 - g.rw : 1;
    dd[m] = g.wrapy && ly == 0 ? (g.rh - 1) * g.rw : -g.rw;
    du[m] = g.wrapy && ly == g.rh - 1 ? (1 - g.rh) * g.rw : g.rw;
    own[m] = -1;
    rpos[m] = 0;
    wall[m] = false;
    if (n >= n_cells) continue;
    const int ux = tx0 + lx - g.hx, uy = ty0 + ly - g.hy;
    int x = ux % g.nx, y = uy % g.ny;
    if (x < 0) x += g.nx;
    if (y < 0) y += g.ny;
    const int xm = x == 0 ? g.nx - 1 : x - 1, xp = x == g.nx - 1 ? 0 : x + 1;
    const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y == g.ny - 1 ? 0 : y + 1;
    const int xs[3] = {xm, x, xp}, ys[3] = {ym * g.rs, y * g.rs, yp * g.rs};
    if (lx >= g.hx && lx < g.hx + g.tw && ux < g.nx && ly >= g.hy && ly < g.hy + g.th && uy < g.ny)
      own[m] = y * g.rs + x;
    rpos[m] = y * g.rec_rs + x;
    wall[m] = x == 0 || x == g.nx - 1;
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      g9[m][i] = Tr::load_raw(ldb<S, false>(rs_src, i * g.ps * int(sizeof(S)),
                                            uint32_t(ys[1 - D * cy(i)] + xs[1 - D * cx(i)]) * uint32_t(sizeof(S))));
    });
    if constexpr (ADJ) {
      const RowRes rr = row_res(rec, recb, 0);
#pragma unroll
      for (int j = 0; j < NREC; ++j)
        rv[m][j] = ldb<T, false>(rr, j * g.ps * int(sizeof(T)), uint32_t(rpos[m]) * uint32_t(sizeof(T)));
    }
    if constexpr (PARK) lds.own[n + 1] = own[m];
  }
  for (int s = 0; s < g.ns; ++s) {
    const int lo = g.wrapy ? 0 : s * g.rw, hi = g.wrapy ? n_cells : n_cells - s * g.rw;
    const bool odd = s & 1, last = s == g.ns - 1;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int n = int(threadIdx.x) + m * NT;
      if (n < lo || n >= hi) continue;
      const int c = n + 1;
      const int cols[3] = {c + dl[m], c, c + dr[m]}, rows[3] = {dd[m], 0, du[m]};
      if (s > 0) {
        if (odd) {
          static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            g9[m][i] = Tr::load(lds.c[opp(i)][cols[1 - D * cx(i)] + rows[1 - D * cy(i)]]);
          });
        } else {
#pragma unroll
          for (int i = 0; i < Q; ++i) g9[m][i] = Tr::load(lds.c[i][c]);
        }
      }
      T out[Q];
      if constexpr (ADJ) {
        T rs9[NREC];
#pragma unroll
        for (int j = 0; j < NREC; ++j) rs9[j] = rv[m][j];
        if (!last) {  // the next step's moments, loaded while this one computes
          const RowRes rr = row_res(rec - (s + 1) * rec_slot, recb, 0);
#pragma unroll
          for (int j = 0; j < NREC; ++j)
            rv[m][j] = ldb<T, false>(rr, j * g.ps * int(sizeof(T)), uint32_t(rpos[m]) * uint32_t(sizeof(T)));
        }
        collide_vjp<T, MODEL>(g9[m], rs9, k, out);
      } else {
        collide<T, MODEL, ConserveMode<S, KIND == TILE_WALLS>::value>(g9[m], out, k, KIND == TILE_REC ? rv[m] : nullptr);
      }
      if constexpr (KIND == TILE_REC) {
        if (own[m] >= 0) {
          const RowRes rr = row_res(rec + s * rec_slot, recb, 0);
#pragma unroll
          for (int j = 0; j < NREC; ++j)
            stb<T, 0>(rr, j * g.ps * int(sizeof(T)), uint32_t(rpos[m]) * uint32_t(sizeof(T)), rv[m][j]);
        }
      }
      if constexpr (KIND == TILE_WALLS) {
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i] = wall[m] ? g9[m][opp(i)] : out[i];
      }
      if (last) {
        if constexpr (PARK) own[m] = lds.own[c];
        if (own[m] >= 0) {
#pragma unroll
          for (int i = 0; i < Q; ++i)
            stb<S, 0>(rs_dst, i * g.ps * int(sizeof(S)), uint32_t(own[m]) * uint32_t(sizeof(S)), Tr::store(out[i]));
        }
      } else if (odd) {
        static_for<0, Q>([&](auto I) {
          constexpr int i = decltype(I)::value;
          lds.c[i][cols[1 + D * cx(i)] + rows[1 + D * cy(i)]] = Tr::store(out[i]);
        });
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) lds.c[opp(i)][c] = Tr::store(out[i]);
      }
    }
    if (!last) __syncthreads();
  }
}

}  // namespace lbm
