// Several A-B time steps (or reverse steps) per launch without LDS or barriers between the
// steps: a wavefront marches up a strip of columns and keeps what the next step needs in
// registers.
//
// Buffers have contiguous rows (node x at in-row position x). A wavefront holds 64 NPL adjacent
// nodes of a row, NPL per lane, and walks the rows of its row block. In iteration r it loads the
// nine populations of row r (those with c_y = +-1 from the rows below and above), runs step 1 on
// row r, step 2 on row r - 1, ..., step NS on row r - NS + 1, and stores the last one. Step s + 1
// on row q pulls from step s's output of rows q - 1, q and q + 1: the populations with c_y = -1
// are the ones just computed, those with c_y = 0 and +1 have waited one and two iterations in
// registers (nine values per node and step; 18 FP32 registers per step at NPL = 2). The
// x-shifts are register renames within a lane and one DPP wave shift per population across
// lanes. Values wait rounded to the storage type, so the result is bit-identical to NS single
// steps.
//
// The strip's edge nodes lose their neighbours, one column per side and step, so a wavefront
// stores the 64 NPL - 2 halo nodes in its middle (halo: kMarchHalo, two in the plan for launches of
// two steps), and a row block recomputes NS - 1 rows of step 1 on either side. Measured on MI355X
// (complete model, us per launch of four steps, per two steps of the LDS-staged pair kernel of
// lbm_pair.h): FP32 4096^2 300 / 197, 8192^2 1102 / 802; FP64 4096^2 531 / 405. The FP32 kernel is
// bound by its instructions: 139 vector instructions per computed node and step, 85 274 per
// wavefront with the surroundings (128 columns for 120 stored, 77 rows for 71), which at 4096^2 are
// 676 000 clocks per SIMD, as many as the launch takes (310 us at the 2.16 GHz that the chip runs at
// then). FP64 fills 0.72 of its issue slots (1.94 GHz), FP16 0.97 (2.34 GHz). Fewer steps leave FP32
// bound by memory (4096^2: 3 steps 280, 2 steps 239-284 us per launch), more need more than 256
// registers. Two nodes per lane halve the halo's share and the DPP shifts of one (4096^2 345 us);
// FP64 has registers for one.
#pragma once

#include "lbm_step.h"

namespace lbm {

constexpr int kMarchMax = 4;    // steps per launch
constexpr int kMarchHalo = 4;   // nodes at either edge of a strip that are not stored (two steps: 2)
constexpr int kMarchWaves = 4;  // strips per block on grids that fill the chip
static_assert(kMarchHalo >= kMarchMax, "a step invalidates one column per side");

template <class S> struct MarchNodes { static constexpr int value = 2; };
template <> struct MarchNodes<double> { static constexpr int value = 1; };
constexpr int kMarchAdjointNodes = 1;

// Strips: column c stores the nodes [x0, min(x0 + w, nx)), x0 = c w, but xlast for the last one.
// A pair of nodes must not straddle the periodic wrap: with an even nx no pair does (x0 and the
// halo are even). With an odd nx the last strip is aligned to the row's end instead (xlast = nx -
// w, odd, so that a pair ends at nx - 1 and the next starts at 0), stores some nodes of its
// neighbour a second time (the same values), and no other strip's halo reaches the row's end.
struct MarchGeo {
  int nx, ny, ps;
  int64_t rs, rec_rs;
  int ncol, w, xlast, halo, nrb;
};

template <class T>
struct MarchRec {
  T* p[kMarchMax];
};

template <int BYTES> struct WordsOf;
template <> struct WordsOf<4> { using V = uint32_t; };
template <> struct WordsOf<8> { using V = unsigned int __attribute__((ext_vector_type(2))); };
template <> struct WordsOf<16> { using V = unsigned int __attribute__((ext_vector_type(4))); };

template <int BYTES, int AUX>
__device__ __forceinline__ typename WordsOf<BYTES>::V ldw(const RowRes& rr, int soff, uint32_t voff) {
  if constexpr (BYTES == 4) return __builtin_amdgcn_raw_buffer_load_b32(rr.r, int(voff), soff, AUX);
  else if constexpr (BYTES == 8) return __builtin_amdgcn_raw_buffer_load_b64(rr.r, int(voff), soff, AUX);
  else return __builtin_amdgcn_raw_buffer_load_b128(rr.r, int(voff), soff, AUX);
}

template <int BYTES, int AUX>
__device__ __forceinline__ void stw(const RowRes& rr, int soff, uint32_t voff, typename WordsOf<BYTES>::V v) {
  if constexpr (BYTES == 4) __builtin_amdgcn_raw_buffer_store_b32(v, rr.r, int(voff), soff, AUX);
  else if constexpr (BYTES == 8) __builtin_amdgcn_raw_buffer_store_b64(v, rr.r, int(voff), soff, AUX);
  else __builtin_amdgcn_raw_buffer_store_b128(v, rr.r, int(voff), soff, AUX);
}

// NPL adjacent elements of type E to and from register words.
template <class E, int NPL, class T>
__device__ __forceinline__ void unpack(typename WordsOf<int(sizeof(E)) * NPL>::V v, T o[NPL]) {
  E e[NPL];
  __builtin_memcpy(e, &v, sizeof(e));
#pragma unroll
  for (int j = 0; j < NPL; ++j) o[j] = StorageTraits<E>::load(e[j]);
}
template <class E, int NPL, class T>
__device__ __forceinline__ typename WordsOf<int(sizeof(E)) * NPL>::V pack(const T o[NPL]) {
  E e[NPL];
#pragma unroll
  for (int j = 0; j < NPL; ++j) e[j] = StorageTraits<E>::store(o[j]);
  typename WordsOf<int(sizeof(E)) * NPL>::V v;
  __builtin_memcpy(&v, e, sizeof(e));
  return v;
}

// v of the lane below (D = 1) or above (D = -1); the edge lane gets 0.
template <int D>
__device__ __forceinline__ float lane_shift(float v) {
  constexpr int ctrl = D > 0 ? 0x138 : 0x130;  // DPP wave_shr:1 / wave_shl:1
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true));
}
template <int D>
__device__ __forceinline__ double lane_shift(double v) {
  constexpr int ctrl = D > 0 ? 0x138 : 0x130;
  using I2 = int __attribute__((ext_vector_type(2)));
  I2 u = __builtin_bit_cast(I2, v);
  u.x = __builtin_amdgcn_update_dpp(0, u.x, ctrl, 0xf, 0xf, true);
  u.y = __builtin_amdgcn_update_dpp(0, u.y, ctrl, 0xf, 0xf, true);
  return __builtin_bit_cast(double, u);
}

// o(x) = v(x - C) over the strip's nodes.
template <int C, int NPL, class T>
__device__ __forceinline__ void strip_shift(const T v[NPL], T o[NPL]) {
  if constexpr (C == 0) {
#pragma unroll
    for (int j = 0; j < NPL; ++j) o[j] = v[j];
  } else if constexpr (C > 0) {
#pragma unroll
    for (int j = NPL - 1; j > 0; --j) o[j] = v[j - 1];
    o[0] = lane_shift<1>(v[NPL - 1]);
  } else {
#pragma unroll
    for (int j = 0; j < NPL - 1; ++j) o[j] = v[j + 1];
    o[NPL - 1] = lane_shift<-1>(v[0]);
  }
}

// The values a buffer of type S would hold, back in the compute type. BF16 pairs share one
// conversion (v_cvt_pk_bf16_f32).
template <class S, int NPL, class T>
__device__ __forceinline__ void stored(T v[NPL]) {
  if constexpr (std::is_same_v<S, bf16_t> && NPL == 2) {
    using F2 = float __attribute__((ext_vector_type(2)));
    using B2 = __bf16 __attribute__((ext_vector_type(2)));
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(F2{v[0], v[1]}, B2));
    v[0] = __uint_as_float(w << 16);
    v[1] = __uint_as_float(w & 0xffff0000u);
  } else if constexpr (sizeof(S) == 2) {
#pragma unroll
    for (int j = 0; j < NPL; ++j) v[j] = StorageTraits<S>::load(StorageTraits<S>::store(v[j]));
  }
}

// A wavefront's strip and row block. Blocks are renumbered so that every XCD works on a
// contiguous range of them, x-neighbours side by side.
struct Strip {
  bool active;
  int lane, x, y0, y1;
  bool store;
};
template <int NPL>
__device__ __forceinline__ Strip strip_of(const MarchGeo& g, int& xw) {
  Strip s;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kLanes));
  const int wpb = int(blockDim.x) / kLanes, ncb = (g.ncol + wpb - 1) / wpb;
  const int t = xcd_order(int(blockIdx.x), int(gridDim.x));
  const int by = t / ncb, col = (t % ncb) * wpb + w;
  s.active = col < g.ncol;
  s.lane = int(threadIdx.x % kLanes);
  const int x0 = col == g.ncol - 1 ? g.xlast : col * g.w;
  s.x = x0 - g.halo + NPL * s.lane;
  xw = s.x % g.nx;
  if (xw < 0) xw += g.nx;
  s.store = s.x >= x0 && s.x < x0 + g.w && s.x < g.nx;
  s.y0 = int(int64_t(by) * g.ny / g.nrb);
  s.y1 = int(int64_t(by + 1) * g.ny / g.nrb);
  return s;
}

// Row r of a periodic column of ny rows, r within [-2 (kMarchMax - 1), ny + kMarchMax) (the reverse
// march reads the records of s rows further down).
__device__ __forceinline__ int wrap_row(int r, int ny) {
  while (r < 0) r += ny;
  while (r >= ny) r -= ny;
  return r;
}

// The direction a population moves by its y-component: D = +1 forward (pull from y - c_y),
// D = -1 in the reverse sweep (gather from y + c_y). AHEAD populations come from the row below in
// marching order and wait two iterations, LEVEL one, BEHIND none.
template <int D> struct MarchOrder;
template <> struct MarchOrder<1> { static constexpr int ahead[3] = {2, 5, 6}, level[3] = {0, 1, 3}, behind[3] = {4, 7, 8}; };
template <> struct MarchOrder<-1> { static constexpr int ahead[3] = {4, 7, 8}, level[3] = {0, 1, 3}, behind[3] = {2, 5, 6}; };

// Queue of a step's outputs between two marching steps.
template <class T, int NPL>
struct MarchQueue {
  T level[3][NPL], ahead1[3][NPL], ahead2[3][NPL];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int j = 0; j < NPL; ++j) level[a][j] = ahead1[a][j] = ahead2[a][j] = T(0);
  }
  // Takes the outputs of one row; returns the next step's inputs for the row before it.
  template <int D>
  __device__ __forceinline__ void push(const T out[Q][NPL], T in[Q][NPL]) {
    using O = MarchOrder<D>;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int j = 0; j < NPL; ++j) {
        in[O::ahead[a]][j] = ahead2[a][j];
        ahead2[a][j] = ahead1[a][j];
        ahead1[a][j] = out[O::ahead[a]][j];
        in[O::level[a]][j] = level[a][j];
        level[a][j] = out[O::level[a]][j];
        in[O::behind[a]][j] = out[O::behind[a]][j];
      }
  }
};

// The block's wavefronts meet once per row: neighbouring strips then touch the cache lines they
// share at about the same time (8192^2 1146 -> 1102 us per launch; at 4096^2 no difference).
__device__ __forceinline__ void march_meet() { __builtin_amdgcn_s_barrier(); }

// NS forward steps; with REC step s also writes its moments to rec.p[s].
template <class S, int MODEL, int NS, bool REC>
__global__ void __launch_bounds__(kMarchWaves * kLanes)
k_march(const S* __restrict__ src, S* __restrict__ dst, MarchGeo g, Coef<typename StorageTraits<S>::T> k,
        MarchRec<typename StorageTraits<S>::T> rec) {
  using T = typename StorageTraits<S>::T;
  constexpr int NPL = MarchNodes<S>::value;
  constexpr int B = NPL * int(sizeof(S)), BR = NPL * int(sizeof(T));
  int xw;
  const Strip st = strip_of<NPL>(g, xw);
  const int r0 = st.y0 - (NS - 1), r1 = st.y1 + (NS - 1);  // rows of step 1
  if (!st.active) {
    for (int r = r0; r < r1; ++r) march_meet();
    return;
  }
  const uint32_t voff = uint32_t(xw) * uint32_t(sizeof(S)), rvoff = uint32_t(xw) * uint32_t(sizeof(T));
  const size_t rsb = size_t(g.rs) * sizeof(S);
  const int psb = g.ps * int(sizeof(S));
  typename WordsOf<B>::V raw[Q];
  auto load = [&](int r) {
    const int y = wrap_row(r, g.ny);
    const int ym = (y == 0) ? g.ny - 1 : y - 1, yp = (y == g.ny - 1) ? 0 : y + 1;
    const RowRes sr[3] = {row_res(src, rsb, ym), row_res(src, rsb, y), row_res(src, rsb, yp)};
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      raw[i] = ldw<B, 0>(sr[-cy(i) + 1], i * psb, voff);
    });
  };
  MarchQueue<T, NPL> queue[NS > 1 ? NS - 1 : 1];
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) queue[s].clear();
  load(r0);
  auto row = [&](const int r) {
    march_meet();
    T in[Q][NPL];
#pragma unroll
    for (int i = 0; i < Q; ++i) unpack<S, NPL>(raw[i], in[i]);
    load(r + 1);  // past the last row as well: a branch would cost a copy of every loaded register
    static_for<0, NS>([&](auto STEP) {
      constexpr int s = decltype(STEP)::value;
      const int yr = r - s;  // this step's row
      const bool own = yr >= st.y0 && yr < st.y1;
      T g9[Q][NPL], out[Q][NPL], rv[NREC][NPL];
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        strip_shift<cx(i), NPL>(in[i], g9[i]);
      });
#pragma unroll
      for (int j = 0; j < NPL; ++j) {
        T a[Q], b[Q], m[NREC];
#pragma unroll
        for (int i = 0; i < Q; ++i) a[i] = g9[i][j];
        collide<T, MODEL, ConserveMode<S>::value>(a, b, k, REC ? m : nullptr);
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i][j] = b[i];
        if constexpr (REC) {
#pragma unroll
          for (int i = 0; i < NREC; ++i) rv[i][j] = m[i];
        }
      }
      if constexpr (REC) {
        if (own && st.store) {
          const RowRes rr = row_res(rec.p[s], size_t(g.rec_rs) * sizeof(T), yr);
#pragma unroll
          for (int i = 0; i < NREC; ++i) stw<BR, 0>(rr, i * g.ps * int(sizeof(T)), rvoff, pack<T, NPL>(rv[i]));
        }
      }
      if constexpr (s < NS - 1) {
#pragma unroll
        for (int i = 0; i < Q; ++i) stored<S, NPL>(out[i]);
        queue[s].template push<1>(out, in);
      } else if (own && st.store) {
        const RowRes dr = row_res(dst, rsb, yr);
#pragma unroll
        for (int i = 0; i < Q; ++i) stw<B, 0>(dr, i * psb, voff, pack<S, NPL>(out[i]));
      }
    });
  };
  for (int r = r0; r < r1; ++r) row(r);
}

// NS reverse steps of the discrete adjoint, fbar^{n+1} -> fbar^{n+1-NS}: the same march with the
// streaming reversed (populations gathered at x + c_i); rec.p[s] holds the moments of time step
// n - s, which reverse step s needs. The compute type throughout. Bound by memory, the records
// above all (20 of the 38 bytes per FP32 node and step). Measured on MI355X, us per reverse step
// of 4096^2, complete model: single steps 244, 2 / 3 / 4 steps per launch 189 / 153 / 138 (two
// nodes per lane 188 / 154 / 136; at 1024^2 12.8 / 12.7 / 13.6 against 12.0 / 11.6 / 12.4).
template <class T, int MODEL, int NS>
__global__ void __launch_bounds__(kMarchWaves * kLanes)
k_march_adjoint(const T* __restrict__ src, T* __restrict__ dst, MarchGeo g, Coef<T> k, MarchRec<const T> rec) {
  constexpr int NPL = kMarchAdjointNodes;
  constexpr int B = NPL * int(sizeof(T));
  int xw;
  const Strip st = strip_of<NPL>(g, xw);
  const int r0 = st.y0 - (NS - 1), r1 = st.y1 + (NS - 1);
  if (!st.active) {
    for (int r = r0; r < r1; ++r) march_meet();
    return;
  }
  const uint32_t voff = uint32_t(xw) * uint32_t(sizeof(T));
  const size_t rsb = size_t(g.rs) * sizeof(T), rrsb = size_t(g.rec_rs) * sizeof(T);
  const int psb = g.ps * int(sizeof(T));
  typename WordsOf<B>::V raw[Q], raw_rec[NS][NREC];
  auto load = [&](int r) {
    const int y = wrap_row(r, g.ny);
    const int ym = (y == 0) ? g.ny - 1 : y - 1, yp = (y == g.ny - 1) ? 0 : y + 1;
    const RowRes sr[3] = {row_res(src, rsb, ym), row_res(src, rsb, y), row_res(src, rsb, yp)};
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      raw[i] = ldw<B, 0>(sr[cy(i) + 1], i * psb, voff);
    });
    static_for<0, NS>([&](auto STEP) {
      constexpr int s = decltype(STEP)::value;
      const RowRes rr = row_res(rec.p[s], rrsb, wrap_row(r - s, g.ny));
#pragma unroll
      for (int i = 0; i < NREC; ++i) raw_rec[s][i] = ldw<B, 0>(rr, i * psb, voff);
    });
  };
  MarchQueue<T, NPL> queue[NS > 1 ? NS - 1 : 1];
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) queue[s].clear();
  load(r0);
  auto row = [&](const int r) {
    march_meet();
    T in[Q][NPL], rv[NS][NREC][NPL];
#pragma unroll
    for (int i = 0; i < Q; ++i) unpack<T, NPL>(raw[i], in[i]);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int i = 0; i < NREC; ++i) unpack<T, NPL>(raw_rec[s][i], rv[s][i]);
    load(r + 1);
    static_for<0, NS>([&](auto STEP) {
      constexpr int s = decltype(STEP)::value;
      const int yr = r - s;
      T g9[Q][NPL], out[Q][NPL];
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        strip_shift<-cx(i), NPL>(in[i], g9[i]);
      });
#pragma unroll
      for (int j = 0; j < NPL; ++j) {
        T a[Q], b[Q], m[NREC];
#pragma unroll
        for (int i = 0; i < Q; ++i) a[i] = g9[i][j];
#pragma unroll
        for (int i = 0; i < NREC; ++i) m[i] = rv[s][i][j];
        collide_vjp<T, MODEL>(a, m, k, b);
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i][j] = b[i];
      }
      if constexpr (s < NS - 1) {
        queue[s].template push<-1>(out, in);
      } else if (yr >= st.y0 && yr < st.y1 && st.store) {
        const RowRes dr = row_res(dst, rsb, yr);
#pragma unroll
        for (int i = 0; i < Q; ++i) stw<B, 0>(dr, i * psb, voff, pack<T, NPL>(out[i]));
      }
    });
  };
  for (int r = r0; r < r1; ++r) row(r);
}

}  // namespace lbm
