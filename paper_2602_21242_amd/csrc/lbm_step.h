// Single-step kernels: the fused stream + collide step (with or without walls) and the adjoint
// step; the two-step adjoint kernel of the AA layout. Instantiated per storage type in
// step_<type>.hip. The kernels that take several steps per launch are in lbm_march.h and
// lbm_tile.h.
//
// Data layout (HBM): shifted populations g_i, row-interleaved structure of arrays: element
// (i, x, y) sits at y * rs + i * ps + pos(x) with ps = pitch = 64 ceil(nx / 64), rs = 9 * pitch.
// The nine population rows of a lattice row are contiguous, which keeps the 18 concurrent
// read/write streams of a step within a compact address window. Rows are padded to whole
// 64-element groups; padding positions are never read by a real node.
//
// A-B buffers have contiguous rows, pos(x) = x: a wavefront that keeps several steps of adjacent
// nodes in registers or LDS (lbm_march.h, lbm_tile.h) needs them adjacent. The single step's
// x-shifted loads then straddle one more cache line, which costs it 1 % (4096^2 183.5 -> 185 us
// per step) in blocks of up to 16 adjacent wavefronts.
//
// AA buffers have lane-strided rows: with S = ceil(nx / 64), node x = lane * S + s is stored at
// pos(x) = 64 s + lane, so the 64 lanes of a wave hold the nodes s, s + S, ..., s + 63 S. The
// x-neighbours of those nodes are again one whole, aligned 64-element group, so the x-shifts of
// the odd steps, which shift stores as well as loads, cost no extra cache lines; only the groups
// s = 0 and s = S - 1 read a group rotated by one lane. (With contiguous rows an odd step's
// stores write parts of lines: 4096^2 282-343 us per odd step instead of 184.) The step kernel
// lets a padding lane read and write its own padding slot (no per-lane guards), the other kernels
// skip padding.
//
// One thread updates NPT nodes (one lane of NPT consecutive groups); a block of 256 threads
// covers 4 NPT groups of one row, so the row, its two periodic neighbours and every
// row/population base address are uniform (scalar registers) and each lane only adds its
// 32-bit in-row offset.
//
// Streaming patterns. The state at time n satisfies f_i^n(x) = buf[s(i)][x - d c_i]:
//   A-B:       d = 1, s(i) = i (the buffer holds post-collision values at their origin;
//              the step pulls from x - c_i and writes in place in the other buffer).
//   AA, even:  d = 0, s(i) = i; the step reads locally and writes f*_i to slot opp(i).
//   AA, odd:   d = 1, s(i) = opp(i); the step pulls and pushes f*_i to x + c_i, slot i.
// Each AA step reads and writes exactly the same set of locations per node, so one buffer
// suffices and threads never race.
#pragma once

#include <type_traits>

#include "lbm_device.h"

namespace lbm {

constexpr int kBlock = 256;
constexpr int kLanes = 64;     // nodes per group of the lane-strided row layout (wavefront)
constexpr int kRowsY = 32768;  // rows per grid y-dimension slice

struct Geo {
  int nx, ny;
  int S;           // groups per row (pitch / 64)
  int ps;          // elements between the rows of two populations of one lattice row
  int64_t rs;      // elements between two lattice rows
  int nseg;        // blocks per lattice row = ceil(S / (4 NPT))
  int plast;       // pos(nx - 1)
  int xcd;         // k_step: blocks in the order of xcd_tile
};

// Largest block of the A-B step kernel: with contiguous rows every group's x-shifted loads
// straddle a line of the next group, which a block's wavefronts share in the compute unit's
// caches, so larger blocks re-read fewer lines (FP32 3000^2 111 us with 256 threads, 108 with
// 512, 105 with 1024; 2048^2 43, 41, 41; BF16 8192^2 393, 392, 388; FP16 3000^2 57.6, 58.4,
// 64.5: 16-bit storage has two to four nodes per thread, and its blocks of 1024 threads too few
// rows in flight).
template <class S> constexpr int kStepBlock = sizeof(S) == 2 ? 512 : 1024;

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Element type the nontemporal builtins accept.
template <class S> struct Bits { using type = S; };
template <> struct Bits<bf16_t> { using type = uint16_t; };

template <class S>
__device__ __forceinline__ S ld1(const S* p) {
  using B = typename Bits<S>::type;
  const B b = __builtin_nontemporal_load(reinterpret_cast<const B*>(p));
  S r;
  __builtin_memcpy(&r, &b, sizeof(r));
  return r;
}

template <class S>
__device__ __forceinline__ void st1(S* p, S v) {
  using B = typename Bits<S>::type;
  B b;
  __builtin_memcpy(&b, &v, sizeof(b));
  __builtin_nontemporal_store(b, reinterpret_cast<B*>(p));
}

// A population load into the register form StorageTraits<S>::Raw (the storage type itself,
// or for FP16 its 16 bits zero-extended to 32).
// NT selects the nontemporal hint (the default) or a plain load.
template <class S, bool NT = true>
__device__ __forceinline__ typename StorageTraits<S>::Raw ld_raw(const S* p) {
  using R = typename StorageTraits<S>::Raw;
  using B = typename Bits<S>::type;
  if constexpr (std::is_same_v<R, S>) {
    if constexpr (NT) {
      return ld1(p);
    } else {
      const B b = *reinterpret_cast<const B*>(p);
      S r;
      __builtin_memcpy(&r, &b, sizeof(r));
      return r;
    }
  } else {
    static_assert(sizeof(S) == 2 && std::is_same_v<R, uint32_t>, "raw registers: 16-bit storage only");
    if constexpr (NT) return R(__builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(p)));
    else return R(*reinterpret_cast<const uint16_t*>(p));
  }
}

// Element at in-row position p of a population row: base (uniform: buffer + row +
// population) plus the lane's 32-bit byte offset.
template <class S>
__device__ __forceinline__ const S* at(const char* base, int p) {
  return reinterpret_cast<const S*>(base + uint32_t(p) * uint32_t(sizeof(S)));
}
template <class S>
__device__ __forceinline__ S* at(char* base, int p) {
  return reinterpret_cast<S*>(base + uint32_t(p) * uint32_t(sizeof(S)));
}

// Buffer-resource accesses. One lattice row of a buffer (its nine population rows, or the five
// rows of a moment record) is described by a buffer resource in scalar registers, rebased to
// that row; an access adds the scalar offset of the population (or record entry) within the
// lattice row and the lane's 32-bit in-row byte offset, which stays in one vector register for
// a whole row loop (plain pointers made the compiler keep nine 64-bit per-population addresses
// and add each row's offset to them in vector arithmetic). AA's adjoint kernels use plain
// pointers: AA's two-step adjoint ran 5 % slower with buffer accesses (433 against 414 us per
// launch at 4096^2). Offsets within a lattice row stay below 2^31 bytes: lbm_init rejects wider
// rows.
constexpr int kRsrcWord3 = 0x00020000;  // resource word 3 of a raw buffer on the gfx9 family
constexpr int kAuxNT = 2;                // cache-policy operand of a nontemporal access (gfx950)
// Cache policy of the single-step kernel (STREAM, chosen by the host from the population buffers'
// size against the last-level cache): on larger grids loads and stores are nontemporal, the
// stores with the SC1 scope bit as well (device scope, written through rather than held in the
// XCD's L2): 4096^2 186.8 -> 183.5 us. SC1 without the nontemporal bit measured 3.5 % slower
// than plain nontemporal stores, stores without either hint 10 % slower. Buffers that stay in the
// last-level cache are read and written plainly: AA, FP32, complete model 3000 x 2000 72 -> 50
// us, 1000^2 15.3 -> 10.5 us (uniform fields; 84 -> 62 us in a Taylor-Green run, XCD order
// included).
constexpr int kAuxStoreWT = kAuxNT | 16;
template <int STREAM> constexpr int kAuxStore = STREAM ? kAuxStoreWT : 0;
// Which loads of a streaming step are nontemporal. A-B: those of the populations that do not move
// along x. The others straddle a line that the next wavefront or block also reads, and a
// nontemporal line is gone by then (us per step, all nontemporal / those / none: FP32 4096^2 186.0
// / 183.4 / 192.4, 8192^2 740 / 730 / 763, FP64 8192 x 4096 793 / 783 / 808, BF16 8192^2 417 / 387
// / 391). AA: all in FP32 and FP64; of 16-bit storage on rows without padding (STREAM_ALL: FP16
// 8192^2 384, plain 410), not on padded ones, whose padding lanes load parts of lines (5200^2 215,
// 190).
enum { STREAM_OFF = 0, STREAM_ON = 1, STREAM_ALL = 2 };
template <class S, int PH, int STREAM, int DX>
constexpr bool kLoadNT = STREAM != STREAM_OFF && (PH == PH_AB ? DX == 0 : sizeof(S) != 2 || STREAM == STREAM_ALL);

struct RowRes {
  __amdgpu_buffer_rsrc_t r;
};

// Lattice row y of a buffer whose lattice rows are row_bytes apart.
__device__ __forceinline__ RowRes row_res(const void* buf, size_t row_bytes, int y) {
  char* base = const_cast<char*>(static_cast<const char*>(buf)) + size_t(y) * row_bytes;
  return RowRes{__builtin_amdgcn_make_buffer_rsrc(base, 0, int(uint32_t(row_bytes)), kRsrcWord3)};
}

// Element (soff + voff bytes into the lattice row) in the register form
// StorageTraits<E>::Raw for storage types, or as E itself for the compute types.
template <class E, bool NT>
__device__ __forceinline__ auto ldb(const RowRes& rr, int soff, uint32_t voff) {
  constexpr int aux = NT ? kAuxNT : 0;
  if constexpr (sizeof(E) == 8) {
    return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b64(rr.r, int(voff), soff, aux));
  } else if constexpr (sizeof(E) == 4) {
    return __builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b32(rr.r, int(voff), soff, aux));
  } else {
    const uint16_t h = __builtin_amdgcn_raw_buffer_load_b16(rr.r, int(voff), soff, aux);
    using R = typename StorageTraits<E>::Raw;
    if constexpr (std::is_same_v<R, uint32_t>) return uint32_t(h);
    else return __builtin_bit_cast(E, h);
  }
}

// Store of one element, nontemporal (every kernel writes each location once per launch), with
// the cache policy AUX.
template <class E, int AUX>
__device__ __forceinline__ void stb(const RowRes& rr, int soff, uint32_t voff, E v) {
  if constexpr (sizeof(E) == 8) {
    using V2 = unsigned int __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, v), rr.r, int(voff), soff, AUX);
  } else if constexpr (sizeof(E) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rr.r, int(voff), soff, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), rr.r, int(voff), soff, AUX);
  }
}

// In-row positions of a node and of its periodic x-neighbours.
struct RowPos {
  int p0, pm, pp;  // pos(x), pos(x - 1), pos(x + 1)
  template <int DX>
  __device__ __forceinline__ int of() const { return DX == 0 ? p0 : (DX < 0 ? pm : pp); }
};

// In-row positions of the node in group s at lane `lane` and of its periodic x-neighbours;
// false past the row (s >= S) and for padding.
__device__ __forceinline__ bool node_pos(const Geo& geo, int s, int lane, RowPos& r) {
  const int q = s * kLanes + lane;
  const int x = lane * geo.S + s;
  if (s >= geo.S || x >= geo.nx) return false;
  r.p0 = q;
  r.pm = s > 0 ? q - kLanes : (lane > 0 ? (geo.S - 1) * kLanes + lane - 1 : geo.plast);
  r.pp = x + 1 == geo.nx ? 0 : (s + 1 < geo.S ? q + kLanes : lane + 1);
  return true;
}

// The same with contiguous rows: position x of group s at lane `lane` is x = 64 s + lane.
__device__ __forceinline__ bool node_pos_contig(const Geo& geo, int s, int lane, RowPos& r) {
  const int x = s * kLanes + lane;
  if (x >= geo.nx) return false;
  r.p0 = x;
  r.pm = x > 0 ? x - 1 : geo.nx - 1;
  r.pp = x + 1 < geo.nx ? x + 1 : 0;
  return true;
}

// The hardware hands consecutive workgroup IDs to the chip's 8 XCDs in turn, and each XCD has
// its own L2. Kernels whose neighbouring blocks read the same lines renumber their blocks so that
// every XCD works on one contiguous range of tiles, x-neighbours side by side. Any value is
// correct (it is a permutation of the tiles); 8 matches MI355X.
constexpr int kXcds = 8;

// Place in that order of the block with linear ID L of n: XCD L % kXcds takes tiles [start,
// start + count) in order, start and count splitting the n tiles as evenly as possible.
__device__ __forceinline__ int xcd_order(int L, int n) {
  const int xcd = L % kXcds;
  return xcd * (n / kXcds) + min(xcd, n % kXcds) + L / kXcds;
}
__device__ __forceinline__ void xcd_tile(int& bx, int& by) {
  const int nx = int(gridDim.x);
  const int t = xcd_order(int(blockIdx.x) + int(blockIdx.y) * nx, nx * int(gridDim.y));
  bx = t % nx;
  by = t / nx;
}

// Block -> lattice row (uniform); the block's wavefronts take NPT consecutive groups each,
// starting at the returned group s0. Grid: (nseg, min(ny, kRowsY), ceil(ny / kRowsY)) with
// nseg = ceil(S / (W NPT)) for blocks of W wavefronts. s0 is uniform across a wavefront and is
// kept in a scalar register. With xcd the blocks of a grid slice are taken in the order of
// xcd_tile.
static_assert(kBlock % kLanes == 0, "a block must consist of whole 64-node groups");
template <int NPT>
__device__ __forceinline__ int first_group(int& y, int& lane, bool xcd, int threads = kBlock) {
  int bx = int(blockIdx.x), by = int(blockIdx.y);
  if (xcd) xcd_tile(bx, by);
  y = int(blockIdx.z) * kRowsY + by;
  lane = int(threadIdx.x % kLanes);
  return (bx * (threads / kLanes) + __builtin_amdgcn_readfirstlane(int(threadIdx.x / kLanes))) * NPT;
}

// One time step; each thread updates NPT nodes (same lane, consecutive groups), issuing the
// loads of all of them before the first collision so that more memory traffic is in flight
// per wavefront. src and dst alias in the AA phases. With REC the moments (rho, u_x, u_y,
// N_xx, N_xy) of every node are written to rec, laid out like the populations with five
// entries per lattice row (row stride rec_rs). With WALLS (A-B) the columns x = 0 and x = nx - 1 are
// solid (fullway bounce-back, the isothermal shocktube of Sec. 5): a wall node pulls its populations
// like any node and, instead of colliding, sends each back the way it came, g*_i = g_opp(i) (exact
// in the shifted storage since w_i = w_opp(i)).
template <class S, int MODEL, int PH, bool REC, int NPT, int STREAM, bool WALLS = false>
__global__ void __launch_bounds__((PH == PH_AB ? kStepBlock<S> : kBlock))
k_step(const S* src, S* dst, Geo geo, Coef<typename StorageTraits<S>::T> k,
       typename StorageTraits<S>::T* rec, int64_t rec_rs) {
  using T = typename StorageTraits<S>::T;
  using Tr = StorageTraits<S>;
  int y, lane;
  const int s0 = first_group<NPT>(y, lane, geo.xcd, PH == PH_AB ? int(blockDim.x) : kBlock);
  // Uniform exits only: the host launches NPT > 1 only when S is a multiple of 4 NPT, so a
  // wavefront's groups are either all inside the row or all past it. Padding lanes
  // (x >= nx) run on their own padding slot for every access (no real node reads those
  // slots and each still has one reader and one writer), so that all loads of the thread
  // stay in one basic block and are issued back to back.
  if (y >= geo.ny || s0 >= geo.S) return;
  RowPos rp[NPT];
#pragma unroll
  for (int n = 0; n < NPT; ++n) {
    const bool node = PH == PH_AB ? node_pos_contig(geo, s0 + n, lane, rp[n]) : node_pos(geo, s0 + n, lane, rp[n]);
    if (!node) rp[n].p0 = rp[n].pm = rp[n].pp = (s0 + n) * kLanes + lane;
  }
  const int ym = (y == 0) ? geo.ny - 1 : y - 1;
  const int yp = (y == geo.ny - 1) ? 0 : y + 1;
  const size_t rsb = size_t(geo.rs) * sizeof(S), psb = size_t(geo.ps) * sizeof(S);
  const char* sr[3] = {reinterpret_cast<const char*>(src) + ym * rsb, reinterpret_cast<const char*>(src) + y * rsb,
                       reinterpret_cast<const char*>(src) + yp * rsb};
  // Stores through buffer descriptors of the three rows (cache policy kAuxStore<STREAM>).
  const RowRes dr[3] = {row_res(dst, rsb, ym), row_res(dst, rsb, y), row_res(dst, rsb, yp)};

  typename Tr::Raw gs[NPT][Q];
#pragma unroll
  for (int n = 0; n < NPT; ++n) {
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr bool shift = (PH != PH_AA_EVEN);
      constexpr int slot = (PH == PH_AA_ODD) ? opp(i) : i;
      constexpr int dx = shift ? -cx(i) : 0;
      constexpr int dy = shift ? -cy(i) : 0;
      gs[n][i] = ld_raw<S, kLoadNT<S, PH, STREAM, dx>>(at<S>(sr[dy + 1] + slot * psb, rp[n].template of<dx>()));
    });
  }

#pragma unroll
  for (int n = 0; n < NPT; ++n) {
    T g[Q], out[Q], rv[NREC];
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = Tr::load_raw(gs[n][i]);
    collide<T, MODEL, ConserveMode<S, WALLS>::value>(g, out, k, REC ? rv : nullptr);
    if constexpr (WALLS) {
      const bool wall = rp[n].p0 == 0 || rp[n].p0 == geo.nx - 1;
#pragma unroll
      for (int i = 0; i < Q; ++i) out[i] = wall ? g[opp(i)] : out[i];
    }
    if constexpr (REC) {
      const RowRes rr = row_res(rec, size_t(rec_rs) * sizeof(T), y);
#pragma unroll
      for (int r = 0; r < NREC; ++r)
        stb<T, kAuxStore<STREAM>>(rr, r * geo.ps * int(sizeof(T)), uint32_t(rp[n].p0) * uint32_t(sizeof(T)), rv[r]);
    }
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr bool shift = (PH == PH_AA_ODD);
      constexpr int slot = (PH == PH_AA_EVEN) ? opp(i) : i;
      constexpr int dx = shift ? cx(i) : 0;
      constexpr int dy = shift ? cy(i) : 0;
      stb<S, kAuxStore<STREAM>>(dr[dy + 1], slot * int(psb), uint32_t(rp[n].template of<dx>()) * uint32_t(sizeof(S)),
                            Tr::store(out[i]));
    });
  }
}

constexpr int kFuseGroups = 8;
constexpr int kFuseRows = 64;
constexpr int kFuseMinRows = 2;
// Blocks of up to kFuseRowsTall rows are taken when the grid then gives each block a compute
// unit of its own (not for FP64): the pair kernel at 4096^2 197 us per launch against 201 with 64
// rows; AA's reverse pair takes the same time with either.
constexpr int kFuseRowsTall = 128;
template <class T> struct FuseTall : std::false_type {};
template <> struct FuseTall<float> : std::true_type {};

// Two reverse steps per launch on AA's lane-strided rows, staged through LDS. A block owns
// kFuseGroups consecutive groups (one interior wavefront each) and the rows [y0, y1), the rows
// split evenly over gridDim.y row blocks (so gridDim.y <= ny); two halo wavefronts compute the
// x-neighbours of its edge groups. The block walks its rows y0 - 1 .. y1 with a ring of three
// rows in LDS. Phase A computes fbar^n of every
// wavefront's node at row r from fbar^{n+1} gathered at x + c_i and the records rec_hi of
// step n; phase B computes fbar^{n-1} of row r - 1 for the interior wavefronts from the
// ring and the records rec_lo of step n - 1, and stores it. The same arithmetic as two
// k_adjoint_step launches (equal up to the compiler's choice of fused multiply-adds, which
// can differ between the two kernels: relative differences of order 1e-16 in FP64 and 1e-7
// in FP32). fbar uses the
// population layout in the compute type; requires nx % 64 == 0 and S % kFuseGroups == 0.
template <class T>
__device__ __forceinline__ void load_gathered(const T* src, const Geo& geo, int r, const RowPos& rp, T fs[Q]) {
  const int y = r < 0 ? r + geo.ny : (r >= geo.ny ? r - geo.ny : r);
  const int ym = (y == 0) ? geo.ny - 1 : y - 1;
  const int yp = (y == geo.ny - 1) ? 0 : y + 1;
  const size_t rsb = size_t(geo.rs) * sizeof(T), psb = size_t(geo.ps) * sizeof(T);
  const char* sr[3] = {reinterpret_cast<const char*>(src) + ym * rsb, reinterpret_cast<const char*>(src) + y * rsb,
                       reinterpret_cast<const char*>(src) + yp * rsb};
  static_for<0, Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    fs[i] = ld1(at<T>(sr[cy(i) + 1] + i * psb, rp.template of<cx(i)>()));
  });
}

template <class T>
__device__ __forceinline__ void load_record(const T* rec, const Geo& geo, int64_t rec_rs, int r, int pos, T rv[NREC]) {
  const int y = r < 0 ? r + geo.ny : (r >= geo.ny ? r - geo.ny : r);
  const char* rrow = reinterpret_cast<const char*>(rec) + y * (size_t(rec_rs) * sizeof(T));
#pragma unroll
  for (int j = 0; j < NREC; ++j) rv[j] = ld1(at<T>(rrow + j * size_t(geo.ps) * sizeof(T), pos));
}

template <class T, int MODEL>
__global__ void __launch_bounds__((kFuseGroups + 2) * kLanes)
k_adjoint_step2(const T* __restrict__ fbar_next, T* __restrict__ fbar, Geo geo, Coef<T> k,
                const T* __restrict__ rec_hi, const T* __restrict__ rec_lo, int64_t rec_rs) {
  constexpr int G = kFuseGroups;
  __shared__ T ring[3][G + 2][Q][kLanes];
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x / kLanes));
  const int lane = int(threadIdx.x % kLanes);
  int bx, by;
  xcd_tile(bx, by);
  const int s0 = bx * G;
  const int y0 = int(int64_t(by) * geo.ny / gridDim.y);
  const int y1 = int(int64_t(by + 1) * geo.ny / gridDim.y);
  RowPos ra;
  if (w == 0 || w == G + 1) {
    RowPos e;
    node_pos(geo, w == 0 ? s0 : s0 + G - 1, lane, e);
    const int p = w == 0 ? e.pm : e.pp;
    node_pos(geo, p / kLanes, p % kLanes, ra);
  } else {
    node_pos(geo, s0 + w - 1, lane, ra);
  }
  const bool interior = w >= 1 && w <= G;
  const int pb = (s0 + w - 1) * kLanes + lane;
  const size_t rsb = size_t(geo.rs) * sizeof(T), psb = size_t(geo.ps) * sizeof(T);

  T fs[Q], rv[NREC], rl[NREC];
  // Phase A of row r: fbar^n of the wavefront's node (gathered fbar^{n+1} in fs, its
  // records in rv) into the ring slot of row r.
  auto phase_a = [&](const int r) {
    const int slot = (r - y0 + 1) % 3;
    T fb[Q];
    collide_vjp<T, MODEL>(fs, rv, k, fb);
#pragma unroll
    for (int i = 0; i < Q; ++i) ring[slot][w][i][lane] = fb[i];
  };
  // Phase B of row yr (interior wavefronts): fbar^{n-1} from the ring rows yr - 1 .. yr + 1
  // and the records of step n - 1 in rl, stored.
  auto phase_b = [&](const int yr) {
    T g[Q], fb[Q];
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      g[i] = ring[(yr + cy(i) - y0 + 1) % 3][w + cx(i)][i][lane];
    });
    collide_vjp<T, MODEL>(g, rl, k, fb);
    char* orow = reinterpret_cast<char*>(fbar) + yr * rsb;
#pragma unroll
    for (int i = 0; i < Q; ++i) st1(at<T>(orow + i * psb, pb), fb[i]);
  };
  auto load_a = [&](const int r) {
    load_gathered<T>(fbar_next, geo, r, ra, fs);
    load_record<T>(rec_hi, geo, rec_rs, r, ra.p0, rv);
  };
  auto load_b = [&](const int yr) { load_record<T>(rec_lo, geo, rec_rs, yr, pb, rl); };

  // Per row r = y0 - 1 .. y1 every wavefront runs phase A of r, issues the loads of r + 1
  // and passes two barriers; between them the interior wavefronts run phase B of r - 1
  // (from r = y0 + 1 on) and then issue the records phase B of r will need (r < y1). The
  // records are loaded one row ahead, after the stores: vector-memory operations complete
  // in issue order, so records loaded after the next row's prefetch would make phase B
  // wait for that prefetch as well.
  load_a(y0 - 1);
  if (!interior) {
    for (int r = y0 - 1; r <= y1; ++r) {
      phase_a(r);
      if (r < y1) load_a(r + 1);
      __syncthreads();
      __syncthreads();
    }
    return;
  }
  // Interior wavefronts: the loop is entered right after the loads of the next row, the most
  // recent operations on every path into it, so both waits in its body (phase B's records,
  // issued before those loads, and phase A's loads, issued before phase B's stores and the
  // next records) leave the later operations in flight.
  phase_a(y0 - 1);
  load_a(y0);
  __syncthreads();
  __syncthreads();
  phase_a(y0);
  load_a(y0 + 1);
  __syncthreads();
  load_b(y0);
  __syncthreads();
  phase_a(y0 + 1);
  if (y0 + 1 < y1) {
    load_a(y0 + 2);
    for (int r = y0 + 2; r < y1; ++r) {
      __syncthreads();
      phase_b(r - 2);
      load_b(r - 1);
      __syncthreads();
      phase_a(r);
      load_a(r + 1);
    }
    __syncthreads();
    phase_b(y1 - 2);
    load_b(y1 - 1);
    __syncthreads();
    phase_a(y1);
  }
  __syncthreads();
  phase_b(y1 - 1);
  __syncthreads();
}

// One reverse step of the discrete adjoint: fbar^n(x) = J(m^n(x))^T fbar*(x) with the
// reverse-streamed fbar*_i(x) = fbar^{n+1}_i(x + c_i). fbar uses the population layout in
// the compute type (geo describes it); rec holds the step's recorded moments. CONTIG: the A-B
// buffers' contiguous rows, else AA's lane-strided ones.
template <class T, int MODEL, bool CONTIG>
__global__ void __launch_bounds__(kBlock)
k_adjoint_step(const T* __restrict__ fbar_next, T* __restrict__ fbar, Geo geo, Coef<T> k,
               const T* __restrict__ rec, int64_t rec_rs) {
  int y, lane;
  const int s0 = first_group<1>(y, lane, CONTIG);
  RowPos rp;
  if (y >= geo.ny || !(CONTIG ? node_pos_contig(geo, s0, lane, rp) : node_pos(geo, s0, lane, rp))) return;
  const int ym = (y == 0) ? geo.ny - 1 : y - 1;
  const int yp = (y == geo.ny - 1) ? 0 : y + 1;
  const size_t rsb = size_t(geo.rs) * sizeof(T), psb = size_t(geo.ps) * sizeof(T);
  const char* nr[3] = {reinterpret_cast<const char*>(fbar_next) + ym * rsb,
                       reinterpret_cast<const char*>(fbar_next) + y * rsb,
                       reinterpret_cast<const char*>(fbar_next) + yp * rsb};
  T fs[Q];
  static_for<0, Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    fs[i] = ld1(at<T>(nr[cy(i) + 1] + i * psb, rp.of<cx(i)>()));
  });
  T rv[NREC];
  const char* rrow = reinterpret_cast<const char*>(rec) + y * (size_t(rec_rs) * sizeof(T));
#pragma unroll
  for (int r = 0; r < NREC; ++r) rv[r] = ld1(at<T>(rrow + r * psb, rp.p0));
  T fb[Q];
  collide_vjp<T, MODEL>(fs, rv, k, fb);
  char* orow = reinterpret_cast<char*>(fbar) + y * rsb;
#pragma unroll
  for (int i = 0; i < Q; ++i) st1(at<T>(orow + i * psb, rp.p0), fb[i]);
}

}  // namespace lbm
