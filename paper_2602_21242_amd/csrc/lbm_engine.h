// Host-callable launchers for one storage type S (explicitly instantiated in
// step_<type>.hip) plus the auxiliary per-node kernels: initialisation at the guided
// equilibrium, population export/import, moments, FP64 invariants, and the adjoint's
// seed and initial-condition kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.h"
#include "lbm_plan.h"

namespace lbm {

// Everything a launcher needs to know about a run (host side). Element (i, x, y) of a buffer is
// at y * row_stride + i * pitch + pos(x): contiguous rows (contig, A-B) have pos(x) = x,
// lane-strided ones (AA) pos(x) = (x mod S) * 64 + floor(x / S), S = pitch / 64.
struct RunDesc {
  int nx, ny, pitch;  // pitch = 64 ceil(nx / 64)
  int64_t rs;         // row stride of the populations and of fbar (9 * pitch)
  int64_t rs_rec;     // row stride of a recorded-moment slot (5 * pitch)
  double theta, nu, rho0, tau;
  int model;         // M_BGK ... M_COMPLETE
  int contig;        // 1: contiguous rows (A-B), 0: lane-strided rows (AA)
  int pair;          // lbm_steps_per_launch reports 2
  int adj_rb;        // AA: row blocks of the two-step adjoint kernel; 0: one reverse step per launch
  int walls;         // 1: solid bounce-back columns at x = 0 and x = nx - 1 (A-B only)
  int xcd;           // 1: the single-step kernel's blocks run in XCD order (see kXcdBytes)
  int stream;        // the single-step kernel's cache policy (STREAM_OFF, _ON, _ALL)
  // A-B: how several forward (march, tile) and reverse (adj_*) steps are launched; steps = 0
  // where a kernel does not apply or is not the fastest.
  MarchPlan march, adj_march;
  TilePlan tile, adj_tile;
  TwoPlan two;  // forward launches of two steps
  int two_rb;   // not 0: the pair kernel takes them (unless recording), over that many row blocks
};

// Where a run's population buffers (both of A-B, the one of AA) stop fitting the 256 MB last-level
// cache well enough for plain accesses to win, us per step plain/streaming: A-B FP32 302 MB 46/48,
// 381 MB 67/62, FP64 324 MB 57/54; AA on rows without padding FP32 326 MB 105/104, 340 MB 111/104,
// FP64 302 MB 92/93, 321 MB 103/102, FP16 302 MB 96/98, 321 MB 118/117. AA's padding lanes keep
// to their own slots while the rest of the group shifts, so padded rows write parts of lines, which
// the caches put together: FP32 358 MB 127/163, 392 MB 140/154, FP64 381 MB 131/122, FP16 348 MB
// 133/133.
constexpr int64_t kStreamBytes = int64_t(304) << 20, kStreamBytesPadded = int64_t(352) << 20;
// Up to here the step's blocks run in XCD order, which keeps a row's neighbours of the previous
// step in the same L2: AA FP32 1000^2 11.7 -> 10.4 us, 2700^2 (267 MB) 68 -> 61, A-B FP32 1700^2
// (212 MB) 27.1 -> 25.2, 2048^2 (302 MB) 40 -> 44. 16-bit storage, whose steps are bound by their
// instructions, gains at small grids alone: BF16 AA 1000^2 (18 MB) 10.5 -> 7.8, FP16 A-B 1000^2
// (37 MB) 10.8 -> 8.6, 1500^2 (83 MB) 16.1 -> 16.9, AA 3000^2 (162 MB) 44 -> 49.
constexpr int64_t kXcdBytes = int64_t(256) << 20, kXcdBytes16 = int64_t(64) << 20;

// State layout at a given time: f_i(x) = buf[swap ? opp(i) : i][x - shift c_i].
struct LayoutSel {
  int shift, swap;
};

constexpr int kReduceBlocks = 1024;  // partial sums of the FP64 invariants

template <class S>
struct Engine {
  using T = typename StorageTraits<S>::T;
  static hipError_t step(const RunDesc& d, int phase, const void* src, void* dst, void* rec, hipStream_t st);
  // ns >= 2 A-B steps in one launch, out of place, by the marching or the tile kernel of the run's
  // plan; rec, when not null, receives the moments of step s at rec + s * rec_slot.
  static hipError_t steps(const RunDesc& d, int ns, const void* src, void* dst, T* rec, int64_t rec_slot,
                          hipStream_t st);
  // Fills the run's plans for the current device (mode: lbm_params.two_step; segment: steps of a
  // recorded run's checkpoint segments, 0: no recording). captured: no plan of single steps alone
  // where lbm_steps_per_launch reports 2 (see lbm_ctx::captured).
  static void plan(RunDesc& d, int mode, int64_t segment, bool captured);
  static hipError_t init(const RunDesc& d, LayoutSel L, void* buf, const double* rho, const double* ux,
                         const double* uy, hipStream_t st);
  static hipError_t get(const RunDesc& d, LayoutSel L, const void* buf, bool out_f64, void* out, hipStream_t st);
  static hipError_t set(const RunDesc& d, LayoutSel L, void* buf, const double* in, hipStream_t st);
  static hipError_t moments(const RunDesc& d, LayoutSel L, const void* buf, bool out_f64, void* rho, void* ux,
                            void* uy, hipStream_t st);
  static hipError_t invariants(const RunDesc& d, LayoutSel L, const void* buf, double* partial, double* result,
                               hipStream_t st);
  static hipError_t seed(const RunDesc& d, LayoutSel L, const void* buf, const T* rhob, const T* uxb,
                         const T* uyb, T* fbar, hipStream_t st);
  static hipError_t fbar_import(const RunDesc& d, const T* dense, T* fbar, hipStream_t st);
  static hipError_t fbar_export(const RunDesc& d, const T* fbar, T* dense, hipStream_t st);
  static hipError_t adjoint_step(const RunDesc& d, const T* fbar_next, T* fbar, const T* rec, hipStream_t st);
  // AA: two reverse steps (fbar^{n+1} -> fbar^{n-1}) over d.adj_rb row blocks; rec_hi holds the
  // records of step n, rec_lo those of step n - 1.
  static hipError_t adjoint_step2(const RunDesc& d, const T* fbar_next, T* fbar, const T* rec_hi, const T* rec_lo,
                                  hipStream_t st);
  // A-B: ns reverse steps in one launch, reverse step s with the moments at rec - s * rec_slot.
  static hipError_t adjoint_march(const RunDesc& d, int ns, const T* fbar_next, T* fbar, const T* rec,
                                  int64_t rec_slot, hipStream_t st);
  static hipError_t adjoint_tile(const RunDesc& d, int ns, const T* fbar_next, T* fbar, const T* rec,
                                 int64_t rec_slot, hipStream_t st);
  static hipError_t ic_adjoint(const RunDesc& d, LayoutSel L, const void* buf0, const T* fbar, T* uxb, T* uyb,
                               hipStream_t st);
};

// Host-side construction of the per-run constants (FP64, rounded once to T).
template <class T>
inline Coef<T> make_coef(const RunDesc& d) {
  Coef<T> k;
  const double th = d.theta;
  k.rho0 = T(d.rho0);
  k.omb = T(1.0 - 1.0 / d.tau);
  k.omb_inv2th2 = T((1.0 - 1.0 / d.tau) / (2.0 * th * th));
  // Per-axis rest factors with r0 + 2 r1 == 1 exactly in T. The product equilibrium carries
  // momentum rho u (r0 + 2 r1) and density excess drho (r0 + 2 r1)^2, so a rounding excess
  // e = r0 + 2 r1 - 1 would scale the momentum field by 1 + e every step (1 + e/tau for LBGK):
  // with FP32 at theta = 1/3, e = 3e-8 and the kinetic energy gains 6e-5 per 1000 steps. The
  // difference that forms the second factor is exact (Sterbenz): 1 - r0 for r0 >= 1/2, and
  // 1 - 2 r1 for 2 r1 >= 1/2.
  if (th <= 0.5) {
    k.r0 = T(1.0 - th);
    k.r1 = (T(1) - k.r0) * T(0.5);
  } else {
    k.r1 = T(0.5 * th);
    k.r0 = T(1) - T(2) * k.r1;
  }
  k.rr0 = T(d.rho0 * double(k.r0));
  k.rr1 = T(d.rho0 * double(k.r1));
  k.inv2th2 = T(1.0 / (2.0 * th * th));
  k.inv4th2 = T(1.0 / (4.0 * th * th));
  k.inv8th2 = T(1.0 / (8.0 * th * th));
  k.a0 = T(th * (1.0 - 3.0 * th));
  k.b0 = T(2.0 * th * (1.0 - th));
  k.c3 = T(1.0 - 3.0 * th);
  // The VJP's theta is that of the rest factors the collision uses, 2 r1 = 1 - r0.
  const double te = 2.0 * double(k.r1);
  k.th = T(te);
  k.c2 = T(1.0 - 2.0 * te);
  k.hc2 = T(0.5 * (1.0 - 2.0 * te));
  k.e0 = T(te * (1.0 - te));
  k.tt2 = T(2.0 * te * te);
  k.omb_inv4th2 = T((1.0 - 1.0 / d.tau) / (4.0 * th * th));
  return k;
}

}  // namespace lbm
