// Host-side choice of how a run's steps are launched: the strips and row blocks of the marching
// kernels (lbm_march.h), the tiles of the LDS kernel (lbm_tile.h), and which of them, or the
// single-step kernel, takes the least time per step on a grid. Plain arithmetic on sizes; no
// device calls.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace lbm {

struct MarchPlan {
  int steps = 0;  // per launch; 0: the kernel does not apply
  int ncol = 0, w = 0, xlast = 0, halo = 0, nrb = 0, waves = 0;
  double us_per_step = 1e30;
};

struct TilePlan {
  int steps = 0;
  int cfg = 0;  // kTileConfigs index
  int tw = 0, th = 0, wrapx = 0, wrapy = 0;
  double us_per_step = 1e30;
};

// Threads and nodes per thread of the tile kernel's instances.
struct TileConfig {
  int threads, nodes;
};
constexpr TileConfig kTileConfigs[] = {{256, 1}, {512, 1}, {1024, 1}, {1024, 2}};
constexpr int kTileConfigCount = 4;
constexpr int kTileWholeSteps = 4096;  // steps per launch where one block holds the whole box

// Costs of the kernels on MI355X in us, by storage type, model and direction; fitted to the
// launch times of 10 000 plans on grids of 64^2 to 1448^2 (FP32, FP64, 16-bit storage, LBGK
// and the complete model, forward, recording and reverse). The fastest plan the model picks is
// within 5 % of the fastest one measured at the median and 12 % at most below 1024^2.
struct CostModel {
  double bytes = 0;      // read and written per node and launch
  double rec_bytes = 0;  // and moments per node and step
  double wave = 0;       // marching and single step: one SIMD's time for a 64-lane collision
  double tile_wave = 0;  // the same inside a tile, LDS accesses included
  double tile_memory = 0;           // bytes per us of a tile's loads and stores
  double march_launch = 0;          // marching: dispatch, the first loads, the last stores
  double march_alone = 0;           // share of a SIMD's cycles that one wavefront issues in
  double march_many = 0;            // and that very many would
  bool march_spread = false;        // three and more wavefronts per SIMD even out over the SIMDs
  double march_memory_alone = 0;    // bytes per us, one wavefront per SIMD: its rows stay close
  double march_memory = 0;          // bytes per us, the halos of the reverse march included
  double single_launch = 0;         // single step: dispatch, first loads, last stores
  double single_issue = 0;          // and the share of a SIMD's cycles it issues in
  double tile_line = 0;             // bytes that a tile's row reads or writes besides its own
  bool tile_uneven = false;         // launches too short for uneven shares of blocks to even out
  int regs[kTileConfigCount] = {};  // vector registers of the tile kernel's instances
  int max_cells = 0;                // largest instance that does not spill
};
constexpr int64_t kEvenNodes = int64_t(1) << 16;  // tiles share steps evenly below
constexpr double kTileLaunch = 4.2;
constexpr double kTileStep = 0.11;     // a step's barrier and LDS latency
constexpr double kTileRound = 0.8;     // a further round of blocks on the same compute unit
constexpr double kTileAlone = 1.12;    // nothing else on the compute unit to fill a block's waits
constexpr double kTileSerial = 1.35;   // blocks one after the other on a compute unit that holds one
constexpr double kCacheBytes = 256e6;  // last-level cache
constexpr double kMemory = 6.5e6;      // bytes per us of the single step

// By bytes per stored value (reverse steps: of the compute type). The wavefront times are vector
// instructions per collision at 2.4 GHz, a quarter of a wavefront per cycle.
inline CostModel cost_model(int bytes, bool bgk, bool adjoint, bool bf16 = false) {
  CostModel c;
  const bool f64 = bytes == 8, half = bytes == 2;
  const double instr = adjoint ? (bgk ? 110 : f64 ? 260 : 200) : f64 ? (bgk ? 120 : 181) : half ? (bgk ? 130 : bf16 ? 150 : 180) : (bgk ? 95 : 145);
  c.wave = instr * 4.0 / 2400.0;
  c.tile_wave = f64 ? (bgk ? 0.19 : 0.25) : half ? (bgk ? 0.19 : 0.23) : (bgk ? 0.135 : 0.17);
  c.tile_memory = adjoint ? 12e6 : half ? 6.5e6 : 9e6;
  c.bytes = 18.0 * bytes;
  c.march_launch = adjoint ? 5.0 : 3.0;
  c.march_alone = adjoint ? 0.7 : f64 ? 0.63 : half && !bf16 ? 0.8 : 0.73;
  c.march_many = adjoint ? 1.0 : f64 ? 0.78 : half ? 1.03 : 0.95;
  c.march_memory = adjoint ? 5.5e6 : half ? (bf16 ? 5.0e6 : 4.6e6) : 4.45e6;
  c.march_memory_alone = adjoint || half ? c.march_memory : f64 ? 4.65e6 : 5.1e6;
  c.march_spread = half;
  c.single_launch = half ? 2.4 : 1.8;
  c.single_issue = half ? 0.69 : 0.6;
  c.rec_bytes = adjoint ? 5.0 * bytes : 0.0;
  const int one = f64 ? 96 : 64, two = f64 ? 128 : adjoint ? 96 : 80;
  c.regs[0] = c.regs[1] = c.regs[2] = one;
  c.regs[3] = two;
  c.max_cells = adjoint && f64 ? 1024 : 2048;
  return c;
}

// ceil of a small non-negative number, without the call into libm that std::ceil is here: lbm_init
// plans in 3 us of host time instead of 8 (with recording 5 instead of 20).
inline double up(double x) {
  const double f = double(int64_t(x));
  return f < x ? f + 1 : f;
}

// Strips of w stored nodes out of `span` (see MarchGeo). False where no strip width works.
inline bool march_strips(int nx, int span, int halo, bool pairs, MarchPlan& p) {
  const int most = span - 2 * halo;
  p.halo = halo;
  if (!pairs || nx % 2 == 0) {
    p.w = most;
    p.ncol = (nx + most - 1) / most;
    p.xlast = (p.ncol - 1) * most;
    return true;
  }
  // Odd width with pairs: the last strip ends at nx, and the one before it keeps its last lane
  // (span - halo - 1 nodes past its first stored one) inside the row.
  if (nx < span - halo) return false;
  for (int w = most; w >= most / 2; w -= 2) {
    const int ncol = std::max(2, (nx + w - 1) / w);
    if (int64_t(ncol - 2) * w + span - halo > nx || nx - w < halo) continue;
    p.w = w;
    p.ncol = ncol;
    p.xlast = nx - w;
    return true;
  }
  return false;
}

// Steps of the next launch when m steps lie ahead. Tiles share them evenly among the launches
// they need, except that on grids too large for the launches to count (even = false) a single step
// left over is a launch of its own: a plan's region for five steps computes as much for three
// (1024^2 FP32, 6 steps as 3 + 3 61 us, as 5 + 1 53). The marching kernel takes as many as it can
// without leaving a single one.
inline int64_t steps_ahead(int64_t m, int march, int tile, bool even = true) {
  if (tile > 0) {
    if (!even && m > tile && m % tile == 1) return tile;
    const int64_t launches = (m + tile - 1) / tile;
    return (m + launches - 1) / launches;
  }
  if (march > 0) return m == march + 1 && march > 2 ? march - 1 : std::min<int64_t>(m, march);
  return 1;
}

// The same where the launches that are left have to be odd or even in number: the call then ends
// in the buffer it started from, or in the other one, whatever the plan. march or tile >= 2; one
// step cannot take an even number of launches.
inline int64_t steps_ahead_parity(int64_t m, int march, int tile, bool odd, bool even = true) {
  const int64_t ns = steps_ahead(m, march, tile, even);
  return ns > 1 && m - ns == int64_t(odd) ? ns - 1 : ns;
}

// Row blocks and steps per launch of least time per step. A SIMD works through its share of the
// strips' row blocks; a block of h rows costs steps * (h + steps - 1) collisions, and more
// wavefronts per SIMD fill more of each other's waits. Fitted to 300 launches from 1000^2 to
// 8192^2 (7 to 9 % off in the mean, the picked plan within 4 % of the fastest one; the largest FP32
// grids are estimated too slow, 89 us per step for 76 at 4096^2 and 328 for 288 at 8192^2): FP16 8192^2
// 388 us per step with two wavefronts per SIMD and two steps, 326 with six and three; BF16 340 and
// 284; FP64 2024^2 40.3 with one wavefront, 38.5 with two; FP32 2048^2 24.4 with three steps, 22.8
// with four; FP32 LBGK 4096^2, bound by memory, 63.6 with one wavefront per SIMD, 72.3 with three.
// horizon: steps come in runs of that many (0: many).
// gain: fewer, longer row blocks and fuller blocks unless others take less than that share of the
// time.
inline MarchPlan plan_march(int nx, int ny, int npl, int halo, int max_steps, int max_waves, int cus, int64_t horizon,
                            const CostModel& cm, double gain = 0.99) {
  MarchPlan best;
  MarchPlan p;
  if (!march_strips(nx, 64 * npl, halo, npl == 2, p)) return best;
  for (int k = 1; k <= 8; ++k) {
    // k strips' row blocks per SIMD, in blocks of max_waves strips or of one.
    for (int waves = max_waves; waves >= 1; waves = waves > 1 ? 1 : 0) {
      const int64_t cols = (int64_t(p.ncol) + waves - 1) / waves;
      const int64_t slots = int64_t(cus) * 4 * k / waves;
      const int64_t nrb = std::min<int64_t>(std::max<int64_t>(1, slots / cols), ny);
      const int64_t rows = (ny + nrb - 1) / nrb;
      const int64_t rounds = (cols * nrb * waves + int64_t(cus) * 4 - 1) / (int64_t(cus) * 4);
      // Time of a launch; `least` where that already exceeds `limit`.
      auto launch = [&](int64_t steps, double limit) {
        const double share = cm.march_spread && rounds > 2 ? double(cols * nrb * waves) / (cus * 4.0) : double(rounds);
        const double rate = cm.march_many - (cm.march_many - cm.march_alone) / double(rounds);
        const double issue = share * double(steps * (rows + steps - 1)) * npl * cm.wave / rate * (waves > 1 ? 1.01 : 1.0);
        // The forward march's halo reads hit the caches; near balance its issue and its accesses
        // delay each other (a norm of order 6), while reverse steps hide one behind the other.
        if (cm.rec_bytes == 0) {
          const double mem = double(nx) * ny * cm.bytes / (rounds < 2 ? cm.march_memory_alone : cm.march_memory);
          const double least = cm.march_launch + std::max({2.0, issue, mem});
          if (least >= limit) return least;
          const double i3 = issue * issue * issue, m3 = mem * mem * mem;
          return cm.march_launch + std::max(2.0, std::cbrt(std::sqrt(i3 * i3 + m3 * m3)));
        }
        const double halo_reads = 64.0 * npl / p.w * double(rows + 2 * (steps - 1)) / double(rows);
        const double mem = double(nx) * ny * (cm.bytes / 2 * (1 + halo_reads) + steps * cm.rec_bytes * halo_reads);
        return cm.march_launch + std::max(issue, mem / cm.march_memory);
      };
      double by_steps[8] = {};
      for (int steps = 2; steps <= max_steps; ++steps) {
        double us;
        if (horizon > 0 && horizon < 64) {
          us = 0;
          for (int64_t m = horizon, ns; m > 0; m -= ns) {
            ns = steps_ahead(m, steps, 0);
            if (!(by_steps[ns] > 0)) by_steps[ns] = launch(ns, 1e30);
            us += by_steps[ns];
          }
          us /= double(horizon);
        } else {
          us = launch(steps, best.us_per_step * gain * steps) / steps;
        }
        if (us < best.us_per_step * gain) {
          best = p;
          best.steps = steps;
          best.nrb = int(nrb);
          best.waves = waves;
          best.us_per_step = us;
        }
      }
    }
  }
  return best;
}

// Blocks of instance c that a compute unit holds at once.
inline int tile_fit(int c, const CostModel& cm) {
  const int by_regs = 512 / cm.regs[c] * 4 * 64 / kTileConfigs[c].threads;
  const int cells = kTileConfigs[c].threads * kTileConfigs[c].nodes;
  return std::max(1, std::min(int(160 * 1024 / (cm.bytes / 2 * (cells + 2))), by_regs));
}

// Time of a launch of ns steps on `tiles` tiles of tw x th nodes, `fit` of them at once on a compute
// unit.
inline double tile_launch_us(int nx, int ny, int cus, int fit, int tiles, int tw, int th, int wx, int wy, int ns,
                             double memory, const CostModel& cm) {
  const int h = ns - 1;
  const double rw = tw + (wx ? 0 : 2 * h), rh = th + (wy ? 0 : 2 * h);
  // Wavefronts of the block (the region shrinks by a row on both sides per step), blocks per
  // compute unit.
  const double wv = up(rw * (wy ? rh : rh - h) / 64.0);
  const double share = double(tiles) / cus, blocks = up(share);
  const double rounds = up(blocks / fit);
  const double per = std::max(up(wv / 4), wv / 4 * (blocks > 2 && !cm.tile_uneven ? share : blocks));
  const double wait = blocks <= 1 ? kTileAlone : fit == 1 ? kTileSerial : 1.0;
  const double region = rw * rh / (double(tw) * th);
  const double line = cm.tile_line / (cm.bytes / 18.0);  // in nodes
  const double mem = double(nx) * ny *
                     (cm.bytes / 2 * (1 + line / tw + region * (1 + line / rw)) + ns * cm.rec_bytes * region) / memory;
  return kTileLaunch + mem + (rounds - 1) * kTileRound + ns * (kTileStep * rounds + cm.tile_wave * per * wait);
}

// Tile shape, instance and steps per launch of least time per step.
inline TilePlan plan_tile(int nx, int ny, int cus, int64_t horizon, const CostModel& cm) {
  TilePlan best;
  const int steps_try[] = {2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32, 48, 64};
  // Records of a segment that do not stay in the last-level cache come from memory, and the
  // marching kernel reads fewer of them twice (gradients, tiles -> march: FP32 1536^2 50 steps 3819
  // -> 3514 us, 1024^2 500 steps 18.2 -> 17.1 ms; in the cache, 1024^2 100 steps: 3440 against
  // 3675).
  const bool spill = double(horizon) * cm.rec_bytes * nx * ny > kCacheBytes;
  const double memory = spill ? std::min(cm.tile_memory, kMemory) : cm.tile_memory;
  for (int c = 0; c < kTileConfigCount; ++c) {
    const int cells = kTileConfigs[c].threads * kTileConfigs[c].nodes;
    if (cells > cm.max_cells) continue;
    int last = 0;  // a short horizon makes several of steps_try the same
    const double side = std::sqrt(double(cells));
    const int fit = tile_fit(c, cm);
    for (int ns : steps_try) {
      int64_t launches = 1, m = ns;
      if (horizon > 0 && horizon < 64) {
        m = horizon;
        launches = (m + ns - 1) / ns;
        ns = int((m + launches - 1) / launches);
        if (ns == last) continue;
        last = ns;
      }
      const int h = ns - 1;
      // No tiles of this many steps can be faster than a launch, its accesses, barriers and
      // collisions of the stored nodes alone.
      const double least = kTileLaunch + double(nx) * ny * (cm.bytes + ns * cm.rec_bytes) / memory +
                           ns * (kTileStep + cm.tile_wave * double(nx) * ny / (256.0 * cus));
      if (least * double(launches) / double(m) >= best.us_per_step * 0.999) continue;
      for (int shape = 0; shape < 9; ++shape) {
        // Shapes: the whole width (0), the whole height (1), else regions of several widths.
        int tw, th, wx = 0, wy = 0;
        if (shape == 0) {
          if (nx > cells) continue;
          wx = 1, tw = nx;
          const int rows = cells / nx;
          if (rows >= ny) wy = 1, th = ny;
          else th = rows - 2 * h;
        } else if (shape == 1) {
          if (ny > cells || cells / ny >= nx) continue;
          wy = 1, th = ny;
          tw = cells / ny - 2 * h;
        } else {
          static const double aspect[] = {0.35, 0.5, 0.7, 1.0, 1.4, 2.0, 2.8};
          const int rw = int(side * aspect[shape - 2]);
          if (rw <= 2 * h) continue;
          tw = std::min(rw - 2 * h, nx);
          th = cells / (tw + 2 * h) - 2 * h;
        }
        if (tw < 1 || th < 1) continue;
        // Even tiles over the box.
        th = std::min(th, ny);
        const int ntx = (nx + tw - 1) / tw, nty = (ny + th - 1) / th;
        tw = (nx + ntx - 1) / ntx;
        th = (ny + nty - 1) / nty;
        const int tiles = ntx * nty;
        const double rw = tw + (wx ? 0 : 2 * h), rh = th + (wy ? 0 : 2 * h);
        if (rw * rh > cells) continue;
        const double us = tile_launch_us(nx, ny, cus, fit, tiles, tw, th, wx, wy, ns, memory, cm) * double(launches) / double(m);
        if (us < best.us_per_step * 0.999) {
          best.steps = ns;
          best.cfg = c;
          best.tw = tw;
          best.th = th;
          best.wrapx = wx;
          best.wrapy = wy;
          best.us_per_step = us;
        }
      }
    }
  }
  // One block that holds the whole box needs no surroundings: any number of steps.
  if (best.wrapx && best.wrapy) best.steps = kTileWholeSteps;
  return best;
}

// Launches of exactly two steps (calls of two, and what longer ones leave over) where the pair
// kernel does not take them: the plan of many steps has tiles for deeper surroundings, and marches
// of 16-bit storage lose two columns per side instead of four. steps = 0 in both and not single: the
// plan of many steps serves as well (to 7 %, which is what the estimates are good for). us per call
// of two by the plan of many steps / by this: FP32 700^2 14.2 / 11.7, 1000^2 24.8 / 17.4; FP16 512^2
// 9.6 / 8.4, 1024^2 21.1 / 18.3, 2048^2 55.6 / 51.8; BF16 768^2 14.9 / 12.7, 2048^2 44.7 / 40.5.
struct TwoPlan {
  MarchPlan march;
  TilePlan tile;
  bool single = false;  // two launches of one step are faster
};
inline double single_step_us(int nx, int ny, int cus, const CostModel& cm);
inline TwoPlan plan_two(int nx, int ny, int npl, int max_waves, int cus, bool march, const TilePlan& many, const CostModel& cost) {
  TwoPlan p;
  const bool half = cost.bytes < 72.0;
  if (!many.steps && !half) return p;
  CostModel cm = cost;
  cm.tile_line = 64.0;
  cm.tile_uneven = true;
  // Fitted to calls of two steps from 128^2 to 1448^2.
  const double scale = double(nx) * ny * cm.bytes < 0.8 * kCacheBytes ? 0.85 : 1.0;
  double now = 1e30;
  if (many.steps) {
    now = 0.5 * scale * tile_launch_us(nx, ny, cus, tile_fit(many.cfg, cm), (nx + many.tw - 1) / many.tw * ((ny + many.th - 1) / many.th),
                                         many.tw, many.th, many.wrapx, many.wrapy, 2, cm.tile_memory, cm);
    p.tile = plan_tile(nx, ny, cus, 2, cm);
    p.tile.us_per_step *= scale;
  }
  if (march) p.march = plan_march(nx, ny, npl, 2, 2, max_waves, cus, 2, cm);
  // 16-bit steps are bound by their instructions, of which surroundings cost more than estimated.
  const double single = std::max(3.3, (half ? 0.95 : 1.05) * single_step_us(nx, ny, cus, cm));
  const double best = std::min({p.march.us_per_step, p.tile.us_per_step, single});
  const bool worth = best < 0.93 * now;
  p.single = worth && single == best;
  if (!worth || p.single || p.march.us_per_step != best) p.march.steps = 0;
  if (!worth || p.single || p.march.steps || p.tile.us_per_step != best) p.tile.steps = 0;
  return p;
}

// Time of a launch of one step.
inline double single_step_us(int nx, int ny, int cus, const CostModel& cm) {
  const double nodes = double(nx) * ny;
  return std::max(2.7, cm.single_launch + nodes * std::max((cm.bytes + cm.rec_bytes) / kMemory, cm.wave / 64.0 / (cus * 4.0) / cm.single_issue));
}

}  // namespace lbm
