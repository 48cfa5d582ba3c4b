"""The host-side launch plans (csrc/lbm_plan.h) over many sizes, without a GPU: a small program
compiled here checks that the marching kernel's strips store every node and that no pair of
nodes straddles the periodic wrap, that the tile kernel's tiles cover the box and their regions
fit the kernel's instance for every number of steps up to the plan's, and that runs of any length
are split into launches that add up to them."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_21242_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lbm_plan.h"
using namespace lbm;
#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf(" fails " #c "\n"); std::exit(1); } } while (0)

static void strips(int nx, int npl) {
  const int span = 64 * npl, halo = 4;
  MarchPlan p;
  if (!march_strips(nx, span, halo, npl == 2, p)) { CHECK(npl == 2 && nx % 2 == 1 && nx < span - halo, "nx %d", nx); return; }
  std::vector<char> stored(nx, 0);
  for (int c = 0; c < p.ncol; ++c) {
    const int x0 = c == p.ncol - 1 ? p.xlast : c * p.w;
    CHECK(p.w <= span - 2 * halo && p.w > 0 && x0 >= 0 && x0 < nx, "nx %d col %d", nx, c);
    for (int l = 0; l < 64; ++l) {
      const int x = x0 - halo + npl * l;
      const int xw = ((x % nx) + nx) % nx;
      CHECK(xw + npl <= nx, "nx %d npl %d col %d lane %d", nx, npl, c, l);
      if (x >= x0 && x < x0 + p.w && x < nx)
        for (int j = 0; j < npl; ++j) stored[xw + j] = 1;
    }
  }
  for (int x = 0; x < nx; ++x) CHECK(stored[x], "nx %d x %d", nx, x);
}

static void plans(int nx, int ny, int64_t horizon) {
  for (int b : {8, 4, 2})
    for (int adj = 0; adj < 2; ++adj) {
      const CostModel cm = cost_model(b, nx % 2, adj);
      const int npl = adj || b == 8 ? 1 : 2;
      const MarchPlan m = plan_march(nx, ny, npl, 4, 4, 4, 256, horizon, cm);
      if (m.steps) {
        CHECK(m.steps >= 2 && m.steps <= 4 && m.nrb >= 1 && m.nrb <= ny && (m.waves == 1 || m.waves == 4), "%d x %d", nx, ny);
        for (int64_t n = 1; n < 40; ++n)
          for (int64_t left = n, s; left > 0; left -= s) {
            s = steps_ahead(left, m.steps, 0);
            CHECK(s >= 1 && s <= m.steps && s <= left && (s > 1 || n == 1 || m.steps == 2), "march steps %ld of %ld", long(s), long(left));
          }
      }
      const TilePlan t = plan_tile(nx, ny, 256, horizon, cm);
      if (!t.steps) continue;
      const int cells = kTileConfigs[t.cfg].threads * kTileConfigs[t.cfg].nodes;
      CHECK(cells <= cm.max_cells && t.tw >= 1 && t.th >= 1 && (!t.wrapx || t.tw == nx) && (!t.wrapy || t.th == ny), "%d x %d", nx, ny);
      for (int64_t n : {1, 2, 3, 7, 11, 63, 64, 65, 200, 10000})
        for (int64_t left = n, s; left > 0; left -= s) {
          s = steps_ahead(left, 0, t.steps);
          CHECK(s >= 1 && s <= t.steps && s <= left, "tile steps %ld of %ld", long(s), long(left));
          const int64_t hx = t.wrapx ? 0 : s - 1, hy = t.wrapy ? 0 : s - 1;
          CHECK((t.tw + 2 * hx) * (t.th + 2 * hy) <= cells, "%d x %d, %ld steps", nx, ny, long(s));
        }
    }
}

int main() {
  for (int nx = 1; nx < 3000; ++nx) strips(nx, 1), strips(nx, 2);
  for (int nx : {1, 2, 3, 5, 31, 64, 65, 100, 123, 124, 125, 200, 255, 512, 777, 1000, 1024, 2041, 2048, 4095, 8192, 40960})
    for (int ny : {1, 2, 3, 7, 64, 100, 200, 513, 1000, 2024, 4096, 8192})
      for (int64_t h : {0, 1, 2, 7, 10, 32, 500}) plans(nx, ny, h);
  std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_plans_cover_the_box_and_fit_the_kernels(tmp_path):
    src = tmp_path / "plan.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
