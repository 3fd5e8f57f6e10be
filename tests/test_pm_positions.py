"""The class-by-class LDS row positions of the parity-major order
(csrc/ee_lanes.hpp: pm_row, make_pm_pos), built for the host and walked as
the sweep kernel walks them: the positions are a permutation of a plane's
rows, every step's two rows are where the walk reads and writes them, and so
are their t, y and glued neighbours."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_03311_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "ee_internal.hpp"
#include "ee_lanes.hpp"
using namespace ee::lanes;

static int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { if (fails < 20) { printf("FAIL line %d ", __LINE__); \
  printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

template <int DIM, int W>
static void walk(const JP& P, int T) {
  const int G = P.G, R = P.R, ly = P.ly, lt = P.lt, half = R / 2;
  std::vector<int> seen((size_t)P.n * R * G, 0);
  const auto at = [&](int r, int t, int y, int w) { return (r * R + pm_row(P, t * ly + y)) * G + w; };
  const int row = (DIM == 2) ? G : ly / 2 * G;  // t + 2 (2D), t + 1 (3D)
  for (int lane = 0; lane < T; ++lane) {
    const LanePM lp = make_lane_pm<DIM, W>(P, lane, T);
    const PmPos pp = make_pm_pos<DIM>(P, lp);
    int step = 0;
    for (int t = lp.t; t < lt; t += lp.dt, ++step) {
      const int r = lp.r0, w = lp.w, p0 = pp.rw + step * pp.step, p1 = p0 + half * G;
      const int t1 = (DIM == 2) ? t + 1 : t;
      CHECK(p0 == at(r, t, lp.y[0], w) && p1 == at(r, t1, lp.y[1], w), "lane %d step %d rows", lane, step);
      if (DIM == 2) {
        CHECK(p1 - row + (t == 0 ? half * G : 0) == at(r, (t + lt - 1) % lt, 0, w), "t - 1");
        CHECK(p0 + row - (t + 2 == lt ? half * G : 0) == at(r, (t + 2) % lt, 0, w), "t + 2");
      } else {
        const int up = row - (t == lt - 1 ? half * G : 0), dn = (t == 0 ? half * G : 0) - row;
        for (int q = 0; q < 2; ++q) {
          const int oth = q ? p0 : p1, y = lp.y[q];
          CHECK(oth + up == at(r, (t + 1) % lt, y, w) && oth + dn == at(r, (t + lt - 1) % lt, y, w), "t -+ 1");
          const int yn = (y & 1) ? (y + 1) % ly : (y + ly - 1) % ly;
          CHECK(oth + pp.yo[q] == at(r, t, yn, w), "lane %d y neighbour of %d", lane, y);
          CHECK(lp.y[q ^ 1] == (y ^ 1), "y pair");
        }
      }
      for (int q = 0; q < 2; ++q) {
        const int tq = q ? t1 : t;
        if (tq <= 1) {
          const int rgl = (tq == 0) ? (r + 1) % P.n : (r + P.n - 1) % P.n;
          CHECK(step == 0 && pp.og[q] == at(rgl, 1 - tq, lp.y[q], w), "lane %d glued row of class %d", lane, q);
        }
        for (int i = 0; i < W; ++i) seen[(size_t)(q ? p1 : p0) + i] += 1;
      }
    }
    CHECK(pp.og[0] >= 0 && pp.og[0] + W <= P.n * R * G && pp.og[1] >= 0 && pp.og[1] + W <= P.n * R * G, "og range");
    CHECK(pp.rw >= 0 && pp.rw + W <= P.n * R * G, "rw range");
  }
  for (size_t i = 0; i < seen.size(); ++i) CHECK(seen[i] == 1, "word %zu visited %d times", i, seen[i]);
}

int main(int argc, char** argv) {
  const int dim = atoi(argv[1]), lt = atoi(argv[2]), lx = atoi(argv[3]), ly = atoi(argv[4]), n = atoi(argv[5]);
  JP P{};
  P.dim = dim; P.n = n; P.lt = lt; P.ly = ly; P.l = 1;
  P.H = lx / 2; P.G = (P.H + 3) / 4; P.G8 = (P.H + 7) >> 3; P.R = lt * ly;
  P.traj_words = 2 * n * P.R * P.G;
  const ee::Magic mr = ee::make_magic((uint32_t)P.R), my = ee::make_magic((uint32_t)ly);
  P.mR = mr.mul; P.sR = mr.shift; P.mLy = my.mul; P.sLy = my.shift;
  int cases = 0;
  for (int T = P.G; T <= 1024; T += (T < 70 ? 1 : 37)) {
    const int W = words_per_lane(P, T);
    if (!use_pm(P, T, W)) continue;
    ++cases;
    const auto go = [&](auto d) {
      constexpr int D = decltype(d)::value;
      if (W == 4) walk<D, 4>(P, T); else if (W == 3) walk<D, 3>(P, T); else if (W == 2) walk<D, 2>(P, T); else walk<D, 1>(P, T);
    };
    if (dim == 2) go(std::integral_constant<int, 2>{}); else go(std::integral_constant<int, 3>{});
  }
  // slots of any size: pm_lanes of them take the rows, the others none
  for (int T = P.G; T <= 1024; T += 29) {
    const int W = words_per_lane(P, T), lanes = pm_lanes(P, T, W);
    CHECK(lanes <= T, "T%d lanes %d", T, lanes);
    CHECK((lanes > 0) || !use_pm(P, T, W), "T%d loses the order", T);
    if (!lanes) continue;
    const auto idle = [&](auto d) {
      constexpr int D = decltype(d)::value;
      for (int lane = lanes; lane < T; ++lane)
        CHECK((W == 4 ? make_lane_pm<D, 4>(P, lane, lanes).t : W == 3 ? make_lane_pm<D, 3>(P, lane, lanes).t
               : W == 2 ? make_lane_pm<D, 2>(P, lane, lanes).t : make_lane_pm<D, 1>(P, lane, lanes).t) >= P.lt,
              "T%d lane %d has rows", T, lane);
      if (W == 4) walk<D, 4>(P, lanes); else if (W == 3) walk<D, 3>(P, lanes);
      else if (W == 2) walk<D, 2>(P, lanes); else walk<D, 1>(P, lanes);
    };
    if (dim == 2) idle(std::integral_constant<int, 2>{}); else idle(std::integral_constant<int, 3>{});
  }
  printf("cases %d fails %d\n", cases, fails);
  return fails || !cases;
}
"""


@pytest.fixture(scope="module")
def walker(tmp_path_factory):
    d = tmp_path_factory.mktemp("pm")
    (d / "walk.cpp").write_text("#include <type_traits>\n" + HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), str(d / "walk.cpp"), "-o", str(d / "walk")], check=True)
    return str(d / "walk")


@pytest.mark.parametrize("shape", [(2, 8, 8, 1, 2), (2, 2, 16, 1, 2), (2, 64, 64, 1, 2), (2, 10, 96, 1, 3),
                                   (2, 24, 24, 1, 2), (3, 8, 8, 2, 2), (3, 32, 32, 32, 2), (3, 24, 24, 24, 2),
                                   (3, 16, 16, 16, 3), (3, 6, 40, 6, 2), (3, 2, 16, 4, 4)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pm_positions(walker, shape):
    r = subprocess.run([walker, *map(str, shape)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
