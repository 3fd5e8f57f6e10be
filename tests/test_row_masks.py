"""The masks and edge words that the sweep kernel's rows use (csrc/ee_lanes.hpp:
glued_bits, ramp_word, ramp_lane, row_pitch, rag_lane), built for the
host, against the sites' coordinates."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_03311_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include "ee_lanes.hpp"
using namespace ee::lanes;

static int fails = 0, cases = 0;
#define CHECK(c, ...) do { if (!(c)) { if (fails < 20) { printf("FAIL line %d ", __LINE__); \
  printf(__VA_ARGS__); printf("\n"); } ++fails; } } while (0)

template <int W>
static void masks(int lx, int pitch, bool rag) {
  const int H = lx / 2;
  JP P{};
  P.H = H; P.G = pitch;
  for (int l = 0; l <= lx; ++l)
    for (int whole = 0; whole < 2; ++whole) {
      P.l = l; P.whole = whole;
      int owners = 0;
      for (int w = 0; w < pitch; w += W) {
        ++cases;
        const bool own = ramp_lane<W>(P, w);
        owners += own;
        for (int p = 0; p < 2; ++p) {
          uint32_t gm[W], off[W];
          glued_bits<W>(P, true, p, w, gm);
          glued_bits<W>(P, false, p, w, off);
          for (int q = 0; q < W; ++q) {
            CHECK((gm[q] & ~0x01010101u) == 0 && off[q] == 0, "bits outside bit 0, or of a row away from the cut");
            for (int i = 0; i < 4; ++i) {
              const int x = 8 * (w + q) + 2 * i + p;
              const bool in_row = 4 * (w + q) + i < H;
              if (in_row)
                CHECK(((gm[q] >> (8 * i)) & 1) == (x < l), "lx %d l %d W %d word %d site %d: glued", lx, l, W, w + q, x);
              // the ramped site: byte (l >> 1) & 3 of word ramp_word of its lane, in the rows of parity l & 1
              const bool here = own && q == ramp_word<W>(P) && i == ((l >> 1) & 3) && p == (l & 1);
              if (in_row || here) CHECK(here == (!whole && x == l), "lx %d l %d W %d site %d: ramp", lx, l, W, x);
            }
          }
        }
      }
      if (l < lx) CHECK(owners == !whole, "lx %d l %d W %d: %d lanes hold the ramped site", lx, l, W, owners);
    }
  if (!rag) return;
  int lasts = 0;
  for (int w = 0; w < pitch; w += W) {
    const RagLane r = rag_lane<W>(H, w);
    for (int q = 0; q < 4; ++q)
      for (int i = 0; i < 4; ++i)
        CHECK(((r.fm[q] >> (8 * i)) & 0xFF) == (q < W && 4 * (w + q) + i < H), "lx %d W %d word %d byte %d: real", lx, W, w + q, i);
    // left of the lane's first site: the row's last site (first lane), else the site before
    const int left = (w == 0) ? H - 1 : 4 * w - 1;
    CHECK(r.wl == left >> 2 && (int)r.e_shift == (w == 0 ? 8 * (3 - (left & 3)) : 0) && 3 - (int)r.e_shift / 8 == (left & 3),
          "lx %d W %d word %d: left edge", lx, W, w);
    const bool last = 4 * w <= H - 1 && H - 1 < 4 * (w + W);
    lasts += last;
    CHECK(r.last == (last ? 0xFFu : 0u) && r.wr == (last ? 0 : w + W), "lx %d W %d word %d: right edge", lx, W, w);
  }
  CHECK(lasts == 1, "lx %d W %d: %d last lanes", lx, W, lasts);
}

static void any(int W, int lx, int pitch, bool rag) {
  if (W == 4) masks<4>(lx, pitch, rag);
  else if (W == 3) masks<3>(lx, pitch, rag);
  else if (W == 2) masks<2>(lx, pitch, rag);
  else masks<1>(lx, pitch, rag);
}

int main() {
  for (int lx = 2; lx <= 200; lx += 2) {
    const int H = lx / 2, G = (H + 3) / 4;
    const RowPitch rp = row_pitch(H, G);
    if (rp.pitch) {
      CHECK(rp.pitch >= G && rp.pitch < G + rp.W && rp.pitch % rp.W == 0 && (rp.W != 3 || rp.pitch == 3), "lx %d pitch", lx);
      any(rp.W, lx, rp.pitch, true);
    } else {
      CHECK((H & 3) == 0 && (rp.W == 1 || G % rp.W == 0), "lx %d as stored", lx);
    }
    any(1, lx, G, false);
    if ((H & 3) == 0)
      for (int W = 2; W <= 4; ++W)
        if (G % W == 0 && (W != 3 || G == 3)) any(W, lx, G, false);
  }
  printf("cases %d fails %d\n", cases, fails);
  return fails || !cases;
}
"""


def test_masks_and_edges_of_every_row_length(tmp_path):
    (tmp_path / "m.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-I", CSRC, str(tmp_path / "m.cpp"),
                    "-o", str(tmp_path / "m")], check=True)
    r = subprocess.run([str(tmp_path / "m")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
