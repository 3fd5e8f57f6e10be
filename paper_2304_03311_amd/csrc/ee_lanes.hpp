// ee_lanes.hpp -- how the lanes of a sweep workgroup enumerate the rows of a
// trajectory's colour planes (the lane-map and parity-major orders), where a
// row's glued partner across the cut lies, and the launch-shape choices that
// depend on them.  Pure index arithmetic on the job constants, compiled into
// the kernels and, for the tests of the enumeration, into host code.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define EE_HDI __host__ __device__ __forceinline__
#else
#define EE_HDI inline
#endif

namespace ee {
namespace lanes {

// q = n / d for n < 2^31 with (mul, shift) from make_magic: the high word
// of n * mul plus n, shifted (it stays below 2^32 for such n).
EE_HDI uint32_t fdiv(uint32_t n, uint32_t mul, uint32_t shift) {
  return ((uint32_t)(((uint64_t)n * mul) >> 32) + n) >> shift;
}

// Per-job constants, held in scalar registers.
struct JP {
  int dim, n, lt, ly, l, N, S, subsets, whole, H, G, G8, R, traj_words, packed_row_words;
  uint32_t key0, key1, thr0, thr1, thr2, reverse, spin_format;
  uint32_t pt_hi0, pt_hi1, pt_lo0, pt_lo1;  // byte tables of (thr[a] >> 16) ^ 0x8000, a = 0..7
  uint32_t mR, sR, mLy, sLy;
  const uint32_t* ramp;
  uint32_t* spins;
  int64_t* work;
};


// Where a trajectory's words lie in device memory: the word at which its
// colour plane c (rows of G words) starts, to be added to a 64-bit pointer,
// and within a plane a 32-bit byte offset.  A trajectory has fewer than 2^31
// words (int indices) and a plane fewer than 2^30, so such an offset reaches
// every word of a plane; counted from the start of the trajectory it would
// wrap in one of more than 4 GiB.
EE_HDI uint32_t plane_start(int rows, int G, int c) { return c ? (uint32_t)rows * (uint32_t)G : 0u; }
EE_HDI uint32_t plane_byte(int word) { return 4u * (uint32_t)word; }

// Per-lane iteration state of one work unit (the same for every sweep): the
// lane owns words w .. w+W-1 of the rows numbered kstart, kstart + kstep,
// ... below kend; wl / wr are the words left and right of that group
// (periodic in x).  The first row is (r0, t0, y0) at word offset rowbase0;
// each next row is dr replicas, dt time slices and dy rows of y further
// on, step words further in storage; when t wraps, r moves by rinc and the
// offset back by wrapadj.
struct Lane {
  int w, wl, wr;
  int kstart, kstep, kend, rowbase0, step;
  int r0, t0, y0;
  int dr, dt, dy;
  int rinc, wrapadj;
};

// Lane map of the rows of one colour plane (n replicas x R = lt*ly rows of G
// words) over T lanes, GW = G/W lanes per row, S = T/GW row slots.
//  * groups and S >= n: slot s takes replica s / B, B = S/n, and rows k, k+B, ... of
//    that replica in the order rho = (k + 2 ly) mod R, so that the rows
//    next to the cut (t = 0, 1) come last: one iteration of the lane's loop
//    meets them instead of one per replica.
//  * otherwise: slot s takes rows s, s+S, ... of the planes in storage order,
//    as the streaming kernel does: its rows come from HBM through the caches,
//    and it measured 11% faster than in the grouped order.
// The rows of a colour are independent within a half-sweep, so the order
// does not change any result.  Divisions by R and ly use the job's magic
// multipliers.
EE_HDI Lane make_lane(const JP& P, int lt_, int T, int W, bool groups) {
  const int GW = P.G / W;
  const int S = T / GW;
  const int slot = lt_ / GW;
  const auto div_ly = [&](int v) { return (int)fdiv((uint32_t)v, P.mLy, P.sLy); };
  const auto div_R = [&](int v) { return (int)fdiv((uint32_t)v, P.mR, P.sR); };
  Lane ln;
  ln.w = (lt_ - slot * GW) * W;
  ln.wl = (ln.w == 0) ? P.G - 1 : ln.w - 1;
  ln.wr = (ln.w + W == P.G) ? 0 : ln.w + W;
  if (groups && S >= P.n) {
    const int B = S / P.n;
    ln.r0 = slot / B;
    const int k0 = slot - ln.r0 * B;
    ln.kstart = k0;
    ln.kstep = B;
    ln.kend = (ln.r0 < P.n) ? P.R : 0;
    int rho = k0 + 2 * P.ly;
    if (rho >= P.R) rho -= P.R;
    ln.t0 = div_ly(rho);
    ln.y0 = rho - ln.t0 * P.ly;
    ln.rowbase0 = (ln.r0 * P.R + rho) * P.G;
    ln.step = B * P.G;
    const int b = B - div_R(B) * P.R;  // B mod R
    ln.dr = 0;
    ln.dt = div_ly(b);
    ln.dy = b - ln.dt * P.ly;
    ln.rinc = 0;
    ln.wrapadj = P.R * P.G;
  } else {
    ln.kstart = slot;
    ln.kstep = S;
    ln.kend = (slot < S) ? P.n * P.R : 0;
    ln.r0 = div_R(slot);
    const int rho = slot - ln.r0 * P.R;
    ln.t0 = div_ly(rho);
    ln.y0 = rho - ln.t0 * P.ly;
    ln.rowbase0 = slot * P.G;
    ln.step = S * P.G;
    ln.dr = div_R(S);
    const int b = S - ln.dr * P.R;
    ln.dt = div_ly(b);
    ln.dy = b - ln.dt * P.ly;
    ln.rinc = 1;
    ln.wrapadj = 0;
  }
  return ln;
}


// Row (in the lane's own trajectory) of the glued partner across the cut of
// row (r, t, y), t in {0, 1}: replica r+1 at t = 1 for t = 0, replica r-1 at
// t = 0 for t = 1.
EE_HDI int glued_row(const JP& P, int r, int t, int y) {
  const int rgl = (t == 0) ? ((r + 1 == P.n) ? 0 : r + 1) : ((r == 0) ? P.n - 1 : r - 1);
  return rgl * P.R + (1 - t) * P.ly + y;
}

// Byte mask of the glued sites (x < l) of a word whose first site has
// x = l - v: bytes i with 2i < v.
EE_HDI uint32_t glued_mask(int v) {
  const int ng = (v <= 0) ? 0 : ((v + 1) >> 1);
  return (ng >= 4) ? 0xFFFFFFFFu : ((1u << (8 * ng)) - 1u);
}


// gm of the W words from word w on: bit 0 of byte i of word q is set where
// its site, x = 8 (w + q) + 2 i + p, has x < l.  The borrow of a byte-wise
// comparison against the number of such sites.
template <int W>
EE_HDI void glued_bits(const JP& P, bool on, int p, int w, uint32_t gm[W]) {
  int n = (P.l - p - 8 * w + 1) >> 1;  // glued sites from word w on
  n = n < 0 ? 0 : (n > 4 * W ? 4 * W : n);
  const uint32_t v = (uint32_t)(on ? n : 0) * 0x01010101u;
#pragma unroll
  for (int q = 0; q < W; ++q) gm[q] = ((v + (0x7C7D7E7Fu - (uint32_t)q * 0x04040404u)) >> 7) & 0x01010101u;
}

// Word of its lane (0 .. W-1) that holds x = l, the same for every lane, and
// whether the lane's words hold it, in the rows of parity l & 1.  The
// whole-region protocol has no single ramped column.
template <int W>
EE_HDI int ramp_word(const JP& P) { return (W == 3) ? (P.l >> 3) : ((P.l >> 3) & (W - 1)); }
template <int W>
EE_HDI bool ramp_lane(const JP& P, int w) { return !P.whole && w == (P.l >> 3) - ramp_word<W>(P); }

// Parity-major row order (grouped lane map, rows of whole words).  The rows
// (t, y) of a replica fall into two classes by the parity q of t + y, and in
// a half-sweep of colour c the sites of the class-q rows have x parity
// p = c ^ q.  Slot k0 of the B slots of its replica takes the class-q rows
// m = k0, k0 + B, ... below R/2 of both classes, one row of each class per
// step: the lanes of a wave meet rows of one class at a time, so p is a
// compile-time constant of each row's code, and the next rows are a fixed
// stride further on.
//   2D: t = 2m + q, so the class-1 row is the row after the class-0 one.
//   3D, ly dividing B: t = m / (ly/2) and y = 2 (m mod ly/2) + ((t + q) & 1):
//   both rows share t, their y differ in bit 0, and t moves by 2B/ly (even)
//   from step to step, so both y stay fixed per lane.
// The rows of one colour are independent within a half-sweep, so the order
// changes no result.  LanePM holds what is fixed for a work unit: the
// lane's first class-0 row (t, word offset rw, Philox counter word 0, y),
// the offsets d_rw, d_c0 of its class-1 partner, the y of both rows and
// their y-neighbour offsets; dt is the t stride (uniform).
// For the lane's rows next to the cut (if any) it also holds their glued
// rows' word offsets og and the byte masks gm[p] of the glued columns x < l
// of its words for x parity p.  The offsets and masks are those of rows in
// storage order, for the test of the enumeration; the kernel takes its own from
// PmPos and glued_bits, and only r0, w, wl, wr, c3, t, dt, y, c0 and d_c0 from
// here.
struct LanePM {
  int w, wl, wr, r0, dt;
  uint32_t c3;  // Philox counter word 3 without the colour bit
  int t, rw, d_rw;
  uint32_t c0, d_c0;
  int y[2], ymo[2], ypo[2];
  int og[2];
  uint32_t gm[2][4];
};

template <int DIM, int W>
EE_HDI LanePM make_lane_pm(const JP& P, int lt_, int T) {
  const int GW = P.G / W;
  const int slot = lt_ / GW;
  const int B = (T / GW) / P.n;
  LanePM L;
  L.w = (lt_ - slot * GW) * W;
  L.wl = (L.w == 0) ? P.G - 1 : L.w - 1;
  L.wr = (L.w + W == P.G) ? 0 : L.w + W;
  L.r0 = slot / B;
  const int k0 = slot - L.r0 * B;
  L.dt = (DIM == 2) ? 2 * B : (int)fdiv((uint32_t)(2 * B), P.mLy, P.sLy);
  L.c3 = (1u << 28) | ((uint32_t)L.r0 << 1);
  int t, y0, y1;
  if (DIM == 2) {
    t = 2 * k0;
    y0 = y1 = 0;
  } else {
    t = (int)fdiv((uint32_t)(2 * k0), P.mLy, P.sLy);
    y0 = 2 * (k0 - t * (P.ly >> 1)) + (t & 1);
    y1 = y0 ^ 1;
  }
  const int rho0 = t * P.ly + y0;
  const int rho1 = (DIM == 2) ? rho0 + 1 : t * P.ly + y1;
  L.t = (L.r0 < P.n) ? t : P.lt;  // a slot past the last replica has no rows
  L.rw = (L.r0 * P.R + rho0) * P.G + L.w;
  L.d_rw = (rho1 - rho0) * P.G;
  L.c0 = (uint32_t)(rho0 * P.G8 + (L.w >> 1));
  L.d_c0 = (uint32_t)((rho1 - rho0) * P.G8);
  L.y[0] = y0;
  L.y[1] = y1;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    L.ymo[q] = (L.y[q] == 0) ? (P.ly - 1) * P.G : -P.G;
    L.ypo[q] = (L.y[q] == P.ly - 1) ? -(P.ly - 1) * P.G : P.G;
    // the class-q row of the lane's first step (2D: t = q, 3D: t), if next to the cut
    const int tq = (DIM == 2) ? t + q : t;
    L.og[q] = (L.t <= 1) ? glued_row(P, L.r0, tq, L.y[q]) * P.G + L.w : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) L.gm[q][i] = (i < W) ? glued_mask(P.l - q - 8 * (L.w + i)) : 0u;
  }
  return L;
}


// Row positions in LDS in parity-major order.  Lanes with consecutive m read
// rows of one class at a time; with the rows in storage order those are two
// rows apart, and 16-byte accesses at such a stride meet every LDS bank
// twice.  So the rows of a (colour, replica) plane are kept class by class:
// row (t, y) of class q = (t + y) & 1 at position q R/2 + m, with m = t / 2
// in 2D and t ly/2 + y/2 in 3D (the order of the lanes' walk).  Consecutive
// lanes then read consecutive words.  Every neighbour of a class-q row is of
// class q ^ 1:
//   2D: t -+ 1 at m - 1 and m (q = 0) or m and m + 1 (q = 1), m mod lt/2;
//   3D: t -+ 1 at m -+ ly/2; the other row of the y pair at m, the y
//       neighbour outside the pair at m -+ 1 (y even: -, odd: +; periodic in
//       y).
EE_HDI int pm_row(const JP& P, int rho) {
  const int half = P.R >> 1;
  if (P.dim == 2) return (rho & 1) * half + (rho >> 1);
  const int t = (int)fdiv((uint32_t)rho, P.mLy, P.sLy), y = rho - t * P.ly;
  return ((t + y) & 1) * half + t * (P.ly >> 1) + (y >> 1);
}

// Word offsets of a lane's rows in that layout: its first class-0 row (the
// class-1 row of the pair is R/2 rows further on), the step between its
// pairs, the y neighbour outside the pair of the class-q row relative to the
// class-(q^1) row of the pair, and the glued partners' rows of its first step
// (0 where that step is not next to the cut).
struct PmPos {
  int rw, step, yo[2], og[2];
};

template <int DIM>
EE_HDI PmPos make_pm_pos(const JP& P, const LanePM& lp) {
  const int hy = P.ly >> 1;
  const bool in = lp.r0 < P.n;  // a slot past the last replica has no rows
  const int m = !in ? 0 : (DIM == 2) ? (lp.t >> 1) : lp.t * hy + (lp.y[0] >> 1);
  PmPos X;
  X.rw = ((in ? lp.r0 : 0) * P.R + m) * P.G + lp.w;
  X.step = ((DIM == 2) ? (lp.dt >> 1) : lp.dt * hy) * P.G;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int yh = lp.y[q] >> 1;
    X.yo[q] = (DIM == 2) ? 0 : ((lp.y[q] & 1) ? ((yh == hy - 1) ? 1 - hy : 1) : ((yh == 0) ? hy - 1 : -1)) * P.G;
    X.og[q] = 0;
    if (in && lp.t <= 1) {
      const int t = (DIM == 2) ? lp.t + q : lp.t;
      const int rgl = (t == 0) ? ((lp.r0 + 1 == P.n) ? 0 : lp.r0 + 1) : ((lp.r0 == 0) ? P.n - 1 : lp.r0 - 1);
      X.og[q] = (rgl * P.R + pm_row(P, (1 - t) * P.ly + lp.y[q])) * P.G + lp.w;
    }
  }
  return X;
}

// Words per lane for a job and slot size of T lanes.  The widest W <= 4
// that divides the row's words and still gives every row a lane group
// (rows of exactly three words take W = 3) needs the fewest passes of the
// slot's lanes over its row groups; of the W that need as many passes, the
// narrowest is taken: each pass is then a shorter instruction chain, and a
// slot with more lanes than wide row groups (a small, latency-bound
// lattice) spreads its rows over all of its lanes.
EE_HDI int words_per_lane(const JP& P, int T) {
  const int nrows = P.n * P.R;  // rows of one colour of a trajectory
  const auto passes = [&](int W) { return (nrows * (P.G / W) + T - 1) / T; };
  int W = 1;
  if ((P.H & 15) == 0 && T / (P.G / 4) >= 1) W = 4;
  else if (P.H == 12) W = 3;
  else if ((P.H & 7) == 0 && T / (P.G / 2) >= 1) W = 2;
  const int p = passes(W);
  if (W == 4 && passes(2) == p) W = 2;
  if (W > 1 && passes(1) == p) W = 1;
  return W;
}

// Whether the rows of a unit go in parity-major order: the grouped lane map
// (at least one row slot per replica), fewer row slots B per replica than
// rows (else half of them would idle there, while the lane-map order gives
// every row its own lane), and, in 3D, ly dividing B.  Uniform over the
// workgroup.
EE_HDI bool use_pm(const JP& P, int T, int W) {
  const int S = T / (P.G / W);
  if (S < P.n) return false;
  const int B = S / P.n;
  return B < P.R && (P.dim == 2 || B % P.ly == 0);
}

// Lanes of a slot of T that take rows in parity-major order, 0 where the rows
// of the unit go in lane-map order: as use_pm, but where ly does not divide
// the B row slots per replica (3D), as many as it does; the other lanes stay
// idle.  24^3 with 512 lanes: B = 256 -> 240, two steps of two rows per
// half-sweep instead of five single rows in lane-map order.  P.G is the row
// pitch, a multiple of W.
EE_HDI int pm_lanes(const JP& P, int T, int W) {
  const int GW = P.G / W;
  const int S = T / GW;
  if (S < P.n) return 0;
  int B = S / P.n;
  if (P.dim == 3 && B > P.ly) B -= B % P.ly;
  const int lanes = (P.dim == 3) ? B * P.n * GW : T;
  return use_pm(P, lanes, W) ? lanes : 0;
}

// Instructions of a pair of rows (2D, parity-major order) on a lane of W words,
// of the compiled loops.
EE_HDI int step_instr(int W) { return W == 4 ? 300 : W == 3 ? 250 : W == 2 ? 165 : 105; }

// Rows whose words do not split evenly into lanes of several words (lx/2 not
// a multiple of 4, or an odd word count) are kept in LDS at a pitch of a
// multiple of the lane's W words; the last lane of a row then has pad sites,
// which never flip.  W by the instructions of a pair of rows (3 only where a
// row is one lane: its Philox calls serve two words each).  22 sites in x: one
// lane of three words instead of three of one, 250 instructions against 315,
// and one edge.
struct RowPitch {
  int W, pitch;  // words per lane; words per row in LDS, 0: as stored
};
EE_HDI RowPitch row_pitch(int H, int G) {
  const auto cost = [&](int W) { return (G + W - 1) / W * step_instr(W); };
  // what words_per_lane takes for whole rows (1 where lx/2 is no multiple of 4)
  const int plain = (H & 15) == 0 ? 4 : H == 12 ? 3 : (H & 7) == 0 ? 2 : 1;
  if ((H & 3) == 0 && G % plain == 0 && plain > 1) return RowPitch{plain, 0};
  int W = 1;
  for (int v = 2; v <= 4; ++v)
    if ((v != 3 || G <= 3) && cost(v) < cost(W)) W = v;
  if (W == 1 && (H & 3) == 0) return RowPitch{1, 0};
  return RowPitch{W, (G + W - 1) / W * W};
}

// What a lane of W words from word w on of a row with pad sites (H real ones)
// needs beside its offsets.
struct RagLane {
  uint32_t fm[4];    // bit 0 of every real site's byte, per word
  uint32_t e_shift;  // brings the last site of the row to the top byte (first lane; 0 elsewhere)
  uint32_t last;     // 0xFF in the lane that holds the row's last site, 0 elsewhere
  int wl, wr;        // words that hold the left and right edge neighbour
};
template <int W>
EE_HDI RagLane rag_lane(int H, int w) {
  RagLane r;
  const int wl = (H - 1) >> 2;  // word of the row's last site
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int n = H - 4 * (w + q);
    r.fm[q] = (q >= W || n <= 0) ? 0u : 0x01010101u >> (n >= 4 ? 0 : 32 - 8 * n);
  }
  const bool last = wl >= w && wl < w + W;
  r.e_shift = (w == 0) ? 8u * (3 - ((H - 1) & 3)) : 0u;
  r.last = last ? 0xFFu : 0u;
  r.wl = (w == 0) ? wl : w - 1;
  r.wr = last ? 0 : w + W;
  return r;
}

}  // namespace lanes
}  // namespace ee
