// ee_kernels.hip -- gfx950 kernels of the non-equilibrium Renyi-entropy
// estimator (Bulgarelli & Panero, arXiv:2304.03311).
//
// sweep_kernel: one workgroup holds k trajectories of one job in LDS
//   (int8 spins, colour-separated rows) and runs, entirely on chip, the
//   initial spins, the thermalisation sweeps and the N protocol sweeps with
//   the integer work (Sec. 3 linear protocol; App. A work-then-update).
//   One lane updates W 32-bit words = 4W same-colour sites of a row.  One
//   Philox4x32-10 call gives a 16-bit field to each of 8 sites; a site
//   accepts when its field is below the top half of its uint32 threshold,
//   and only a tie (probability 2^-16) draws the low 16 bits from a second
//   call.  In batch mode the workgroups are persistent and pull work units
//   (job, block of trajectories) from a device queue.
// estimate_kernel, est_*_kernel: Jarzynski estimator (App. A): integer
//   max/min of I_j, FP64 sum of exp(beta (I_j - I_max)/N), log-sum-exp,
//   delete-one jackknife.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <vector>

#include "ee_dd.hpp"
#include "ee_internal.hpp"
#include "ee_lanes.hpp"
#include "ee_rows.hpp"

namespace {

typedef __attribute__((address_space(3))) uint32_t lds_u32;

__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const lds_u32*)(const uint32_t*)p;
}

// The Metropolis update of the sites of one row of colour c that a lane owns
// (words w .. w+W-1 of the row), parity of the row known only at run time.
//   aC, aO  locations of word w of the row in its own colour plane and in the
//           other one
//   tmo, tpo, ymo, ypo  word offsets from aO of the same words in rows t-1,
//           t+1, y-1 and y+1 (periodic)
//   gmem, ag  where the glued partner row is (CUT; a location that may be
//           read also for rows away from the cut)
//   (r, t, y)  the row; c0, c3 Philox counter words 0 and 3 of its first call
// FULL: lx/2 is a multiple of 4 (no pad bytes, x-neighbours by byte
// alignment of two words).  W: consecutive words per lane (2 or 4 need
// FULL and a word count that W divides; 3 needs FULL and rows of exactly
// three words, so that w = 0 and words 0, 1 share a Philox call while word
// 2 takes the next one).  CUT: the code for rows next to the cut (t = 0, 1)
// is compiled in; without it the row must have t > 1.
template <int DIM, bool FULL, int W, bool CUT, bool LA, typename M, typename GM>
__device__ __forceinline__ void update_row(const JP& P, const PhKey& K, const M& mem, const uint32_t aC,
                                           const uint32_t aO, const GM& gmem, const uint32_t ag, const int w,
                                           const int wl, const int wr, const uint32_t* __restrict__ thr, const int c,
                                           const uint32_t g, const uint32_t j, const int pos, const int dpos,
                                           const bool work, int& dI, const int t, const int y, const int tmo,
                                           const int tpo, const int ymo, const int ypo, const uint32_t c0,
                                           const uint32_t c3, uint32_t* nextU = nullptr) {
  static_assert(W == 1 || ((W == 2 || W == 3 || W == 4) && FULL), "several words per lane need whole rows");
  const int G = P.G;
  const int tailsh = 8 * ((P.H - 1) & 3);
  const uint32_t valid = (!FULL && w == G - 1 && tailsh != 24) ? ((1u << (tailsh + 8)) - 1u) : 0xFFFFFFFFu;
  const uint32_t fmask = valid & 0x01010101u;  // bit 0 of every real site's byte
  const int p = (c + t + y) & 1;               // x parity of this row's sites
  const auto at = [&](int words) { return aO + 4u * (uint32_t)words; };
  uint32_t A[W], B[W], S[1][W], Tm[W], Tp[W], idx[1][W], Sn[1][W];
  CutRow<W> cr[1];
  // towards the cut and away from it, by address: the sum is symmetric
  const int toff0 = (CUT && t == 1) ? tmo : tpo, toff1 = (CUT && t == 1) ? tpo : tmo;
  ld_words<W>(mem, aO, A);
  const uint32_t E = ld_word(mem, at((p ? wr : wl) - w));
  ld_words<W>(mem, aC, S[0]);
  ld_words<W>(mem, at(toff0), Tp);
  ld_words<W>(mem, at(toff1), Tm);
  if constexpr (CUT) ld_words<W>(gmem, ag, cr[0].Tg);
  uint32_t Ym[W], Yp[W];
  if constexpr (DIM == 3) {
    ld_words<W>(mem, at(ymo), Ym);
    ld_words<W>(mem, at(ypo), Yp);
  } else {
#pragma unroll
    for (int q = 0; q < W; ++q) Ym[q] = Yp[q] = 0;
  }
  // LA (lookahead): K is the keys of the next half-sweep; this row's Philox
  // outputs come in nextU, computed during the previous half-sweep, and the
  // next ones replace them.  They do not depend on spins, so that chain
  // overlaps this row's loads and decisions instead of lengthening the next
  // half-sweep.
  constexpr int NC = (W + 1) / 2;
  uint32_t U[NC][4], Un[NC][4];
  fields_of_row<W>(K, c0, Un);
#pragma unroll
  for (int k = 0; k < NC; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      U[k][e] = LA ? nextU[4 * k + e] : Un[k][e];
      if (LA) nextU[4 * k + e] = Un[k][e];
    }
  if constexpr (CUT) {
    cr[0].on = t <= 1;
    cr[0].p = p;
    cr[0].y = y;
    cr[0].ramp = cr[0].on && p == (P.l & 1) && ramp_lane<W>(P, w);
#pragma unroll
    for (int q = 0; q < W; ++q) cr[0].Tc[q] = Tp[q];
    uint32_t gm[W];
    glued_bits<W>(P, cr[0].on && !P.whole, p, w, gm);
    cut_partner<W>(cr[0], gm, Tp);
  }
  if (FULL) {
    x_words<W, -1>(A, E, p, B);
  } else {
    const uint32_t rshift = (w == G - 1) ? (uint32_t)tailsh : 24u;
    const uint32_t Br = (A[0] >> 8) | ((E & 0xFFu) << rshift);
    const uint32_t Bl = (A[0] << 8) | ((w == 0) ? ((E >> tailsh) & 0xFFu) : (E >> 24));
    B[0] = p ? Br : Bl;
  }
#pragma unroll
  for (int q = 0; q < W; ++q) idx[0][q] = nbr_index<DIM>(S[0][q], A[q], B[q], Tm[q], Tp[q], Ym[q], Yp[q]);
  uint32_t fm[W];
#pragma unroll
  for (int q = 0; q < W; ++q) fm[q] = fmask;
  decide_rows<DIM, W, 1, CUT>(P, U, &c0, c3, g, j, w, fm, thr, S, idx, cr, pos, dpos, work, dI, Sn,
                              [&](int, uint32_t* Tc, uint32_t* Tg) {
                                ld_words<W>(mem, at(toff0), Tc);
                                ld_words<W>(gmem, ag, Tg);
                              });
  st_words<W>(mem, aC, Sn[0]);
}

// One half-sweep of colour c over the lane's rows of one trajectory, in the
// order of the lane map (any map; the streaming path's and the general
// on-chip one).  base: location of the trajectory (two colour planes).
template <int DIM, bool FULL, int W, typename M>
__device__ __forceinline__ void half_sweep(const JP& P, PhKey& K, const Lane& ln, const M& mem, const uint32_t base,
                                           const uint32_t* __restrict__ thr, const int c, const uint32_t g,
                                           const uint32_t j, const int pos, const int dpos, const bool work, int& dI) {
  const int G = P.G;
  const int cw = P.n * P.R * G;  // words per colour plane
  const uint32_t bC = base + 4u * (uint32_t)(c * cw), bO = base + 4u * (uint32_t)((c ^ 1) * cw);
  const int LyG = P.ly * G;
  const int ltLyG = P.lt * LyG;
  const int ywrap = (P.ly - 1) * G;
  const uint32_t ctr3 = (1u << 28) | (uint32_t)c;
  const int w = ln.w;
  int r = ln.r0, t = ln.t0, y = ln.y0;
  int rowbase = ln.rowbase0;
  for (int kk = ln.kstart; kk < ln.kend; kk += ln.kstep) {
    // the periodic wrap in t adds or removes one replica's rows; the one
    // below t = 0 belongs to a row next to the cut (cut variant only)
    const int tpo = LyG - ((t == P.lt - 1) ? ltLyG : 0);
    const int ymo = (y == 0) ? ywrap : -G;
    const int ypo = (y == P.ly - 1) ? -ywrap : G;
    const uint32_t c0 = (uint32_t)((t * P.ly + y) * P.G8 + (w >> 1));
    const uint32_t c3 = ctr3 | ((uint32_t)r << 1);
    K.x0 = c3 ^ P.key1;
    const uint32_t off = 4u * (uint32_t)(rowbase + w);
    const auto row = [&](auto cut) {
      constexpr bool CUT = decltype(cut)::value;
      const int tmo = -LyG + ((CUT && t == 0) ? ltLyG : 0);
      const uint32_t ag = (CUT && t <= 1) ? bO + 4u * (uint32_t)(glued_row(P, r, t, y) * G + w) : bO + off;
      update_row<DIM, FULL, W, CUT, false>(P, K, mem, bC + off, bO + off, mem, ag, w, ln.wl, ln.wr, thr, c, g, j, pos,
                                           dpos, work, dI, t, y, tmo, tpo, ymo, ypo, c0, c3);
    };
    // the code for rows next to the cut runs only where some lane of the
    // wave has such a row
    if (__builtin_amdgcn_ballot_w64(t <= 1) != 0) row(std::true_type{});
    else row(std::false_type{});
    // next row of this lane
    rowbase += ln.step;
    if (DIM == 3) {
      y += ln.dy;
      if (y >= P.ly) { y -= P.ly; ++t; }
    }
    t += ln.dt;
    if (t >= P.lt) {
      t -= P.lt;
      r += ln.rinc;
      rowbase -= ln.wrapadj;
    }
    r += ln.dr;
  }
}

// half_sweep for lanes that own at most one row (small, latency-bound
// lattices): the row's Philox outputs U were computed during the previous
// half-sweep, and this one computes those of the next (keys Kn) into U.
template <int DIM, bool FULL, int W>
__device__ __forceinline__ void half_sweep_la(const JP& P, const Lane& ln, const uint32_t base,
                                              const uint32_t* __restrict__ thr, const int c, const uint32_t g,
                                              const uint32_t j, const int pos, const int dpos, const bool work, int& dI,
                                              uint32_t* U, const PhKey& Kn) {
  if (ln.kstart >= ln.kend) return;
  const LdsMem mem;
  const int G = P.G;
  const int cw = P.n * P.R * G;  // words per colour plane
  const uint32_t bC = base + 4u * (uint32_t)(c * cw), bO = base + 4u * (uint32_t)((c ^ 1) * cw);
  const int LyG = P.ly * G;
  const int ltLyG = P.lt * LyG;
  const int ywrap = (P.ly - 1) * G;
  const int w = ln.w, r = ln.r0, t = ln.t0, y = ln.y0;
  const int tpo = LyG - ((t == P.lt - 1) ? ltLyG : 0);
  const int ymo = (y == 0) ? ywrap : -G;
  const int ypo = (y == P.ly - 1) ? -ywrap : G;
  const uint32_t off = 4u * (uint32_t)(ln.rowbase0 + w);
  const uint32_t c0 = (uint32_t)((t * P.ly + y) * P.G8 + (w >> 1));
  const uint32_t c3 = (1u << 28) | ((uint32_t)r << 1) | (uint32_t)c;
  const auto row = [&](auto cut) {
    constexpr bool CUT = decltype(cut)::value;
    const int tmo = -LyG + ((CUT && t == 0) ? ltLyG : 0);
    const uint32_t ag = (CUT && t <= 1) ? bO + 4u * (uint32_t)(glued_row(P, r, t, y) * G + w) : bO + off;
    update_row<DIM, FULL, W, CUT, true>(P, Kn, mem, bC + off, bO + off, mem, ag, w, ln.wl, ln.wr, thr, c, g, j, pos,
                                        dpos, work, dI, t, y, tmo, tpo, ymo, ypo, c0, c3, U);
  };
  if (__builtin_amdgcn_ballot_w64(t <= 1) != 0) row(std::true_type{});
  else row(std::false_type{});
}

// Word left of (p = 0) or right of (p = 1) the lane's W words of a row that is
// one lane or an aligned pair of lanes wide (GW = 1, 2): from the lane's or
// its neighbour's registers.
template <int W, int PAR, int GW>
__device__ __forceinline__ uint32_t edge_word(const uint32_t A[W]) {
  if constexpr (GW == 1) return PAR ? A[0] : A[W - 1];
  return __builtin_amdgcn_mov_dpp(PAR ? A[0] : A[W - 1], 0xB1, 0xF, 0xF, true);  // quad_perm [1, 0, 3, 2]: lane ^ 1
}

// Rows of colour C of the lane in parity-major order: class 0 (x parity C)
// and class 1 (x parity C ^ 1) together in each step.  The two rows are
// neighbours of each other (2D: t and t + 1; 3D: the two y of a pair), so
// each one's words of the other colour serve both, and their two to four
// Philox calls run side by side.  The rows lie in LDS class by class
// (PmPos), which makes every access of a wave consecutive.
// Bound by VALU issue: 280 instructions for the 32 sites of a step (bulk, 2D;
// 298 in 3D), of which 148 are the four Philox calls.  Measured against one
// row at a time with scalar keys and the rows in storage order: 2D 64x64, 64
// jobs x 1024 trajectories 151 against 177 ms (10.6 against 12.3
// instructions per attempt), 3D 32^3 x 512 trajectories 21.4 against 25.1 ms.
// has_cut: some lane of the wave starts with rows next to the cut.  cut_mask:
// the lane's glued_bits in its rows next to the cut (0 if it has none), of
// word q and x parity p moved to bit 4 p + q of each byte.  has_ramp: these
// rows hold the ramped site.
// RAG: rows with pad sites (row_pitch; P.G is the pitch), whose lanes have
// what RagLane says.
struct RagLane {
  uint32_t fm[4];    // bit 0 of every real site's byte, per word
  uint32_t e_shift;  // brings the last site of the row to the top byte (first lane; 0 elsewhere)
  uint32_t last;     // 0xFF in the lane that holds the row's last site, 0 elsewhere
  int wl, wr;        // words that hold the left and right edge neighbour
};
template <int W>
__device__ __forceinline__ RagLane rag_lane(int H, int w) {
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

template <int DIM, int W, int GW, int C, bool RAG = false>
__device__ __forceinline__ void rows_pm(const JP& P, PhKey& K, const LanePM& lp, const PmPos& pp, const RagLane& rl,
                                        const uint32_t base,
                                        const uint32_t* __restrict__ thr, const uint32_t ones, const uint32_t g,
                                        const uint32_t j, const int pos, const int dpos, const bool work, int& dI,
                                        const bool has_cut, const uint32_t cut_mask, const bool has_ramp) {
  const LdsMem mem;
  const int cw4 = 4 * P.n * P.R * P.G;           // bytes per colour plane
  const int d4 = 2 * P.R * P.G;                  // class-0 row to class-1 row
  const int row4 = (DIM == 2) ? 4 * P.G : 2 * P.ly * P.G;  // m to the m of t + 2 (2D), t + 1 (3D)
  const int wrap4 = d4;
  const uint32_t da = 4u * (uint32_t)pp.step;
  const uint32_t dc0 = (uint32_t)(lp.dt * P.ly * P.G8);
  const uint32_t c3 = lp.c3 | (uint32_t)C;
  K.x0 = c3 ^ P.key1;
  const uint32_t bO = base + (uint32_t)(C ? 0 : cw4);
  const int wl = RAG ? rl.wl : lp.wl, wr = RAG ? rl.wr : lp.wr;
  const int e0 = 4 * ((C ? wr : wl) - lp.w), e1 = 4 * ((C ? wl : wr) - lp.w);
  uint32_t fm[W];
#pragma unroll
  for (int q = 0; q < W; ++q) fm[q] = RAG ? rl.fm[q] : ones;
  // x neighbours of a row of parity p
  const auto x_row = [&](auto par, const uint32_t A[W], uint32_t E, uint32_t B[W]) {
    constexpr int PAR = decltype(par)::value;
    if constexpr (!RAG) {
      x_words<W, PAR>(A, E, PAR, B);
    } else {
      // E: a word whose top byte (p = 0, after the shift) is the left
      // neighbour of the first site, or whose bottom byte is the right one of
      // the last site: beyond the last real site of the row it takes the place
      // of the pad byte
      uint32_t A2[W];
#pragma unroll
      for (int q = 0; q < W; ++q) A2[q] = A[q];
      if (GW == 1) {
        uint32_t Ew = A[0];
#pragma unroll
        for (int q = 1; q < W; ++q)
          if (PAR == 0 && q == ((P.H - 1) >> 2)) Ew = A[q];
        E = Ew;
      }
      if (PAR == 0) {
        E <<= rl.e_shift;
      } else {
        const uint32_t in = (E & rl.last) << (8 * (P.H & 3));
#pragma unroll
        for (int q = 0; q < W; ++q)
          if (q == ((P.H >> 2) & (W == 3 ? 3 : W - 1))) A2[q] |= in;
      }
      x_words<W, PAR>(A2, E, PAR, B);
    }
  };
  // The two row locations and the counter are opaque to the compiler at each
  // step (the empty asm statement emits nothing): every access is then one
  // register plus at most one offset, instead of one induction variable per
  // access, and nothing of the first step is carried over from sweep to sweep
  // (in registers that the loop lacks).
  uint32_t aO = bO + 4u * (uint32_t)pp.rw;
  uint32_t aC = aO + (uint32_t)(C ? cw4 : -cw4);
  uint32_t c0 = lp.c0;
  int t = lp.t;
  const auto step = [&](auto cut) {
    constexpr bool CUT = decltype(cut)::value;
    asm volatile("" : "+v"(aC), "+v"(aO), "+v"(c0));
    uint32_t A0[W], A1[W], B0[W], B1[W], S[2][W], idx[2][W], Sn[2][W];
    const uint32_t cc[2] = {c0, c0 + lp.d_c0};
    uint32_t U[2 * ((W + 1) / 2)][4], E0, E1;
    CutRow<W> cr[2];
    const uint32_t aO1 = aO + (uint32_t)d4, aC1 = aC + (uint32_t)d4;
    // What only the cut needs is made anew from values that the compiler
    // cannot see through: hoisted out of the sweep loop it would take
    // registers from every step.
    int w = lp.w, og0 = pp.og[0], og1 = pp.og[1];
    if constexpr (CUT) {
      asm volatile("" : "+v"(w), "+v"(og0), "+v"(og1));
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        cr[r].on = t <= 1;
        cr[r].p = C ^ r;
        cr[r].y = lp.y[r];
        cr[r].ramp = has_ramp && cr[r].p == (P.l & 1);
      }
    }
    // 2D: rows t (even) and t + 1.  3D: both rows at t; towards the cut
    // (t + 1 for t = 0, t - 1 for t = 1) and away from it by address.  The
    // wrap below t = 0 belongs to a row next to the cut, so only the cut
    // variant has it.
    const uint32_t up = (uint32_t)(row4 - ((DIM == 3 && t == P.lt - 1) ? wrap4 : 0));
    const uint32_t dn = (uint32_t)(((CUT && t == 0) ? wrap4 : 0) - row4);
    const uint32_t tc = (CUT && t == 1) ? dn : up, ta = (CUT && t == 1) ? up : dn;
    const uint32_t tp = (uint32_t)(row4 - ((DIM == 2 && t + 2 == P.lt) ? wrap4 : 0));
    // Row 0: its words are loaded, its Philox outputs made while they
    // arrive, then they are summed; then the same for row 1.  (All loads
    // first, for both rows, took too many registers: the spills cost more
    // than the one latency saved.)
    uint32_t T0[W], T1[W], Y[W];
    ld_words<W>(mem, aO, A0);
    ld_words<W>(mem, aO1, A1);
    ld_words<W>(mem, aC, S[0]);
    if constexpr (CUT) ld_words<W>(mem, bO + 4u * (uint32_t)og0, cr[0].Tg);
    if constexpr (DIM == 2) {
      ld_words<W>(mem, aO1 + dn, T0);  // t - 1
    } else {
      ld_words<W>(mem, aO1 + tc, T1);
      ld_words<W>(mem, aO1 + ta, T0);
      ld_words<W>(mem, aO1 + 4u * (uint32_t)pp.yo[0], Y);
    }
    if constexpr (GW == 0) { E0 = ld_word(mem, aO + (uint32_t)e0); E1 = ld_word(mem, aO1 + (uint32_t)e1); }
    fields_of_row<W>(K, cc[0], U);
    if constexpr (GW != 0 && !RAG) { E0 = edge_word<W, C, GW>(A0); E1 = edge_word<W, C ^ 1, GW>(A1); }
    x_row(std::integral_constant<int, C>{}, A0, E0, B0);
    if constexpr (DIM == 2) {
#pragma unroll
      for (int q = 0; q < W; ++q) T1[q] = A1[q];
    }
    if constexpr (CUT) {
#pragma unroll
      for (int q = 0; q < W; ++q) cr[0].Tc[q] = T1[q];
      uint32_t gm[W];
#pragma unroll
      for (int q = 0; q < W; ++q) gm[q] = cut_mask >> (4 * cr[0].p + q);
      cut_partner<W>(cr[0], gm, T1);
    }
#pragma unroll
    for (int q = 0; q < W; ++q) idx[0][q] = nbr_index<DIM>(S[0][q], A0[q], B0[q], T0[q], T1[q], A1[q], Y[q]);
    ld_words<W>(mem, aC1, S[1]);
    if constexpr (CUT) ld_words<W>(mem, bO + 4u * (uint32_t)og1, cr[1].Tg);
    if constexpr (DIM == 2) {
      ld_words<W>(mem, aO + tp, T0);  // t + 2
    } else {
      ld_words<W>(mem, aO + tc, T1);
      ld_words<W>(mem, aO + ta, T0);
      ld_words<W>(mem, aO + 4u * (uint32_t)pp.yo[1], Y);
    }
    fields_of_row<W>(K, cc[1], U + (W + 1) / 2);
    x_row(std::integral_constant<int, C ^ 1>{}, A1, E1, B1);
    if constexpr (DIM == 2) {
#pragma unroll
      for (int q = 0; q < W; ++q) T1[q] = A0[q];
    }
    if constexpr (CUT) {
#pragma unroll
      for (int q = 0; q < W; ++q) cr[1].Tc[q] = T1[q];
      uint32_t gm[W];
#pragma unroll
      for (int q = 0; q < W; ++q) gm[q] = cut_mask >> (4 * cr[1].p + q);
      cut_partner<W>(cr[1], gm, T1);
    }
#pragma unroll
    for (int q = 0; q < W; ++q) idx[1][q] = nbr_index<DIM>(S[1][q], A1[q], B1[q], T0[q], T1[q], A0[q], Y[q]);
    decide_rows<DIM, W, 2, CUT>(P, U, cc, c3, g, j, w, fm, thr, S, idx, cr, pos, dpos, work, dI, Sn,
                                [&](int r, uint32_t* Tc, uint32_t* Tg) {
                                  ld_words<W>(mem, (r ? aO : aO1) + ((DIM == 3) ? tc : 0u), Tc);
                                  ld_words<W>(mem, bO + 4u * (uint32_t)(r ? og1 : og0), Tg);
                                });
    st_words<W>(mem, aC, Sn[0]);
    st_words<W>(mem, aC1, Sn[1]);
    t += lp.dt;
    aC += da;
    aO += da;
    c0 += dc0;
  };
  // Rows next to the cut are met in the first step only (t grows); outside
  // the loop, what that step needs does not weigh on the others.
  if (has_cut && t < P.lt) step(std::true_type{});
  while (t < P.lt) step(std::false_type{});
}

// Initial spins (phase 0 of the Philox streams): +1 iff u < 2^31.  PM: into
// the class-by-class rows of the parity-major order, pitch words each.
template <bool PM, typename M>
__device__ void init_spins(const JP& P, const M& mem, uint32_t base, uint32_t j, int lt_, int T, int pitch) {
  const int nR = P.n * P.R;
  for (int q = lt_; q < P.traj_words; q += T) {
    const int w = q % P.G;
    const int rowg = q / P.G;
    const int c = rowg / nR;
    const int row = rowg - c * nR;
    const int r = row / P.R;
    const int rho = row - r * P.R;
    uint32_t u[4];
    philox10((uint32_t)(rho * P.G + w), 0u, j, ((uint32_t)r << 1) | (uint32_t)c, P.key0, P.key1, u);
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * w + i < P.H) word |= (uint32_t)(u[i] < 0x80000000u) << (8 * i);
    const int at = PM ? (rowg - rho + pm_row(P, rho)) * pitch + w : q;
    st_words<1>(mem, base + 4u * (uint32_t)at, &word);
  }
}

// Row (over colours and replicas) rowg of the storage order in LDS.
template <bool PM>
__device__ __forceinline__ int lds_row(const JP& P, int rowg) {
  if (!PM) return rowg;
  const int rho = rowg - (int)fdiv((uint32_t)rowg, P.mR, P.sR) * P.R;
  return rowg - rho + pm_row(P, rho);
}

template <bool PM>
__device__ void load_spins(const JP& P, uint32_t base, uint32_t j, int lt_, int T, int pitch) {
  const LdsMem mem;
  const bool int8 = P.spin_format == EE_SPINS_INT8;
  const int PW = P.packed_row_words;
  const uint32_t* src = P.spins + (size_t)j * (int8 ? P.traj_words : 2 * P.n * P.R * PW);
  for (int q = lt_; q < P.traj_words; q += T) {
    const int rowg = q / P.G;
    const int w = q - rowg * P.G;
    uint32_t word;
    if (int8) {
      word = src[q];
    } else {
      const uint32_t nib = (src[rowg * PW + (w >> 3)] >> (4 * (w & 7))) & 0xFu;
      word = (nib * 0x00204081u) & 0x01010101u;  // 4 bits -> 4 bytes
    }
    st_words<1>(mem, base + 4u * (uint32_t)(lds_row<PM>(P, rowg) * pitch + w), &word);
  }
}

template <bool PM>
__device__ void store_spins(const JP& P, uint32_t base, uint32_t j, int lt_, int T, int pitch) {
  const LdsMem mem;
  if (P.spin_format == EE_SPINS_INT8) {
    uint32_t* dst = P.spins + (size_t)j * P.traj_words;
    for (int q = lt_; q < P.traj_words; q += T) {
      const int rowg = q / P.G;
      dst[q] = ld_word(mem, base + 4u * (uint32_t)(lds_row<PM>(P, rowg) * pitch + q - rowg * P.G));
    }
  } else {
    const int PW = P.packed_row_words;
    const int total = 2 * P.n * P.R * PW;
    uint32_t* dst = P.spins + (size_t)j * total;
    for (int q = lt_; q < total; q += T) {
      const int rowg = q / PW;
      const int wb = q - rowg * PW;
      const uint32_t row = base + 4u * (uint32_t)(lds_row<PM>(P, rowg) * pitch);
      uint32_t packed = 0;
      for (int k = 0; k < 8; ++k) {
        const int w = 8 * wb + k;
        if (w < P.G) packed |= (((ld_word(mem, row + 4u * (uint32_t)w) * 0x01020408u) >> 24) & 0xFu) << (4 * k);
      }
      dst[q] = packed;
    }
  }
}

// Words (from the end of the trajectory slots) of the workgroup's small
// tables in dynamic LDS: unit index, per-slot work sums, threshold table.
constexpr int kTabUnit = 0, kTabWork = 4, kTabThr = 4 + ee::kMaxSlots;

// All sweeps of one work unit: cnt trajectories of one job, one per LDS slot
// of T lanes.  PM: the rows in parity-major order (rows_pm; GW as in
// edge_word) over pm of the lanes, else in the order of the lane map.  A function of its own (one call per unit, which
// lives for milliseconds): its registers are allocated for this variant
// alone.  Inlined into one kernel, the variants' uniform values shared 100
// scalar registers and 1250 of them were spilled.
template <int DIM, bool FULL, int W, bool PM, int GW = 0, bool RAG = false>
__device__ __noinline__ void run_unit(const JobDev* J_, uint32_t lds, uint32_t tab, int T_, int pm_, int j0_,
                                      int cnt_, uint32_t flags_, int n_therm_, int g0_) {
  static_assert(!PM || FULL || RAG, "the parity-major order needs rows of whole words");
  const JobDev* const J = uni_ptr(J_);
  const JP P = load_jp(J);
  const int pitch = RAG ? uni(J->rag_pitch) : P.G;
  const int slot_words = uni(J->lds_words);
  JP PP = P;  // the rows as they lie in LDS
  PP.G = pitch;
  const int T = uni(T_), j0 = uni(j0_), cnt = uni(cnt_), n_therm = uni(n_therm_);
  const uint32_t flags = uni(flags_);
  lds = uni(lds);
  tab = uni(tab);
  const LdsMem mem;
  int* const s_dI = (int*)mem.at<int>(tab + 4u * kTabWork);
  uint32_t* const s_thr = (uint32_t*)mem.at<uint32_t>(tab + 4u * kTabThr);
  const int tid = threadIdx.x;
  const int slot = tid / T;
  const int lt_ = tid - slot * T;
  const bool active = slot < cnt;
  const uint32_t L = lds + 4u * (uint32_t)(slot * slot_words);
  // one trajectory per wave or more: its index is uniform
  const uint32_t j = ((T & 63) == 0) ? uni((uint32_t)(j0 + slot)) : (uint32_t)(j0 + slot);
  if (tid < ee::kMaxSlots) s_dI[tid] = 0;
  if (tid < 8) s_thr[tid] = thr_entry(P, DIM, tid);
  if (active) {
    if (pitch != P.G) {  // the pad words
      const uint32_t zero = 0;
      for (int q = lt_; q < 2 * P.n * P.R * pitch; q += T) st_words<1>(mem, L + 4u * (uint32_t)q, &zero);
    }
  }
  if (pitch != P.G) __syncthreads();
  if (active) {
    if (flags & ee::kFlagInit) init_spins<PM>(P, mem, L, j, lt_, T, pitch);
    else load_spins<PM>(P, L, j, lt_, T, pitch);
  }
  PhKey K;
  key_unit(K, P);
  const uint32_t ones = in_vgpr(0x01010101u);
  __syncthreads();

  int dI = 0;
  uint32_t g = (uint32_t)uni(g0_);
  const int pos0 = P.reverse ? P.N : 0;
  // n_therm sweeps at the starting position, then (protocol) the N sweeps
  // k = 0 .. N-1 at positions k+1 (forward) or N-1-k (reverse); the work
  // is taken at the colour-0 half of each protocol sweep.
  const bool proto = (flags & ee::kFlagProto) != 0;
  const int n_sweeps = n_therm + (proto ? P.N : 0);
  const int dpos_p = P.reverse ? -1 : 1;
  const auto sweeps = [&](auto half) {
    for (int s = 0; s < n_sweeps; ++s, ++g) {
      const int k = s - n_therm;
      const bool in_proto = k >= 0;
      const int pos = in_proto ? (P.reverse ? P.N - 1 - k : k + 1) : pos0;
      half(pos, in_proto ? dpos_p : 0, in_proto);
    }
  };
  if constexpr (PM) {
    LanePM lp = make_lane_pm<DIM, W>(PP, lt_, uni(pm_));
    const bool has_cut = __builtin_amdgcn_ballot_w64(lp.t <= 1) != 0;
    const PmPos pp = make_pm_pos<DIM>(PP, lp);
    const RagLane rl = RAG ? rag_lane<W>(P.H, lp.w) : RagLane{};
    uint32_t cut_mask = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      uint32_t gm[W];
      glued_bits<W>(P, lp.t <= 1 && !P.whole, p, lp.w, gm);
#pragma unroll
      for (int q = 0; q < W; ++q) cut_mask |= gm[q] << (4 * p + q);
    }
    const bool has_ramp = lp.t <= 1 && ramp_lane<W>(P, lp.w);
    if (!active) lp.t = P.lt;  // no rows
    sweeps([&](int pos, int dpos, bool in_proto) {
      key_sweep(K, P, g, j);
      rows_pm<DIM, W, GW, 0, RAG>(PP, K, lp, pp, rl, L, s_thr, ones, g, j, pos, dpos, in_proto, dI, has_cut, cut_mask, has_ramp);
      __syncthreads();
      rows_pm<DIM, W, GW, 1, RAG>(PP, K, lp, pp, rl, L, s_thr, ones, g, j, pos, dpos, false, dI, has_cut, cut_mask, has_ramp);
      __syncthreads();
    });
  } else {
    const Lane ln = make_lane(P, lt_, T, W, true);
    const bool on = active && ln.kstart < ln.kend;
    // Lane-map order with at most one row per lane (uniform, from the shape:
    // the row slots of a replica cover its rows): the Philox outputs of each
    // half-sweep are computed during the one before.
    const int slots = T / (P.G / W);
    const bool lookahead = n_sweeps > 0 && ((slots >= P.n) ? (slots / P.n >= P.R) : (slots >= P.n * P.R));
    if (lookahead) {
      constexpr int NC = (W + 1) / 2;
      uint32_t U[4 * NC];
      // K runs one half-sweep ahead
      K.x0 = ((1u << 28) | ((uint32_t)ln.r0 << 1)) ^ P.key1;  // colour 0
      key_sweep(K, P, g, j);
      if (on) {
        uint32_t c0[NC], u[NC][4];
#pragma unroll
        for (int k = 0; k < NC; ++k) c0[k] = (uint32_t)((ln.t0 * P.ly + ln.y0) * P.G8 + (ln.w >> 1)) + k;
        philox_rows<NC>(K, c0, u);
#pragma unroll
        for (int k = 0; k < NC; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) U[4 * k + e] = u[k][e];
      }
      sweeps([&](int pos, int dpos, bool in_proto) {
#pragma unroll 1
        for (int c = 0; c < 2; ++c) {
          K.x0 ^= 1u;
          if (c == 1) key_sweep(K, P, g + 1, j);
          if (on)
            half_sweep_la<DIM, FULL, W>(P, ln, L, s_thr, c, g, j, pos, dpos, in_proto && c == 0, dI, U, K);
          __syncthreads();
        }
      });
    } else {
      sweeps([&](int pos, int dpos, bool in_proto) {
        key_sweep(K, P, g, j);
#pragma unroll 1
        for (int c = 0; c < 2; ++c) {
          if (on)
            half_sweep<DIM, FULL, W>(P, K, ln, mem, L, s_thr, c, g, j, pos, dpos, in_proto && c == 0, dI);
          __syncthreads();
        }
      });
    }
  }
  if (proto) {
    if (dI != 0) atomicAdd(&s_dI[slot], dI);
    __syncthreads();
    if (active && lt_ == 0) P.work[j] = (int64_t)s_dI[slot];
  }
  if (active) store_spins<PM>(P, L, j, lt_, T, pitch);
  __syncthreads();
}

// The variant of a work unit: the dimension, the words per lane, the row
// order (all uniform over the workgroup).
template <int DIM>
__device__ __forceinline__ void run_unit_dispatch(const JobDev* J, uint32_t lds, uint32_t tab, int j0, int cnt,
                                                  int kslots, uint32_t flags, int n_therm, int g0) {
  JP P;
  P.dim = DIM;
  P.n = uni(J->n); P.ly = uni(J->ly); P.H = uni(J->H); P.G = uni(J->G); P.R = uni(J->R);
  const int T = blockDim.x / kslots;
  const int W = words_per_lane(P, T);
  if (const int rp = uni(J->rag_pitch)) {
    // rows with pad sites: in parity-major order, or lane by word as below
    const int rW = uni(J->rag_W), G = P.G;
    P.G = rp;
    const int pm = pm_lanes(P, T, rW);
    const bool one = rp == rW;
#define EE_RAG(...) return run_unit<DIM, false, __VA_ARGS__, true>(J, lds, tab, T, pm, j0, cnt, flags, n_therm, g0)
    if (pm && rW == 4 && one) EE_RAG(4, true, 1);
    if (pm && rW == 4) EE_RAG(4, true, 0);
    if (pm && rW == 3) EE_RAG(3, true, 1);
    if (pm && rW == 2 && one) EE_RAG(2, true, 1);
    if (pm && rW == 2) EE_RAG(2, true, 0);
    if (pm) EE_RAG(1, true, 0);
#undef EE_RAG
    P.G = G;
  }
  const int pm = (P.H & 3) == 0 ? pm_lanes(P, T, W) : 0;
  // lanes per row, where the row's edge words come from registers (a pair of
  // lanes only if the slot's lanes start at an even lane)
  const int gw = P.G / W;
  const bool one = gw == 1, two = gw == 2 && (T & 1) == 0;
#define EE_RUN(...) return run_unit<__VA_ARGS__>(J, lds, tab, T, pm, j0, cnt, flags, n_therm, g0)
  if (W == 4) {
    if (pm && one) EE_RUN(DIM, true, 4, true, 1);
    if (pm && two) EE_RUN(DIM, true, 4, true, 2);
    if (pm) EE_RUN(DIM, true, 4, true);
    EE_RUN(DIM, true, 4, false);
  }
  if (W == 3) {
    if (pm) EE_RUN(DIM, true, 3, true, 1);
    EE_RUN(DIM, true, 3, false);
  }
  if (W == 2) {
    if (pm && one) EE_RUN(DIM, true, 2, true, 1);
    if (pm) EE_RUN(DIM, true, 2, true);
    EE_RUN(DIM, true, 2, false);
  }
  if (pm) EE_RUN(DIM, true, 1, true);
  if ((P.H & 3) == 0) EE_RUN(DIM, true, 1, false);
  EE_RUN(DIM, false, 1, false);
#undef EE_RUN
}

// Per-job mode (units == nullptr): workgroup b runs trajectories
// [b*single_k, b*single_k + single_k) of single_job.  Batch mode: persistent
// workgroups draw units from the queue until it is empty.  The dimension of
// each unit's job selects the 2D or 3D sweep (uniform per workgroup).
// tail: word offset, in the dynamic LDS, of the workgroup's small tables,
// which follow the trajectory slots.  The kernel has no static LDS.  4 waves
// per SIMD (128 VGPRs) and up to four words per lane, so that the per-row
// address and loop work is spread over 16 sites.
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
sweep_kernel(const JobDev* single_job, int single_k, const Unit* units, int n_units, int* queue,
             const JobDev* const* jobtab, uint32_t flags, int n_therm, int g0, int tail) {
  extern __shared__ __align__(16) uint32_t lds_raw[];
  const uint32_t lds = lds_address(lds_raw);
  const uint32_t tab = lds + 4u * (uint32_t)tail;
  int* const s_unit = reinterpret_cast<int*>(lds_raw + tail + kTabUnit);
  for (int iter = 0;; ++iter) {
    const JobDev* J;
    int j0, cnt, kslots;
    if (units != nullptr) {
      if (threadIdx.x == 0) *s_unit = atomicAdd(queue, 1);
      __syncthreads();
      const int u = uni(*s_unit);
      if (u >= n_units) break;
      const Unit U = units[u];
      J = uni_ptr(jobtab[uni(U.job)]);
      j0 = uni(U.j0);
      cnt = uni(U.count);
      kslots = uni(U.slots);
    } else {
      if (iter > 0) break;
      J = single_job;
      kslots = single_k;
      j0 = blockIdx.x * kslots;
      cnt = min(kslots, J->n_traj - j0);
    }
    if (uni(J->dim) == 3) run_unit_dispatch<3>(J, lds, tab, j0, cnt, kslots, flags, n_therm, g0);
    else run_unit_dispatch<2>(J, lds, tab, j0, cnt, kslots, flags, n_therm, g0);
  }
}

// ---------------------------------------------------------------------------
// Streaming path: lattices larger than one workgroup's LDS.  The spins stay
// in HBM (INT8 colour planes); one launch updates one colour of every
// trajectory of a job.  Block (x, y) covers lanes of trajectory y; a
// trajectory has `lanes` lanes, each walking its rows as in the on-chip
// path.  The neighbour rows are read through the vector caches, and the
// integer work goes to HBM with 64-bit atomics.
// ---------------------------------------------------------------------------
// Workgroups are dispatched to the XCDs (kXcd of them, each with its own L2)
// in turn by workgroup id.  The grid is one-dimensional, bx blocks per
// trajectory; the physical id is mapped to a logical (trajectory, block)
// such that each XCD gets one contiguous run of logical blocks, i.e. whole
// trajectories and neighbouring rows, which then meet in one L2.  The map
// is a bijection of [0, total), so results do not depend on it.
constexpr int kXcd = 8;
__device__ __forceinline__ void xcd_block(int bx, int total, int& j, int& b) {
  const int id = blockIdx.x;
  const int q = total / kXcd, rem = total - q * kXcd;
  const int x = id % kXcd, k = id / kXcd;
  const int logical = (x < rem) ? x * (q + 1) + k : rem * (q + 1) + (x - rem) * q + k;
  j = logical / bx;
  b = logical - j * bx;
}

template <int DIM, bool FULL, int W>
__device__ __forceinline__ void stream_half(const JP& P, uint32_t* s_thr, int lanes, int c, uint32_t g, int pos,
                                            int dpos, bool work) {
  const int bx = (lanes + 255) / 256;
  int jj, b;
  xcd_block(bx, (int)gridDim.x, jj, b);
  const int lt_ = b * blockDim.x + threadIdx.x;
  const uint32_t j = (uint32_t)jj;
  const HbmMem mem{P.spins + (size_t)j * P.traj_words};
  int dI = 0;
  PhKey K;
  key_unit(K, P);
  key_sweep(K, P, g, j);
  const Lane ln = make_lane(P, lt_ < lanes ? lt_ : 0, lanes, W, false);
  if (lt_ < lanes && ln.kstart < ln.kend)
    half_sweep<DIM, FULL, W>(P, K, ln, mem, 0u, s_thr, c, g, j, pos, dpos, work, dI);
  if (dI != 0) atomicAdd(reinterpret_cast<unsigned long long*>(&P.work[j]), (unsigned long long)(long long)dI);
}

// Body of the streaming launches: the widest lane width (words per lane)
// that the job's rows allow.
__device__ __forceinline__ void stream_body(const JobDev* J, int lanes, int c, uint32_t g, int pos, int dpos,
                                            int work) {
  __shared__ uint32_t s_thr[8];
  const JP P = load_jp(J);
  const int dim = uni(J->dim);
  if (threadIdx.x < 8)
    s_thr[threadIdx.x] = thr_entry(P, dim, threadIdx.x);
  __syncthreads();
  const bool full = (P.H & 3) == 0;
  const bool w = work != 0;
  switch (words_per_lane(P, lanes)) {
    case 4:
      if (dim == 3) stream_half<3, true, 4>(P, s_thr, lanes, c, g, pos, dpos, w);
      else stream_half<2, true, 4>(P, s_thr, lanes, c, g, pos, dpos, w);
      return;
    case 3:
      if (dim == 3) stream_half<3, true, 3>(P, s_thr, lanes, c, g, pos, dpos, w);
      else stream_half<2, true, 3>(P, s_thr, lanes, c, g, pos, dpos, w);
      return;
    case 2:
      if (dim == 3) stream_half<3, true, 2>(P, s_thr, lanes, c, g, pos, dpos, w);
      else stream_half<2, true, 2>(P, s_thr, lanes, c, g, pos, dpos, w);
      return;
    default:
      if (dim == 3) {
        if (full) stream_half<3, true, 1>(P, s_thr, lanes, c, g, pos, dpos, w);
        else stream_half<3, false, 1>(P, s_thr, lanes, c, g, pos, dpos, w);
      } else {
        if (full) stream_half<2, true, 1>(P, s_thr, lanes, c, g, pos, dpos, w);
        else stream_half<2, false, 1>(P, s_thr, lanes, c, g, pos, dpos, w);
      }
  }
}

// 4 waves per SIMD (128 VGPRs), up to four words per lane.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
stream_sweep_kernel(const JobDev* J, int lanes, int c, uint32_t g, int pos, int dpos, int work) {
  stream_body(J, lanes, c, g, pos, dpos, work);
}

// ---------------------------------------------------------------------------
// Plane-marching streaming path: lattices larger than one workgroup's LDS,
// jobs with enough trajectories to fill the GPU with long marches.  One
// sweep is one launch of march_kernel and one of march_fixup_kernel.
//
// A plane is every site of one replica with one t (all y, both colours).
// A sweep updates colour 0 everywhere with colour 1 unchanged, then colour
// 1 with colour 0 new (the oracle's order; sites of one colour are
// independent).  Workgroup (j, r, s) marches the planes of segment s of
// replica r of trajectory j through a ring of kMarchSlots plane slots in
// LDS: at step p it updates colour 0 of plane p (colour 1 of planes p-1, p,
// p+1 still old) and then colour 1 of plane p-1 (colour 0 of planes p-2,
// p-1, p already new), while plane p+2 is loaded and plane p-2, final,
// written back.  Each plane is read and written once per sweep, 2 B per
// site.  Colour 1 of a segment's first and last plane needs colour 0 of the
// neighbouring segments' planes, so it is left to march_fixup_kernel; the
// main pass only reads colour 1 of the neighbouring segments' boundary
// planes, which nobody writes during it.  Segments cover the unwrapped
// planes [1, lt + 1) (plane lt is t = 0), so planes t = 1 and t = 0, the
// rows next to the cut, are always boundary planes: the main pass updates
// only their colour 0, whose glued partners (colour 1 of replica r +- 1 in
// plane 1 - t) it reads from HBM, unchanged by the main pass.
// ---------------------------------------------------------------------------
constexpr int kMarchSlots = 5;
__device__ __forceinline__ void segment_bounds(int lt, int nseg, int s, int& t0, int& t1) {
  t0 = 1 + (int)((int64_t)lt * s / nseg);
  t1 = 1 + (int)((int64_t)lt * (s + 1) / nseg);
}

// Plane transfers between replica r of the trajectory in HBM (colour-plane
// storage) and a ring slot ([colour][y][word], the rows of the plane in
// storage order, so that slot unit i is simply the i-th unit of the slot).
// A unit is four words when the row length G is a multiple of 4, else one
// word; GV units per row.  The HBM side goes through global-address-space
// pointers: flat accesses would also count against the LDS wait counter, so
// that every LDS wait of the compute phases would wait for the transfers
// in flight.  A 16-byte unit is a native four-word vector.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
template <typename V>
using gptr = __attribute__((address_space(1))) V*;

// HBM word offset, at t = 0, of unit u of a plane of replica r.
__device__ __forceinline__ int unit_offset(const JP& P, int r, int u, int GV, int uw) {
  const int q = u / GV, wv = u - q * GV;
  const int c = q / P.ly, y = q - c * P.ly;
  return ((c * P.n + r) * P.R + y) * P.G + uw * wv;
}

template <bool TO_LDS, typename V>
__device__ __forceinline__ void plane_copy_v(const JP& P, uint32_t* traj, uint32_t* slot, int r, int t, int i_lo,
                                             int i_hi, int GV) {
  constexpr int UW = sizeof(V) / 4;
  V* sv = reinterpret_cast<V*>(slot);
  const gptr<uint32_t> base = (gptr<uint32_t>)(traj + t * P.ly * P.G);
  for (int i = i_lo + (int)threadIdx.x; i < i_hi; i += blockDim.x) {
    const gptr<V> g = (gptr<V>)(base + unit_offset(P, r, i, GV, UW));
    if (TO_LDS) sv[i] = *g;
    else *g = sv[i];
  }
}

// Copy colours [c_lo, c_hi) of plane t (synchronously: each unit's load or
// store is followed by its use).
template <bool TO_LDS>
__device__ __forceinline__ void plane_copy(const JP& P, uint32_t* traj, uint32_t* slot, int r, int t, int c_lo,
                                           int c_hi) {
  if ((P.G & 3) == 0) {
    const int GV = P.G >> 2;
    plane_copy_v<TO_LDS, v4u>(P, traj, slot, r, t, c_lo * P.ly * GV, c_hi * P.ly * GV, GV);
  } else {
    plane_copy_v<TO_LDS, uint32_t>(P, traj, slot, r, t, c_lo * P.ly * P.G, c_hi * P.ly * P.G, P.G);
  }
}

// This thread's share of the plane transfers: 16-byte units u0 + k T
// (k < 4) of a plane, with their HBM word offsets at t = 0 (the units of
// plane t sit at the same offsets plus t ly G words), computed once per
// launch.  A load is split in two: xfer_fetch() issues the loads into
// registers, xfer_put() writes them to the slot; between the two the loads
// are in flight while the workgroup computes.  Units from 4 T on, and
// planes whose rows are not a multiple of four words, are copied at once.
struct Xfer {
  int o0, o1, o2, o3;  // HBM word offsets (t = 0) of units u0 + k T
  int u0, T, U, U0;    // first unit, stride, units per plane, units of colour 0
  int GV, tw, r;       // units per row, HBM words per plane step (ly G), replica
  bool vec;            // rows of a multiple of four words
};

__device__ __forceinline__ Xfer make_xfer(const JP& P, int r) {
  Xfer X;
  X.vec = (P.G & 3) == 0;
  X.GV = P.G >> 2;
  X.U = 2 * P.ly * X.GV;
  X.U0 = P.ly * X.GV;
  X.T = blockDim.x;
  X.u0 = threadIdx.x;
  X.tw = P.ly * P.G;
  X.r = r;
  const auto off = [&](int u) { return (X.vec && u < X.U) ? unit_offset(P, r, u, X.GV, 4) : 0; };
  X.o0 = off(X.u0);
  X.o1 = off(X.u0 + X.T);
  X.o2 = off(X.u0 + 2 * X.T);
  X.o3 = off(X.u0 + 3 * X.T);
  return X;
}

// Issue the loads of colours [c_lo, 2) of plane t.
__device__ __forceinline__ void xfer_fetch(const Xfer& X, const JP& P, uint32_t* traj, uint32_t* slot, int t,
                                           int c_lo, v4u& v0, v4u& v1, v4u& v2, v4u& v3) {
  if (!X.vec) {
    plane_copy<true>(P, traj, slot, X.r, t, c_lo, 2);
    return;
  }
  const int lo = c_lo * X.U0;
  const gptr<uint32_t> base = (gptr<uint32_t>)(traj + t * X.tw);
  const auto ld = [&](int k, int o, v4u& v) {
    const int u = X.u0 + k * X.T;
    if (u >= lo && u < X.U) v = *(gptr<v4u>)(base + o);
  };
  ld(0, X.o0, v0);
  ld(1, X.o1, v1);
  ld(2, X.o2, v2);
  ld(3, X.o3, v3);
  if (4 * X.T < X.U) plane_copy_v<true, v4u>(P, traj, slot, X.r, t, max(lo, 4 * X.T), X.U, X.GV);
}

__device__ __forceinline__ void xfer_put(const Xfer& X, uint32_t* slot, int c_lo, const v4u& v0, const v4u& v1,
                                         const v4u& v2, const v4u& v3) {
  if (!X.vec) return;
  const int lo = c_lo * X.U0;
  v4u* sv = reinterpret_cast<v4u*>(slot);
  const auto st = [&](int k, const v4u& v) {
    const int u = X.u0 + k * X.T;
    if (u >= lo && u < X.U) sv[u] = v;
  };
  st(0, v0);
  st(1, v1);
  st(2, v2);
  st(3, v3);
}

// Write colours [0, c_hi) of plane t back to HBM.
__device__ __forceinline__ void xfer_store(const Xfer& X, const JP& P, uint32_t* traj, uint32_t* slot, int t,
                                           int c_hi) {
  if (!X.vec) {
    plane_copy<false>(P, traj, slot, X.r, t, 0, c_hi);
    return;
  }
  const int hi = c_hi * X.U0;
  const gptr<uint32_t> base = (gptr<uint32_t>)(traj + t * X.tw);
  const v4u* sv = reinterpret_cast<const v4u*>(slot);
  const auto st = [&](int k, int o) {
    const int u = X.u0 + k * X.T;
    if (u < hi) *(gptr<v4u>)(base + o) = sv[u];
  };
  st(0, X.o0);
  st(1, X.o1);
  st(2, X.o2);
  st(3, X.o3);
  if (4 * X.T < hi) plane_copy_v<false, v4u>(P, traj, slot, X.r, t, 4 * X.T, hi, X.GV);
}

// A row of a plane's colour: y and first word w.
struct RowDesc {
  int y, w;
};

__device__ __forceinline__ RowDesc row_desc(int it, int GW, int W) {
  RowDesc d;
  d.y = it / GW;
  d.w = (it - d.y * GW) * W;
  return d;
}

// Colour c of plane t of replica r (unwrapped plane index p: slots of p-1,
// p, p+1 are sm, s0, sp) from the ring; PW words per slot.  d0: this
// thread's first row (the same in every plane).  Rows next to the cut
// (t <= 1) come here with c = 0 only.
template <int DIM, bool FULL, int W>
__device__ __forceinline__ void march_colour(const JP& P, PhKey& K, uint32_t* win, uint32_t* traj, int PW, int sm, int s0,
                                             int sp, int c, int r, int t, const uint32_t* thr, uint32_t g,
                                             uint32_t j, int pos, int dpos, bool work, int& dI, const RowDesc& d0) {
  const int G = P.G, GW = G / W, ly = P.ly;
  const LdsMem mem;
  const HbmMem hbm{traj};
  const uint32_t ring = lds_address(win);
  const uint32_t own = ring + 4u * (uint32_t)(s0 * PW + c * ly * G);
  const uint32_t oth = ring + 4u * (uint32_t)(s0 * PW + (c ^ 1) * ly * G);
  const int tmo = (sm - s0) * PW, tpo = (sp - s0) * PW;
  const uint32_t c3 = (1u << 28) | ((uint32_t)r << 1) | (uint32_t)c;
  K.x0 = c3 ^ P.key1;
  const auto rows = [&](auto cut) {
    constexpr bool CUT = decltype(cut)::value;
    // glued partners: colour 1 of replica r+1 in plane 1 (t = 0) or of
    // replica r-1 in plane 0 (t = 1), in HBM
    const int rgl = (t == 0) ? ((r + 1 == P.n) ? 0 : r + 1) : ((r == 0) ? P.n - 1 : r - 1);
    const int ogl = ((P.n + rgl) * P.R + (1 - t) * ly) * G;
    RowDesc d = d0;
    for (int it = threadIdx.x; it < ly * GW;) {
      const int y = d.y, w = d.w;
      const int wl = (w == 0) ? G - 1 : w - 1, wr = (w + W == G) ? 0 : w + W;
      const int ymo = (y == 0) ? (ly - 1) * G : -G, ypo = (y == ly - 1) ? -(ly - 1) * G : G;
      const uint32_t c0 = (uint32_t)((t * ly + y) * P.G8 + (w >> 1));
      const uint32_t off = 4u * (uint32_t)(y * G + w);
      update_row<DIM, FULL, W, CUT, false>(P, K, mem, own + off, oth + off, hbm, CUT ? 4u * (uint32_t)ogl + off : 0u,
                                           w, wl, wr, thr, c, g, j, pos, dpos, work, dI, t, y, tmo, tpo, ymo, ypo,
                                           c0, c3);
      it += blockDim.x;
      if (it < ly * GW) d = row_desc(it, GW, W);
    }
  };
  if (t <= 1) rows(std::true_type{});
  else rows(std::false_type{});
}

template <int DIM, bool FULL, int W>
__device__ __forceinline__ void march_segment(const JP& P, uint32_t* win, const uint32_t* thr, int nseg, uint32_t g,
                                              int pos, int dpos, bool work) {
  int jj, rs;
  xcd_block(P.n * nseg, (int)gridDim.x, jj, rs);
  const int r = rs / nseg, seg = rs - r * nseg;
  const uint32_t j = (uint32_t)jj;
  uint32_t* traj = P.spins + (size_t)j * P.traj_words;
  const int PW = 2 * P.ly * P.G;
  int t0, t1;
  segment_bounds(P.lt, nseg, seg, t0, t1);
  // ring of kMarchSlots slots: plane p in slot (p - t0 + 1) mod kMarchSlots
  const auto slot = [&](int p) { return (p - t0 + 1) % kMarchSlots; };
  const auto phys = [&](int p) { return (p >= P.lt) ? p - P.lt : p; };  // 0 <= p < 2 lt
  const Xfer X = make_xfer(P, r);
  const RowDesc d0 = row_desc(threadIdx.x, P.G / W, W);
  int dI = 0;
  PhKey K;
  key_unit(K, P);
  key_sweep(K, P, g, j);
  v4u v0 = {}, v1 = {}, v2 = {}, v3 = {};
  // planes t0-1 .. t0+1; a neighbouring segment's boundary plane
  // contributes only its colour 1
  for (int p = t0 - 1; p <= t0 + 1; ++p) {
    const int c_lo = (p < t0 || p >= t1) ? 1 : 0;
    xfer_fetch(X, P, traj, win + slot(p) * PW, phys(p), c_lo, v0, v1, v2, v3);
    xfer_put(X, win + slot(p) * PW, c_lo, v0, v1, v2, v3);
  }
  __syncthreads();
  for (int p = t0; p < t1; ++p) {
    // step p: colour 0 of plane p (planes p-1 .. p+1 in the ring), then
    // colour 1 of plane p-1 (planes p-2 .. p).  Meanwhile plane p+2 is
    // fetched (into registers, then into its slot, free since plane p-3
    // was written back) and the final plane p-2 is written back.
    const bool fetch = p + 2 <= t1;
    const int c_lo = (p + 2 == t1) ? 1 : 0;
    if (fetch) xfer_fetch(X, P, traj, win + slot(p + 2) * PW, phys(p + 2), c_lo, v0, v1, v2, v3);
    march_colour<DIM, FULL, W>(P, K, win, traj, PW, slot(p - 1), slot(p), slot(p + 1), 0, r, phys(p), thr, g, j, pos,
                               dpos, work, dI, d0);
    __syncthreads();
    // plane p-2 is final (colour 1 of the segment's first plane waits for
    // the fix-up pass)
    if (p - 2 >= t0) xfer_store(X, P, traj, win + slot(p - 2) * PW, phys(p - 2), (p - 2 > t0) ? 2 : 1);
    if (p - 1 >= t0 + 1)
      march_colour<DIM, FULL, W>(P, K, win, traj, PW, slot(p - 2), slot(p - 1), slot(p), 1, r, phys(p - 1), thr, g, j,
                                 pos, dpos, false, dI, d0);
    if (fetch) xfer_put(X, win + slot(p + 2) * PW, c_lo, v0, v1, v2, v3);
    __syncthreads();
  }
  if (t1 - 2 >= t0) xfer_store(X, P, traj, win + slot(t1 - 2) * PW, phys(t1 - 2), (t1 - 2 > t0) ? 2 : 1);
  xfer_store(X, P, traj, win + slot(t1 - 1) * PW, phys(t1 - 1), 1);
  if (dI != 0) atomicAdd(reinterpret_cast<unsigned long long*>(&P.work[j]), (unsigned long long)(long long)dI);
}

// Colour 1 of each segment's first and last plane, every replica, from HBM
// (block: one plane of one segment of one trajectory).
template <int DIM, bool FULL, int W>
__device__ __forceinline__ void fixup_plane(const JP& P, const uint32_t* thr, int nseg, uint32_t g, int pos,
                                            int dpos) {
  const int b = blockIdx.x;
  const int jj = b / (2 * nseg), rem = b - jj * 2 * nseg, seg = rem >> 1, last = rem & 1;
  int t0, t1;
  segment_bounds(P.lt, nseg, seg, t0, t1);
  if (last && t1 - 1 == t0) return;  // a one-plane segment has one boundary plane
  const int t = (last ? t1 - 1 : t0) % P.lt;
  const uint32_t j = (uint32_t)jj;
  uint32_t* traj = P.spins + (size_t)j * P.traj_words;
  const int G = P.G, GW = G / W, ly = P.ly, R = P.R;
  const HbmMem mem{traj};
  PhKey K;
  key_unit(K, P);
  key_sweep(K, P, g, j);
  const uint32_t bC = 4u * (uint32_t)(P.n * R * G);  // colour 1; colour 0 is at 0
  const int LyG = ly * G, ltLyG = P.lt * LyG;
  const int tpo = LyG - ((t == P.lt - 1) ? ltLyG : 0);
  const int tmo = -LyG + ((t == 0) ? ltLyG : 0);
  int dI = 0;
  const auto rows = [&](auto cut) {
    constexpr bool CUT = decltype(cut)::value;
    for (int it = threadIdx.x; it < P.n * ly * GW; it += blockDim.x) {
      const int rr = it / GW, w = (it - rr * GW) * W;
      const int r = rr / ly, y = rr - r * ly;
      const int wl = (w == 0) ? G - 1 : w - 1, wr = (w + W == G) ? 0 : w + W;
      const int ymo = (y == 0) ? (ly - 1) * G : -G, ypo = (y == ly - 1) ? -(ly - 1) * G : G;
      const int rowbase = (r * R + t * ly + y) * G;
      const uint32_t c0 = (uint32_t)((t * ly + y) * P.G8 + (w >> 1));
      const uint32_t c3 = (1u << 28) | ((uint32_t)r << 1) | 1u;
      K.x0 = c3 ^ P.key1;
      const uint32_t off = 4u * (uint32_t)(rowbase + w);
      const uint32_t ag = CUT ? 4u * (uint32_t)(glued_row(P, r, t, y) * G + w) : off;
      update_row<DIM, FULL, W, CUT, false>(P, K, mem, bC + off, off, mem, ag, w, wl, wr, thr, 1, g, j, pos, dpos,
                                           false, dI, t, y, tmo, tpo, ymo, ypo, c0, c3);
    }
  };
  if (t <= 1) rows(std::true_type{});
  else rows(std::false_type{});
}

// Words per lane of the marching kernels: as the on-chip kernel chooses for
// a workgroup of blockDim lanes per plane.
template <bool MAIN>
__device__ __forceinline__ void march_body(const JobDev* J, int nseg, uint32_t g, int pos, int dpos, int work) {
  extern __shared__ __align__(16) uint32_t march_lds[];
  const JP P = load_jp(J);
  const int dim = uni(J->dim);
  const int PW = 2 * P.ly * P.G;
  uint32_t* thr = MAIN ? march_lds + kMarchSlots * PW : march_lds;  // after the ring (main pass) or alone (fix-up)
  if (threadIdx.x < 8)
    thr[threadIdx.x] = thr_entry(P, dim, threadIdx.x);
  __syncthreads();
  const bool full = (P.H & 3) == 0;
  const bool w = work != 0;
  const auto go = [&](auto dimc, auto fullc, auto wc) {
    constexpr int D = decltype(dimc)::value;
    constexpr bool F = decltype(fullc)::value;
    constexpr int WW = decltype(wc)::value;
    if (MAIN) march_segment<D, F, WW>(P, march_lds, thr, nseg, g, pos, dpos, w);
    else fixup_plane<D, F, WW>(P, thr, nseg, g, pos, dpos);
  };
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using T_ = std::true_type;
  using F_ = std::false_type;
  switch (words_per_lane(P, (int)blockDim.x)) {
    case 4:
      if (dim == 3) go(I3{}, T_{}, std::integral_constant<int, 4>{});
      else go(I2{}, T_{}, std::integral_constant<int, 4>{});
      return;
    case 3:
      if (dim == 3) go(I3{}, T_{}, std::integral_constant<int, 3>{});
      else go(I2{}, T_{}, std::integral_constant<int, 3>{});
      return;
    case 2:
      if (dim == 3) go(I3{}, T_{}, std::integral_constant<int, 2>{});
      else go(I2{}, T_{}, std::integral_constant<int, 2>{});
      return;
    default:
      if (dim == 3) {
        if (full) go(I3{}, T_{}, std::integral_constant<int, 1>{});
        else go(I3{}, F_{}, std::integral_constant<int, 1>{});
      } else {
        if (full) go(I2{}, T_{}, std::integral_constant<int, 1>{});
        else go(I2{}, F_{}, std::integral_constant<int, 1>{});
      }
  }
}

__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
march_kernel(const JobDev* J, int nseg, uint32_t g, int pos, int dpos, int work) {
  march_body<true>(J, nseg, g, pos, dpos, work);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
march_fixup_kernel(const JobDev* J, int nseg, uint32_t g, int pos, int dpos) {
  march_body<false>(J, nseg, g, pos, dpos, 0);
}

// Initial spins of every trajectory, written straight to HBM.
__global__ void __launch_bounds__(256) stream_init_kernel(const JobDev* J, int lanes) {
  const JP P = load_jp(J);
  const uint32_t j = blockIdx.y;
  const int lt_ = blockIdx.x * blockDim.x + threadIdx.x;
  if (lt_ < lanes) init_spins<false>(P, HbmMem{P.spins + (size_t)j * P.traj_words}, 0u, j, lt_, lanes, P.G);
}

__global__ void zero_work_kernel(const JobDev* J) {
  const int n = J->n_traj;
  int64_t* w = J->work;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) w[i] = 0;
}

__global__ void queue_reset_kernel(int* queue) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *queue = 0;
}

// ---------------------------------------------------------------------------
// Estimator (App. A, Jarzynski's equality).
//
// Every floating-point result is formed by the same operations in the same
// order as the plain definition: the n_t exponentials e_j are summed one
// after the other in ascending j, each leave-one-out sum is its own
// ascending sum over j != i, and the mean and variance of W are sums of the
// terms -(beta/S) I_j in ascending j.  exp and log are the correctly
// rounded ones of ee_dd.hpp.
//
// What bounds it is then the chain of dependent FP64 adds (some 17 cycles a
// term for a wave alone on its SIMD), and how many of the n^2 adds of the leave-one-out sums run beside
// each other.  Up to kEstSmall trajectories one workgroup does a job
// (estimate_kernel): lane i forms sum i, lane n the full sum, all in one walk
// over the e_j in LDS, and one more wave the other sums.  Above, four
// launches: the exponentials over many workgroups (est_exp_kernel), the plain
// sums in one wave per job (est_sum_kernel), the leave-one-out sums in one
// wave per 64 of them (est_loo_kernel) and their spread (est_err_kernel).
// Sums i of a wave start from the full sum's prefix, which is their own
// beginning.  16384 trajectories: 0.64 against 9.8 ms in one workgroup; 64
// jobs of 1024: 59 against 145 us; 8 trajectories: 9 against 29 us.
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)
constexpr int kEstTileN = 256;  // e_j per workgroup of est_exp_kernel

// Integer minimum and maximum over the block: butterfly shuffles within each
// wave, then the waves' results through LDS (sh: 32 entries).
__device__ __forceinline__ void block_min_max(long long& mn, long long& mx, long long* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const long long a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  const int nw = (blockDim.x + 63) >> 6, wave = threadIdx.x >> 6;
  if (nw == 1) return;
  if ((threadIdx.x & 63) == 0) {
    sh[2 * wave] = mn;
    sh[2 * wave + 1] = mx;
  }
  __syncthreads();
  for (int k = 0; k < nw; ++k) {
    mn = sh[2 * k] < mn ? sh[2 * k] : mn;
    mx = sh[2 * k + 1] > mx ? sh[2 * k + 1] : mx;
  }
}

// Visit load(0), load(1), ... load(n-1) in order with add(j, v), loading
// kEstGroup values ahead of their adds.
constexpr int kEstGroup = 16;
template <typename Load, typename Add>
__device__ __forceinline__ void for_groups(int n, Load load, Add add) {
  // pairs of groups: each group's registers are loaded again while the other
  // one is added
  const int full = n / (2 * kEstGroup) * (2 * kEstGroup);
  if (full > 0) {
    double a[kEstGroup], b[kEstGroup];
#pragma unroll
    for (int k = 0; k < kEstGroup; ++k) a[k] = load(k);
    for (int j = 0; j < full; j += 2 * kEstGroup) {
#pragma unroll
      for (int k = 0; k < kEstGroup; ++k) b[k] = load(j + kEstGroup + k);
#pragma unroll
      for (int k = 0; k < kEstGroup; ++k) add(j + k, a[k]);
      const int jn = (j + 2 * kEstGroup < full) ? j + 2 * kEstGroup : j;
#pragma unroll
      for (int k = 0; k < kEstGroup; ++k) a[k] = load(jn + k);
#pragma unroll
      for (int k = 0; k < kEstGroup; ++k) add(j + kEstGroup + k, b[k]);
    }
  }
  for (int j = full; j < n; ++j) add(j, load(j));
}

// The same for a workgroup of one wave and terms in device memory: the lanes
// load tiles of kTileTerms terms, one tile ahead, and every lane then reads
// them in order from LDS (buf: two tiles).  Read through the scalar cache, 16
// terms ahead, a term took 32 cycles.
constexpr int kTileTerms = 512;
template <typename Load, typename Add>
__device__ __forceinline__ void for_tiles(int n, double* buf, Load load, Add add) {
  constexpr int K = kTileTerms / 64;
  const int lane = threadIdx.x;
  double v[K];
  const auto fetch = [&](int j0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int j = j0 + 64 * k + lane;
      v[k] = (j < n) ? load(j) : 0.0;
    }
  };
  const auto put = [&](double* b) {
#pragma unroll
    for (int k = 0; k < K; ++k) b[64 * k + lane] = v[k];
  };
  __syncthreads();
  fetch(0);
  put(buf);
  int cur = 0;
  for (int j0 = 0; j0 < n; j0 += kTileTerms, cur ^= 1) {
    __syncthreads();
    if (j0 + kTileTerms < n) fetch(j0 + kTileTerms);
    const double* b = buf + cur * kTileTerms;
    for_groups(min(kTileTerms, n - j0), [&](int j) { return b[j]; }, [&](int j, double x) { add(j0 + j, x); });
    if (j0 + kTileTerms < n) put(buf + (cur ^ 1) * kTileTerms);
  }
}

struct EstJob {
  int n;
  double beta, N;  // W_j = -(beta/N) I_j
  const int64_t* I;
  double *e, *loo;
  ee_result* res;
  int replicas;
};
__device__ __forceinline__ EstJob est_job(const JobDev* J) {
  EstJob E;
  E.n = uni(J->n_traj);
  E.beta = J->beta;
  E.N = (double)uni(J->S);
  E.I = uni_ptr(J->work);
  E.e = reinterpret_cast<double*>(uni_ptr(J->work) + E.n);  // n doubles: e_j
  E.loo = E.e + E.n;                                        // n doubles: leave-one-out estimates
  E.res = uni_ptr(J->result);
  E.replicas = uni(J->n);
  return E;
}

// The jackknife error from the leave-one-out estimates, visited in ascending
// i by visit(add).
template <typename Visit>
__device__ __forceinline__ double jackknife(int n, Visit visit) {
  if (n < 2) return __builtin_nan("");
  double mean = 0.0;
  visit([&](int, double v) { mean += v; });
  mean /= n;
  double acc = 0.0;
  visit([&](int, double v) { acc += (v - mean) * (v - mean); });
  return sqrt((double)(n - 1) / (double)n * acc);
}

// One job per workgroup, n <= kEstSmall; blockDim.x: n + 1 rounded up to
// whole waves, and one wave more.
__global__ void __launch_bounds__(1024) estimate_kernel(const JobDev* const* jobtab) {
  __shared__ double se[ee::kEstSmall], sl[ee::kEstSmall];
  __shared__ long long shl[32];
  __shared__ double shd[8];
  const EstJob E = est_job(jobtab[blockIdx.x]);
  const int tid = threadIdx.x, n = E.n;
  const bool stat = (tid >> 6) == ((int)blockDim.x >> 6) - 1;  // the last wave
  const bool mine = tid < n;  // never in the last wave
  const long long Ii = mine ? E.I[tid] : 0;
  long long mn = mine ? Ii : LLONG_MAX, mx = mine ? Ii : LLONG_MIN;
  block_min_max(mn, mx, shl);
  const double w = -(E.beta / E.N);
  if (mine) {
    se[tid] = ee::dd::exp_cr((E.beta * (double)(Ii - mx)) / E.N);
    sl[tid] = w * (double)Ii;  // W_j
  }
  __syncthreads();
  const double shift = (E.beta * (double)mx) / E.N;
  const int lane = tid & 63;
  double acc = 0.0, lg = 0.0;
  if (stat) {
    // lane 0: sum of e^2, lane 1: the mean and variance of W; lanes 2 and 3:
    // log n, log (n - 1)
    const bool sq = lane == 0;
    for_groups(n, [&](int j) { return sq ? se[j] : sl[j]; }, [&](int, double v) { acc += sq ? v * v : v; });
    if (lane == 0) shd[1] = acc;
    const double wm = acc / n;
    double wv = 0.0;
    for_groups(n, [&](int j) { return sl[j]; }, [&](int, double v) { wv += (v - wm) * (v - wm); });
    if (lane == 1) {
      shd[2] = wm;
      shd[3] = wv / n;
    }
    lg = ee::dd::log_cr((double)((lane == 3 && n >= 2) ? n - 1 : n));
    if (lane == 2) shd[4] = lg;
    if (lane == 3) shd[5] = lg;
  } else {
    // lane i: the sum over j != i (adding +0.0 for j = i leaves a sum of
    // non-negative terms unchanged); lane n: the full sum
    for_groups(n, [&](int j) { return se[j]; }, [&](int j, double v) { acc += (j == tid) ? 0.0 : v; });
    if (tid <= n && !(n == 1 && tid == 0)) lg = ee::dd::log_cr(acc);
    if (tid == n) {
      shd[0] = acc;
      shd[6] = lg;
    }
  }
  __syncthreads();
  if (mine) sl[tid] = -(shift + lg - shd[5]);
  __syncthreads();
  if (tid == 0) {
    const double dF = -(shift + shd[6] - shd[4]);
    const double err = jackknife(n, [&](auto add) { for_groups(n, [&](int i) { return sl[i]; }, add); });
    ee_result* res = E.res;
    res->dF = dF;
    res->dS = dF / (double)(E.replicas - 1);
    res->dF_err = err;
    res->w_mean = shd[2];
    res->w_var = shd[3];
    res->ess = shd[0] * shd[0] / shd[1];
    res->i_min = mn;
    res->i_max = mx;
    res->n_traj = n;
  }
}

// e_j of kEstTileN trajectories (y) of job x; every workgroup finds the
// extreme works itself.
__global__ void __launch_bounds__(kEstTileN) est_exp_kernel(const JobDev* const* jobtab) {
  __shared__ long long shl[32];
  const EstJob E = est_job(jobtab[blockIdx.x]);
  const int i = blockIdx.y * kEstTileN + threadIdx.x;
  if (blockIdx.y * kEstTileN >= E.n) return;
  long long mn = LLONG_MAX, mx = LLONG_MIN;
  for (int q = threadIdx.x; q < E.n; q += kEstTileN) {
    const long long v = E.I[q];
    mn = v < mn ? v : mn;
    mx = v > mx ? v : mx;
  }
  block_min_max(mn, mx, shl);
  if (i < E.n) E.e[i] = ee::dd::exp_cr((E.beta * (double)(E.I[i] - mx)) / E.N);
  if (i == 0) {
    E.res->i_min = mn;
    E.res->i_max = mx;
    E.res->n_traj = E.n;
  }
}

// The plain sums of job x, one per lane: 0 of e (its prefix before every 64th
// term goes to loo, where the leave-one-out sums of those 64 begin), 1 of
// e^2, 2 of W, which then does the variance.
__global__ void __launch_bounds__(64) est_sum_kernel(const JobDev* const* jobtab) {
  const EstJob E = est_job(jobtab[blockIdx.x]);
  const int lane = threadIdx.x, n = E.n;
  __shared__ double buf[2 * kTileTerms];
  const double w = -(E.beta / E.N);
  double acc = 0.0;
  if (blockIdx.y == 0) {
    for_tiles(n, buf, [&](int j) { return E.e[j]; }, [&](int j, double v) {
      if ((j & 63) == 0 && lane == 0) E.loo[j] = acc;
      acc += (lane == 1) ? v * v : v;
    });
    const double s2 = __shfl(acc, 1, 64), s = __shfl(acc, 0, 64);
    const double lg = ee::dd::log_cr(lane == 0 ? s : (double)n);
    const double log_n = __shfl(lg, 1, 64);
    if (lane == 0) {
      const double shift = (E.beta * (double)E.res->i_max) / E.N;
      const double dF = -(shift + lg - log_n);
      E.res->dF = dF;
      E.res->dS = dF / (double)(E.replicas - 1);
      E.res->ess = s * s / s2;
    }
  } else {
    const auto load = [&](int j) { return w * (double)E.I[j]; };
    for_tiles(n, buf, load, [&](int, double v) { acc += v; });
    const double wm = acc / n;
    double wv = 0.0;
    for_tiles(n, buf, load, [&](int, double v) { wv += (v - wm) * (v - wm); });
    if (lane == 0) {
      E.res->w_mean = wm;
      E.res->w_var = wv / n;
    }
  }
}

// Leave-one-out estimates 64 y .. 64 y + 63 of job x, one per lane.
__global__ void __launch_bounds__(64) est_loo_kernel(const JobDev* const* jobtab) {
  const EstJob E = est_job(jobtab[blockIdx.x]);
  const int n = E.n, i0 = blockIdx.y * 64, i = i0 + (int)threadIdx.x;
  if (i0 >= n || n < 2) return;
  __shared__ double buf[2 * kTileTerms];
  const double* e = E.e + i0;
  double acc = E.loo[i0];
  const int own = min(64, n - i0);
  for (int j = 0; j < own; ++j) acc += (j == (int)threadIdx.x) ? 0.0 : e[j];
  for_tiles(n - i0 - own, buf, [&](int j) { return e[64 + j]; }, [&](int, double v) { acc += v; });
  const double shift = (E.beta * (double)E.res->i_max) / E.N;
  const double log_n1 = ee::dd::log_cr((double)(n - 1));
  if (i < n) E.loo[i] = -(shift + ee::dd::log_cr(acc) - log_n1);
}

__global__ void __launch_bounds__(64) est_err_kernel(const JobDev* const* jobtab) {
  const EstJob E = est_job(jobtab[blockIdx.x]);
  __shared__ double buf[2 * kTileTerms];
  const double err =
      jackknife(E.n, [&](auto add) { for_tiles(E.n, buf, [&](int i) { return E.loo[i]; }, add); });
  if (threadIdx.x == 0) E.res->dF_err = err;
}

}  // namespace

// Fixed device scratch of the allocation-free batch entry point: the queue
// counter, the job table and the work units of one launch.  Each GPU holds
// its own copy until the process ends.  In host code the array's name is
// only a stand-in: its device address comes from hipGetSymbolAddress.
constexpr size_t kScratchBytes = size_t(2) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

extern "C" {

int ee_k_max_lds_bytes() { return 160 * 1024 - 256; }

size_t ee_k_scratch_bytes() { return kScratchBytes; }

// Device address of the current device's copy of the scratch array, looked
// up once per device (with that device current) and kept.
int ee_k_scratch_ptr(void** out) {
  static std::mutex mu;
  static std::vector<void*> ptrs;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  std::lock_guard<std::mutex> lk(mu);
  if ((int)ptrs.size() <= dev) ptrs.resize(dev + 1, nullptr);
  if (ptrs[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    ptrs[dev] = p;
  }
  *out = ptrs[dev];
  return 0;
}

static hipError_t set_lds_attr(const void* fn) {
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                             ee_k_max_lds_bytes() + ee::kSweepTailBytes);
}

int ee_k_sweep_kernel_ptr(const void** fn) {
  *fn = reinterpret_cast<const void*>(&sweep_kernel);
  return (int)set_lds_attr(*fn);
}
int ee_k_queue_reset_ptr(const void** fn) {
  *fn = reinterpret_cast<const void*>(&queue_reset_kernel);
  return 0;
}
// The launches of the estimator of `count` jobs of at most max_n
// trajectories, in order; each takes the job table.  Returns their number.
int ee_k_estimate_plan(int count, int max_n, ee::EstLaunch out[4]) {
  if (max_n <= ee::kEstSmall) {
    out[0] = {reinterpret_cast<const void*>(&estimate_kernel), count, 1, (max_n + 64) / 64 * 64 + 64};
    return 1;
  }
  out[0] = {reinterpret_cast<const void*>(&est_exp_kernel), count, (max_n + kEstTileN - 1) / kEstTileN, kEstTileN};
  out[1] = {reinterpret_cast<const void*>(&est_sum_kernel), count, 2, 64};
  out[2] = {reinterpret_cast<const void*>(&est_loo_kernel), count, (max_n + 63) / 64, 64};
  out[3] = {reinterpret_cast<const void*>(&est_err_kernel), count, 1, 64};
  return 4;
}

int ee_k_launch_sweep(const ee::JobDev* single_job, int single_k, const ee::Unit* units, int n_units, int* queue,
                      const ee::JobDev* const* jobtab, uint32_t flags, int n_therm, int g0, int grid, int block,
                      int lds_bytes, void* stream) {
  const void* fn = nullptr;
  hipError_t e = (hipError_t)ee_k_sweep_kernel_ptr(&fn);
  if (e != hipSuccess) return (int)e;
  const int tail = ee::sweep_tail_words(lds_bytes);
  const int bytes = lds_bytes + ee::kSweepTailBytes;
  hipLaunchKernelGGL(sweep_kernel, dim3(grid), dim3(block), bytes, (hipStream_t)stream, single_job, single_k, units,
                     n_units, queue, jobtab, flags, n_therm, g0, tail);
  return (int)hipGetLastError();
}

int ee_k_launch_stream_sweep(const ee::JobDev* job, int n_traj, int lanes, int c, uint32_t g, int pos, int dpos,
                             int work, void* stream) {
  const int bx = (lanes + 255) / 256;
  // one-dimensional grid: bx blocks per trajectory, remapped per XCD in the kernel
  hipLaunchKernelGGL(stream_sweep_kernel, dim3(bx * n_traj), dim3(256), 0, (hipStream_t)stream, job, lanes, c, g,
                     pos, dpos, work);
  return (int)hipGetLastError();
}

int ee_k_march_lds_bytes(int plane_words) { return kMarchSlots * plane_words * 4 + 32; }

int ee_k_launch_march(const ee::JobDev* job, int n_traj, int n_replicas, int nseg, int block, int plane_words,
                      uint32_t g, int pos, int dpos, int work, void* stream) {
  const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&march_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, ee_k_max_lds_bytes());
  if (attr != hipSuccess) return (int)attr;
  hipLaunchKernelGGL(march_kernel, dim3(n_traj * n_replicas * nseg), dim3(block), ee_k_march_lds_bytes(plane_words),
                     (hipStream_t)stream, job, nseg, g, pos, dpos, work);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL(march_fixup_kernel, dim3(n_traj * nseg * 2), dim3(256), 32, (hipStream_t)stream, job, nseg, g,
                     pos, dpos);
  return (int)hipGetLastError();
}

int ee_k_launch_stream_init(const ee::JobDev* job, int n_traj, int lanes, void* stream) {
  const int bx = (lanes + 255) / 256;
  hipLaunchKernelGGL(stream_init_kernel, dim3(bx, n_traj), dim3(256), 0, (hipStream_t)stream, job, lanes);
  return (int)hipGetLastError();
}

int ee_k_launch_zero_work(const ee::JobDev* job, int n_traj, void* stream) {
  const int bx = (n_traj + 255) / 256;
  hipLaunchKernelGGL(zero_work_kernel, dim3(bx), dim3(256), 0, (hipStream_t)stream, job);
  return (int)hipGetLastError();
}

int ee_k_launch_queue_reset(int* queue, void* stream) {
  hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, queue);
  return (int)hipGetLastError();
}

int ee_k_launch_estimate(const ee::JobDev* const* jobtab, int count, int max_n, void* stream) {
  ee::EstLaunch L[4];
  const int k = ee_k_estimate_plan(count, max_n, L);
  void* args[] = {&jobtab};
  for (int i = 0; i < k; ++i) {
    const hipError_t e = hipLaunchKernel(L[i].fn, dim3(L[i].gx, L[i].gy), dim3(L[i].block), args, 0, (hipStream_t)stream);
    if (e != hipSuccess) return (int)e;
  }
  return (int)hipGetLastError();
}

}  // extern "C"
