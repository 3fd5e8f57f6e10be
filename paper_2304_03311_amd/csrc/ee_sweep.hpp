// ee_sweep.hpp -- the on-chip sweep kernel: one workgroup holds k trajectories
// of one job in LDS (int8 spins, colour-separated rows) and runs, entirely on
// chip, the initial spins, the thermalisation sweeps and the N protocol sweeps
// with the integer work (Sec. 3 linear protocol; App. A work-then-update).
// Compiled twice, with and without the whole-region protocol (EE_WHOLE); the
// including file names the kernel with EE_SWEEP_KERNEL.
#pragma once
#include "ee_rows.hpp"

namespace {

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
    update_row<DIM, FULL, W, CUT, true>(P, Kn, mem, bC + off, mem, bO + off, mem, ag, w, ln.wl, ln.wr, thr, c, g, j, pos,
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
// jobs x 1024 trajectories 151 against 177 ms (145 with the whole-region
// protocol in a kernel of its own), 3D 32^3 x 512 trajectories 21.4 (20.9)
// against 25.1 ms.
// has_cut: some lane of the wave starts with rows next to the cut.  cut_mask:
// the lane's glued_bits in its rows next to the cut (0 if it has none), of
// word q and x parity p moved to bit 4 p + q of each byte.  has_ramp: these
// rows hold the ramped site.
// RAG: rows with pad sites (row_pitch; P.G is the pitch), whose lanes have
// what RagLane says.
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

// Row (over colours and replicas) rowg of the storage order in LDS.
template <bool PM>
__device__ __forceinline__ int lds_row(const JP& P, int rowg) {
  if (!PM) return rowg;
  const int rho = rowg - (int)fdiv((uint32_t)rowg, P.mR, P.sR) * P.R;
  return rowg - rho + pm_row(P, rho);
}

// Initial spins into LDS (PM: into the class-by-class rows of the parity-major
// order), pitch words per row.
template <bool PM>
__device__ void init_spins(const JP& P, uint32_t base, uint32_t j, int lt_, int T, int pitch) {
  const LdsMem mem;
  for (int q = lt_; q < P.traj_words; q += T) {
    const InitWord I = init_word(P, j, q);
    const int at = PM ? (I.rowg - I.rho + pm_row(P, I.rho)) * pitch + I.w : q;
    st_words<1>(mem, base + 4u * (uint32_t)at, &I.word);
  }
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
    if (flags & ee::kFlagInit) init_spins<PM>(P, L, j, lt_, T, pitch);
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
EE_SWEEP_KERNEL(const JobDev* single_job, int single_k, const Unit* units, int n_units, int* queue,
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

}  // namespace
