// ee_rows.hpp -- the Metropolis update of rows of one colour, shared by the
// on-chip sweep kernel and the HBM-streaming kernels: the random numbers, the
// neighbour counts, the acceptance, the rows next to the cut.
//
// What bounds this code is the VALU issue: a wave64 instruction takes four
// cycles of its SIMD whatever it does (two for a plain 32-bit xor, add, and,
// right shift or three-input bitwise operation on vector registers, if another
// wave has such an instruction ready at the same time; a scalar-register
// operand loses that).  So the sequence below is chosen for few instructions
// first, and keeps what is uniform but used in three-input operations (the
// Philox keys) in vector registers.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ee_internal.hpp"
#include "ee_lanes.hpp"

// Whether the whole-region protocol is compiled in.  Its code takes registers
// from the rows next to the cut in every protocol, so the on-chip kernel
// exists without it and with it.
#ifndef EE_WHOLE
#define EE_WHOLE 1
#endif

namespace {

using ee::JobDev;
using ee::Unit;
using namespace ee::lanes;

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T* uni_ptr(T* p) {
  uint64_t v = reinterpret_cast<uint64_t>(p);
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ JP load_jp(const JobDev* J) {
  JP P;
  P.dim = uni(J->dim);
  P.n = uni(J->n); P.lt = uni(J->lt); P.ly = uni(J->ly); P.l = uni(J->l); P.N = uni(J->N);
  P.S = uni(J->S); P.subsets = uni(J->subsets); P.whole = EE_WHOLE ? uni(J->whole) : 0;
  P.H = uni(J->H); P.G = uni(J->G); P.R = uni(J->R); P.traj_words = uni(J->traj_words);
  P.G8 = (P.H + 7) >> 3;
  P.packed_row_words = (P.H + 31) >> 5;
  P.key0 = uni(J->key0); P.key1 = uni(J->key1);
  P.thr0 = uni(J->thr_bulk[0]); P.thr1 = uni(J->thr_bulk[1]); P.thr2 = uni(J->thr_bulk[2]);
  P.reverse = uni(J->reverse); P.spin_format = uni(J->spin_format);
  P.pt_hi0 = uni(J->pt[0]); P.pt_hi1 = uni(J->pt[1]);
  P.pt_lo0 = uni(J->pt[2]); P.pt_lo1 = uni(J->pt[3]);
  P.mR = uni(J->magic_R); P.sR = uni(J->shift_R); P.mLy = uni(J->magic_Ly); P.sLy = uni(J->shift_Ly);
  P.ramp = uni_ptr(J->ramp_thr);
  P.spins = uni_ptr(J->spins);
  P.work = uni_ptr(J->work);
  return P;
}

// Full 32-bit thresholds by neighbour index (see nbr_index): entry i of the
// LDS table that the tie path reads.
__device__ __forceinline__ uint32_t thr_entry(const JP& P, int dim, int i) {
  if (dim == 2 && i >= 4) i = 7 - i;
  return (i == 0) ? P.thr0 : (i == 1) ? P.thr1 : (i == 2 && dim == 3) ? P.thr2 : 0xFFFFFFFFu;
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 products;
// the two xors of each output word are one 3-input bitwise op (table 0x96).
// ---------------------------------------------------------------------------
constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
constexpr uint32_t kHalfBias = 0x80008000u;  // v ^ 0x8000 of both 16-bit fields of a word

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const uint64_t p0 = (uint64_t)kM0 * c0;
    const uint64_t p1 = (uint64_t)kM1 * c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += kW0;
    k1 += kW1;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// A value kept in a vector register as it is (the empty asm statement emits
// nothing): the compiler would otherwise keep a uniform value in a scalar
// register, or recompute it at each use.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The part of the sweep calls (counter (c0, g, j, c3)) that is the same for
// all calls of a lane in one half-sweep: the round keys, and of the first
// rounds what depends on g and j only.  The first round's second product
// (M1 j) and the second round's first one (M0 n0, n0 from g and j) are done
// once per sweep; a call is left with 18 of the 20 products.
//   x0  c3 ^ key1 (per half-sweep: c3 holds the colour)
//   x1, x2, x3  round 1: the word that joins hi(p1), the one that joins
//       lo(M0 c0), and round 2: the one that joins hi(p0)
//   a, b  the keys of rounds 2..9 and 3..9; the last ones carry the field
//       bias of the output words 0 and 2
struct PhKey {
  uint32_t x0, x1, x2, x3, a[8], b[7];
};

__device__ __forceinline__ void key_unit(PhKey& K, const JP& P) {
#pragma unroll
  for (int i = 0; i < 8; ++i) K.a[i] = in_vgpr((P.key0 + (uint32_t)(i + 2) * kW0) ^ (i == 7 ? kHalfBias : 0u));
#pragma unroll
  for (int i = 0; i < 7; ++i) K.b[i] = in_vgpr((P.key1 + (uint32_t)(i + 3) * kW1) ^ (i == 6 ? kHalfBias : 0u));
}

__device__ __forceinline__ void key_sweep(PhKey& K, const JP& P, uint32_t g, uint32_t j) {
  const uint64_t p = (uint64_t)kM1 * j;
  const uint64_t q = (uint64_t)kM0 * xor3((uint32_t)(p >> 32), g, P.key0);
  K.x1 = in_vgpr((uint32_t)p ^ (P.key0 + kW0));
  K.x2 = in_vgpr((uint32_t)(q >> 32) ^ (P.key1 + kW1));
  K.x3 = in_vgpr((uint32_t)q ^ (P.key1 + 2 * kW1));
}

// NC calls side by side (two to four independent chains: a single call's
// rounds wait for its own products), every 16-bit field as v ^ 0x8000.
// Measured on its own at four waves per SIMD: 198 cycles a call one at a time
// with scalar keys, 155 two at a time and 150 four at a time with the keys in
// vector registers.
template <int NC>
__device__ __forceinline__ void philox_rows(const PhKey& K, const uint32_t c0[NC], uint32_t u[NC][4]) {
  uint32_t w0[NC], w1[NC], w2[NC], w3[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const uint64_t p0 = (uint64_t)kM0 * c0[k];
    const uint64_t p1 = (uint64_t)kM1 * ((uint32_t)(p0 >> 32) ^ K.x0);
    w0[k] = (uint32_t)(p1 >> 32) ^ K.x1;
    w1[k] = (uint32_t)p1;
    w2[k] = (uint32_t)p0 ^ K.x2;
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const uint64_t p0 = (uint64_t)kM0 * w0[k];
    const uint64_t p1 = (uint64_t)kM1 * w2[k];
    w0[k] = xor3((uint32_t)(p1 >> 32), w1[k], K.a[0]);
    w2[k] = (uint32_t)(p0 >> 32) ^ K.x3;
    w1[k] = (uint32_t)p1;
    w3[k] = (uint32_t)p0;
  }
#pragma unroll
  for (int i = 0; i < 7; ++i) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const uint64_t p0 = (uint64_t)kM0 * w0[k];
      const uint64_t p1 = (uint64_t)kM1 * w2[k];
      w0[k] = xor3((uint32_t)(p1 >> 32), w1[k], K.a[i + 1]);
      w2[k] = xor3((uint32_t)(p0 >> 32), w3[k], K.b[i]);
      w1[k] = (uint32_t)p1;
      w3[k] = (uint32_t)p0;
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    u[k][0] = w0[k];
    u[k][1] = w1[k] ^ kHalfBias;
    u[k][2] = w2[k];
    u[k][3] = w3[k] ^ kHalfBias;
  }
}

// Output word o (0..3, possibly not a compile-time constant) of a Philox
// result, by selects rather than a dynamically indexed register array.
__device__ __forceinline__ uint32_t pick4(const uint32_t u[4], int o) {
  const uint32_t lo = (o & 1) ? u[1] : u[0];
  const uint32_t hi = (o & 1) ? u[3] : u[2];
  return (o & 2) ? hi : lo;
}

// 16-bit half hi (0 low, 1 high) of a Philox output word.
__device__ __forceinline__ uint32_t half16(uint32_t word, int hi) { return hi ? (word >> 16) : (word & 0xFFFFu); }

// Ramp position (0..S) of row y when the protocol stands at position pos
// (0..N): every row follows pos, or (subset protocol) row y moves during
// steps [y S, (y+1) S).
__device__ __forceinline__ int row_m(const JP& P, int y, int pos) {
  if (!P.subsets) return pos;
  const int m = pos - y * P.S;
  return m < 0 ? 0 : (m > P.S ? P.S : m);
}

// Two 16-bit lanes per 32-bit word: saturating signed difference a - b, and
// unsigned minimum (v_pk_sub_i16 with clamp, v_pk_min_u16).
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t sub_sat_s16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(s16x2, a),
                                                                    __builtin_bit_cast(s16x2, b)));
}
__device__ __forceinline__ uint32_t min_u16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ bool tied(uint32_t d) { return ((d & 0xFFFFu) == 0) | ((d >> 16) == 0); }

// ---------------------------------------------------------------------------
// Spin words in memory.  A location is a byte address: in LDS, or relative to
// the start of a colour plane of the trajectory in device memory (ee_lanes.hpp:
// plane_start, plane_byte).  The W consecutive words of
// a lane are one 4W-byte access.  Where W is 2 or 4, the address is 4W-byte
// aligned (the row pitch G and every plane and trajectory offset are
// multiples of W), and the lanes of a wave cover consecutive LDS banks; W
// separate dword accesses at a lane stride of W words would conflict W-fold.
// W = 3 (rows of three words, one lane per row) reads dwords: an odd lane
// stride does not conflict.  Device memory is reached through the global
// address space: a flat access, which is what a pointer of unknown space
// compiles to, also counts against the LDS/scalar wait counter.
// ---------------------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct LdsMem {
  template <typename T>
  using ptr = __attribute__((address_space(3))) T*;
  template <typename T>
  __device__ __forceinline__ ptr<T> at(uint32_t a) const { return (ptr<T>)(uintptr_t)a; }
};
struct HbmMem {
  uint32_t* base;  // a colour plane of the trajectory (uniform)
  template <typename T>
  using ptr = __attribute__((address_space(1))) T*;
  template <typename T>
  __device__ __forceinline__ ptr<T> at(uint32_t a) const { return (ptr<T>)((ptr<uint8_t>)base + a); }
};

template <typename M>
__device__ __forceinline__ uint32_t ld_word(const M& m, uint32_t a) { return *m.template at<const uint32_t>(a); }

template <int W, typename M>
__device__ __forceinline__ void ld_words(const M& m, uint32_t a, uint32_t v[W]) {
  if constexpr (W == 4) {
    const u32x4 x = *m.template at<const u32x4>(a);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  } else if constexpr (W == 2) {
    const u32x2 x = *m.template at<const u32x2>(a);
    v[0] = x.x; v[1] = x.y;
  } else {
#pragma unroll
    for (int q = 0; q < W; ++q) v[q] = ld_word(m, a + 4u * q);
  }
}
template <int W, typename M>
__device__ __forceinline__ void st_words(const M& m, uint32_t a, const uint32_t v[W]) {
  if constexpr (W == 4) {
    *m.template at<u32x4>(a) = u32x4{v[0], v[1], v[2], v[3]};
  } else if constexpr (W == 2) {
    *m.template at<u32x2>(a) = u32x2{v[0], v[1]};
  } else {
#pragma unroll
    for (int q = 0; q < W; ++q) *m.template at<uint32_t>(a + 4u * q) = v[q];
  }
}

// ---------------------------------------------------------------------------
// Neighbour index of the four sites of a word (one per byte), from the words
// of the neighbours (bit 0 of each byte is 1 for spin +1) and of the sites
// themselves.  The index selects the site's threshold.
//   2D: the sum of the four neighbours plus 3 s.  For s = 0 it is the number
//       a of anti-aligned neighbours, for s = 1 it is 7 - a; of the values
//       that both give (3 and 4) all stand for a >= 2, so the threshold table
//       [t0 t1 F F F F t1 t0] serves both (F: every attempt accepted).
//   3D: a itself, as ((sum of the six neighbours) + s) ^ 7 s.
// ---------------------------------------------------------------------------
template <int DIM>
__device__ __forceinline__ uint32_t nbr_index(uint32_t S, uint32_t A, uint32_t B, uint32_t T0, uint32_t T1,
                                              uint32_t Y0, uint32_t Y1) {
  if constexpr (DIM == 2) return (A + B + T0) + (T1 + (S << 1)) + S;
  // perm: byte 0 -> 0, 1 -> 7
  return ((A + B + T0) + T1 + Y0 + Y1 + S) ^ __builtin_amdgcn_perm(0u, 0x00000700u, S);
}

// Anti-aligned counts per byte from the index.
template <int DIM>
__device__ __forceinline__ uint32_t anti_count(uint32_t idx, uint32_t S) {
  if constexpr (DIM == 2) return idx ^ __builtin_amdgcn_perm(0u, 0x00000700u, S);
  return idx;
}

// x neighbours (the word of the other side; the near side is A itself): the
// sites' x-1 (p = 0) or x+1 (p = 1) neighbours straddle two words.  E: the
// word left of (p = 0) or right of (p = 1) the lane's words.
template <int W, int PAR>
__device__ __forceinline__ void x_words(const uint32_t A[W], uint32_t E, int p, uint32_t B[W]) {
  if (PAR >= 0) p = PAR;
  const uint32_t sh = p ? 1u : 3u;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    const uint32_t nxt = (q + 1 < W) ? A[q + 1] : E;
    const uint32_t prv = (q > 0) ? A[q - 1] : E;
    B[q] = __builtin_amdgcn_alignbyte(p ? nxt : A[q], p ? A[q] : prv, sh);
  }
}

// What the rows next to the cut (t = 0, 1) add, per row of a lane.
//   on   the row is one of them;  p its x parity;  y its y
//   ramp it holds the ramped site x = l among the lane's words
//   Tc   own-replica partner words across the cut, Tg the glued partners'
template <int W>
struct CutRow {
  bool on, ramp;
  int p, y;
  uint32_t Tc[W], Tg[W];
};

// The partners counted in the bulk sum: the glued ones where bit 0 of the
// bytes of gm[q] (glued_bits; other bits do not matter) is set.
template <int W>
__device__ __forceinline__ void cut_partner(const CutRow<W>& cr, const uint32_t gm[W], uint32_t Te[W]) {
#pragma unroll
  for (int q = 0; q < W; ++q) Te[q] = __builtin_amdgcn_bitop3_b32(gm[q], cr.Tg[q], cr.Tc[q], 0xCA);
}

// The Philox outputs of one row of a lane.  Callers make them between the
// loads of the rows' words and their first use: some 300 cycles in which the
// loads complete.
template <int W>
__device__ __forceinline__ void fields_of_row(const PhKey& K, const uint32_t c0, uint32_t U[(W + 1) / 2][4]) {
  constexpr int NC = (W + 1) / 2;
  uint32_t cc[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) cc[k] = c0 + k;
  __builtin_amdgcn_sched_barrier(0);
  philox_rows<NC>(K, cc, U);
  __builtin_amdgcn_sched_barrier(0);
}

// The acceptance of NR rows of a lane, W words (4W sites) each.
//   S, idx  the spins and neighbour indices; Sn gets the new spins
//   c0, c3  Philox counter words 0 (of each row's first call) and 3
//   w       first word of the lane in its rows;  fmask: bit 0 of every real
//           site's byte, per word
//   thr     LDS table of full thresholds by neighbour index
//   cr      rows next to the cut (CUT only)
//   pos, dpos, work, dI  protocol position, its step (0 while thermalising),
//           whether the work is taken, and the lane's work
//   U       the rows' Philox outputs (fields_of_row)
//   partners(r, Tc, Tg)  loads row r's partner words across the cut again
//           (for the whole-region protocol; in registers they would have to
//           be kept over the whole update, in every protocol)
template <int DIM, int W, int NR, bool CUT, typename Partners>
__device__ __forceinline__ void decide_rows(const JP& P, const uint32_t U[NR * ((W + 1) / 2)][4],
                                            const uint32_t c0[NR], const uint32_t c3, const uint32_t g,
                                            const uint32_t j, const int w, const uint32_t fmask[W],
                                            const uint32_t* __restrict__ thr, const uint32_t S[NR][W],
                                            const uint32_t idx[NR][W], const CutRow<W>* cr, const int pos,
                                            const int dpos, const bool work, int& dI, uint32_t Sn[NR][W],
                                            Partners partners) {
  constexpr int NC = (W + 1) / 2;  // Philox calls per row: 8 sites each
  // Word q of the lane has its fields in call q >> 1 from output word
  // (ob + 2q) & 3 on: sites 0, 1 in one output word, sites 2, 3 in the next.
  const int ob = (W == 1) ? 2 * (w & 1) : 0;

  // Rows next to the cut: the threshold of the ramped site x = l (one lane
  // per row), K = s (S a_fix + (S-m) s_intra + m s_inter) in units of beta/S,
  // is read before the bulk decision, which hides its latency.
  const int ramp_sh = 8 * ((P.l >> 1) & 3);
  const int rq = ramp_word<W>(P);
  uint32_t Ur[NR];
  if constexpr (CUT) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      Ur[r] = 0;
      if (cr[r].ramp) {
        const int m = row_m(P, cr[r].y, pos);
        int dm2 = 0;
        if (work) dm2 = 2 * (m - row_m(P, cr[r].y, pos - dpos));
#pragma unroll
        for (int q = 0; q < W; ++q) {
          if (rq != q) continue;
          const uint32_t bw = cr[r].Tc[q] ^ S[r][q], cw = cr[r].Tg[q] ^ S[r][q];
          // x = l is not glued: its partner across the cut counted in idx is
          // the own replica's
          const uint32_t fa = ((anti_count<DIM>(idx[r][q], S[r][q]) >> ramp_sh) & 0xFFu) - ((bw >> ramp_sh) & 1u);
          const uint32_t bb = (bw >> ramp_sh) & 1u;
          const uint32_t cc = (cw >> ramp_sh) & 1u;
          Ur[r] = P.ramp[m * (8 * DIM) + fa * 4 + bb * 2 + cc];
          // the ramped site of colour 0 sees phi_k: its bonds' weights moved
          // by (m - m_prev), so the D_k term is (m - m_prev) 2 (b - c)
          if (work) dI += dm2 * ((int)bb - (int)cc);
        }
      }
    }
  }

  // The decision u <= U with u = 2^16 v + w is v < U >> 16 unless v equals
  // U >> 16; only then is w (a phase-2 call) needed.  Both sides are
  // compared two sites at a time as 16-bit lanes: d = sat(v' - t) with
  // v' = v ^ 0x8000 and t = (U >> 16) ^ 0x8000 has the sign of
  // v - (U >> 16), and d = 0 marks a tie.  t of the four sites comes from
  // byte tables selected by the index; a byte permute spreads the four signs
  // over their bytes.
  uint32_t f[NR][W];   // per site: 0xFF flip, 0 keep
  uint32_t dmk[NR * NC];  // per call: minimum of its d's (a zero half marks a tie)
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const uint32_t* u = U[r * NC + k];
      uint32_t dm = 0xFFFFFFFFu;
#pragma unroll
      for (int q = 2 * k; q < 2 * k + 2 && q < W; ++q) {
        const uint32_t th = __builtin_amdgcn_perm(P.pt_hi1, P.pt_hi0, idx[r][q]);
        const uint32_t tl = __builtin_amdgcn_perm(P.pt_lo1, P.pt_lo0, idx[r][q]);
        const int o = (ob + 2 * q) & 3;
        const uint32_t d01 = sub_sat_s16x2(pick4(u, o), __builtin_amdgcn_perm(th, tl, 0x05010400u));
        const uint32_t d23 = sub_sat_s16x2(pick4(u, o + 1), __builtin_amdgcn_perm(th, tl, 0x07030602u));
        const uint32_t mn = min_u16x2(d01, d23);
        dm = (q == 2 * k) ? mn : min_u16x2(dm, mn);
        f[r][q] = __builtin_amdgcn_perm(d23, d01, 0x0B0A0908u);  // sign of each 16-bit half
      }
      dmk[r * NC + k] = dm;
    }
  uint32_t dmin = dmk[0];
#pragma unroll
  for (int k = 1; k < NR * NC; ++k) dmin = min_u16x2(dmin, dmk[k]);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(tied(dmin)) != 0, 0)) {
    // rare (2^-16 per site): decide the tied sites on u = 2^16 v + w, with
    // the phase-2 call of only the calls that have a tie
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        if (!tied(dmk[r * NC + k])) continue;
        uint32_t u2[4];
        philox10(c0[r] + k, g, j, c3 + (1u << 28), P.key0, P.key1, u2);
#pragma unroll
        for (int q = 2 * k; q < 2 * k + 2 && q < W; ++q) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t th = thr[(idx[r][q] >> (8 * i)) & 0xFFu];
            const int o = ((ob + 2 * q) & 3) + (i >> 1);
            if ((half16(pick4(U[r * NC + k], o), i & 1) ^ 0x8000u) == (th >> 16)) {
              const bool acc = half16(pick4(u2, o), i & 1) <= (th & 0xFFFFu);
              f[r][q] = (f[r][q] & ~(0xFFu << (8 * i))) | (acc ? 0xFFu << (8 * i) : 0u);
            }
          }
        }
      }
  }

  if constexpr (CUT) {
    // the ramped sites (one column, or with the whole-region protocol every
    // column x < l), decided after the bulk and tie decisions, which they
    // replace for their bytes
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (cr[r].ramp) {
#pragma unroll
        for (int q = 0; q < W; ++q) {
          if (rq != q) continue;
          const int ri = ramp_sh >> 3;
          const int o = ((ob + 2 * q) & 3) + (ri >> 1);
          const uint32_t vr = half16(pick4(U[r * NC + (q >> 1)], o), ri & 1) ^ 0x8000u;
          bool acc = vr < (Ur[r] >> 16);
          if (vr == (Ur[r] >> 16)) {
            uint32_t u2[4];
            philox10(c0[r] + (q >> 1), g, j, c3 + (1u << 28), P.key0, P.key1, u2);
            acc = half16(pick4(u2, o), ri & 1) <= (Ur[r] & 0xFFFFu);
          }
          f[r][q] = (f[r][q] & ~(0xFFu << ramp_sh)) | (acc ? 0xFFu << ramp_sh : 0u);
        }
      }
      if (P.whole && cr[r].on && 8 * w + cr[r].p < P.l) {
        // whole-region protocol: every site x < l of a row next to the cut is
        // ramped and none is glued.  Per site K = s (S a_fix + (S-m) s_intra +
        // m s_inter) from the ramp table, replacing the bulk decision.
        const int m = row_m(P, cr[r].y, pos);
        const uint32_t* __restrict__ Um = P.ramp + m * (8 * DIM);
        uint32_t Tc[W], Tg[W], gm[W];
        partners(r, Tc, Tg);
        glued_bits<W>(P, true, cr[r].p, w, gm);
        // word by word: the four sites' thresholds first (sites that are not
        // ramped read one too), so that their loads are in flight together
#pragma unroll
        for (int q = 0; q < W; ++q) {
          if (gm[q] == 0) continue;
          const uint32_t bw = Tc[q] ^ S[r][q];  // intra partner anti-aligned (bit 0 of each byte)
          const uint32_t cw = Tg[q] ^ S[r][q];  // inter partner anti-aligned
          const uint32_t fw = anti_count<DIM>(idx[r][q], S[r][q]) - bw;  // the 2 dim - 1 fixed neighbours
          const uint32_t at = 4u * fw + 2u * bw + cw;                     // table index per byte
          uint32_t Uw[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) Uw[i] = Um[min((at >> (8 * i)) & 0xFFu, 8u * DIM - 1u)];
          if (work) {
            // colour-0 ramped sites see phi_k; each adds (m - m_prev) 2 (b - c)
            const int dm = m - row_m(P, cr[r].y, pos - dpos);
            dI += dm * 2 * (__popc(bw & gm[q]) - __popc(cw & gm[q]));
          }
          uint32_t acc = 0, ties = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int o = ((ob + 2 * q) & 3) + (i >> 1);
            const uint32_t vr = half16(pick4(U[r * NC + (q >> 1)], o), i & 1) ^ 0x8000u;
            acc |= (vr < (Uw[i] >> 16)) ? 0xFFu << (8 * i) : 0u;
            ties |= (vr == (Uw[i] >> 16)) ? 1u << (8 * i) : 0u;
          }
          if ((ties & gm[q]) != 0) {
            uint32_t u2[4];
            philox10(c0[r] + (q >> 1), g, j, c3 + (1u << 28), P.key0, P.key1, u2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int o = ((ob + 2 * q) & 3) + (i >> 1);
              const bool up = half16(pick4(u2, o), i & 1) <= (Uw[i] & 0xFFFFu);
              if ((ties >> (8 * i)) & 1u) acc = (acc & ~(0xFFu << (8 * i))) | (up ? 0xFFu << (8 * i) : 0u);
            }
          }
          f[r][q] = __builtin_amdgcn_bitop3_b32(gm[q] * 0xFFu, acc, f[r][q], 0xCA);
        }
      }
    }
  }
  // S ^ (f & fmask) in one three-input op (table 0x78 = a ^ (b & c))
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int q = 0; q < W; ++q) Sn[r][q] = __builtin_amdgcn_bitop3_b32(S[r][q], f[r][q], fmask[q], 0x78);
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;

__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const lds_u32*)(const uint32_t*)p;
}

// The Metropolis update of the sites of one row of colour c that a lane owns
// (words w .. w+W-1 of the row), parity of the row known only at run time.
//   own, aC and oth, aO  locations of word w of the row in its own colour
//           plane and in the other one
//   tmo, tpo, ymo, ypo  word offsets from aO of the same words in rows t-1,
//           t+1, y-1 and y+1 (periodic)
//   glu, ag  where the glued partner row is (CUT; a location that may be
//           read also for rows away from the cut)
//   (r, t, y)  the row; c0, c3 Philox counter words 0 and 3 of its first call
// FULL: lx/2 is a multiple of 4 (no pad bytes, x-neighbours by byte
// alignment of two words).  W: consecutive words per lane (2 or 4 need
// FULL and a word count that W divides; 3 needs FULL and rows of exactly
// three words, so that w = 0 and words 0, 1 share a Philox call while word
// 2 takes the next one).  CUT: the code for rows next to the cut (t = 0, 1)
// is compiled in; without it the row must have t > 1.
template <int DIM, bool FULL, int W, bool CUT, bool LA, typename M, typename GM>
__device__ __forceinline__ void update_row(const JP& P, const PhKey& K, const M& own, const uint32_t aC, const M& oth,
                                           const uint32_t aO, const GM& glu, const uint32_t ag, const int w,
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
  ld_words<W>(oth, aO, A);
  const uint32_t E = ld_word(oth, at((p ? wr : wl) - w));
  ld_words<W>(own, aC, S[0]);
  ld_words<W>(oth, at(toff0), Tp);
  ld_words<W>(oth, at(toff1), Tm);
  if constexpr (CUT) ld_words<W>(glu, ag, cr[0].Tg);
  uint32_t Ym[W], Yp[W];
  if constexpr (DIM == 3) {
    ld_words<W>(oth, at(ymo), Ym);
    ld_words<W>(oth, at(ypo), Yp);
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
                                ld_words<W>(oth, at(toff0), Tc);
                                ld_words<W>(glu, ag, Tg);
                              });
  st_words<W>(own, aC, Sn[0]);
}

// One half-sweep of colour c over the lane's rows of one trajectory on chip, in
// the order of the lane map.  base: location of the trajectory (two colour
// planes).
template <int DIM, bool FULL, int W>
__device__ __forceinline__ void half_sweep(const JP& P, PhKey& K, const Lane& ln, const LdsMem& mem, const uint32_t base,
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
      update_row<DIM, FULL, W, CUT, false>(P, K, mem, bC + off, mem, bO + off, mem, ag, w, ln.wl, ln.wr, thr, c, g, j, pos,
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

// Initial spins (phase 0 of the Philox streams) of word q of trajectory j in
// storage order: +1 iff u < 2^31.  Word w of row rho of its replica, row rowg
// over colours and replicas.
struct InitWord {
  uint32_t word;
  int w, rowg, rho;
};
__device__ __forceinline__ InitWord init_word(const JP& P, uint32_t j, int q) {
  const int nR = P.n * P.R;
  InitWord I;
  I.w = q % P.G;
  I.rowg = q / P.G;
  const int c = I.rowg / nR;
  const int row = I.rowg - c * nR;
  const int r = row / P.R;
  I.rho = row - r * P.R;
  uint32_t u[4];
  philox10((uint32_t)(I.rho * P.G + I.w), 0u, j, ((uint32_t)r << 1) | (uint32_t)c, P.key0, P.key1, u);
  I.word = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * I.w + i < P.H) I.word |= (uint32_t)(u[i] < 0x80000000u) << (8 * i);
  return I;
}

}  // namespace
