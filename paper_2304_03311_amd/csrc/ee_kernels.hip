// ee_kernels.hip -- gfx950 kernels of the non-equilibrium Renyi-entropy
// estimator (Bulgarelli & Panero, arXiv:2304.03311).
//
// sweep_kernel (ee_sweep.hpp): one workgroup holds k trajectories of one job
//   in LDS and runs all their sweeps on chip.  One lane updates W 32-bit
//   words = 4W same-colour sites of a row.  One Philox4x32-10 call gives a
//   16-bit field to each of 8 sites; a site accepts when its field is below
//   the top half of its uint32 threshold, and only a tie (probability 2^-16)
//   draws the low 16 bits from a second call.  In batch mode the workgroups
//   are persistent and pull work units (job, block of trajectories) from a
//   device queue.
// stream_row_kernel: one colour of every trajectory of a job that stays in
//   HBM; march_kernel and march_fixup_kernel: the same jobs plane by plane
//   through LDS, on request.
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

// ---------------------------------------------------------------------------
// Streaming path: lattices larger than one workgroup's LDS.  The spins stay
// in HBM (INT8 colour planes); one launch updates one colour of every
// trajectory of a job.  The grid is one-dimensional, `blocks` workgroups per
// trajectory, mapped to trajectories as below; of a trajectory's row slots,
// slot s takes the rows s, s + slots, ... in storage order, one lane per W
// words.  The neighbour rows are read through the vector caches, and the
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

// The trajectory, row slot and first word of a lane of a streaming
// launch; false for a lane past the last slot.
__device__ __forceinline__ bool stream_lane(const ee::StreamArgs& a, int W, uint32_t& j, int& slot, int& w) {
  const int id = blockIdx.x, x = id % kXcd, k = id / kXcd;
  const int logical = x * a.q8 + min(x, a.rem8) + k;  // as xcd_block
  const int jj = (int)fdiv((uint32_t)logical, a.bx.mul, a.bx.shift);
  const int lane = (logical - jj * a.blocks) * 256 + (int)threadIdx.x;
  j = (uint32_t)jj;
  slot = (int)fdiv((uint32_t)lane, a.gw.mul, a.gw.shift);
  w = (lane - slot * (a.P.G / W)) * W;
  return lane < a.lanes;
}

// One row at a time, in storage order over the lanes: consecutive lanes read
// consecutive words.  (Pairs of neighbouring rows per lane, as on chip, cost
// 150 instead of 190 instructions a row but read every other row: 4.9 against
// 3.7 ms on 96^3 and 9.2 against 7.1 ms on the cylinder below, though 5.3
// against 5.5 ms on 48^3.)  Bound by memory on large jobs: 3D 96^3 x 32
// trajectories 17.0 us a launch, 5.0 TB/s on its 3 B per attempt, as fast as a
// large copy.  What is the same for every lane comes by value in the
// arguments, with the multipliers of its divisions, and the lanes have no
// barrier; made from the job's description in memory, behind one dependent
// load after the other, it was a fifth of the time and kept small jobs at four
// rows per lane: 96^3 x 32, 110 sweeps 4.05 -> 3.75 ms, 48^3 x 16, 600 sweeps
// 7.72 -> 5.52 ms, the 2D L = 128 cylinder x 256, 200 sweeps 7.95 -> 7.12 ms.
// Each colour plane has a base of its own, since a trajectory may pass 4 GiB:
// 3.73, 5.24 and 7.09 ms, 2D 1760 x 220 x 20, 158 sweeps 3.42 -> 3.36 ms.
template <int DIM, bool FULL, int W>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
stream_row_kernel(ee::StreamArgs a, int c, uint32_t g, int pos, int dpos, int work) {
  const JP& P = a.P;
  uint32_t j;
  int slot, w;
  if (!stream_lane(a, W, j, slot, w)) return;
  uint32_t* const traj = P.spins + (uint64_t)j * (uint32_t)P.traj_words;
  const HbmMem own{traj + plane_start(a.rows, P.G, c)}, oth{traj + plane_start(a.rows, P.G, c ^ 1)};
  PhKey K;
  key_unit(K, P);
  key_sweep(K, P, g, j);
  const int G = P.G, LyG = P.ly * G, ltLyG = P.lt * LyG;
  const int wl = (w == 0) ? G - 1 : w - 1, wr = (w + W == G) ? 0 : w + W;
  int dI = 0;
  for (int m = slot; m < a.rows; m += a.slots) {
    const int r = (int)fdiv((uint32_t)m, P.mR, P.sR);
    const int rho = m - r * P.R;
    const int t = (DIM == 2) ? rho : (int)fdiv((uint32_t)rho, P.mLy, P.sLy);
    const int y = (DIM == 2) ? 0 : rho - t * P.ly;
    const int tpo = LyG - ((t == P.lt - 1) ? ltLyG : 0);
    const int ymo = (y == 0) ? (P.ly - 1) * G : -G;
    const int ypo = (y == P.ly - 1) ? -(P.ly - 1) * G : G;
    const uint32_t c0 = (uint32_t)(rho * P.G8 + (w >> 1));
    const uint32_t c3 = (1u << 28) | ((uint32_t)r << 1) | (uint32_t)c;
    K.x0 = c3 ^ P.key1;
    // opaque to the compiler (the empty asm statement emits nothing): it would
    // carry an induction variable per access, some 30 instructions more
    uint32_t off = plane_byte(m * G + w);
    asm volatile("" : "+v"(off));
    const auto row = [&](auto cut) {
      constexpr bool CUT = decltype(cut)::value;
      const int tmo = -LyG + ((CUT && t == 0) ? ltLyG : 0);
      const uint32_t ag = (CUT && t <= 1) ? plane_byte(glued_row(P, r, t, y) * G + w) : off;
      update_row<DIM, FULL, W, CUT, false>(P, K, own, off, oth, off, oth, ag, w, wl, wr, a.thr, c, g, j, pos, dpos,
                                           work != 0, dI, t, y, tmo, tpo, ymo, ypo, c0, c3);
    };
    if (__builtin_amdgcn_ballot_w64(t <= 1) != 0) row(std::true_type{});
    else row(std::false_type{});
  }
  if (dI != 0) atomicAdd(reinterpret_cast<unsigned long long*>(&P.work[j]), (unsigned long long)(long long)dI);
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
  const HbmMem hbm{traj + plane_start(P.n * P.R, G, 1)};  // the glued partners' plane
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
    const int ogl = (rgl * P.R + (1 - t) * ly) * G;
    RowDesc d = d0;
    for (int it = threadIdx.x; it < ly * GW;) {
      const int y = d.y, w = d.w;
      const int wl = (w == 0) ? G - 1 : w - 1, wr = (w + W == G) ? 0 : w + W;
      const int ymo = (y == 0) ? (ly - 1) * G : -G, ypo = (y == ly - 1) ? -(ly - 1) * G : G;
      const uint32_t c0 = (uint32_t)((t * ly + y) * P.G8 + (w >> 1));
      const uint32_t off = 4u * (uint32_t)(y * G + w);
      update_row<DIM, FULL, W, CUT, false>(P, K, mem, own + off, mem, oth + off, hbm, CUT ? plane_byte(ogl) + off : 0u,
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
  const HbmMem own{traj + plane_start(P.n * R, G, 1)}, oth{traj};
  PhKey K;
  key_unit(K, P);
  key_sweep(K, P, g, j);
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
      const uint32_t off = plane_byte(rowbase + w);
      const uint32_t ag = CUT ? plane_byte(glued_row(P, r, t, y) * G + w) : off;
      update_row<DIM, FULL, W, CUT, false>(P, K, own, off, oth, off, oth, ag, w, wl, wr, thr, 1, g, j, pos, dpos,
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
  if (lt_ >= lanes) return;
  uint32_t* const traj = P.spins + (size_t)j * P.traj_words;
  // unsigned: the last step may pass 2^31
  for (uint32_t q = (uint32_t)lt_; q < (uint32_t)P.traj_words; q += (uint32_t)lanes)
    traj[q] = init_word(P, j, (int)q).word;
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
// term for a wave alone on its SIMD), and how many of the n^2 adds of the
// leave-one-out sums run beside each other.  Up to kEstSmall trajectories one workgroup does a job
// (estimate_kernel): lane i forms sum i, lane n the full sum, all in one walk
// over the e_j in LDS, and one more wave the other sums.  Above, four
// launches: the exponentials over many workgroups (est_exp_kernel), the plain
// sums in one wave per job (est_sum_kernel), the leave-one-out sums in one
// wave per 64 of them (est_loo_kernel) and their spread (est_err_kernel).
// Sums i of a wave start from the full sum's prefix, which is their own
// beginning.  16384 trajectories: 0.64 against 9.8 ms in one workgroup; 64
// jobs of 1024: 59 against 145 us; 8 trajectories: 9 against 29 us.  From the
// first launch's start to the last one's end, one workgroup / four launches:
// 64 trajectories 8 / 45 us, 512 34 / 51, 640 41 / 54, 768 54 / 52, 895 66 / 65,
// 958 70 / 67: they meet at 700 to 900, and the line (kEstSmall) lies there.
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

// The on-chip sweep kernel, with the whole-region protocol where a job of the
// launch needs it.
int ee_k_sweep_kernel_ptr(int whole, const void** fn) {
  return whole ? ee_k_sweep_whole_ptr(fn) : ee_k_sweep_plain_ptr(fn);
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

int ee_k_launch_sweep(int whole, const ee::JobDev* single_job, int single_k, const ee::Unit* units, int n_units,
                      int* queue, const ee::JobDev* const* jobtab, uint32_t flags, int n_therm, int g0, int grid,
                      int block, int lds_bytes, void* stream) {
  const void* fn = nullptr;
  hipError_t e = (hipError_t)ee_k_sweep_kernel_ptr(whole, &fn);
  if (e != hipSuccess) return (int)e;
  int tail = ee::sweep_tail_words(lds_bytes);
  void* args[] = {&single_job, &single_k, &units, &n_units, &queue, &jobtab, &flags, &n_therm, &g0, &tail};
  return (int)hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds_bytes + ee::kSweepTailBytes, (hipStream_t)stream);
}

int ee_k_launch_stream(const ee::StreamArgs* a, int W, int n_traj, int c, uint32_t g, int pos, int dpos, int work,
                       void* stream) {
  const auto go = [&](auto dim, auto w, auto full) {
    hipLaunchKernelGGL((stream_row_kernel<decltype(dim)::value, decltype(full)::value, decltype(w)::value>),
                       dim3(a->blocks * n_traj), dim3(256), 0, (hipStream_t)stream, *a, c, g, pos, dpos, work);
  };
  const auto width = [&](auto dim) {
    using T_ = std::true_type;
    if ((a->P.H & 3) != 0) go(dim, std::integral_constant<int, 1>{}, std::false_type{});
    else if (W == 4) go(dim, std::integral_constant<int, 4>{}, T_{});
    else if (W == 3) go(dim, std::integral_constant<int, 3>{}, T_{});
    else if (W == 2) go(dim, std::integral_constant<int, 2>{}, T_{});
    else go(dim, std::integral_constant<int, 1>{}, T_{});
  };
  if (a->P.dim == 3) width(std::integral_constant<int, 3>{});
  else width(std::integral_constant<int, 2>{});
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
