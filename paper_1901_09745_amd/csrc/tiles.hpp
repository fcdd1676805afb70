// Device helpers shared by the step and adjoint kernels: nearest-image
// arithmetic, the Table 1 pair fraction, the LDS image of a tile's particle
// list and its per-cell slot search, tile geometry, and lattice links.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.hpp"

namespace psclbm {

// Minimum-image separation along one axis, as selects (no branch): the
// same sums d - L or d + L as a branch would take, d + 0 otherwise.
__device__ __forceinline__ double min_image(double d, int periodic, int L) {
  const double Ld = (double)L;
  const double hL = 0.5 * Ld;
  double t = d > hL ? -Ld : 0.0;
  t = d < -hL ? Ld : t;
  return periodic ? d + t : d;
}

// The same in FP32 for c - xh, c an integer cell coordinate and xh the FP32
// high part of a centre in [0, L): the difference and the shift by L are
// exact (both are multiples of xh's last place and no larger than L), so the
// arm c - x = min_image(c - xh) - xl rounds once.
__device__ __forceinline__ float min_image_f(float d, int periodic, int L) {
  const float Lf = (float)L;
  const float hL = 0.5f * Lf;
  float t = d > hL ? -Lf : 0.0f;
  t = d < -hL ? Lf : t;
  return periodic ? d + t : d;
}

// ---------------------------------------------------------------------------
// Solid fraction of one (cell, particle) pair, the inside/outside rule of Table 1 with
// Eq. 15/18: eps = V_a(r) + 1/2 - d inside the shell r +- h.
// ---------------------------------------------------------------------------
__device__ inline double pair_eps(double d, double r, double cs, double h) {
  double e;
  if (d >= r + h) e = 0.0;
  else if (d <= r - h) e = 1.0;
  else e = cs - d;
  if (e <= 0.0) e = 0.0;
  if (e >= 1.0) e = 1.0;
  return e;
}

// Square root of v > 0 to FP64 accuracy from the hardware FP32 root, refined
// by one Newton step in FP64 (relative error about 1e-15: the square of the
// FP32 root's), in place of the longer correctly rounded FP64 sequence.
__device__ __forceinline__ double sqrt_nr(double v) {
  const float s = __builtin_amdgcn_sqrtf((float)v);
  const double s0 = (double)s;
  const double res = fma(-s0, s0, v);
  return s > 0.0f ? s0 + res * (double)(0.5f * __builtin_amdgcn_rcpf(s)) : 0.0;
}

// LDS image of a tile's particle list: 96 bytes an entry in either form.
template <typename E>
struct LdsEntryT;
template <>
struct LdsEntryT<double> {
  double x, y, z;
  double r, cs;
  double u[3], w[3];
  int id;
  int pad;
};
template <>
struct LdsEntryT<float> {
  double x, y, z;
  double r, cs;
  // the centre as an FP32 pair, x = xh + xl to FP64 accuracy, and U and
  // Omega rounded to FP32: the FP32 arithmetic forms take u_s = U + Omega x r
  // from these
  float xh[3], xl[3];
  float uf[3], wf[3];
  int id;
  int pad;
};
using LdsEntry = LdsEntryT<double>;

template <typename E>
__device__ __forceinline__ void fill_entry(LdsEntryT<E>& L, const PSnap& P, int id) {
  L.x = P.x[0];
  L.y = P.x[1];
  L.z = P.x[2];
  L.r = P.r;
  L.cs = P.cs;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if constexpr (std::is_same<E, float>::value) {
      L.xh[a] = (float)P.x[a];
      L.xl[a] = (float)(P.x[a] - (double)L.xh[a]);
      L.uf[a] = (float)P.u[a];
      L.wf[a] = (float)P.w[a];
    } else {
      L.u[a] = P.u[a];
      L.w[a] = P.w[a];
    }
  }
  L.id = id;
}

// A tile's particle list: `cnt` particles, the first `held` of them in LDS.  A
// row tile's are all held.  A flat tile meets the particles of several row tiles
// and its list has room for all of theirs, but LDS for half as much again as one
// of them, which is what the lists of most packings reach; the particles past
// that are read from their snapshots at each use.  (300x180x190 with 8000 spheres
// and lists of 64, FP64 / FP32 / FP16: 607 / 350 / 264 us a step, 602 / 344 / 250
// without the look-ups, 614 / 378 / 328 with up to 206 entries in LDS, 723 / 445 /
// 340 in row tiles.)
template <typename E>
struct TileListT {
  LdsEntryT<E>* lds;
  int cnt, held;
  int over;         // the list is longer than what is held (scalar)
  const int* rest;  // ids of the entries from `held` on
  const PSnap* snap;
  __device__ __forceinline__ int id_past(int e) const { return rest[e - held]; }
};
using TileList = TileListT<double>;

// Entry e of the list: the one in LDS, or (MORE: the list may be longer than
// what is held) one filled here.  GUARD: the waves of shorter lists branch over
// the lane's test (the adjoint 76 -> 74 us, 100x80x80; the step, which it costs a
// spilled register, without).
template <bool MORE, bool GUARD = false, typename E>
__device__ __forceinline__ typename std::conditional<MORE, LdsEntryT<E>, const LdsEntryT<E>&>::type
tile_entry(const TileListT<E>& tl, int e) {
  if constexpr (MORE) {
    if ((!GUARD || tl.over) && e >= tl.held) {
      LdsEntryT<E> L;
      fill_entry(L, tl.snap[tl.id_past(e)], tl.id_past(e));
      return L;
    }
  }
  return tl.lds[e];
}

// Slots of one cell: up to KSLOTS particles with eps > 0, ascending particle
// id (lds[e[k]].id).  The fractions are evaluated in FP64 and held as E (FP64,
// or FP32 for the FP32 arithmetic forms, whose weights are formed in FP32).
template <typename E>
struct SlotsT {
  int n;
  int e[KSLOTS];  // index in the tile list
  E eps[KSLOTS];
};
using Slots = SlotsT<double>;

// Workgroup LDS of the slot search: per cell, the slots found so far.
template <typename E>
struct SlotLdsT {
  int n[BLOCK];
  unsigned short e[KSLOTS][BLOCK];  // list entries (a list holds less than 2^15)
  E eps[KSLOTS][BLOCK];
};
using SlotLds = SlotLdsT<double>;

// Inclusive prefix sum of an int over the 64 lanes of a wave, in DPP steps:
// shifts by 1, 2, 4 and 8 within each row of 16 lanes, then the row totals
// carried up by the row broadcasts of lanes 15 and 31.  Every lane of the
// wave must be active.
__device__ __forceinline__ int wave_scan_incl(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 -> rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 -> rows 2, 3
  return v;
}

// The cells of one wave: 64 of a row (row tiles), or 64 consecutive cells of a
// plane in one or more rows (FLAT).  All values are uniform over the wave.
template <bool FLAT>
struct WaveCells {
  int x0, y0, z;  // the first cell
  int rows;       // rows the wave's cells lie in (1 for row tiles)
  int last;       // last lane with a cell, negative when there is none
};

// A list entry's y and z separations are the same for all of a row's cells.
// Phase 1: each lane takes one (list entry, row of the wave) item and, when
// the entry's shell r + h reaches the row, the chord of the row the shell can
// cover (the lanes whose cell centres lie within sqrt((r + h)^2 - dy^2 -
// dz^2) of the centre's nearest image, bounded in FP32 and widened by 1e-3
// lanes, since it only limits the cells examined; on periodic x narrower than
// 64 + 2 (r + h) + 2 the whole row).  Phase 2: the (entry, cell) pairs of all
// chords, laid out item by item by a prefix scan, are taken 64 at a time, one
// per lane: Table 1 for the pair in FP64, and a slot of its cell in LDS when
// the fraction is positive.  Phase 3: each cell reads its slots and orders
// them by particle id.  At most KSLOTS slots are kept per cell (more set
// ERR_SLOTS).  All 64 lanes must call this.
static_assert(SEG == 64, "64 cells a wave");

template <int D, bool FLAT, bool MORE, typename E>
__device__ inline void collect_slots_of(const Geom& g, const WaveCells<FLAT>& wc, bool active,
                                     const TileListT<E>& tl, double h, SlotsT<E>& s,
                                     unsigned* err, SlotLdsT<E>& sl) {
  const int px = g.periodic[0], py = g.periodic[1], pz = g.periodic[2];
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int z = wc.z;
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wbase = tid - lane;
  const int last = wc.last;  // uniform over the wave
  const double Lx = (double)nx;
  // item t: entry t / rows, row t % rows (the quotient is exact: rows <= 64, so
  // (t + 1/2) / rows stays 2^-7 from a whole number, which the product's error,
  // 2^-22 of its value, does not reach below 2^15 entries: a list's limit)
  const int rows = FLAT ? wc.rows : 1;
  const float per_row = FLAT ? __builtin_amdgcn_rcpf((float)rows) : 1.0f;
  auto entry_of = [&](int t) { return FLAT ? (int)(((float)t + 0.5f) * per_row) : t; };
  const int items = tl.cnt * rows;
  sl.n[tid] = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int base = 0; last >= 0 && base < items; base += 64) {
    // phase 1: chords
    const int it = base + lane;
    int chord = 0, lo = 0, wrap = 0, shc = 0, row = 0;
    double dyz2 = 0.0;
    if (it < items) {
      const int ec = entry_of(it);
      row = FLAT ? it - ec * rows : 0;
      // the row's lanes la .. lb; lane l is its cell x = xr + l
      const int xr = wc.x0 - row * nx;
      const int la = FLAT && xr < 0 ? -xr : 0;
      const int lb = FLAT && nx - 1 - xr < last ? nx - 1 - xr : last;
      const auto& P = tile_entry<MORE>(tl, ec);
      const double dy = min_image((double)(wc.y0 + row) - P.y, py, ny);
      dyz2 = dy * dy;
      if constexpr (D == 3) {
        const double dz = min_image((double)z - P.z, pz, nz);
        dyz2 += dz * dz;
      }
      const double rh = P.r + h;
      if (dyz2 < rh * rh) {
        // x-image of the centre nearest the row's middle: shc 1 is -Lx, 2 is +Lx
        const double ddx = (FLAT ? (double)xr + 0.5 * (double)(la + lb) : (double)xr + 31.5) - P.x;
        if (px) shc = ddx > 0.5 * Lx ? 1 : (ddx < -0.5 * Lx ? 2 : 0);
        wrap = px && Lx < 66.0 + 2.0 * rh;
        int hi;
        if (wrap) {
          lo = la;
          hi = lb;
        } else {
          // the chord only bounds the cells examined (their membership is
          // decided in phase 2), so FP32 with a margin of 1e-3 lanes will do
          const double sh = shc == 1 ? -Lx : (shc == 2 ? Lx : 0.0);
          const float half = __builtin_amdgcn_sqrtf((float)(rh * rh - dyz2));
          const float c0 = (float)((P.x - sh) - (double)xr);  // centre's image, in lanes
          const float l = ceilf(c0 - half - 1e-3f), u = floorf(c0 + half + 1e-3f);
          lo = l < (float)la ? la : (int)l;
          hi = u > (float)lb ? lb : (int)u;
        }
        chord = hi >= lo ? hi - lo + 1 : 0;
      }
    }
    const int incl = wave_scan_incl(chord);
    const int off = incl - chord;
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const unsigned long long cmask = __ballot(chord > 0);
    // lo (6 bits), wrap, shc (2 bits), off (at most 64 x 63) and the row in one
    // word for the broadcast (lo past the last lane only where the chord is empty)
    const int pk = (lo & 63) | (wrap << 6) | (shc << 7) | (off << 9) | (row << 22);
    // phase 2: one (entry, cell) pair per lane
    for (int jb = 0; jb < total; jb += 64) {
      const int j = jb + lane;
      int b = 0;
      for (unsigned long long m = cmask; m; m &= m - 1) {
        const int c = __ffsll(m) - 1;
        if (j >= __builtin_amdgcn_readlane(off, c)) b = c;
      }
      const int pkb = __shfl(pk, b, 64);
      const double dyz2b = __shfl(dyz2, b, 64);
      const int lob = pkb & 63, wrapb = (pkb >> 6) & 1, offb = (pkb >> 9) & 0x1fff;
      const double shb = ((pkb >> 7) & 3) == 1 ? -Lx : (((pkb >> 7) & 3) == 2 ? Lx : 0.0);
      const int cl = lob + (j - offb);  // cell lane of the pair
      const bool valid = j < total && (unsigned)cl < 64u;
      const int e = entry_of(base + b);
      const auto& P = tile_entry<MORE>(tl, valid ? e : 0);
      const int xr = FLAT ? wc.x0 - (pkb >> 22) * nx : wc.x0;
      double dx = (double)(xr + cl) - P.x;
      dx = wrapb ? min_image(dx, px, nx) : dx + shb;
      const double d2 = dx * dx + dyz2b;
      // the Table 1 rule on d = sqrt(d2)
      const double rh = P.r + h;
      const bool in_shell = valid && d2 < rh * rh;
      double eps = 0.0;
      if constexpr (std::is_same<E, float>::value) {
        // the FP32 arithmetic forms: the refined FP32 root for every pair in
        // the shell (a wave with one lane in the band takes the root for all
        // its lanes anyway), the rule's clamps giving 0 and 1.  The fraction
        // itself stays accurate to FP64: near eps = 1 the weight B amplifies
        // its error about (1 + tau - 1/2) / (tau - 1/2) times
        if (in_shell) eps = pair_eps(sqrt_nr(d2), P.r, P.cs, h);
      } else {
        // FP64: the root only where the fraction is not already fixed at 0
        // or 1 by the shell or the clamp
        const double rl = P.r - h;
        const double c1 = P.cs - 1.0;
        const bool inner = (rl >= 0.0 && d2 <= rl * rl) || (c1 >= 0.0 && d2 <= c1 * c1);
        const bool outer = P.cs <= 0.0 || d2 >= P.cs * P.cs;
        eps = inner ? 1.0 : 0.0;
        if (in_shell && !inner && !outer) eps = pair_eps(sqrt(d2), P.r, P.cs, h);
      }
      if (in_shell && eps > 0.0) {
        const int c = wbase + cl;
        const int k = atomicAdd(&sl.n[c], 1);
        if (k < KSLOTS) {
          sl.e[k][c] = (unsigned short)e;
          sl.eps[k][c] = (E)eps;
        } else if (err) {
          atomicOr(err, ERR_SLOTS);
        }
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // phase 3: this cell's slots, in ascending particle id
  int n = sl.n[tid];
  n = n < KSLOTS ? n : KSLOTS;
  if (!active) n = 0;
  s.n = n;
#pragma unroll
  for (int k = 0; k < KSLOTS; ++k) {
    const bool has = k < n;
    s.e[k] = has ? sl.e[k][tid] : 0;
    s.eps[k] = has ? sl.eps[k][tid] : (E)0;
  }
  // the ids are read and compared only where some cell of the wave holds two
  // slots or more, and the full network only where one holds three or more
  if (__any(n > 1)) {
    int id[KSLOTS];
#pragma unroll
    for (int k = 0; k < KSLOTS; ++k) id[k] = k < n ? tile_entry<MORE>(tl, s.e[k]).id : 0x7fffffff;
    // compare-exchange network on (id, e, eps): (0,1) (2,3) (0,2) (1,3) (1,2)
    auto cx = [&](int i, int k) {
      const bool sw = id[k] < id[i];
      const int ti = id[i], te = s.e[i];
      const E tp = s.eps[i];
      id[i] = sw ? id[k] : ti;
      s.e[i] = sw ? s.e[k] : te;
      s.eps[i] = sw ? s.eps[k] : tp;
      id[k] = sw ? ti : id[k];
      s.e[k] = sw ? te : s.e[k];
      s.eps[k] = sw ? tp : s.eps[k];
    };
    static_assert(KSLOTS == 4, "sorting network for four slots");
    cx(0, 1);
    if (__any(n > 2)) {
      cx(2, 3);
      cx(0, 2);
      cx(1, 3);
      cx(1, 2);
    }
  }
}

// MORE: the tile's list may be longer than what LDS holds; those that are take a
// copy of the search of their own.
template <int D, bool FLAT, bool MORE, typename E>
__device__ __forceinline__ void collect_slots(const Geom& g, const WaveCells<FLAT>& wc, bool active,
                                              const TileListT<E>& tl, double h, SlotsT<E>& s,
                                              unsigned* err, SlotLdsT<E>& sl) {
  if constexpr (MORE) {
    if (tl.over) {
      collect_slots_of<D, FLAT, true>(g, wc, active, tl, h, s, err, sl);
      return;
    }
  }
  collect_slots_of<D, FLAT, false>(g, wc, active, tl, h, s, err, sl);
}

// Loads the tile's particle list into LDS (in list order: the slot search
// orders each cell's slots by particle id), as far as LDS holds it, and clears
// the force accumulators of the entries held.  The list length is uniform over
// the block; when it is positive the block has passed a barrier after the fill.
// Must be called by the whole block.
// `issue` is called once the loads of the count and the first ids are under
// way: loads a kernel starts there travel beside the list's own chain (count
// and ids, snapshots, LDS).
template <typename E, typename Issue>
__device__ inline TileListT<E> load_tile_list(const int* tile_count, const TileLists& ls,
                                              const PSnap* snap, int tile, LdsEntryT<E>* lds,
                                              double* acc, int np, Issue issue) {
  // each thread's first list entry is read alongside the count (entries past
  // the count are stale ids or zeros inside the list buffer, never used)
  const int* lst = ls.ids + (size_t)tile * ls.cap;
  const int e0 = (int)threadIdx.x;
  const int pre = np > 0 && e0 < ls.cap ? lst[e0] : 0;
  int cnt = np > 0 ? tile_count[tile] : 0;
  issue();
  if (cnt > ls.cap + ls.more_cap) cnt = ls.cap + ls.more_cap;
  const int held = cnt < ls.cap ? cnt : ls.cap;
  const int over = __builtin_amdgcn_readfirstlane((int)(cnt > held));
  const TileListT<E> tl{lds, cnt, held, over, ls.more + (size_t)tile * ls.more_cap, snap};
  if (cnt == 0) return tl;
  // (the first entry apart from the loop: its id is waited for by itself, not
  // with every load issued after it)
  if (e0 < held) fill_entry(lds[e0], snap[pre], pre);
  for (int e = e0 + BLOCK; e < held; e += BLOCK) fill_entry(lds[e], snap[lst[e]], lst[e]);
  if (acc)
    for (int k = threadIdx.x; k < 6 * held; k += BLOCK) acc[k] = 0.0;
  __syncthreads();
  return tl;
}
template <typename E>
__device__ inline TileListT<E> load_tile_list(const int* tile_count, const TileLists& ls,
                                              const PSnap* snap, int tile, LdsEntryT<E>* lds,
                                              double* acc, int np) {
  return load_tile_list(tile_count, ls, snap, tile, lds, acc, np, [] {});
}

// The calling wave's cells in a tile.
template <bool FLAT>
__device__ inline WaveCells<FLAT> wave_cells(const Geom& g, int tile) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tx = tile % g.ntx;
  const int r = tile / g.ntx;
  WaveCells<FLAT> c;
  if constexpr (FLAT) {
    const int p0 = BLOCK * tx + SEG * w;  // the wave's first cell in the plane
    const int left = g.nx * g.ny - p0;
    c.y0 = __builtin_amdgcn_readfirstlane(p0 / g.nx);
    c.x0 = __builtin_amdgcn_readfirstlane(p0 - c.y0 * g.nx);
    c.z = __builtin_amdgcn_readfirstlane(r);
    c.last = __builtin_amdgcn_readfirstlane((left < SEG ? left : SEG) - 1);
    c.rows = __builtin_amdgcn_readfirstlane((c.x0 + c.last) / g.nx + 1);
  } else {
    const int ty = r % g.nty;
    const int segs = g.twx >> 6;  // segments per tile row
    c.x0 = __builtin_amdgcn_readfirstlane(tx * g.twx + SEG * (w % segs));
    c.y0 = __builtin_amdgcn_readfirstlane(ty * g.twy + w / segs);
    c.z = __builtin_amdgcn_readfirstlane(r / g.nty);
    c.rows = 1;
    const int left = g.nx - c.x0;
    c.last = c.y0 < g.ny && c.z < g.nz ? (left < SEG ? left : SEG) - 1 : -1;
  }
  if (c.last < 0) c.x0 = c.y0 = c.z = 0;  // no cell: the lattice's first, for its loads
  return c;
}

// The calling lane's cell; a lane past c.last, which has none, takes the last
// lane's (the first when there is no cell at all), so that its loads are in
// range.
struct LaneCell {
  int x, y;
};
template <bool FLAT>
__device__ __forceinline__ LaneCell lane_cell(const Geom& g, const WaveCells<FLAT>& c) {
  const int lane = (int)(threadIdx.x & 63), last = c.last > 0 ? c.last : 0;
  const int t = c.x0 + (lane < last ? lane : last);
  LaneCell l;
  l.x = t;
  l.y = c.y0;
  if constexpr (FLAT) {
    // t < nx + 63: t / nx is 0 or 1 in rows of 64 or more, and in shorter
    // ones the product with 2^16 / nx rounded up is exact (t nx < 2^16)
    const unsigned k = g.nx >= SEG ? (t >= g.nx ? 1u : 0u)
                                   : ((unsigned)t * (65536u / (unsigned)g.nx + 1u)) >> 16;
    l.x = t - (int)k * g.nx;
    l.y = c.y0 + (int)k;
  }
  return l;
}


// Workgroup -> tile map.  The dispatcher deals consecutive workgroups round-
// robin to the 8 XCDs; this bijection gives each XCD one contiguous run of
// tiles so that the halo lines shared by neighbouring tiles stay in one L2.
__device__ inline int xcd_tile(int b, int nb) {
  constexpr int NX = 8;
  const int per = nb / NX, rem = nb % NX;
  const int xcd = b % NX, k = b / NX;
  return xcd * per + (xcd < rem ? xcd : rem) + k;
}
__device__ inline int tile_of(const Geom& g, int b, int nb) { return g.remap ? xcd_tile(b, nb) : b; }

// Lattice extents and periodicity as plain scalars (no arrays: every access
// stays a register or a kernel-argument load).
struct Dims {
  int nx, ny, nz;
  int px, py, pz;
  unsigned sy, sz;  // strides of y and z
};

__device__ __forceinline__ Dims dims_of(const Geom& g) {
  Dims d;
  d.nx = g.nx;
  d.ny = g.ny;
  d.nz = g.nz;
  d.px = g.periodic[0];
  d.py = g.periodic[1];
  d.pz = g.periodic[2];
  d.sy = (unsigned)g.nx;
  d.sz = (unsigned)g.nx * (unsigned)g.ny;
  return d;
}

// The neighbour of row y's cell at the x face `face` is in another flat wave.
__device__ __forceinline__ bool at_wave_edge(const Dims& d, int face, int y) {
  const unsigned p = (unsigned)(face ? d.nx - 1 : 0) + d.sy * (unsigned)y;
  return p % SEG == (face ? 0u : SEG - 1u);
}

// Element `e` of a per-direction array through a 32-bit byte offset, in the
// global address space, so the access is the scalar base plus one 32-bit
// vector offset.
template <typename S>
using GlobalT = __attribute__((address_space(1))) S;
template <typename S>
__device__ __forceinline__ GlobalT<S>& elem(S* base, unsigned e) {
  auto* gb = (__attribute__((address_space(1))) char*)base;
  return *(GlobalT<S>*)(gb + (e * (unsigned)sizeof(S)));
}

// The same element read or written with a non-temporal hint when NT (the line
// is streamed through the caches rather than kept in them) and through a 64-bit
// offset when WIDE (arrays of 4 GiB or more).
template <bool NT, bool WIDE = false, typename S>
__device__ __forceinline__ S elem_ld(S* base, unsigned e) {
  auto& v = WIDE ? *(GlobalT<S>*)(base + e) : elem(base, e);
  if constexpr (NT) return __builtin_nontemporal_load(&v);
  else return v;
}
template <bool NT, bool WIDE = false, typename S>
__device__ __forceinline__ void elem_st(S* base, unsigned e, S v) {
  auto& to = WIDE ? *(GlobalT<S>*)(base + e) : elem(base, e);
  if constexpr (NT) __builtin_nontemporal_store(v, &to);
  else to = v;
}

// The links of one cell: its neighbours through the periodic wrap, and the
// non-periodic faces it lies at.  y and z are uniform over the wave, so a
// link's y and z part is a scalar that goes into the base pointer, and its x
// part is one of three lane offsets: no arithmetic per link.  (In a FLAT wave
// y varies and joins the lane part, one addition a link.)  Only in a wave
// with a cell at a wall do the lanes choose an address each (`at`); that path
// is taken by the waves along the faces alone.  Resolving each link through
// the faces by itself, with a branch around each load, cost the odd steps
// 100-260 VALU and 50-510 SALU instructions a wave (384x192x192 with walls,
// FP64: 890 us against 822 for the even step; the 10x51x51 FP32 duct 10.8
// against 6.2 us).
template <int Q, bool WALLS, bool FLAT>
struct CellLinks {
  using L = Lattice<Q>;
  unsigned n, xm, xp;  // the cell and its x neighbours
  int ym, yp, zm, zp;  // offsets to its y and z neighbours (uniform but for y in a FLAT wave)
  unsigned wall;       // bit f: the cell lies at the non-periodic face f
  bool inner;          // no cell of the wave lies at one (uniform)

  __device__ __forceinline__ CellLinks(const Dims& d, int x, int y, int z) {
    n = (unsigned)x + d.sy * (unsigned)y + d.sz * (unsigned)z;
    xm = x == 0 ? n + (unsigned)(d.nx - 1) : n - 1u;
    xp = x == d.nx - 1 ? n - (unsigned)(d.nx - 1) : n + 1u;
    ym = y == 0 ? (d.ny - 1) * (int)d.sy : -(int)d.sy;
    yp = y == d.ny - 1 ? -(d.ny - 1) * (int)d.sy : (int)d.sy;
    zm = zp = 0;
    if constexpr (L::D == 3) {
      zm = z == 0 ? (int)(d.sz * (unsigned)(d.nz - 1)) : -(int)d.sz;
      zp = z == d.nz - 1 ? -(int)(d.sz * (unsigned)(d.nz - 1)) : (int)d.sz;
    }
    wall = 0;
    inner = true;
    if constexpr (WALLS) {
      if (!d.px) wall |= (x == 0 ? 1u : 0u) | (x == d.nx - 1 ? 2u : 0u);
      if (!d.py) wall |= (y == 0 ? 4u : 0u) | (y == d.ny - 1 ? 8u : 0u);
      if (L::D == 3 && !d.pz) wall |= (z == 0 ? 16u : 0u) | (z == d.nz - 1 ? 32u : 0u);
      inner = __ballot(wall != 0) == 0;
    }
  }
  // the faces a link along e_i crosses when it leaves the lattice
  __device__ static constexpr unsigned faces(int i) {
    return (L::ex(i) < 0 ? 1u : 0u) | (L::ex(i) > 0 ? 2u : 0u) | (L::ey(i) < 0 ? 4u : 0u) |
           (L::ey(i) > 0 ? 8u : 0u) | (L::ez(i) < 0 ? 16u : 0u) | (L::ez(i) > 0 ? 32u : 0u);
  }
  // the non-periodic faces the cell's link along e_i leaves through
  __device__ __forceinline__ unsigned out(int i) const { return wall & faces(i); }
  __device__ __forceinline__ unsigned lane_part(int i) const {
    const unsigned v = L::ex(i) > 0 ? xp : (L::ex(i) < 0 ? xm : n);
    return FLAT ? v + (unsigned)y_part(i) : v;
  }
  __device__ __forceinline__ int y_part(int i) const {
    return L::ey(i) > 0 ? yp : (L::ey(i) < 0 ? ym : 0);
  }
  __device__ __forceinline__ int row_part(int i) const {
    return (FLAT ? 0 : y_part(i)) + (L::ez(i) > 0 ? zp : (L::ez(i) < 0 ? zm : 0));
  }
  // Where the population that leaves along e_i goes (N cells per direction
  // array): array i of the neighbour, or, when the link leaves through a
  // non-periodic face, the cell's own slot of the opposite direction.  The
  // odd step reads what arrives along e_o from the same place, i = opp(o).
  template <typename S>
  __device__ __forceinline__ S* at(S* A, unsigned N, int i) const {
    S* in = A + (size_t)i * N + (ptrdiff_t)row_part(i) + lane_part(i);
    if constexpr (WALLS) {
      if (out(i)) in = A + (size_t)L::opp(i) * N + n;
    }
    return in;
  }
};

// The link from cell (x, y, z) along (dx, dy, dz): sets the neighbour's cell
// offset m (periodic wrap applied) and returns the mask of non-periodic faces
// the link leaves through (bit f for face f; 0 when the neighbour exists).
// WALLS == false: every axis is periodic and no link ever leaves.
template <bool WALLS>
__device__ __forceinline__ unsigned link(const Dims& d, int x, int y, int z, int dx, int dy,
                                         int dz, unsigned n, unsigned& m) {
  unsigned out = 0;
  int off = 0;
  if (dx) {
    const int v = x + dx;
    int o = dx;
    if (v < 0) {
      if (!WALLS || d.px) o += d.nx; else out |= 1u;
    } else if (v >= d.nx) {
      if (!WALLS || d.px) o -= d.nx; else out |= 2u;
    }
    off += o;
  }
  if (dy) {
    const int v = y + dy;
    int o = dy;
    if (v < 0) {
      if (!WALLS || d.py) o += d.ny; else out |= 4u;
    } else if (v >= d.ny) {
      if (!WALLS || d.py) o -= d.ny; else out |= 8u;
    }
    off += o * (int)d.sy;
  }
  if (dz) {
    const int v = z + dz;
    int o = dz;
    if (v < 0) {
      if (!WALLS || d.pz) o += d.nz; else out |= 16u;
    } else if (v >= d.nz) {
      if (!WALLS || d.pz) o -= d.nz; else out |= 32u;
    }
    off += o * (int)d.sz;
  }
  m = (unsigned)((int)n + off);
  return WALLS ? out : 0u;
}

// ---------------------------------------------------------------------------
// Particle snapshot and tile binning (the candidate box of Table 1), shared by the
// rasterisation and by the DEM kernel that rasterises the next step.
// ---------------------------------------------------------------------------
__device__ inline double va2d(double r) {  // Eq. 19
  const double s = sqrt(r * r - 0.25);
  return 0.5 * s + r * r * atan(0.5 / s);
}
__device__ inline double va3d(double r) {  // Eq. 17 (principal-value arctangents)
  const double r2 = r * r;
  const double s = sqrt(r2 - 0.5);
  return (1.0 / 12.0 - r2) * atan(0.5 * s / (0.5 - r2)) + s / 3.0 +
         (r2 - 1.0 / 12.0) * atan(0.5 / s) - (4.0 / 3.0) * r2 * r * atan(0.25 / (r * s));
}

// Snapshot of a particle; false when the radius is outside the domain of
// Eq. 17 / 19 (the snapshot then covers no cell).  c_s = V_a(r) + 1/2 is
// taken from (r_known, cs_known) when r equals r_known (a previous snapshot
// of the same particle).
__device__ inline bool make_snap(int three_d, const double* x, const double* u, const double* w,
                                 double r, PSnap& P, double r_known = -1.0,
                                 double cs_known = 0.0) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    P.x[a] = x[a];
    P.u[a] = u[a];
    P.w[a] = w[a];
  }
  if (!three_d) {
    P.x[2] = 0.0;
    P.u[2] = 0.0;
    P.w[0] = P.w[1] = 0.0;
  }
  P.r = r;
  P.pad = 0.0;
  const bool ok = P.r * P.r > (three_d ? 0.5 : 0.25) && P.r < 1e300;
  if (!ok) {
    P.cs = -1e300;
    P.r = 0.0;
  } else if (r == r_known) {
    P.cs = cs_known;
  } else {
    P.cs = (three_d ? va3d(P.r) : va2d(P.r)) + 0.5;
  }
  return ok;
}

// Tiles (of 2^sh cells) touched along one axis by the cell range [lo, hi]: at
// most two runs of tile indices (the second after a periodic wrap).
struct AxisRuns {
  int a0, a1, b0, b1;  // runs [a0, a1] and [b0, b1] (b0 > b1 when absent)
};

__device__ inline AxisRuns axis_runs(int lo, int hi, int L, int sh, int periodic) {
  AxisRuns r;
  r.b0 = 1;
  r.b1 = 0;
  const int last = (L - 1) >> sh;
  if (!periodic) {
    if (lo < 0) lo = 0;
    if (hi > L - 1) hi = L - 1;
    if (lo > hi) {
      r.a0 = 1;
      r.a1 = 0;
      return r;
    }
    r.a0 = lo >> sh;
    r.a1 = hi >> sh;
    return r;
  }
  if (hi - lo + 1 >= L) {
    r.a0 = 0;
    r.a1 = last;
    return r;
  }
  int wl, wh;
  if (lo >= -L && hi < 2 * L) {  // the box of a centre in [0, L): no division
    wl = lo < 0 ? lo + L : (lo >= L ? lo - L : lo);
    wh = hi < 0 ? hi + L : (hi >= L ? hi - L : hi);
  } else {
    wl = ((lo % L) + L) % L;
    wh = ((hi % L) + L) % L;
  }
  if (wl <= wh) {
    r.a0 = wl >> sh;
    r.a1 = wh >> sh;
  } else {
    const int t0 = wl >> sh, t1 = wh >> sh;
    if (t1 >= t0) {
      r.a0 = 0;
      r.a1 = last;
    } else {
      r.a0 = t0;
      r.a1 = last;
      r.b0 = 0;
      r.b1 = t1;
    }
  }
  return r;
}

// Lanes a particle where only its rasterisation needs several (measured at the
// DEM kernel).
constexpr int RASTER_LANES = 32;

// k / n for 0 <= k < 2^20 and n >= 1 in FP32: (k + 1/2) / n stays 1 / (2 n) from a
// whole number, the product is off by less than 2^-22 of its value, so the
// quotient is exact while k < 2^20 (larger: by division).
struct SmallDiv {
  int n;
  float r;
  __device__ explicit SmallDiv(int v) : n(v), r(__builtin_amdgcn_rcpf((float)v)) {}
  __device__ int quot(int k) const {
    return k < (1 << 20) ? (int)(((float)k + 0.5f) * r) : k / n;
  }
};

// Enters particle s (snapshot P) in the list of every tile that its shell box
// X +- (r + h) touches; LPP consecutive lanes of the calling wave (this one's
// number among them: lane) stride over the tiles.  An atomic's return and the
// store after it are 1-2 us, and a sphere of the 256^3 workload enters about
// 200 tiles, so each lane starts four tiles' atomics before it waits for the
// first.  (The scattered entries themselves bound it on large sets: counts spread
// over lines of their own took 55 us against 22 for the 8000 spheres, and
// leaving out the box corners' tiles, a fifth, gained nothing.)
template <int LPP>
__device__ inline void bin_tiles(const Geom& g, int three_d, double h, const PSnap& P, int s,
                                 int lane, int* count, const TileLists& ls, unsigned* err) {
  const double R = P.r + h;
  const int L[3] = {g.nx, g.ny, g.nz};
  // (flat tiles: runs of x cells and of rows)
  const int sx = g.flat ? 0 : 31 - __builtin_clz((unsigned)g.twx);
  const int sh[3] = {sx, g.flat ? 0 : 8 - sx, 0};
  static_assert(BLOCK == 256, "twx * twy == 2^8");
  AxisRuns runs[3];
  int la[3], lt[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int lo, hi;
    if (a == 2 && !three_d) {
      lo = hi = 0;
    } else {
      lo = (int)ceil(P.x[a] - R);
      hi = (int)floor(P.x[a] + R);
    }
    runs[a] = axis_runs(lo, hi, L[a], sh[a], g.periodic[a]);
    la[a] = runs[a].a1 >= runs[a].a0 ? runs[a].a1 - runs[a].a0 + 1 : 0;
    lt[a] = la[a] + (runs[a].b1 >= runs[a].b0 ? runs[a].b1 - runs[a].b0 + 1 : 0);
  }
  if (lt[0] <= 0 || lt[1] <= 0 || lt[2] <= 0) return;
  // tile_at(k): the k-th candidate tile, or -1; `total` candidates
  auto enter_all = [&](auto batch, int total, auto tile_at) {
    constexpr int U = decltype(batch)::value;
    for (int k0 = lane; k0 < total; k0 += LPP * U) {
      int t[U], slot[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int k = k0 + LPP * j;
        t[j] = k < total ? tile_at(k) : -1;
        slot[j] = t[j] >= 0 ? atomicAdd(&count[t[j]], 1) : 0;
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if (t[j] < 0) continue;
        if (slot[j] < ls.cap)
          ls.ids[(size_t)t[j] * ls.cap + slot[j]] = s;
        else if (slot[j] - ls.cap < ls.more_cap)
          ls.more[(size_t)t[j] * ls.more_cap + (slot[j] - ls.cap)] = s;
        else
          atomicOr(err, ERR_SLOTS);
      }
    }
  };
  if (g.flat) {
    // per plane, the tiles from the first row of the box to its last (both
    // runs of a wrapped box, the tile they may share counted once), each entered
    // if one of its rows within the box holds one of the box's cells
    const bool two = runs[1].b1 >= runs[1].b0;
    auto first = [&](int y) { return (int)((unsigned)y * (unsigned)g.nx / BLOCK); };
    auto final = [&](int y) { return (int)(((unsigned)(y + 1) * (unsigned)g.nx - 1u) / BLOCK); };
    const int a0 = first(runs[1].a0), a1 = final(runs[1].a1);
    int b0 = two ? first(runs[1].b0) : 1;
    int b1 = two ? final(runs[1].b1) : 0;
    if (two && b1 >= a0) b1 = a0 - 1;  // run b (from row 0) ends below run a
    const int na = a1 - a0 + 1;
    const SmallDiv per(na + (b1 >= b0 ? b1 - b0 + 1 : 0));
    // (fewer candidates, each with more work: one at a time)
    enter_all(std::integral_constant<int, 1>{}, per.n * lt[2], [&](int k) {
      const int iz = per.quot(k), kt = k - iz * per.n;
      const int tx = kt < na ? a0 + kt : b0 + (kt - na);
      const int tz = iz < la[2] ? runs[2].a0 + iz : runs[2].b0 + (iz - la[2]);
      const int p0 = BLOCK * tx, p1 = p0 + BLOCK - 1;
      bool hit = false;
      const int y1 = p1 / g.nx < g.ny - 1 ? p1 / g.nx : g.ny - 1;
      for (int y = p0 / g.nx; y <= y1; ++y) {
        if (!((y >= runs[1].a0 && y <= runs[1].a1) || (y >= runs[1].b0 && y <= runs[1].b1))) continue;
        const int c0 = p0 - y * g.nx, c1 = p1 - y * g.nx;  // the tile's x range in row y
        hit |= runs[0].a0 <= c1 && runs[0].a1 >= c0;
        hit |= runs[0].b1 >= runs[0].b0 && runs[0].b0 <= c1 && runs[0].b1 >= c0;
      }
      return hit ? tx + g.ntx * tz : -1;
    });
    return;
  }
  const SmallDiv dx(lt[0]), dy(lt[1]);
  enter_all(std::integral_constant<int, 4>{}, lt[0] * lt[1] * lt[2], [&](int k) {
    const int q = dx.quot(k), ix = k - q * lt[0];
    const int iz = dy.quot(q), iy = q - iz * lt[1];
    const int tx = ix < la[0] ? runs[0].a0 + ix : runs[0].b0 + (ix - la[0]);
    const int ty = iy < la[1] ? runs[1].a0 + iy : runs[1].b0 + (iy - la[1]);
    const int tz = iz < la[2] ? runs[2].a0 + iz : runs[2].b0 + (iz - la[2]);
    return tx + g.ntx * (ty + g.nty * tz);
  });
}

// DEM bin of a position along axis a (uniform bins of width bin_size).
__device__ inline int dem_bin_coord(double x, int L, int periodic, int nbin, double bin_size) {
  double v = x;
  if (periodic && !(x >= 0.0 && x < (double)L)) {  // (fmod is a long loop: only when it acts)
    v = fmod(v, (double)L);
    if (v < 0) v += L;
  }
  int b = (int)floor(v / bin_size);
  if (b < 0) b = 0;
  if (b >= nbin) b = nbin - 1;
  return b;
}

// A place for a particle at position x in its DEM bin of the target set: the bin
// and the slot in it, bin_cap or more when the bin is full (called by one lane per
// particle, early: the atomic's return is waited for at the record's store).
struct DemPlace {
  int bin, slot;
};
__device__ inline DemPlace dem_bin_place(const DemBinOut& b, int three_d, const Geom& g,
                                         const double* x) {
  const int bx = dem_bin_coord(x[0], g.nx, g.periodic[0], b.nbin[0], b.bin_size[0]);
  const int by = dem_bin_coord(x[1], g.ny, g.periodic[1], b.nbin[1], b.bin_size[1]);
  const int bz = three_d ? dem_bin_coord(x[2], g.nz, g.periodic[2], b.nbin[2], b.bin_size[2]) : 0;
  DemPlace p;
  p.bin = bx + b.nbin[0] * (by + b.nbin[1] * bz);
  p.slot = atomicAdd(&b.count[p.bin], 1);
  return p;
}

// The record of particle s (position x, velocity u, radius r) at its place.
__device__ inline void dem_bin_store(const DemBinOut& b, const DemPlace& p, int s,
                                     const double* x, const double* u, double r, unsigned* err) {
  if (p.slot < b.bin_cap) {
    double* rc = b.rec + ((size_t)p.bin * b.bin_cap + p.slot) * 8;
    rc[0] = x[0];
    rc[1] = x[1];
    rc[2] = x[2];
    rc[3] = u[0];
    rc[4] = u[1];
    rc[5] = u[2];
    rc[6] = r;
    rc[7] = (double)s;
  } else {
    atomicOr(err, ERR_CONTACTS);
  }
}

}  // namespace psclbm
