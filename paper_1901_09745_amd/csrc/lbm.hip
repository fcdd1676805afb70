// Lattice kernels of the gfx950 PSC-LBM library.
//
// Storage: one structure-of-arrays distribution array A[i][n] (n = x + nx*(y +
// ny*z)) updated in place with the two-parity "AA" streaming pattern, so each
// time step reads and writes every population exactly once:
//   even step (parity 0): cell n reads A[i][n] and writes its post-collision
//                          f*_i to A[opp(i)][n];
//   odd step  (parity 1): cell n reads f_i from A[opp(i)][n - e_i] and writes
//                          f*_i to A[i][n + e_i].
// A third form (ring step, used to recompute states for the adjoint) reads a
// canonical FP64 array and writes the canonical result into another:
//   ring step (parity 2): cell n reads src[i][n] and writes f*_i to dst[i][n + e_i].
// A link that leaves the domain through a non-periodic face is reflected into
// the cell itself (halfway bounce-back, Eq. 6), which in both parities lands
// on the location the same cell reads back next step; every location is read
// and written by one thread per step, so the update needs no second copy.
//
// Per-cell physics (Sec. 2.1-2.3): moments with the half-force shift (Eq. 5),
// BGK with Guo forcing (Eqs. 2-4), and in cells covered by particles the
// modified partially-saturated-cell collision (Eqs. 10, 12, 13) with the
// per-particle momentum exchange of Eq. 14.  The solid fractions (Eqs. 15-19,
// Table 1) are evaluated per cell from the workgroup tile's particle list held
// in LDS, so no per-cell solid data is stored in HBM.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <type_traits>

#include "common.hpp"
#include "dem.hpp"
#include "tiles.hpp"

namespace psclbm {

static_assert(Lattice<9>::opp(1) == 3 && Lattice<9>::opp(6) == 8 && Lattice<9>::opp(7) == 5,
              "D2Q9 opposite table");

template <int Q>
__host__ __device__ constexpr bool check_lattice() {
  for (int i = 0; i < Q; ++i) {
    const int o = Lattice<Q>::opp(i);
    if (Lattice<Q>::ex(o) != -Lattice<Q>::ex(i) || Lattice<Q>::ey(o) != -Lattice<Q>::ey(i) ||
        Lattice<Q>::ez(o) != -Lattice<Q>::ez(i))
      return false;
  }
  return true;
}
static_assert(check_lattice<9>() && check_lattice<19>(), "opposite directions");

// ---------------------------------------------------------------------------
// FP32 arithmetic that keeps the collision free of systematic rounding.
// ---------------------------------------------------------------------------
// w_i x in the compute type.  In FP32 the weights are not representable: 4/9,
// 1/9, 1/18 and 1/36 all round with one relative error of about 7.5e-9 (1/3
// with 3e-8), which scales the mass and momentum of every equilibrium the
// collision relaxes towards, and the relaxation then adds that excess to the
// flow again at every step.  The product is taken with the weight split into
// its FP32 rounding and the remainder, so that it carries one ordinary
// rounding of the result instead.
template <int Q, typename C>
__device__ __forceinline__ C wmul(int i, C x) {
  if constexpr (std::is_same<C, double>::value) {
    return (C)Lattice<Q>::w(i) * x;
  } else {
    const float hi = (float)Lattice<Q>::w(i);
    const float lo = (float)(Lattice<Q>::w(i) - (double)hi);
    return __builtin_fmaf(x, hi, x * lo);
  }
}

// The FP16 storage form keeps a cell's populations in registers as it stores
// them, h_i = g_i / w_i: the collision then takes no weight per direction,
// and the weights enter the moments once per weight class.
template <int PREC>
constexpr bool scaled_form() {
  return PREC == PSCLBM_FP32_FP16STORE;
}
// w_i x, or x itself in the scaled form
template <int Q, bool SC, typename C>
__device__ __forceinline__ C wq(int i, C x) {
  if constexpr (SC) return x;
  else return wmul<Q>(i, x);
}
// The density deviation sum_i g_i and the momentum sum_i e_i g_i of a cell;
// in the scaled form as sum_c w_c (sums over the rest, axis and diagonal
// classes of h_i).
template <int Q, bool SC, typename C>
__device__ __forceinline__ void cell_moments(const C (&g)[Q], C& r, C& jx, C& jy, C& jz) {
  using L = Lattice<Q>;
  if constexpr (!SC) {
    r = jx = jy = jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      r += g[i];
      if (L::ex(i) > 0) jx += g[i];
      if (L::ex(i) < 0) jx -= g[i];
      if (L::ey(i) > 0) jy += g[i];
      if (L::ey(i) < 0) jy -= g[i];
      if (L::ez(i) > 0) jz += g[i];
      if (L::ez(i) < 0) jz -= g[i];
    }
  } else {
    C R[3] = {0, 0, 0}, X[3] = {0, 0, 0}, Y[3] = {0, 0, 0}, Z[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int c = L::ex(i) * L::ex(i) + L::ey(i) * L::ey(i) + L::ez(i) * L::ez(i);
      R[c] += g[i];
      if (L::ex(i) > 0) X[c] += g[i];
      if (L::ex(i) < 0) X[c] -= g[i];
      if (L::ey(i) > 0) Y[c] += g[i];
      if (L::ey(i) < 0) Y[c] -= g[i];
      if (L::ez(i) > 0) Z[c] += g[i];
      if (L::ez(i) < 0) Z[c] -= g[i];
    }
    constexpr int axis = 1, diag = Q == 9 ? 5 : 7;  // a direction of each class
    r = wmul<Q>(0, R[0]) + (wmul<Q>(axis, R[1]) + wmul<Q>(diag, R[2]));
    jx = wmul<Q>(axis, X[1]) + wmul<Q>(diag, X[2]);
    jy = wmul<Q>(axis, Y[1]) + wmul<Q>(diag, Y[2]);
    jz = wmul<Q>(axis, Z[1]) + wmul<Q>(diag, Z[2]);
  }
}

// Velocity of Eq. 5, u = (j + F/2) / rho, in the compute type, from the
// momentum component j, the half force h and q = drho / rho.  In FP32 the half
// force (of order 1e-7 against a momentum of order 1e-3 in a slowly developing
// flow) loses its low bits when added to j, the same bits step after step,
// which biases the force the flow receives; the sum is therefore kept as its
// rounded value s and the exact remainder e (Knuth's two-sum), and 1/rho as
// (1 - q) / rho0, so that the rounding of rho only touches the small
// correction: u = (s + (e - s q)) / rho0.
template <typename C>
__device__ __forceinline__ C eq5_velocity(C j, C h, C q, C inv_rho, C inv_rho0) {
  if constexpr (std::is_same<C, double>::value) {
    (void)q;
    (void)inv_rho0;
    return (j + h) * inv_rho;
  } else {
    (void)inv_rho;
    const C s = j + h;
    const C bp = s - j;
    const C e = (j - (s - bp)) + (h - bp);
    return (s + (e - s * q)) * inv_rho0;
  }
}

// The same without a body force: the sum j + F/2 is j itself, so the FP32
// form is one fused multiply-add, u = (j - j q) / rho0.
template <typename C>
__device__ __forceinline__ C eq5_velocity_unforced(C j, C q, C inv_rho, C inv_rho0) {
  if constexpr (std::is_same<C, double>::value) {
    (void)q;
    (void)inv_rho0;
    return j * inv_rho;
  } else {
    (void)inv_rho;
    return __builtin_fmaf(-j, q, j) * inv_rho0;
  }
}

// 1/rho for Eq. 5: exact in FP64. The FP32 forms use it only for q = drho /
// rho, the small correction in both velocities above, where the hardware
// reciprocal's last bit stays below the velocity's own rounding.
template <typename C>
__device__ __forceinline__ C inv_density(C rho) {
  if constexpr (std::is_same<C, double>::value) return 1.0 / rho;
  else return __builtin_amdgcn_rcpf(rho);
}

// ---------------------------------------------------------------------------
// Storage conversion: deviation g_i = f_i - w_i rho0 in the compute type (in
// the FP16 form g_i / w_i, as stored).
// ---------------------------------------------------------------------------
// Direction i's array of a state with N cells, as a base the compiler holds
// in scalar registers and cannot re-derive from the others. Where all Q
// accesses of a cell share one offset (the even step's own-cell accesses) it
// otherwise forms each 64-bit address with a vector add from the previous one.
template <typename S>
__device__ __forceinline__ S* dir_ptr(S* A, int i, unsigned N) {
  S* p = A + (size_t)i * N;
  asm("" : "+s"(p));
  return p;
}
template <int PREC, int Q>
struct Store {
  using S = typename Form<PREC>::S;
  using C = typename Form<PREC>::C;
  // the deviation g_i of a stored value in the compute type (g_i / w_i as
  // stored in the scaled, FP16, form)
  __device__ static C deviation(S v, int i, double rho0) {
    if constexpr (PREC == PSCLBM_FP64) {
      return v - Lattice<Q>::w(i) * rho0;
    } else if constexpr (PREC == PSCLBM_FP32) {
      return v;
    } else {
      (void)i;
      return static_cast<float>(v);
    }
  }
  // deviation g of direction i (g / w_i in the scaled form) as stored
  __device__ static S stored(int i, C g, double rho0) {
    if constexpr (PREC == PSCLBM_FP64) return Lattice<Q>::w(i) * rho0 + g;
    else return static_cast<S>(g);
  }
  // the deviation memory then holds, in FP64 (exactly, and in the FP16 form to
  // the rounding of h w_i: the per-cell part of the mass sum)
  __device__ static double held(int i, C g, double rho0) {
    const S v = stored(i, g, rho0);
    if constexpr (PREC == PSCLBM_FP64) return v - Lattice<Q>::w(i) * rho0;
    else if constexpr (PREC == PSCLBM_FP32) return static_cast<double>(v);
    else return static_cast<double>(static_cast<float>(v)) * Lattice<Q>::w(i);
  }
  // Exact canonical FP64 value of stored population i.
  __device__ static double to_f64(const S* a, size_t idx, int i, double rho0) {
    if constexpr (PREC == PSCLBM_FP64) {
      return a[idx];
    } else if constexpr (PREC == PSCLBM_FP32) {
      return Lattice<Q>::w(i) * rho0 + static_cast<double>(a[idx]);
    } else {
      // h w added to w rho0 in one rounding (left to the compiler, the rest
      // population's w rho0 was the fused product and h w rounded by itself)
      return fma(static_cast<double>(static_cast<float>(a[idx])), Lattice<Q>::w(i),
                 Lattice<Q>::w(i) * rho0);
    }
  }
  __device__ static void from_f64(S* a, size_t idx, int i, double f, double rho0) {
    const double g = f - Lattice<Q>::w(i) * rho0;
    if constexpr (PREC == PSCLBM_FP64) {
      a[idx] = f;
    } else if constexpr (PREC == PSCLBM_FP32) {
      a[idx] = static_cast<float>(g);
    } else {
      a[idx] = static_cast<_Float16>(static_cast<float>(g / Lattice<Q>::w(i)));
    }
  }
};

// ---------------------------------------------------------------------------
// The fused collide-stream step.
// ---------------------------------------------------------------------------
// Waves per SIMD of each form, the register budget of the tiles (which the
// contact workgroups' code must fit as well), each as measured fastest: 2D
// FP32 / FP16 8 (their slot fractions held in FP32, so that eight
// workgroups' LDS fits a CU), walled 3D FP32 / FP16 7 in row tiles and 6 in flat
// ones (whose look-ups past LDS spill 10 registers at 7: FP16, 300x180x190 286
// us against 265), periodic 3D FP32 / FP16 6 (the per-cell moments keep their
// registers lower), 2D FP64 5, 3D FP64 4.  The reduced 3D forms are bound by instruction issue, and more
// waves hide more of the loads' and the tile list's latency under it, up to
// the point where spills cost more.
template <int Q, int PREC, bool WALLS, bool FLAT>
constexpr int step_waves() {
  if (PREC == PSCLBM_FP64) return Q == 9 ? 5 : 4;
  if (Q == 9) return 8;
  return WALLS && !FLAT ? 7 : 6;
}

// Forms whose loads of f start before the tile's list is waited for rather
// than after it: FP64 in 3D on periodic lattices, whose four waves per SIMD
// hide the least (256^3 940 -> 925 us; between walls 90 -> 92, the 2D channel
// 9.2 -> 9.6, the reduced forms within 1 %).
template <int Q, int PREC, bool WALLS>
constexpr bool EARLY_LOADS = Q == 19 && PREC == PSCLBM_FP64 && !WALLS;

// Where the contact workgroups stand among the tiles.  Their waves wait on
// chains of scattered loads; as the grid's first workgroups they have the chip
// to themselves, and memory idle, for some 25 us (20,000 spheres).  The 3D
// FP64 and FP32 forms, whose lattices leave issue slots free, spread them:
// groups of 8 workgroups (one an XCD, so that the round robin of the tile
// workgroups is that of their own index), one in 2^shift, the largest power
// with which they end before the grid does.  384x192x192 with 20,000 spheres:
// FP64 867 -> 854 us a coupled step, FP32 452 -> 443.  The FP16 form (352 ->
// 355), bound by issue, and 2D (28.1 -> 28.6) keep them first, and so do grids
// below SPREAD_TILES, 16 tiles a CU: 6912 tiles gain 1 % in both forms, 2048
// lose 0.7 % in FP32.
constexpr int SPREAD_TILES = 4096;
template <int Q, int PREC>
constexpr bool SPREAD_CONTACTS = Q == 19 && PREC != PSCLBM_FP32_FP16STORE;

template <bool SPREAD>
struct ContactBlocks {
  int groups, shift, g;  // groups of 8; the calling workgroup's group
  __device__ __forceinline__ ContactBlocks(int blocks, int s)
      : groups(blocks >> 3), shift(SPREAD ? s : 0), g((int)blockIdx.x >> 3) {}
  // the calling workgroup is a contact workgroup, and its index among them
  __device__ __forceinline__ bool contact() const {
    if constexpr (!SPREAD) return g < groups;
    return (g & ((1 << shift) - 1)) == 0 && (g >> shift) < groups;
  }
  __device__ __forceinline__ int index() const {
    if constexpr (!SPREAD) return (int)blockIdx.x;
    return ((g >> shift) << 3) + (int)(blockIdx.x & 7);
  }
  // contact workgroups before a tile workgroup
  __device__ __forceinline__ int before() const {
    if constexpr (!SPREAD) return 8 * groups;
    const int n = (g + (1 << shift) - 1) >> shift;
    return 8 * (n < groups ? n : groups);
  }
};

// NT: the accesses to the own cell's slots (the even step's, and the ring
// step's loads), each line by one wave, are streamed with non-temporal hints.
// MORE: the tiles' lists may be longer than what LDS holds (flat tiles).
template <int Q, int PREC, int PAR, bool WALLS, bool FLAT, bool MORE = false, bool NT = false>
__global__ void __launch_bounds__(BLOCK)
    __attribute__((amdgpu_waves_per_eu(step_waves<Q, PREC, WALLS, FLAT>())))
    k_step(const StepArgs a) {
  static_assert(!NT || PAR != 1, "non-temporal streaming of the own cell's slots only");
  using L = Lattice<Q>;
  using C = typename Form<PREC>::C;
  using S = typename Form<PREC>::S;
  using ST = Store<PREC, Q>;
  constexpr int D = L::D;
  // slot fractions held in FP32 by the FP32 arithmetic forms
  using E = typename std::conditional<PREC == PSCLBM_FP64, double, float>::type;
  constexpr bool SC = scaled_form<PREC>();
  constexpr bool EARLY = EARLY_LOADS<Q, PREC, WALLS>;
  extern __shared__ double smem_d[];
  __shared__ SlotLdsT<E> slot_lds;
  const ContactBlocks<SPREAD_CONTACTS<Q, PREC>> cbs(a.dem_blocks, a.dem_shift);
  if (cbs.contact()) {
    // contact workgroup of the coupled step: one wave per particle gathers
    // its DEM contact force from the binning of the step's start
    const int i = __builtin_amdgcn_readfirstlane((int)(cbs.index() * (BLOCK / 64) + threadIdx.x / 64));
    if (i < a.dem.n) {
      const int lane = (int)(threadIdx.x & 63);
      double xs[3], us[3], fs[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        xs[k] = a.px[3 * i + k];
        us[k] = a.pu[3 * i + k];
      }
      // (the slot search's LDS is free here)
      static_assert(sizeof(slot_lds) >= BLOCK / 64 * CONTACT_LDS * sizeof(int), "contact lists");
      dem_contact_wave(a.dem, i, lane, xs, us, a.pr[i], fs,
                       reinterpret_cast<int*>(&slot_lds) + CONTACT_LDS * (int)(threadIdx.x / 64));
      if (lane == 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) a.fc[3 * i + k] = fs[k];
    }
    return;
  }
  S* __restrict__ A = static_cast<S*>(a.f);
  // the tiles: the other workgroups
  const int nb = (int)gridDim.x - a.dem_blocks;
  const int bid = (int)blockIdx.x - cbs.before();
  const int tile = tile_of(a.g, bid, nb);

  // particle list of the tile (LDS) and its force accumulators
  using Entry = LdsEntryT<E>;
  Entry* lds = reinterpret_cast<Entry*>(smem_d);
  double* acc = reinterpret_cast<double*>(lds + a.lists.cap);
  const Dims d = dims_of(a.g);
  // the wave's cells; z, and y unless FLAT, are uniform over the wave (scalar)
  const WaveCells<FLAT> wc = wave_cells<FLAT>(a.g, tile);
  const LaneCell cell = lane_cell<FLAT>(a.g, wc);
  const int x = cell.x, y = cell.y, z = wc.z;
  const bool active = (int)(threadIdx.x & 63) <= wc.last;
  const unsigned N = (unsigned)a.g.N;

  // ---- f as stored: started before the tile's list is waited for in the forms
  // EARLY_LOADS names, after it in the others ----
  S raw[Q];
  auto load = [&] {
    // (lanes without a cell load too: no branch, so that the number of loads
    // under way is known when the list's ids are waited for; lane_cell has
    // their cell in range, at x0 again in walled rows, where the select costs
    // fewer registers than the lane's minimum kept: 4 spilled, not 8)
    const CellLinks<Q, WALLS, FLAT> lk(d, WALLS && !FLAT && !active ? wc.x0 : x, y, z);
    if constexpr (PAR == 1) {
      if (lk.inner) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const int o = L::opp(i);  // arrives along e_i: leaves along e_o seen from here
          raw[i] = elem(A + (size_t)o * N + (ptrdiff_t)lk.row_part(o), lk.lane_part(o));
        }
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) raw[i] = *lk.at(A, N, L::opp(i));
      }
    } else {
      S* from = PAR == 2 ? const_cast<S*>(static_cast<const S*>(a.src)) : A;
#pragma unroll
      for (int i = 0; i < Q; ++i) raw[i] = elem_ld<NT>(dir_ptr(from, i, N), lk.n);
    }
  };
  const TileListT<E> tl = load_tile_list(a.tile_count, a.lists, a.snap, tile, lds, acc, a.np,
                                         [&] { if constexpr (EARLY) load(); });
  const int cnt = tl.cnt;
  const double rho0 = a.g.rho0;
  // ---- solid fractions of the covering particles (Table 1), whole wave; in
  // 3D after the loads of f are issued, so that their latency overlaps the
  // slot search (in 2D the registers this holds cost more than it saves) ----
  SlotsT<E> s;
  s.n = 0;
  if constexpr (Q == 9) {
    if (cnt > 0) collect_slots<D, FLAT, MORE>(a.g, wc, active, tl, a.h, s, a.err, slot_lds);
  }

  C g[Q];
  C rho = (C)1, ux = 0, uy = 0, uz = 0, uu = 0;
  C Bn_cell = 0;
  // uniform parameters in the compute type (the FP32 copies are rounded on
  // the host, to the values a conversion here would give)
  auto uni = [](double v, float vf) -> C {
    if constexpr (std::is_same<C, double>::value) { (void)vf; return v; }
    else { (void)v; return vf; }
  };
  const C F0 = uni(a.force[0], a.force_f[0]), F1 = uni(a.force[1], a.force_f[1]),
          F2 = uni(a.force[2], a.force_f[2]);
  const C rho0c = uni(a.g.rho0, a.rho0_f), inv_rho0 = uni(a.inv_rho0, a.inv_rho0_f);
  const double tm = a.tau - 0.5;
  E bscale = 1;  // B_s / eps_{n,s} of the cell (Eq. 13), formed with the weights
  if constexpr (!EARLY) load();
  if constexpr (Q == 19) {
    if (cnt > 0) collect_slots<D, FLAT, MORE>(a.g, wc, active, tl, a.h, s, a.err, slot_lds);
  }
  // deviations g_i = f_i - w_i rho0 (in the scaled form g_i / w_i)
#pragma unroll
  for (int i = 0; i < Q; ++i) g[i] = ST::deviation(raw[i], i, rho0);
  // the slots' list entries, two to a register (entries < 2^15): registers held
  // through the collision
  const unsigned e01 = (unsigned)s.e[0] | ((unsigned)s.e[1] << 16);
  const unsigned e23 = (unsigned)s.e[2] | ((unsigned)s.e[3] << 16);
  auto slot_e = [&](int k) {
    return (int)(((k < 2 ? e01 : e23) >> (16 * (k & 1))) & 0xffffu);
  };
  static_assert(KSLOTS == 4, "entries packed for four slots");

  // ---- the covering particles, slot by slot ----
  // the row's y and z as FP64, converted from their scalar registers at each
  // use: an empty asm makes each use opaque, so the compiler does not hold
  // (or spill) one converted copy across the slots
  auto row_coord = [](int v) {
    if constexpr (!FLAT) asm volatile("" : "+s"(v));
    return (double)v;
  };
  constexpr int NV = D == 3 ? 6 : 3;
  // particle s of slot k at this cell: its share B_s, the weight of its
  // momentum exchange (Eq. 14 weighs it by B_s, Eq. 11 by the cell's B_n),
  // u_s - u and u_s + u with u_s the rigid-body velocity at the cell centre,
  // and the cell centre's offset from the particle centre
  struct SlotKin {
    C Bs, Bm, dv[3], sv[3], r[3];
  };
  auto slot_kin = [&](int k) {
    SlotKin t;
    t.Bs = a.original ? (C)(s.eps[k] * tm / ((1.0 - s.eps[k]) + tm)) : (C)(s.eps[k] * bscale);
    t.Bm = a.original ? Bn_cell : t.Bs;
    const auto& P = tile_entry<MORE>(tl, slot_e(k));
    // u_s = U + Omega x r in the arithmetic precision: the arm from its FP64
    // nearest image, or in the FP32 forms from the centre's FP32 pair
    C cx, cy, cz;
    if constexpr (PREC == PSCLBM_FP64) {
      cx = min_image((double)x - P.x, d.px, d.nx);
      cy = min_image(row_coord(y) - P.y, d.py, d.ny);
      cz = D == 3 ? min_image(row_coord(z) - P.z, d.pz, d.nz) : 0.0;
    } else {
      cx = min_image_f((float)x - P.xh[0], d.px, d.nx) - P.xl[0];
      cy = min_image_f((float)y - P.xh[1], d.py, d.ny) - P.xl[1];
      cz = D == 3 ? min_image_f((float)z - P.xh[2], d.pz, d.nz) - P.xl[2] : 0.0f;
    }
    C U[3], W[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (PREC == PSCLBM_FP64) {
        U[c] = P.u[c];
        W[c] = P.w[c];
      } else {
        U[c] = P.uf[c];
        W[c] = P.wf[c];
      }
    }
    const C usx = U[0] + W[1] * cz - W[2] * cy;
    const C usy = U[1] + W[2] * cx - W[0] * cz;
    const C usz = D == 3 ? U[2] + W[0] * cy - W[1] * cx : (C)0;
    t.dv[0] = usx - ux;
    t.dv[1] = usy - uy;
    t.dv[2] = usz - uz;
    t.sv[0] = usx + ux;
    t.sv[1] = usy + uy;
    t.sv[2] = usz + uz;
    t.r[0] = cx;
    t.r[1] = cy;
    t.r[2] = cz;
    return t;
  };
  // the negated momentum exchange of Eq. 14, m_s = B [rho (u_s - u) + F]:
  // force, then torque about the particle centre
  auto exchange = [&](const SlotKin& t, C (&mv)[NV]) {
    const C mx = t.Bm * (rho * t.dv[0] + F0);
    const C my = t.Bm * (rho * t.dv[1] + F1);
    mv[0] = -mx;
    mv[1] = -my;
    if constexpr (D == 3) {
      const C mz = t.Bm * (rho * t.dv[2] + F2);
      mv[2] = -mz;
      mv[3] = -(t.r[1] * mz - t.r[2] * my);
      mv[4] = -(t.r[2] * mx - t.r[0] * mz);
      mv[5] = -(t.r[0] * my - t.r[1] * mx);
    } else {
      mv[2] = -(t.r[0] * my - t.r[1] * mx);
    }
  };
  // added to the list entry's FP64 accumulators in LDS, or (an entry that LDS
  // does not hold) to the particle's
  auto accumulate = [&](int e, const C (&mv)[NV]) {
    auto add = [&](double* ac) {
      atomicAdd(ac + 0, (double)mv[0]);
      atomicAdd(ac + 1, (double)mv[1]);
      if constexpr (D == 3) {
        atomicAdd(ac + 2, (double)mv[2]);
        atomicAdd(ac + 3, (double)mv[3]);
        atomicAdd(ac + 4, (double)mv[4]);
        atomicAdd(ac + 5, (double)mv[5]);
      } else {
        atomicAdd(ac + 5, (double)mv[2]);
      }
    };
    if constexpr (MORE) {
      if (e >= tl.held) {
        add(a.facc + 6 * (size_t)tl.id_past(e));
        return;
      }
    }
    add(acc + 6 * e);
  };
  // periodic 3D reduced-precision forms: the particles' equilibrium difference
  // enters the collision through ten per-cell moments (one pass over the
  // directions); the others add it slot by slot after the collision (with
  // walls, the moments' registers cost spills of loaded populations)
  constexpr bool FOLD = D == 3 && PREC != PSCLBM_FP64 && !WALLS;
  // no body force: the Guo terms vanish (uniform over the launch)
  const bool forced = a.forced != 0;

  if (active) {
    // ---- inlet / outlet layers: reset to an equilibrium before collision ----
    if (WALLS && a.open_mask) {
      bool reset = false;
      double ub0 = 0.0, ub1 = 0.0, ub2 = 0.0;
      // x-face outlets: the velocity of the interior neighbour at this time
      // level, from the neighbour's lane of this wave
      double wu0 = 0.0, wu1 = 0.0, wu2 = 0.0;
      const int lane = (int)(threadIdx.x & 63);
      if (a.outlet_wave && __any(x == 0 || x == d.nx - 1)) {
        C r_, j0, j1, j2;
        cell_moments<Q, SC>(g, r_, j0, j1, j2);
        int src = lane;
        if ((a.outlet_wave & 1u) && x == 0) src = lane + 1;
        if ((a.outlet_wave & 2u) && x == d.nx - 1) src = lane - 1;
        r_ = __shfl(r_, src);
        j0 = __shfl(j0, src);
        j1 = __shfl(j1, src);
        j2 = __shfl(j2, src);
        const C ir = inv_density(rho0c + r_);
        const C qr = r_ * ir, ir0 = inv_rho0;
        wu0 = (double)eq5_velocity(j0, (C)0.5 * F0, qr, ir, ir0);
        wu1 = (double)eq5_velocity(j1, (C)0.5 * F1, qr, ir, ir0);
        wu2 = (double)eq5_velocity(j2, (C)0.5 * F2, qr, ir, ir0);
      }
#pragma unroll
      for (int f = 0; f < 6; ++f) {  // outlets first, an inlet wins on a corner
        const bool on = f == 0 ? x == 0 : f == 1 ? x == d.nx - 1 : f == 2 ? y == 0
                      : f == 3 ? y == d.ny - 1 : f == 4 ? z == 0 : z == d.nz - 1;
        if (((a.outlet_mask >> f) & 1u) && on) {
          // (a flat wave's first or last lane may have its neighbour in the next wave)
          if (((a.outlet_wave >> f) & 1u) && !(FLAT && lane == (f == 0 ? SEG - 1 : 0))) {
            ub0 = wu0;
            ub1 = wu1;
            ub2 = wu2;
          } else {
            const unsigned k = f < 2 ? (unsigned)y + (unsigned)d.ny * z
                                     : (f < 4 ? (unsigned)x + (unsigned)d.nx * z
                                              : (unsigned)x + (unsigned)d.nx * y);
            const double* o = a.outlet_u + ((size_t)f * a.face_stride + k) * 3;
            ub0 = o[0];
            ub1 = o[1];
            ub2 = o[2];
          }
          reset = true;
        }
      }
#pragma unroll
      for (int f = 0; f < 6; ++f) {
        const bool on = f == 0 ? x == 0 : f == 1 ? x == d.nx - 1 : f == 2 ? y == 0
                      : f == 3 ? y == d.ny - 1 : f == 4 ? z == 0 : z == d.nz - 1;
        if (((a.inlet_mask >> f) & 1u) && on) {
          ub0 = a.g.face_u[f][0];
          ub1 = a.g.face_u[f][1];
          ub2 = a.g.face_u[f][2];
          reset = true;
        }
      }
      if (reset) {
        const C u0 = (C)ub0, u1 = (C)ub1, u2 = (C)ub2;
        const C uq = u0 * u0 + u1 * u1 + u2 * u2;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const C eu = edot(L::ex(i), L::ey(i), L::ez(i), u0, u1, u2);
          g[i] = wq<Q, SC>(i, (C)rho0 * ((C)3 * eu + (C)4.5 * eu * eu - (C)1.5 * uq));
        }
      }
    }

    // ---- moments with the half-force shift (Eq. 5) ----
    C drho, jx, jy, jz;
    cell_moments<Q, SC>(g, drho, jx, jy, jz);
    rho = rho0c + drho;
    const C inv_rho = inv_density(rho);
    const C q_rho = drho * inv_rho;
    if (forced) {
      ux = eq5_velocity(jx, (C)0.5 * F0, q_rho, inv_rho, inv_rho0);
      uy = eq5_velocity(jy, (C)0.5 * F1, q_rho, inv_rho, inv_rho0);
      uz = eq5_velocity(jz, (C)0.5 * F2, q_rho, inv_rho, inv_rho0);
    } else {
      ux = eq5_velocity_unforced(jx, q_rho, inv_rho, inv_rho0);
      uy = eq5_velocity_unforced(jy, q_rho, inv_rho, inv_rho0);
      uz = eq5_velocity_unforced(jz, q_rho, inv_rho, inv_rho0);
    }
    uu = ux * ux + uy * uy + uz * uz;
    const C omega = uni(a.omega, a.omega_f);
    const C kguo = (C)1 - (C)0.5 * omega;
    const C uF = ux * F0 + uy * F1 + uz * F2;

    // Weights (Eq. 13 with the cell total clamped at one, Table 1): B_n from
    // the clamped cell total, each particle's share B_s per slot.  The
    // original weighting (Eq. 9) takes each particle's B_s from its own
    // fraction and B_n as their sum.
    // In the precision the fractions are held in: FP64, or FP32 with the
    // hardware reciprocal (1 ulp) for the FP32 arithmetic forms; the
    // denominators are at least tau - 1/2 > 0.
    auto recip = [](E v) -> E {
      if constexpr (PREC == PSCLBM_FP64) return 1.0 / v;
      else return __builtin_amdgcn_rcpf(v);
    };
    E S_ = 0;
#pragma unroll
    for (int k = 0; k < KSLOTS; ++k)
      if (k < s.n) S_ += s.eps[k];
    const E tme = uni(tm, a.tm_f);  // E is the compute type
    const E en = S_ < (E)1 ? S_ : (E)1;
    const E den = ((E)1 - en) + tme;
    E inv_den = 1;
    if (s.n > 0) inv_den = recip(den);
    // share of each particle: Eq. 13 when the fractions sum to at most one,
    // else eps_{n,s} / sum (the clamped total has B_n = 1)
    bscale = tme * inv_den;
    if (S_ > (E)1) bscale = recip(S_);
    E Bn_e = s.n > 0 ? en * tme * inv_den : (E)0;
    // a covered cell (en = 1) has B_n = 1 exactly, which the reciprocal's
    // last bit must not undo (no BGK part may act there)
    if constexpr (PREC != PSCLBM_FP64)
      if (en >= (E)1) Bn_e = (E)1;
    if (a.original) {
      double Bn_d = 0.0;
#pragma unroll
      for (int k = 0; k < KSLOTS; ++k)
        if (k < s.n) Bn_d += s.eps[k] * tm / ((1.0 - s.eps[k]) + tm);
      Bn_e = (E)Bn_d;
    }
    const C Bn = (C)Bn_e;
    Bn_cell = Bn;
    const C omB = (C)1 - Bn;
    const C relax = omB * omega;

    // The weights multiply each direction's own sum (the FP32 forms' split
    // product, wmul): formed once per cell and shared by the directions, with
    // opposite pairs relaxed in their sums and differences, the same terms took
    // 1-3 % less time but correlated the cell's equilibrium errors over its
    // directions (FP32 open box with a sphere: velocity error 4.03e-7 -> 4.29e-7
    // against FP64, torque errors of single placements doubled).
    if constexpr (FOLD) {
      // ---- the slots: the moments A = sum_s B_s (u_s - u) and the symmetric
      // M = sum_s B_s (u_s u_s - u u) (diagonal in mD, off-diagonal doubled
      // in mH, formed as B_s [(u_s - u)(u_s + u)^T + transpose] / 2), and the
      // momentum exchange ----
      C mA[3] = {0, 0, 0}, mD[3] = {0, 0, 0}, mH[3] = {0, 0, 0};
      if (s.n > 0) {
#pragma unroll
        for (int k = 0; k < KSLOTS; ++k) {
          if (k >= s.n) continue;
          const SlotKin t = slot_kin(k);
          C b[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            b[c] = t.Bs * t.dv[c];
            mA[c] += b[c];
            mD[c] += b[c] * t.sv[c];
          }
          mH[0] += b[0] * t.sv[1] + b[1] * t.sv[0];
          mH[1] += b[0] * t.sv[2] + b[2] * t.sv[0];
          mH[2] += b[1] * t.sv[2] + b[2] * t.sv[1];
          if (a.facc) {
            C mv[NV];
            exchange(t, mv);
            accumulate(slot_e(k), mv);
          }
        }
      }
      // ---- one pass over the directions: BGK + Guo weighted by 1 - B_n, the
      // bounce-back of the non-equilibrium part, B_n (fneq_{-i} - fneq_i), and
      // the particles' sum_s B_s [f^eq_i(rho, u_s) - f^eq_i(rho, u)], which is
      // w_i rho [3 e_i.A + 4.5 e_i.M.e_i - 1.5 tr M] (Eqs. 2-4, 10-12) ----
      const C r3 = (C)3 * rho, r45 = (C)4.5 * rho;
      const C pA[3] = {r3 * mA[0], r3 * mA[1], r3 * mA[2]};
      const C pD[3] = {r45 * mD[0], r45 * mD[1], r45 * mD[2]};
      const C pH[3] = {r45 * mH[0], r45 * mH[1], r45 * mH[2]};
      const C p0 = (C)-1.5 * rho * (mD[0] + mD[1] + mD[2]);
      auto collide = [&](auto guo) {
        constexpr bool GUO = decltype(guo)::value;
        // (opaque: what the two copies share is not hoisted above the branch,
        // where it spilled 2-6 registers: 256^3 FP16 8.05 -> 7.79 ms in 20 steps)
        C vx = ux, vy = uy, vz = uz;
        asm volatile("" : "+v"(vx), "+v"(vy), "+v"(vz));
        const C gk = omB * kguo;
        // g_i - relax fneq_i + B_n (fneq_-i - fneq_i) as g_i - (relax + B_n)
        // fneq_i + B_n fneq_-i: the non-equilibrium parts stay explicit, so an
        // equilibrium is kept exactly (no rounding of 1 - relax - B_n enters)
        const C rB = relax + Bn;
        {
          C x0 = p0;
          if constexpr (GUO) x0 -= gk * (C)3 * uF;
          const C fneq = g[0] - wq<Q, SC>(0, drho - rho * (C)1.5 * uu);
          g[0] = g[0] - relax * fneq + wq<Q, SC>(0, x0);
        }
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const int o = L::opp(i);
          if (o < i) continue;
          const int ex = L::ex(i), ey = L::ey(i), ez = L::ez(i);
          const C eu = edot(ex, ey, ez, vx, vy, vz);
          const C sym = drho + rho * ((C)4.5 * eu * eu - (C)1.5 * uu);
          const C fn_i = g[i] - wq<Q, SC>(i, sym + rho * (C)3 * eu);
          const C fn_o = g[o] - wq<Q, SC>(i, sym - rho * (C)3 * eu);
          // the even and odd parts under e -> -e of the particles' term and
          // of the Guo term (Eq. 4)
          C ps = p0;
          eacc(ex * ex, ps, pD[0]);
          eacc(ey * ey, ps, pD[1]);
          eacc(ez * ez, ps, pD[2]);
          eacc(ex * ey, ps, pH[0]);
          eacc(ex * ez, ps, pH[1]);
          eacc(ey * ez, ps, pH[2]);
          C pa = edot(ex, ey, ez, pA[0], pA[1], pA[2]);
          if constexpr (GUO) {
            const C eF = edot(ex, ey, ez, F0, F1, F2);
            ps += gk * ((C)9 * eu * eF - (C)3 * uF);
            pa += gk * ((C)3 * eF);
          }
          g[i] = g[i] - rB * fn_i + Bn * fn_o + wq<Q, SC>(i, ps + pa);
          g[o] = g[o] - rB * fn_o + Bn * fn_i + wq<Q, SC>(i, ps - pa);
        }
      };
      if (forced)
        collide(std::true_type{});
      else
        collide(std::false_type{});
    } else {
      // ---- pass 1: BGK + Guo weighted by (1 - B_n), plus the bounce-back of
      // the non-equilibrium part, B_n (fneq_{-i} - fneq_i); one opposite pair
      // at a time (Eqs. 2-4, 10, 12), the relaxation and the bounce-back
      // applied as in the folded collision above ----
      const C rB = relax + Bn;
      {
        const C wi = SC ? (C)1 : (C)L::w(0);
        const C fneq = g[0] - wq<Q, SC>(0, drho - rho * (C)1.5 * uu);
        g[0] = g[0] - relax * fneq - omB * kguo * wi * (C)3 * uF;
      }
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const int o = L::opp(i);
        if (o < i) continue;
        const C wi = SC ? (C)1 : (C)L::w(i);
        const C eu = edot(L::ex(i), L::ey(i), L::ez(i), ux, uy, uz);
        const C eF = edot(L::ex(i), L::ey(i), L::ez(i), F0, F1, F2);
        const C sym = drho + rho * ((C)4.5 * eu * eu - (C)1.5 * uu);
        const C fn_i = g[i] - wq<Q, SC>(i, sym + rho * (C)3 * eu);
        const C fn_o = g[o] - wq<Q, SC>(i, sym - rho * (C)3 * eu);
        // Guo term (Eq. 4): even and odd parts under e -> -e
        const C Fsym = kguo * wi * ((C)9 * eu * eF - (C)3 * uF);
        const C Fant = kguo * wi * ((C)3 * eF);
        g[i] = g[i] - rB * fn_i + Bn * fn_o + omB * (Fsym + Fant);
        g[o] = g[o] - rB * fn_o + Bn * fn_i + omB * (Fsym - Fant);
      }
    }
  }

  // ---- pass 2 (covered cells of the other forms): sum_s B_s [f^eq_i(rho,
  // u_s) - f^eq_i(rho, u)] and the momentum exchange ----
  if constexpr (!FOLD) {
    // slot k of this cell: the equilibrium difference into g and, unless the
    // step accumulates no force (the ring step), the negated exchange into mv
    auto slot_update = [&](int k, C (&mv)[NV]) {
      const SlotKin t = slot_kin(k);
      const C du2 = t.dv[0] * t.sv[0] + t.dv[1] * t.sv[1] + t.dv[2] * t.sv[2];  // |u_s|^2 - |u|^2
      const C rB = rho * t.Bs;
      g[0] -= wq<Q, SC>(0, rB * (C)1.5 * du2);
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const int o = L::opp(i);
        if (o < i) continue;
        const C de = edot(L::ex(i), L::ey(i), L::ez(i), t.dv[0], t.dv[1], t.dv[2]);
        const C se = edot(L::ex(i), L::ey(i), L::ez(i), t.sv[0], t.sv[1], t.sv[2]);
        // 4.5 [(e.u_s)^2 - (e.u)^2] - 1.5 (|u_s|^2 - |u|^2), and 3 e.(u_s - u)
        const C ds_s = (C)4.5 * de * se - (C)1.5 * du2;
        const C ds_a = (C)3 * de;
        g[i] += wq<Q, SC>(i, rB * (ds_s + ds_a));
        g[o] += wq<Q, SC>(i, rB * (ds_s - ds_a));
      }
      if (a.facc) exchange(t, mv);
    };
    if constexpr (PREC == PSCLBM_FP64 || D == 3) {
      // every covered lane adds its own exchange (the LDS unit serialises
      // lanes of one entry; the block sums below would cost FP64 registers)
      if (s.n > 0) {
#pragma unroll
        for (int k = 0; k < KSLOTS; ++k) {
          if (k >= s.n) continue;
          C mv[NV];
          slot_update(k, mv);
          if (a.facc) accumulate(slot_e(k), mv);
        }
      }
    } else {
      // slot by slot over the wave: the exchange is first summed over
      // aligned blocks of up to 8 lanes whose slot holds the same entry, and
      // only each block's leader adds it to LDS
      const int lane = (int)(threadIdx.x & 63);
#pragma unroll
      for (int k = 0; k < KSLOTS; ++k) {
        const bool has = k < s.n;
        if (!__any(has)) break;  // uniform over the wave
        C mv[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) mv[j] = 0;
        if (has) slot_update(k, mv);
        if (a.facc) {
          bool lead;
          const unsigned mf = merge_flags(has ? slot_e(k) : -1, lane, lead);
#pragma unroll
          for (int j = 0; j < NV; ++j) mv[j] = merge_sum(mv[j], mf);
          if (lead) accumulate(slot_e(k), mv);
        }
      }
    }
  }

  if (active) {
    // ---- stream (Eq. 1) with halfway bounce-back (Eq. 6) ----
    // the cell's index and links formed again from x (an empty asm keeps the
    // compiler from reusing, and so holding or spilling, those of the loads)
    int xo = x;
    asm volatile("" : "+v"(xo));  // (FLAT: y stays held)
    if constexpr (WALLS) {
      if (a.moving_mask) {  // moving walls: -2 w_i rho (e_i . u_w) / c_s^2
        const CellLinks<Q, true, FLAT> lk(d, xo, y, z);
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const unsigned mw = lk.out(i) & a.moving_mask;
          if (mw) {
            double uw0 = 0.0, uw1 = 0.0, uw2 = 0.0;
#pragma unroll
            for (int f = 0; f < 6; ++f)
              if ((mw >> f) & 1u) {
                uw0 += a.g.face_u[f][0];
                uw1 += a.g.face_u[f][1];
                uw2 += a.g.face_u[f][2];
              }
            const double eu = edot(L::ex(i), L::ey(i), L::ez(i), uw0, uw1, uw2);
            g[i] -= (C)(6.0 * (SC ? 1.0 : L::w(i)) * eu) * rho;
          }
        }
      }
    }
    if constexpr (PAR == 0) {  // own cell, opposite slot
      const unsigned no = (unsigned)xo + d.sy * (unsigned)y + d.sz * (unsigned)z;
#pragma unroll
      for (int i = 0; i < Q; ++i)
        elem_st<NT>(dir_ptr(A, L::opp(i), N), no, ST::stored(i, g[i], rho0));
    } else {
      const CellLinks<Q, WALLS, FLAT> lk(d, xo, y, z);
      if (lk.inner) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
          elem_st<false>(A + (size_t)i * N + (ptrdiff_t)lk.row_part(i), lk.lane_part(i),
                         ST::stored(i, g[i], rho0));
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) *lk.at(A, N, i) = ST::stored(i, g[i], rho0);
      }
    }
  }

  // ---- per-workgroup FP64 mass partial (sum of the stored deviations), after
  // the last step of a call ----
  __shared__ double wsum[BLOCK / 64];
  if (a.mass_part) {
    double mass_dev = 0.0;
    if (active)
#pragma unroll
      for (int i = 0; i < Q; ++i) mass_dev += ST::held(i, g[i], rho0);
    mass_dev = wave_sum(mass_dev);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = mass_dev;
  }
  __syncthreads();
  if (a.mass_part && threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < BLOCK / 64; ++k) t += wsum[k];
    a.mass_part[bid] = t;
  }

  // ---- flush the tile's force / torque partials (FP64), one (entry,
  // component) pair per thread so that a tile's atomics are issued together
  // rather than six in turn by each entry's thread (256^3 FP32 step 576 ->
  // 541 us); the barrier of the mass reduction above orders the LDS
  // accumulation before this read ----
  if (cnt > 0 && a.facc) {
    for (int t = threadIdx.x; t < 6 * tl.held; t += BLOCK) {
      const int e = t / 6, k = t - 6 * e;
      const double v = acc[t];
      if (v != 0.0) atomicAdd(a.facc + 6 * (size_t)lds[e].id + k, v);
    }
  }
  // ---- clear the other force buffer for the next step ----
  if (a.np > 0 && a.fzero) {
    const unsigned tot = 6u * (unsigned)a.np;
    for (unsigned k = (unsigned)bid * BLOCK + threadIdx.x; k < tot; k += (unsigned)nb * BLOCK)
      a.fzero[k] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Outlet layers: velocity (Eq. 5) of the interior neighbour of every outlet
// cell at the current time level, read before the step kernel runs.
// ---------------------------------------------------------------------------
// Storage index of canonical population i of the cell (x, y, z) = n at
// streaming parity PAR, as (direction array, element).
template <int Q, int PAR>
__device__ __forceinline__ size_t canonical_slot(const Dims& d, unsigned N, int x, int y, int z,
                                                 unsigned n, int i) {
  using L = Lattice<Q>;
  if constexpr (PAR == 0) return (size_t)i * N + n;
  unsigned m = n;
  const bool out = link<true>(d, x, y, z, -L::ex(i), -L::ey(i), -L::ez(i), n, m) != 0;
  return (size_t)(out ? i : L::opp(i)) * N + (out ? n : m);  // reflected at a face: the own slot
}

// Latency-bound (a few ten thousand cells): one thread per cell of each face
// that is asked for, all Q loads independent and in flight together.  With the
// directions in a rolled loop and 64-bit index divisions the loads went one
// after another: four faces of a 200x100x100 box took 19.3 us a step.
template <int Q, int PREC, int PAR>
__global__ void __launch_bounds__(256) k_outlet_velocity(Geom g, const void* f, double fx,
                                                         double fy, double fz, double* out,
                                                         long long stride, unsigned faces,
                                                         unsigned edges) {
  using L = Lattice<Q>;
  using ST = Store<PREC, Q>;
  using S = typename Form<PREC>::S;
  using C = typename Form<PREC>::C;
  unsigned left = faces;  // this block's face: the blockIdx.y-th set bit
  for (unsigned k = 0; k < blockIdx.y; ++k) left &= left - 1;
  const int face = __ffs((int)left) - 1;
  const Dims d = dims_of(g);
  const int ax = face / 2;
  const unsigned w1 = (unsigned)(ax == 0 ? d.ny : d.nx);
  const unsigned cells = w1 * (unsigned)(ax == 2 ? d.ny : d.nz);
  const int inner = (face % 2 == 0) ? 1 : (ax == 0 ? d.nx : ax == 1 ? d.ny : d.nz) - 2;
  const unsigned N = (unsigned)g.N;
  const S* A = static_cast<const S*>(f);
  for (unsigned k = blockIdx.x * 256u + threadIdx.x; k < cells; k += gridDim.x * 256u) {
    const int b = (int)(k / w1), a = (int)(k - (unsigned)b * w1);
    const int x = ax == 0 ? inner : a;
    const int y = ax == 0 ? a : ax == 1 ? inner : b;
    const int z = ax == 2 ? inner : b;
    // edges: x faces whose cells take the velocity from the neighbour's lane but
    // for those whose neighbour is in the next flat wave
    if (((edges >> face) & 1u) && !at_wave_edge(d, face, y)) continue;
    const unsigned n = (unsigned)x + d.sy * (unsigned)y + d.sz * (unsigned)z;
    S v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = A[canonical_slot<Q, PAR>(d, N, x, y, z, n, i)];
    double* o = out + ((size_t)face * stride + k) * 3;
    if ((edges >> face) & 1u) {  // in the step's arithmetic, as the face's other cells have it
      C h[Q], r, j0, j1, j2;
#pragma unroll
      for (int i = 0; i < Q; ++i) h[i] = ST::deviation(v[i], i, g.rho0);
      cell_moments<Q, scaled_form<PREC>()>(h, r, j0, j1, j2);
      const C ir = inv_density((C)g.rho0 + r), ir0 = (C)(1.0 / g.rho0);
      const C qr = r * ir;
      o[0] = (double)eq5_velocity(j0, (C)0.5 * (C)fx, qr, ir, ir0);
      o[1] = (double)eq5_velocity(j1, (C)0.5 * (C)fy, qr, ir, ir0);
      o[2] = (double)eq5_velocity(j2, (C)0.5 * (C)fz, qr, ir, ir0);
      continue;
    }
    double rho = 0, j0 = 0, j1 = 0, j2 = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const double fi = ST::to_f64(v, (size_t)i, i, g.rho0);
      rho += fi;
      eacc(L::ex(i), j0, fi);
      eacc(L::ey(i), j1, fi);
      eacc(L::ez(i), j2, fi);
    }
    o[0] = (j0 + 0.5 * fx) / rho;
    o[1] = (j1 + 0.5 * fy) / rho;
    o[2] = (j2 + 0.5 * fz) / rho;
  }
}

// ---------------------------------------------------------------------------
// State I/O
// ---------------------------------------------------------------------------
template <int Q, int PREC>
__global__ void k_set_equilibrium(Geom g, void* f, const double* rho, const double* u) {
  using L = Lattice<Q>;
  using S = typename Form<PREC>::S;
  for (long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x; n < g.N;
       n += (long long)gridDim.x * blockDim.x) {
    const double r = rho ? rho[n] : g.rho0;
    double ub[3] = {0, 0, 0};
    if (u) {
      ub[0] = u[3 * n];
      ub[1] = u[3 * n + 1];
      ub[2] = u[3 * n + 2];
    }
    const double uu = ub[0] * ub[0] + ub[1] * ub[1] + ub[2] * ub[2];
    for (int i = 0; i < Q; ++i) {
      const double eu = L::ex(i) * ub[0] + L::ey(i) * ub[1] + L::ez(i) * ub[2];
      const double fe = r * L::w(i) * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
      Store<PREC, Q>::from_f64(static_cast<S*>(f), (size_t)i * g.N + n, i, fe, g.rho0);
    }
  }
}

template <int Q, int PREC>
__global__ void k_set_f(Geom g, void* f, const double* src) {
  using S = typename Form<PREC>::S;
  for (long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x; n < g.N;
       n += (long long)gridDim.x * blockDim.x)
    for (int i = 0; i < Q; ++i)
      Store<PREC, Q>::from_f64(static_cast<S*>(f), (size_t)i * g.N + n, i,
                               src[(size_t)i * g.N + n], g.rho0);
}

// The state in the canonical layout (dst), or its density and velocity (rho,
// u; either null), one cell per thread: bound by its bytes, so the index
// arithmetic is 32-bit, all Q loads are in flight together, and u's three
// values a cell go through LDS to be written as whole lines.  256^3 fields:
// FP32 605 -> 320 us (5.7 TB/s), FP16 568 -> 205-270 us; with 64-bit index
// divisions the directions' loads went one after another.
template <int Q, int PREC, int PAR, bool FIELDS>
__global__ void __launch_bounds__(256) k_get_f(Geom g, const void* f, double* dst, double* rho,
                                               double* u, double fx, double fy, double fz) {
  using L = Lattice<Q>;
  using ST = Store<PREC, Q>;
  using S = typename Form<PREC>::S;
  const Dims d = dims_of(g);
  const unsigned N = (unsigned)g.N;
  const unsigned n0 = blockIdx.x * 256u, n = n0 + threadIdx.x;
  double j0 = 0, j1 = 0, j2 = 0, m = 1;
  if (n < N) {
    int x = 0, y = 0, z = 0;
    if constexpr (PAR == 1) {
      const unsigned r = n / d.sy;
      x = (int)(n - r * d.sy);
      z = (int)(r / (unsigned)d.ny);
      y = (int)(r - (unsigned)z * (unsigned)d.ny);
    }
    const S* A = static_cast<const S*>(f);
    S v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = A[canonical_slot<Q, PAR>(d, N, x, y, z, n, i)];
    if constexpr (!FIELDS) {
#pragma unroll
      for (int i = 0; i < Q; ++i)
        __builtin_nontemporal_store(ST::to_f64(v, (size_t)i, i, g.rho0), dst + (size_t)i * N + n);
    } else {
      m = 0;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const double fi = ST::to_f64(v, (size_t)i, i, g.rho0);
        m += fi;
        eacc(L::ex(i), j0, fi);
        eacc(L::ey(i), j1, fi);
        eacc(L::ez(i), j2, fi);
      }
      if (rho) rho[n] = m;
    }
  }
  if constexpr (FIELDS) {
    if (!u) return;
    __shared__ double su[3 * 256];
    su[3 * threadIdx.x] = (j0 + 0.5 * fx) / m;
    su[3 * threadIdx.x + 1] = (j1 + 0.5 * fy) / m;
    su[3 * threadIdx.x + 2] = (j2 + 0.5 * fz) / m;
    __syncthreads();
    const unsigned rest = 3u * (N - n0 < 256u ? N - n0 : 256u);
    double* ub = u + 3 * (size_t)n0;
#pragma unroll
    for (unsigned k = 0; k < 3; ++k) {
      const unsigned e = threadIdx.x + 256u * k;
      if (e < rest) ub[e] = su[e];
    }
  }
}

// The force / torque rows [n][6] as two [n][3] arrays (either null).  One
// launch: as two strided copies of the runtime they took 2.7 us on the GPU
// but 10 us of the host, longer than a small lattice's step (200x100 FP64).
__global__ void __launch_bounds__(256) k_read_forces(const double* rows, unsigned total,
                                                     double* force, double* torque) {
  const unsigned t = blockIdx.x * 256u + threadIdx.x;
  if (t >= total) return;
  const unsigned s = t / 6, k = t - 6 * s;
  double* dst = k < 3 ? force : torque;
  if (dst) dst[3 * (size_t)s + (k < 3 ? k : k - 3)] = rows[t];
}

// Mass of the current state, per workgroup (sum of stored deviations).
template <int Q, int PREC>
__global__ void __launch_bounds__(256) k_mass_direct(Geom g, const void* f, double* part) {
  using S = typename Form<PREC>::S;
  double t = 0.0;
  for (long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x; n < g.N;
       n += (long long)gridDim.x * blockDim.x)
    for (int i = 0; i < Q; ++i)
      t += Store<PREC, Q>::to_f64(static_cast<const S*>(f), (size_t)i * g.N + n, i, g.rho0) -
           Lattice<Q>::w(i) * g.rho0;
  for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
  __shared__ double ws[4];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Deterministic two-level reduction of the per-workgroup mass partials.
__global__ void k_reduce(const double* part, int n, double* out) {
  __shared__ double s[256];
  double t = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) t += part[k];
  s[threadIdx.x] = t;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = s[0];
}

// ---------------------------------------------------------------------------
// Rasterisation: particle snapshot, then tile binning (the candidate box X +- (r + h) of Table 1).
// ---------------------------------------------------------------------------
// RASTER_LANES lanes per particle: its snapshot (with V_a of Eq. 17 / 19),
// its force / torque rows cleared in both buffers, and its entry in the list
// of every tile of its shell box (at most two runs per axis after a periodic
// wrap), the lanes striding over the tiles.  The list counts are double
// buffered: this launch fills `count` (all zero on entry) and clears `stale`,
// the counts of the previous rasterisation, for the next one.
__global__ void __launch_bounds__(256) k_rasterize(Geom g, int n, int three_d, double h,
                                                   const double* x, const double* u,
                                                   const double* w, const double* r,
                                                   PSnap* snap, int* count, int* stale,
                                                   TileLists lists, double* f0,
                                                   double* f1, unsigned* err, DemBinOut db) {
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long k = gid; k < g.ntx * (long long)g.nty * g.ntz;
       k += (long long)gridDim.x * blockDim.x)
    stale[k] = 0;
  if (db.count)
    for (long long k = gid; k < db.nbins; k += (long long)gridDim.x * blockDim.x) db.stale[k] = 0;
  const int s = (int)(gid / RASTER_LANES);
  const int lane = (int)(threadIdx.x % RASTER_LANES);
  if (s >= n) return;
  PSnap P;
  const bool ok = make_snap(three_d, x + 3 * s, u + 3 * s, w + 3 * s, r[s], P);
  // the bin's and the tiles' atomics first, then the stores that need them
  const bool bin = db.count && lane == 0;
  DemPlace place = {0, 0};
  if (bin) place = dem_bin_place(db, three_d, g, x + 3 * s);
  if (lane < 6) f0[6 * s + lane] = 0.0;
  else if (lane < 12) f1[6 * s + lane - 6] = 0.0;
  if (ok) bin_tiles<RASTER_LANES>(g, three_d, h, P, s, lane, count, lists, err);
  if (lane == 0) {
    snap[s] = P;
    if (!ok) atomicOr(err, ERR_RADIUS);
  }
  if (bin) dem_bin_store(db, place, s, x + 3 * s, u + 3 * s, r[s], err);
}

template <int D, bool FLAT>
__global__ void __launch_bounds__(BLOCK) k_solid_fraction(Geom g, double h, int np,
                                                        const int* tile_count, TileLists lists,
                                                        const PSnap* snap, double* eps_total,
                                                        int* ids, double* seps, int kout,
                                                        unsigned* err) {
  extern __shared__ double smem_d[];
  __shared__ SlotLds slot_lds;
  LdsEntry* lds = reinterpret_cast<LdsEntry*>(smem_d);
  const int tile = blockIdx.x;
  const TileList tl = load_tile_list(tile_count, lists, snap, tile, lds, nullptr, np);
  const WaveCells<FLAT> wc = wave_cells<FLAT>(g, tile);
  const LaneCell cell = lane_cell<FLAT>(g, wc);
  const bool active = (int)(threadIdx.x & 63) <= wc.last;
  const long long n = cell.x + (long long)g.nx * (cell.y + (long long)g.ny * wc.z);
  Slots s;
  s.n = 0;
  if (tl.cnt > 0) collect_slots<D, FLAT, FLAT>(g, wc, active, tl, h, s, err, slot_lds);
  if (!active) return;
  double S_ = 0.0;
#pragma unroll
  for (int k = 0; k < KSLOTS; ++k)
    if (k < s.n) S_ += s.eps[k];
  if (eps_total) eps_total[n] = S_ < 1.0 ? S_ : 1.0;
  // the recorded slots (static register indices), then padding
#pragma unroll
  for (int k = 0; k < KSLOTS; ++k) {
    if (k >= kout) break;
    if (ids) ids[(size_t)n * kout + k] = k < s.n ? tile_entry<FLAT>(tl, s.e[k]).id : -1;
    if (seps) seps[(size_t)n * kout + k] = k < s.n ? s.eps[k] : 0.0;
  }
  for (int k = KSLOTS; k < kout; ++k) {
    if (ids) ids[(size_t)n * kout + k] = -1;
    if (seps) seps[(size_t)n * kout + k] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static int grid_for(long long n, int block = 256) {
  long long b = (n + block - 1) / block;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (int)b;
}

template <int Q, int PREC, bool WALLS, bool FLAT, bool MORE>
static int dispatch_step(psclbm_ctx* c, const StepArgs& a, int par, size_t lds_bytes) {
  const int nb = c->ntiles + a.dem_blocks;
  if (par == 2) {  // ring step: canonical FP64 in and out
    if constexpr (PREC == PSCLBM_FP64) {
      // The state read is streamed where it is a little larger than the 256 MB
      // last-level cache, which then holds more of the state written, the next
      // step's source: 192x96x96 (256 MB) 113 -> 99 us, 2048^2 (288 MB) 127 ->
      // 111, 128^3 (304 MB) 130 -> 121; above that the hints cost: 192x128x128
      // (456 MB) 201 -> 203, 384x192x192 891 -> 942 (256^3 0.99-1.05 times), and
      // flat tiles, whose waves share lines, 1.06-1.14 times at any size.
      const double mb = (double)c->geom.N * Q * sizeof(double) / (1024 * 1024);
      if constexpr (!FLAT) {
        if (mb > 256.0 && mb <= 352.0) {
          k_step<Q, PREC, 2, WALLS, FLAT, MORE, true><<<nb, BLOCK, lds_bytes, c->stream>>>(a);
          return hip_ok(hipGetLastError());
        }
      }
      k_step<Q, PREC, 2, WALLS, FLAT, MORE><<<nb, BLOCK, lds_bytes, c->stream>>>(a);
    } else {
      return PSCLBM_EINVAL;
    }
  } else if (par == 1) {
    k_step<Q, PREC, 1, WALLS, FLAT, MORE><<<nb, BLOCK, lds_bytes, c->stream>>>(a);
  } else if (c->geom.nt_even) {
    k_step<Q, PREC, 0, WALLS, FLAT, MORE, true><<<nb, BLOCK, lds_bytes, c->stream>>>(a);
  } else {
    k_step<Q, PREC, 0, WALLS, FLAT, MORE><<<nb, BLOCK, lds_bytes, c->stream>>>(a);
  }
  return hip_ok(hipGetLastError());
}

template <int Q, int PREC, bool FLAT, bool MORE>
static int dispatch_step(psclbm_ctx* c, const StepArgs& a, int par, size_t lds) {
  const bool walls = !(c->geom.periodic[0] && c->geom.periodic[1] && c->geom.periodic[2]);
  return walls ? dispatch_step<Q, PREC, true, FLAT, MORE>(c, a, par, lds)
               : dispatch_step<Q, PREC, false, FLAT, MORE>(c, a, par, lds);
}

template <int Q, int PREC>
static int dispatch_step(psclbm_ctx* c, const StepArgs& a, int par, size_t lds) {
  if (!c->geom.flat) return dispatch_step<Q, PREC, false, false>(c, a, par, lds);
  return a.np > 0 && a.lists.more_cap > 0 ? dispatch_step<Q, PREC, true, true>(c, a, par, lds)
                                          : dispatch_step<Q, PREC, true, false>(c, a, par, lds);
}

template <int PREC>
static int dispatch_step_q(psclbm_ctx* c, const StepArgs& a, int par, size_t lds) {
  return c->geom.q == 9 ? dispatch_step<9, PREC>(c, a, par, lds)
                        : dispatch_step<19, PREC>(c, a, par, lds);
}

#define PSCLBM_DISPATCH(QV, PV, CALL)                                       \
  do {                                                                      \
    if ((QV) == 9) {                                                        \
      if ((PV) == PSCLBM_FP64) { constexpr int Q = 9, P = PSCLBM_FP64; CALL; } \
      else if ((PV) == PSCLBM_FP32) { constexpr int Q = 9, P = PSCLBM_FP32; CALL; } \
      else { constexpr int Q = 9, P = PSCLBM_FP32_FP16STORE; CALL; }        \
    } else {                                                                \
      if ((PV) == PSCLBM_FP64) { constexpr int Q = 19, P = PSCLBM_FP64; CALL; } \
      else if ((PV) == PSCLBM_FP32) { constexpr int Q = 19, P = PSCLBM_FP32; CALL; } \
      else { constexpr int Q = 19, P = PSCLBM_FP32_FP16STORE; CALL; }       \
    }                                                                       \
  } while (0)

int launch_zero(psclbm_ctx* c, void* p, size_t bytes) {
  return hip_ok(hipMemsetAsync(p, 0, bytes, c->stream));
}

int launch_init_equilibrium(psclbm_ctx* c, const double* rho, const double* u) {
  const int grid = grid_for(c->geom.N);
  PSCLBM_DISPATCH(c->geom.q, c->prec,
                  (k_set_equilibrium<Q, P><<<grid, 256, 0, c->stream>>>(c->geom, c->f, rho, u)));
  return hip_ok(hipGetLastError());
}

int launch_set_f(psclbm_ctx* c, const double* f) {
  const int grid = grid_for(c->geom.N);
  PSCLBM_DISPATCH(c->geom.q, c->prec,
                  (k_set_f<Q, P><<<grid, 256, 0, c->stream>>>(c->geom, c->f, f)));
  return hip_ok(hipGetLastError());
}

template <bool FIELDS>
static int read_state(psclbm_ctx* c, double* f, double* rho, double* u) {
  const unsigned grid = (unsigned)((c->geom.N + 255) / 256);  // N < 2^31: storage under 4 GiB
  const double* F = c->cfg.body_force;
  if (c->steps & 1)
    PSCLBM_DISPATCH(c->geom.q, c->prec,
                    (k_get_f<Q, P, 1, FIELDS><<<grid, 256, 0, c->stream>>>(
                        c->geom, c->f, f, rho, u, F[0], F[1], F[2])));
  else
    PSCLBM_DISPATCH(c->geom.q, c->prec,
                    (k_get_f<Q, P, 0, FIELDS><<<grid, 256, 0, c->stream>>>(
                        c->geom, c->f, f, rho, u, F[0], F[1], F[2])));
  return hip_ok(hipGetLastError());
}

int launch_read_forces(psclbm_ctx* c, double* force, double* torque) {
  const unsigned total = 6u * (unsigned)c->np;
  k_read_forces<<<(total + 255) / 256, 256, 0, c->stream>>>(c->facc[c->force_buf], total, force,
                                                           torque);
  return hip_ok(hipGetLastError());
}

int launch_get_f(psclbm_ctx* c, double* f) { return read_state<false>(c, f, nullptr, nullptr); }

int launch_get_macros(psclbm_ctx* c, double* rho, double* u) {
  return read_state<true>(c, nullptr, rho, u);
}

int launch_rasterize(psclbm_ctx* c, const psclbm_particles* p, bool dem_bins) {
  const int three_d = c->geom.q == 19;
  const int next = c->tile_cur ^ 1;
  DemBinOut db = dem_bin_out(c, dem_bins);
  long long blocks = ((long long)p->n * RASTER_LANES + 255) / 256;
  long long clear = c->ntiles > db.nbins ? c->ntiles : db.nbins;
  const long long clear_blocks = (clear + 255) / 256;
  if (blocks < clear_blocks) blocks = clear_blocks < 4096 ? clear_blocks : 4096;
  if (blocks < 1) blocks = 1;
  k_rasterize<<<(unsigned)blocks, 256, 0, c->stream>>>(
      c->geom, p->n, three_d, c->cfg.shell_h, p->x, p->u, p->omega, p->radius, c->snap,
      c->tile_count_buf[next], c->tile_count_buf[c->tile_cur], c->lists, c->facc[0], c->facc[1], c->err, db);
  const int rc = hip_ok(hipGetLastError());
  if (rc) return rc;
  c->tile_cur = next;
  c->tile_count = c->tile_count_buf[next];
  if (dem_bins) dem_bins_advance(c);
  return PSCLBM_OK;
}

template <int D, bool FLAT>
static int solid_fraction(psclbm_ctx* c, double* eps, int* ids, double* seps, int k) {
  const size_t lds = (sizeof(LdsEntry) + sizeof(double)) * (size_t)c->lists.cap;
  k_solid_fraction<D, FLAT><<<c->ntiles, BLOCK, lds, c->stream>>>(
      c->geom, c->cfg.shell_h, c->np, c->tile_count, c->lists, c->snap, eps, ids,
      seps, k, c->err);
  return hip_ok(hipGetLastError());
}

int launch_solid_fraction(psclbm_ctx* c, double* eps, int* ids, double* seps, int k) {
  if (c->geom.q == 9)
    return c->geom.flat ? solid_fraction<2, true>(c, eps, ids, seps, k)
                        : solid_fraction<2, false>(c, eps, ids, seps, k);
  return c->geom.flat ? solid_fraction<3, true>(c, eps, ids, seps, k)
                      : solid_fraction<3, false>(c, eps, ids, seps, k);
}

// Arguments of one step from the context (state, forces and mass in place).
static StepArgs step_args(psclbm_ctx* c) {
  StepArgs a;
  a.g = c->geom;
  a.f = c->f;
  a.src = nullptr;
  a.tau = c->cfg.tau;
  for (int k = 0; k < 3; ++k) a.force[k] = c->cfg.body_force[k];
  a.h = c->cfg.shell_h;
  a.np = c->np;
  a.tile_count = c->tile_count;
  a.lists = c->lists;
  a.snap = c->snap;
  const int next = c->force_buf ^ 1;
  a.facc = c->facc[next];
  a.fzero = c->facc[next ^ 1];
  a.mass_part = c->mass_part;
  a.outlet_u = c->outlet_u;
  a.face_stride = c->face_stride;
  a.err = c->err;
  a.omega = 1.0 / c->cfg.tau;
  a.inv_rho0 = 1.0 / c->geom.rho0;
  for (int k = 0; k < 3; ++k) a.force_f[k] = (float)a.force[k];
  a.forced = a.force[0] != 0.0 || a.force[1] != 0.0 || a.force[2] != 0.0;
  a.omega_f = (float)a.omega;
  a.inv_rho0_f = (float)a.inv_rho0;
  a.rho0_f = (float)c->geom.rho0;
  a.tm_f = (float)(a.tau - 0.5);
  a.inlet_mask = a.outlet_mask = a.moving_mask = 0;
  for (int f = 0; f < 6; ++f) {
    if (c->geom.face[f] == PSCLBM_INLET_EQ) a.inlet_mask |= 1u << f;
    if (c->geom.face[f] == PSCLBM_OUTLET_EQ) a.outlet_mask |= 1u << f;
    if (c->geom.face[f] == PSCLBM_MOVING_WALL) a.moving_mask |= 1u << f;
  }
  a.open_mask = a.inlet_mask | a.outlet_mask;
  a.outlet_wave = outlet_wave_mask(c->geom, a.outlet_mask);
  a.original = c->cfg.weighting == PSCLBM_WEIGHT_ORIGINAL;
  a.dem_blocks = a.dem_shift = 0;
  std::memset(&a.dem, 0, sizeof(a.dem));
  a.px = a.pu = a.pr = nullptr;
  a.fc = nullptr;
  return a;
}

int launch_outlet_velocity(psclbm_ctx* c, const void* f, int prec, int par, unsigned faces,
                           unsigned edges) {
  const double* F = c->cfg.body_force;
  if (!faces) return PSCLBM_OK;
  const dim3 grid((unsigned)grid_for(c->face_stride), (unsigned)__builtin_popcount(faces));
  if (par)
    PSCLBM_DISPATCH(c->geom.q, prec,
                    (k_outlet_velocity<Q, P, 1><<<grid, 256, 0, c->stream>>>(
                        c->geom, f, F[0], F[1], F[2], c->outlet_u, c->face_stride, faces, edges)));
  else
    PSCLBM_DISPATCH(c->geom.q, prec,
                    (k_outlet_velocity<Q, P, 0><<<grid, 256, 0, c->stream>>>(
                        c->geom, f, F[0], F[1], F[2], c->outlet_u, c->face_stride, faces, edges)));
  return hip_ok(hipGetLastError());
}

static size_t step_lds(const psclbm_ctx* c) {
  return c->np > 0 ? (sizeof(LdsEntry) + 6 * sizeof(double)) * (size_t)c->lists.cap : 0;
}

int launch_step(psclbm_ctx* c, bool mass) {
  return launch_step_contacts(c, mass, nullptr, nullptr, nullptr, nullptr);
}

// mass: the state is the call's result, so its mass partials are formed.  The
// partials of the steps before it were overwritten unread; without their
// conversions and FP64 sums (57 of some 730 vector instructions a wave in the
// FP16 form) a step takes 339, not 352 us (FP16 spheres, 256^3), 54.2, not
// 55.4 (FP32 open box 200x100x100), 21.3, not 22.0 (FP32 disks, 1024^2).
int launch_step_contacts(psclbm_ctx* c, bool mass, const DemArgs* dem, const double* x,
                         const double* u, const double* r) {
  const int par = (int)(c->steps & 1);
  StepArgs a = step_args(c);
  if (!mass) a.mass_part = nullptr;
  if (dem && dem->n > 0) {
    a.dem_blocks = ((dem->n + BLOCK / 64 - 1) / (BLOCK / 64) + 7) / 8 * 8;
    if (c->ntiles >= SPREAD_TILES)
      while (((long long)a.dem_blocks << (a.dem_shift + 1)) <= (c->ntiles + a.dem_blocks) / 8 * 8)
        ++a.dem_shift;
    a.dem = *dem;
    a.px = x;
    a.pu = u;
    a.pr = r;
    a.fc = c->fcontact;
  }
  // outlets whose neighbour is in another wave: velocities before the step
  const unsigned edges = outlet_edges(a.g, a.outlet_wave);
  int rc = launch_outlet_velocity(c, c->f, c->prec, par, (a.outlet_mask & ~a.outlet_wave) | edges,
                                  edges);
  if (rc) return rc;
  const size_t lds = step_lds(c);
  if (c->prec == PSCLBM_FP64)
    rc = dispatch_step_q<PSCLBM_FP64>(c, a, par, lds);
  else if (c->prec == PSCLBM_FP32)
    rc = dispatch_step_q<PSCLBM_FP32>(c, a, par, lds);
  else
    rc = dispatch_step_q<PSCLBM_FP32_FP16STORE>(c, a, par, lds);
  if (rc) return rc;
  c->force_buf ^= 1;
  c->steps += 1;
  c->mass_valid = mass;
  return PSCLBM_OK;
}

int launch_recompute(psclbm_ctx* c, const double* f0, int nsteps, double* ring) {
  StepArgs a = step_args(c);
  a.facc = nullptr;
  a.fzero = nullptr;
  a.mass_part = nullptr;
  const size_t lds = step_lds(c);
  const size_t QN = (size_t)c->geom.q * (size_t)c->geom.N;
  const unsigned edges = outlet_edges(a.g, a.outlet_wave);
  for (int k = 0; k < nsteps; ++k) {
    const double* src = k == 0 ? f0 : ring + (size_t)(k - 1) * QN;
    int rc = launch_outlet_velocity(c, src, PSCLBM_FP64, 0,
                                    (a.outlet_mask & ~a.outlet_wave) | edges, edges);
    if (rc) return rc;
    a.src = src;
    a.f = ring + (size_t)k * QN;
    rc = dispatch_step_q<PSCLBM_FP64>(c, a, 2, lds);
    if (rc) return rc;
  }
  return PSCLBM_OK;
}

int launch_mass(psclbm_ctx* c, double* h_mass) {
  // After a step the fused per-workgroup partials already hold the sum of
  // the stored state; otherwise reduce the state directly.
  if (!c->mass_valid) {
    PSCLBM_DISPATCH(c->geom.q, c->prec,
                    (k_mass_direct<Q, P><<<c->nblocks, 256, 0, c->stream>>>(c->geom, c->f,
                                                                            c->mass_part)));
    int rc0 = hip_ok(hipGetLastError());
    if (rc0) return rc0;
    c->mass_valid = 1;
  }
  double* tmp = c->scalar;
  k_reduce<<<1, 256, 0, c->stream>>>(c->mass_part, c->nblocks, tmp);
  int rc = hip_ok(hipGetLastError());
  if (rc) return rc;
  double dev = 0.0;
  rc = hip_ok(hipMemcpyAsync(&dev, tmp, sizeof(double), hipMemcpyDeviceToHost, c->stream));
  if (rc) return rc;
  rc = hip_ok(hipStreamSynchronize(c->stream));
  if (rc) return rc;
  *h_mass = (double)c->geom.N * c->geom.rho0 + dev;
  return PSCLBM_OK;
}

}  // namespace psclbm
