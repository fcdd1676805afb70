// Hand-written adjoint of one PSC-LBM step (FP64), the transpose of the
// per-cell Jacobian of the step of lbm.hip applied to a given sensitivity.
//
// Notation per cell n (all FP64): f the state entering the step (after the
// inlet / outlet reset), lam*_i = dJ/df*_i the sensitivity of the post-
// collision population (read where that population streams to), B_n and the
// per-particle shares B_s (Eq. 13 with the clamped cell total of Table 1), and
//   f*_i = f_i - (1 - B_n) [w (f_i - f^eq_i) - F_i]
//          + sum_s B_s [f_{-i} - f^eq_{-i}(rho,u) + f^eq_i(rho,u_s) - f_i]   (Eqs. 10, 12)
//   m_s  = B_s [rho (u_s - u) + F],  F_s -= m_s,  T_s -= r_s x m_s       (Eq. 14)
// with w = 1/tau, rho = sum f, u = (sum f e + F/2)/rho (Eq. 5),
// u_s = U_s + Omega_s x r_s, r_s = x_n - X_s (nearest image), and the Table 1
// fraction eps_s = V_a(r) + 1/2 - |r_s| inside its linear band.
// Given dJ/dF_s and dJ/dT_s (the seeds of this step), q_s = dJ/dm_s =
// -dJ/dF_s - dJ/dT_s x r_s.  Then
//   lam_j = alpha lam*_j + B_n lam*_{-j} + kappa + a_rho + a_u . (e_j - u)/rho
// with alpha = 1 - (1 - B_n) w - B_n, kappa the moving-wall term and
//   a_rho = sum_i lam*_i [(1-B_n) w f^eq_i - B_n f^eq_{-i} + sum_s B_s f^eq_i(u_s)] / rho
//           + sum_s B_s q_s . (u_s - u)
//   a_u   = sum_i lam*_i [(1-B_n) w df^eq_i/du - B_n df^eq_{-i}/du + (1-B_n) dF_i/du]
//           - sum_s B_s rho q_s
// and for each covering particle
//   dJ/du_s = B_s [sum_i lam*_i rho w_i (3 e_i + 9 (e_i.u_s) e_i - 3 u_s) + rho q_s]
//   dJ/deps_t = B_n'(S) (lam* . P) + c(S) G_t + c'(S) sum_s eps_s G_s,
//     P_i = w (f_i - f^eq_i) - F_i,  G_s = lam* . Omega^s + q_s . [rho (u_s - u) + F],
//     c = tm/den, c' = tm/den^2 (sum eps <= 1) or c = 1/S, c' = -1/S^2,
//     B_n' = tm (1 + tm)/den^2 (sum eps < 1) else 0, tm = tau - 1/2, den = 1 - S + tm,
//   dJ/dX_s += dJ/deps_s r_s/|r_s| (linear band only) - (dJ/du_s x Omega_s + dJ/dT_s x m_s)
//   dJ/dU_s += dJ/du_s,  dJ/dOmega_s += r_s x dJ/du_s.
// Inlet cells (reset to f^eq(rho0, u_in)) pass lam through df^eq/du_in to the
// face velocity and have zero sensitivity of their own state; outlet cells
// pass it through u of their interior neighbour (a second kernel).  Moving
// walls pass lam of the reflected population to the wall velocity.
#include <hip/hip_runtime.h>

#include <cmath>

#include "common.hpp"
#include "tiles.hpp"

namespace psclbm {

struct AdjArgs {
  Geom g;
  double tau, omega;
  double force[3];
  double h;
  int np;
  const int* tile_count;
  TileLists lists;
  const PSnap* snap;
  const double* f;        // canonical FP64 state entering the step
  const double* lam_in;   // dJ/df(t+1), canonical
  double* lam_out;        // dJ/df(t), canonical
  const double* gF;       // dJ/dF_s of this step [3n] or null
  const double* gT;       // dJ/dT_s of this step [3n] or null
  double* gX;             // += [3n]
  double* gU;             // += [3n]
  double* gW;             // += [3n]
  double* gface;          // += [6][3]
  const double* outlet_u; // [6][face cells][3], velocity of each outlet's neighbour
  double* outlet_g;       // [6][face cells][3], dJ/du of that velocity
  long long face_stride;
  unsigned inlet_mask, outlet_mask, moving_mask;
  unsigned outlet_wave;   // outlet faces (x only) served from the neighbour's lane
};

template <int Q>
__device__ __forceinline__ double feq_i(int i, double rho, double ux, double uy, double uz,
                                        double uu) {
  using L = Lattice<Q>;
  const double eu = L::ex(i) * ux + L::ey(i) * uy + L::ez(i) * uz;
  return rho * L::w(i) * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
}

// Bytes: the state and the sensitivity read, the sensitivity written.  Bound
// by them in 3D with non-temporal hints (NT: the two aligned streams, when
// they are larger than the last-level cache), else by the latency of its chain
// at two or three waves per SIMD.  192x96x96 with 2000 spheres between walls:
// 195 us as one wave's list, search, loads and arithmetic in turn; 186 with the
// loads started first, 180 with the slots' gradients summed over lanes before
// the LDS atomics, 162 with the hints (5.0 TB/s).  1024^2 with 1600 disks 60
// -> 52 us (open faces compiled out, three waves); the 512x256 channel 17.0 ->
// 13.1 (the inlet's gradient summed per tile).  The open 200x100x100 box in flat
// tiles 319 -> 235 (x outlets from the neighbour's lane, as in row tiles; faces'
// passes with a cell's loads in flight together).
// WIDE: arrays of 4 GiB or more a direction (the reduced forms hold up to 2^31
// cells, and the sensitivities are FP64 in every form), addressed in 64 bits.
template <int Q, bool WALLS, bool FLAT, bool NT, bool WIDE = false>
__global__ void __launch_bounds__(BLOCK)
    __attribute__((amdgpu_waves_per_eu(Q == 9 && !WALLS ? 3 : 2))) k_adjoint(const AdjArgs a) {
  using L = Lattice<Q>;
  constexpr int D = L::D;
  extern __shared__ double smem_d[];
  __shared__ SlotLds slot_lds;
  const Geom& G = a.g;
  const int tile = tile_of(G, (int)blockIdx.x, (int)gridDim.x);
  // the wave's cells; z, and y unless FLAT, are uniform over the wave (scalar)
  const WaveCells<FLAT> wc = wave_cells<FLAT>(G, tile);
  const LaneCell cell = lane_cell<FLAT>(G, wc);
  const int x = cell.x, y = cell.y, z = wc.z;
  const bool active = (int)(threadIdx.x & 63) <= wc.last;
  const unsigned N = (unsigned)G.N;
  const Dims d = dims_of(G);
  const CellLinks<Q, WALLS, FLAT> lk(d, x, y, z);
  const unsigned n = lk.n;

  // The sensitivity of each post-collision population, read where it streams
  // to, and the state entering the step: all 2 Q loads of a cell are started
  // before the tile's list is waited for and used after the slot search.
  double ls[Q], fv[Q];
  auto issue = [&] {
    // (lanes without a cell read the last one's: no branch, so that the
    // number of loads under way is known when the list's ids are waited for)
    if (lk.inner) {
#pragma unroll
      for (int i = 0; i < Q; ++i)
        ls[i] = elem_ld<false, WIDE>(a.lam_in + (size_t)i * N + (ptrdiff_t)lk.row_part(i),
                                     lk.lane_part(i));
    } else {
#pragma unroll
      for (int i = 0; i < Q; ++i) ls[i] = *lk.at(a.lam_in, N, i);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) fv[i] = elem_ld<NT, WIDE>(a.f + (size_t)i * N, n);
  };
  LdsEntry* lds = reinterpret_cast<LdsEntry*>(smem_d);
  double* acc = reinterpret_cast<double*>(lds + a.lists.cap);  // [lists.cap][9]
  // dJ/d(face velocity) of the tile: every cell of an inlet adds to the same
  // three numbers, and atomics of one address are taken in turn
  __shared__ double face_acc[18];
  const bool faces = WALLS && a.gface;  // (a periodic lattice has no such face)
  if (faces && threadIdx.x < 18) face_acc[threadIdx.x] = 0.0;
  const TileList tl = load_tile_list(a.tile_count, a.lists, a.snap, tile, lds, nullptr, a.np, issue);
  const int cnt = tl.cnt;
  for (int k = threadIdx.x; k < 9 * tl.held; k += BLOCK) acc[k] = 0.0;
  if (cnt > 0 || faces) __syncthreads();
  Slots s;
  s.n = 0;
  if (cnt > 0) collect_slots<D, FLAT, FLAT>(G, wc, active, tl, a.h, s, nullptr, slot_lds);

  // from here on every lane computes (those without a cell the wave's last
  // one, without slots and without output), so that lanes can exchange values
  {
    const double rho0 = G.rho0;
    const double F0 = a.force[0], F1 = a.force[1], F2 = a.force[2];
    const int lane = (int)(threadIdx.x & 63);

    // kappa is the moving-wall term -6 w_i rho (e_i . u_w): d/df_j = -6 w_i (e_i . u_w)
    double kappa = 0.0;
    if (WALLS && a.moving_mask) {
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const unsigned mw = lk.out(i) & a.moving_mask;
        if (mw) {
          double uw0 = 0.0, uw1 = 0.0, uw2 = 0.0;
#pragma unroll
          for (int fc = 0; fc < 6; ++fc)
            if ((mw >> fc) & 1u) {
              uw0 += G.face_u[fc][0];
              uw1 += G.face_u[fc][1];
              uw2 += G.face_u[fc][2];
            }
          kappa -= 6.0 * L::w(i) * edot(L::ex(i), L::ey(i), L::ez(i), uw0, uw1, uw2) * ls[i];
        }
      }
    }

    // the state entering the step: its moments and the two sums through which
    // it enters the adjoint, Sf = sum_i lam*_i f_i and So = sum_i lam*_{-i} f_i
    // (= sum_i lam*_i f_{-i}); an x-face outlet whose interior neighbour is in
    // this wave takes that neighbour's velocity from its lane
    double rho_in = 0.0, j0 = 0.0, j1 = 0.0, j2 = 0.0, Sf = 0.0, So = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const double fi = fv[i];
      rho_in += fi;
      eacc(L::ex(i), j0, fi);
      eacc(L::ey(i), j1, fi);
      eacc(L::ez(i), j2, fi);
      Sf += ls[i] * fi;
      So += ls[L::opp(i)] * fi;
    }
    double uin0 = 0.0, uin1 = 0.0, uin2 = 0.0;
    double wu0 = 0.0, wu1 = 0.0, wu2 = 0.0;
    if (WALLS && a.outlet_wave) {
      uin0 = (j0 + 0.5 * F0) / rho_in;
      uin1 = (j1 + 0.5 * F1) / rho_in;
      uin2 = (j2 + 0.5 * F2) / rho_in;
      int src = lane;
      if ((a.outlet_wave & 1u) && x == 0) src = lane + 1;
      if ((a.outlet_wave & 2u) && x == d.nx - 1) src = lane - 1;
      wu0 = __shfl(uin0, src);
      wu1 = __shfl(uin1, src);
      wu2 = __shfl(uin2, src);
    }

    // inlet / outlet reset (as in the forward: outlets first, an inlet wins)
    int reset = 0, rface = 0;
    bool by_lane = false;  // of an outlet: its neighbour is in this wave
    double ub0 = 0.0, ub1 = 0.0, ub2 = 0.0;
    double rho = rho_in, jx = j0, jy = j1, jz = j2;
    if (WALLS && active && (a.inlet_mask | a.outlet_mask)) {
#pragma unroll
      for (int fc = 0; fc < 6; ++fc) {
        const bool on = fc == 0 ? x == 0 : fc == 1 ? x == d.nx - 1 : fc == 2 ? y == 0
                      : fc == 3 ? y == d.ny - 1 : fc == 4 ? z == 0 : z == d.nz - 1;
        if (((a.outlet_mask >> fc) & 1u) && on) {
          by_lane = ((a.outlet_wave >> fc) & 1u) && !(FLAT && lane == (fc == 0 ? SEG - 1 : 0));
          if (by_lane) {
            ub0 = wu0; ub1 = wu1; ub2 = wu2;
          } else {
            const unsigned k = fc < 2 ? (unsigned)y + (unsigned)d.ny * z
                                      : (fc < 4 ? (unsigned)x + (unsigned)d.nx * z
                                                : (unsigned)x + (unsigned)d.nx * y);
            const double* o = a.outlet_u + ((size_t)fc * a.face_stride + k) * 3;
            ub0 = o[0]; ub1 = o[1]; ub2 = o[2];
          }
          reset = 2;
          rface = fc;
        }
      }
#pragma unroll
      for (int fc = 0; fc < 6; ++fc) {
        const bool on = fc == 0 ? x == 0 : fc == 1 ? x == d.nx - 1 : fc == 2 ? y == 0
                      : fc == 3 ? y == d.ny - 1 : fc == 4 ? z == 0 : z == d.nz - 1;
        if (((a.inlet_mask >> fc) & 1u) && on) {
          ub0 = G.face_u[fc][0]; ub1 = G.face_u[fc][1]; ub2 = G.face_u[fc][2];
          reset = 1;
          rface = fc;
        }
      }
      if (reset) {  // the state is f^eq(rho0, u_b)
        const double uq = ub0 * ub0 + ub1 * ub1 + ub2 * ub2;
        rho = jx = jy = jz = Sf = So = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          const double fi = feq_i<Q>(i, rho0, ub0, ub1, ub2, uq);
          rho += fi;
          eacc(L::ex(i), jx, fi);
          eacc(L::ey(i), jy, fi);
          eacc(L::ez(i), jz, fi);
          Sf += ls[i] * fi;
          So += ls[L::opp(i)] * fi;
        }
      }
    }

    // moving walls: d/du_w of -6 w_i rho (e_i . u_w)
    if (active && faces && a.moving_mask) {
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const unsigned mw = lk.out(i) & a.moving_mask;
        if (!mw) continue;
        const double cw = -6.0 * L::w(i) * rho * ls[i];
#pragma unroll
        for (int fc = 0; fc < 6; ++fc)
          if ((mw >> fc) & 1u) {
            if (L::ex(i)) atomicAdd(face_acc + 3 * fc, cw * L::ex(i));
            if (L::ey(i)) atomicAdd(face_acc + 3 * fc + 1, cw * L::ey(i));
            if (L::ez(i)) atomicAdd(face_acc + 3 * fc + 2, cw * L::ez(i));
          }
      }
    }

    const double ux = (jx + 0.5 * F0) / rho, uy = (jy + 0.5 * F1) / rho, uz = (jz + 0.5 * F2) / rho;
    const double uu = ux * ux + uy * uy + uz * uz;
    const double w = a.omega;
    const double kg = 1.0 - 0.5 * w;

    // weights
    double S = 0.0;
#pragma unroll
    for (int k = 0; k < KSLOTS; ++k)
      if (k < s.n) S += s.eps[k];
    const double tm = a.tau - 0.5;
    const double en = S < 1.0 ? S : 1.0;
    const double den = (1.0 - en) + tm;
    const double Bn = s.n > 0 ? en * tm / den : 0.0;
    const double c = S <= 1.0 ? tm / den : 1.0 / S;
    const double cp = S <= 1.0 ? tm / (den * den) : -1.0 / (S * S);
    const double Bnp = S < 1.0 ? tm * (1.0 + tm) / (den * den) : 0.0;

    // base adjoint terms; LP = sum_i lam*_i (w (f_i - f^eq_i) - F_i) and
    // L0 = sum_i lam*_i (f_{-i} - f^eq_{-i} - f_i), the part of lam* . Omega^s
    // common to every particle, start from the state sums Sf, So; and the
    // moments of w_i lam*_i (orders 0, 1, 2 in e_i), through which the
    // particle terms close
    // Moments of w_i lam*_i (orders 0, 1, 2 in e_i; only the nonzero
    // components of e_i are added).  Every sum over directions of the base
    // adjoint closes on them, since f^eq_i and F_i are polynomials of degree
    // two in e_i with the weight w_i, and e_{-i} = -e_i, w_{-i} = w_i:
    //   sum_i lam*_i    f^eq_i / rho = m0 (1 - 1.5 u^2) + 3 u.m1 + 4.5 u.M2.u  (Qp)
    //   sum_i lam*_{-i} f^eq_i / rho = m0 (1 - 1.5 u^2) - 3 u.m1 + 4.5 u.M2.u  (Qm)
    //   sum_i lam*_i F_i / k = 3 (F.m1 - (u.F) m0) + 9 u.M2.F
    double m0 = 0.0, m1x = 0.0, m1y = 0.0, m1z = 0.0;
    double mxx = 0.0, myy = 0.0, mzz = 0.0, mxy = 0.0, mxz = 0.0, myz = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int ex = L::ex(i), ey = L::ey(i), ez = L::ez(i);
      const double wl = L::w(i) * ls[i];
      m0 += wl;
      eacc(ex, m1x, wl);
      eacc(ey, m1y, wl);
      eacc(ez, m1z, wl);
      if (ex != 0) mxx += wl;
      if (ey != 0) myy += wl;
      if (ez != 0) mzz += wl;
      eacc(ex * ey, mxy, wl);
      eacc(ex * ez, mxz, wl);
      eacc(ey * ez, myz, wl);
    }
    const double irho = 1.0 / rho;
    const double uF = ux * F0 + uy * F1 + uz * F2;
    const double Mux = mxx * ux + mxy * uy + mxz * uz;  // M2 u
    const double Muy = mxy * ux + myy * uy + myz * uz;
    const double Muz = mxz * ux + myz * uy + mzz * uz;
    const double MFx = mxx * F0 + mxy * F1 + mxz * F2;  // M2 F
    const double MFy = mxy * F0 + myy * F1 + myz * F2;
    const double MFz = mxz * F0 + myz * F1 + mzz * F2;
    const double um1 = ux * m1x + uy * m1y + uz * m1z;
    const double uMu = ux * Mux + uy * Muy + uz * Muz;
    const double even = m0 * (1.0 - 1.5 * uu) + 4.5 * uMu;
    const double Qp = even + 3.0 * um1, Qm = even - 3.0 * um1;
    const double lF = kg * (3.0 * ((F0 * m1x + F1 * m1y + F2 * m1z) - uF * m0) +
                            9.0 * (ux * MFx + uy * MFy + uz * MFz));
    // LP = sum_i lam*_i (w (f_i - f^eq_i) - F_i) and L0 = sum_i lam*_i
    // (f_{-i} - f^eq_{-i} - f_i), the part of lam* . Omega^s common to every
    // particle, from the state sums Sf, So
    const double LP = w * (Sf - rho * Qp) - lF;
    const double L0 = So - Sf - rho * Qm;
    // the coefficient of f^eq_i is cf_i = (1-B_n) w lam*_i - B_n lam*_{-i}:
    // sum_i cf_i f^eq_i / rho, and the velocity gradient
    //   sum_i cf_i df^eq_i/du + (1-B_n) lam*_i dF_i/du
    //   = rho (3 c1 m1 + 9 c2 M2 u - 3 c2 m0 u) + (1-B_n) k (9 M2 F - 3 m0 F)
    // with c1 = (1-B_n) w + B_n, c2 = (1-B_n) w - B_n
    double ar = (1.0 - Bn) * w * Qp - Bn * Qm;
    const double c1 = (1.0 - Bn) * w + Bn, c2 = (1.0 - Bn) * w - Bn;
    const double kF = (1.0 - Bn) * kg;
    double aux = rho * (3.0 * c1 * m1x + 9.0 * c2 * Mux - 3.0 * c2 * m0 * ux) + kF * (9.0 * MFx - 3.0 * m0 * F0);
    double auy = rho * (3.0 * c1 * m1y + 9.0 * c2 * Muy - 3.0 * c2 * m0 * uy) + kF * (9.0 * MFy - 3.0 * m0 * F1);
    double auz = rho * (3.0 * c1 * m1z + 9.0 * c2 * Muz - 3.0 * c2 * m0 * uz) + kF * (9.0 * MFz - 3.0 * m0 * F2);

    // covering particles, first pass: G_s = lam* . Omega^s + q_s . M_s with
    //   lam* . f^eq(rho, u_s) = rho [m0 (1 - 1.5 u_s^2) + 3 u_s . m1 + 4.5 u_s.M2.u_s]
    //   sum_i lam*_i df^eq_i(u_s)/du_s = rho [3 m1 + 9 M2 u_s - 3 m0 u_s]
    // and every particle gradient term but the one carrying sum_s eps_s G_s;
    // dJ/deps_s = B_n' (lam* . P) + c G_s + c' sum_t eps_t G_t enters dJ/dX_s
    // through d eps / d X = r / |r| on the linear band of Table 1 (zero where
    // clamped)
    double SG = 0.0;
    const double BLP = Bnp * LP;
    const bool several = s.n > 1;
    // the gradient of one slot (9 values: X, U, Omega) into the entry's LDS
    // accumulators: summed first over aligned blocks of up to 8 lanes whose
    // slot holds the same entry, so that the LDS unit, which takes lanes of one
    // address in turn, sees a block's leader only
    // (or, for an entry that LDS does not hold, the particle's own)
    auto add = [&](int e, int j, double t) {
      if constexpr (FLAT) {
        if (tl.over && e >= tl.held) {
          double* dst = j < 3 ? a.gX : (j < 6 ? a.gU : a.gW);
          if (dst) atomicAdd(dst + 3 * tl.id_past(e) + (j % 3), t);
          return;
        }
      }
      atomicAdd(acc + 9 * e + j, t);
    };
    auto accumulate = [&](int e, bool has, auto& v) {
      constexpr int NV = sizeof(v) / sizeof(v[0]);
      bool lead;
      const unsigned mf = merge_flags(has ? e : -1, lane, lead);
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if (D == 2 && (j == 2 || (j > 4 && j < 8))) continue;  // out of the plane
        const double t = merge_sum(v[j], mf);
        if (lead) add(e, j, t);
      }
    };
#pragma unroll
    for (int k = 0; k < KSLOTS; ++k) {
      const bool has = k < s.n;
      if (!__any(has)) break;  // uniform over the wave
      double v[9];
#pragma unroll
      for (int j = 0; j < 9; ++j) v[j] = 0.0;
      const int e = has ? s.e[k] : 0;
      if (has) {
        const double epsk = s.eps[k];
        const auto& P = tile_entry<FLAT, true>(tl, e);
        const double rx = min_image((double)x - P.x, d.px, d.nx);
        const double ry = min_image((double)y - P.y, d.py, d.ny);
        const double rz = D == 3 ? min_image((double)z - P.z, d.pz, d.nz) : 0.0;
        const double usx = P.u[0] + P.w[1] * rz - P.w[2] * ry;
        const double usy = P.u[1] + P.w[2] * rx - P.w[0] * rz;
        const double usz = P.u[2] + P.w[0] * ry - P.w[1] * rx;
        const double us2 = usx * usx + usy * usy + usz * usz;
        const double Bs = epsk * c;
        // q = dJ/dm = -dJ/dF - dJ/dT x r
        double qx = 0.0, qy = 0.0, qz = 0.0;
        const int id = P.id;
        if (a.gF) {
          qx -= a.gF[3 * id];
          qy -= a.gF[3 * id + 1];
          qz -= a.gF[3 * id + 2];
        }
        double tx = 0.0, ty = 0.0, tz = 0.0;
        if (a.gT) {
          tx = a.gT[3 * id];
          ty = a.gT[3 * id + 1];
          tz = a.gT[3 * id + 2];
          qx -= ty * rz - tz * ry;
          qy -= tz * rx - tx * rz;
          qz -= tx * ry - ty * rx;
        }
        const double Mx = rho * (usx - ux) + F0, My = rho * (usy - uy) + F1, Mz = rho * (usz - uz) + F2;
        const double M2x = mxx * usx + mxy * usy + mxz * usz;
        const double M2y = mxy * usx + myy * usy + myz * usz;
        const double M2z = mxz * usx + myz * usy + mzz * usz;
        // (sum_i lam*_i f^eq_i(u_s)) / rho
        const double Lfr = m0 * (1.0 - 1.5 * us2) + 3.0 * (usx * m1x + usy * m1y + usz * m1z) +
                           4.5 * (usx * M2x + usy * M2y + usz * M2z);
        const double dsx = rho * (3.0 * m1x + 9.0 * M2x - 3.0 * usx * m0);
        const double dsy = rho * (3.0 * m1y + 9.0 * M2y - 3.0 * usy * m0);
        const double dsz = rho * (3.0 * m1z + 9.0 * M2z - 3.0 * usz * m0);
        const double Gs = L0 + rho * Lfr + qx * Mx + qy * My + qz * Mz;
        SG += epsk * Gs;
        ar += Bs * Lfr + Bs * (qx * (usx - ux) + qy * (usy - uy) + qz * (usz - uz));
        aux -= Bs * rho * qx;
        auy -= Bs * rho * qy;
        auz -= Bs * rho * qz;
        // dJ/du_s, and through u_s = U + Omega x r and m = B_s M: the parts of
        // dJ/dr that are dJ/du_s x Omega and dJ/dT x m
        const double ax = Bs * (dsx + rho * qx), ay = Bs * (dsy + rho * qy), az = Bs * (dsz + rho * qz);
        const double mx = Bs * Mx, my = Bs * My, mz = Bs * Mz;
        const double dist = sqrt(rx * rx + ry * ry + rz * rz);
        const double lin = P.cs - dist;
        const bool band = dist < P.r + a.h && dist > P.r - a.h && lin > 0.0 && lin < 1.0;
        // (the c' sum_t eps_t G_t part here when this is the cell's only particle)
        const double own = several ? 0.0 : cp * epsk * Gs;
        const double gd = band ? (BLP + c * Gs + own) / dist : 0.0;
        v[0] = gd * rx - ((ay * P.w[2] - az * P.w[1]) + (ty * mz - tz * my));
        v[1] = gd * ry - ((az * P.w[0] - ax * P.w[2]) + (tz * mx - tx * mz));
        v[2] = gd * rz - ((ax * P.w[1] - ay * P.w[0]) + (tx * my - ty * mx));
        v[3] = ax;
        v[4] = ay;
        v[5] = az;
        v[6] = ry * az - rz * ay;
        v[7] = rz * ax - rx * az;
        v[8] = rx * ay - ry * ax;
      }
      accumulate(e, has, v);
    }

    // second pass, for cells that several particles share: the c' sum_t eps_t
    // G_t part of dJ/deps_s
    if (__any(several)) {
      const double cSG = cp * SG;
#pragma unroll
      for (int k = 0; k < KSLOTS; ++k) {
        if (!several || k >= s.n) continue;
        const int e = s.e[k];
        const auto& P = tile_entry<FLAT, true>(tl, e);
        const double rx = min_image((double)x - P.x, d.px, d.nx);
        const double ry = min_image((double)y - P.y, d.py, d.ny);
        const double rz = D == 3 ? min_image((double)z - P.z, d.pz, d.nz) : 0.0;
        const double dist = sqrt(rx * rx + ry * ry + rz * rz);
        const double lin = P.cs - dist;
        const bool band = dist < P.r + a.h && dist > P.r - a.h && lin > 0.0 && lin < 1.0;
        if (!band) continue;
        const double gd = cSG / dist;
        add(e, 0, gd * rx);
        add(e, 1, gd * ry);
        if constexpr (D == 3) add(e, 2, gd * rz);
      }
    }

    // sensitivity of the state entering the step; a reset cell passes it to
    // the boundary velocity (f = f^eq(rho0, u_b)):
    //   dJ/du_b = sum_j lam_j rho0 w_j (3 e_j + 9 (e_j.u_b) e_j - 3 u_b)
    // and keeps none of its own
    const double alpha = 1.0 - (1.0 - Bn) * w - Bn;
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    if (reset) {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        const double ex = L::ex(j), ey = L::ey(j), ez = L::ez(j);
        const double lj = alpha * ls[j] + Bn * ls[L::opp(j)] + kappa + ar +
                          (aux * (ex - ux) + auy * (ey - uy) + auz * (ez - uz)) * irho;
        const double eu = ex * ub0 + ey * ub1 + ez * ub2;
        const double rw = lj * rho0 * L::w(j);
        g0 += rw * (3.0 * ex + 9.0 * eu * ex - 3.0 * ub0);
        g1 += rw * (3.0 * ey + 9.0 * eu * ey - 3.0 * ub1);
        g2 += rw * (3.0 * ez + 9.0 * eu * ez - 3.0 * ub2);
      }
      if (reset == 1) {
        if (faces) {
          atomicAdd(face_acc + 3 * rface, g0);
          atomicAdd(face_acc + 3 * rface + 1, g1);
          atomicAdd(face_acc + 3 * rface + 2, g2);
        }
      } else if (!by_lane) {
        const unsigned k = rface < 2 ? (unsigned)y + (unsigned)d.ny * z
                                     : (rface < 4 ? (unsigned)x + (unsigned)d.nx * z
                                                  : (unsigned)x + (unsigned)d.nx * y);
        double* o = a.outlet_g + ((size_t)rface * a.face_stride + k) * 3;
        o[0] = g0;
        o[1] = g1;
        o[2] = g2;
      }
    }
    // in-wave outlets: the neighbour lane takes the outlet's dJ/du_b through
    // its own u = (sum f e + F/2)/rho: lam_j += g . (e_j - u)/rho
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (WALLS && a.outlet_wave) {
#pragma unroll
      for (int fc = 0; fc < 2; ++fc) {
        if (!((a.outlet_wave >> fc) & 1u)) continue;
        const bool mine = reset == 2 && rface == fc && by_lane;
        const int nbx = fc == 0 ? 1 : d.nx - 2;
        const int src = x == nbx ? (fc == 0 ? lane - 1 : lane + 1) : lane;
        const double v0 = __shfl(mine ? g0 : 0.0, src);
        const double v1 = __shfl(mine ? g1 : 0.0, src);
        const double v2 = __shfl(mine ? g2 : 0.0, src);
        if (x == nbx) {
          s0 += v0 / rho_in;
          s1 += v1 / rho_in;
          s2 += v2 / rho_in;
        }
      }
    }
    const double sb = -(s0 * uin0 + s1 * uin1 + s2 * uin2);
    // lam_j = alpha lam*_j + B_n lam*_{-j} + kappa + ar + au.(e_j - u)/rho:
    // the part common to every j, and au/rho dotted with e_j's nonzero
    // components
    const double qx = aux * irho, qy = auy * irho, qz = auz * irho;
    const double base = kappa + ar - (qx * ux + qy * uy + qz * uz);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int ex = L::ex(j), ey = L::ey(j), ez = L::ez(j);
      double lj = alpha * ls[j] + Bn * ls[L::opp(j)] + base + edot(ex, ey, ez, qx, qy, qz);
      if (reset) lj = 0.0;
      lj += edot(ex, ey, ez, s0, s1, s2) + sb;
      if (active) elem_st<NT, WIDE>(a.lam_out + (size_t)j * N, n, lj);
    }
  }

  // flush the tile's particle gradients, one (entry, component) pair per
  // thread so that a tile's atomics are issued together
  __syncthreads();
  if (faces && threadIdx.x < 18) {
    const double v = face_acc[threadIdx.x];
    if (v != 0.0) atomicAdd(a.gface + threadIdx.x, v);
  }
  for (int t = threadIdx.x; t < 9 * tl.held; t += BLOCK) {
    const int e = t / 9, k = t - 9 * e;
    const double v = acc[t];
    if (v == 0.0) continue;
    const int id = lds[e].id;
    double* dst = k < 3 ? a.gX : (k < 6 ? a.gU : a.gW);
    if (dst) atomicAdd(dst + 3 * id + (k % 3), v);
  }
}

// Outlet cells: the sensitivity of the reset velocity goes to the interior
// neighbour's state through u = (sum f e + F/2)/rho: lam_j += g . (e_j - u)/rho.
// One face a launch, since two faces may have a neighbour in common; all Q loads
// of a cell in flight together.  edge: only the cells at the waves' edges.
template <int Q>
__global__ void __launch_bounds__(256) k_outlet_adjoint(Geom g, int face, int edge, const double* f,
                                                        const double* gu, double* lam, double fx,
                                                        double fy, double fz, long long stride) {
  using L = Lattice<Q>;
  const Dims d = dims_of(g);
  const int ax = face / 2;
  const unsigned w1 = (unsigned)(ax == 0 ? d.ny : d.nx);
  const unsigned cells = w1 * (unsigned)(ax == 2 ? d.ny : d.nz);
  const int inner = (face % 2 == 0) ? 1 : (ax == 0 ? d.nx : ax == 1 ? d.ny : d.nz) - 2;
  const unsigned N = (unsigned)g.N;
  for (unsigned k = blockIdx.x * 256u + threadIdx.x; k < cells; k += gridDim.x * 256u) {
    const int b = (int)(k / w1), a = (int)(k - (unsigned)b * w1);
    const int x = ax == 0 ? inner : a;
    const int y = ax == 0 ? a : ax == 1 ? inner : b;
    const int z = ax == 2 ? inner : b;
    if (edge && !at_wave_edge(d, face, y)) continue;
    const unsigned n = (unsigned)x + d.sy * (unsigned)y + d.sz * (unsigned)z;
    double v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = f[(size_t)i * N + n];
    double rho = 0.0, j0 = 0.0, j1 = 0.0, j2 = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      rho += v[i];
      eacc(L::ex(i), j0, v[i]);
      eacc(L::ey(i), j1, v[i]);
      eacc(L::ez(i), j2, v[i]);
    }
    const double ux = (j0 + 0.5 * fx) / rho, uy = (j1 + 0.5 * fy) / rho, uz = (j2 + 0.5 * fz) / rho;
    const double* gv = gu + ((size_t)face * stride + k) * 3;
    const double g0 = gv[0], g1 = gv[1], g2 = gv[2];
#pragma unroll
    for (int j = 0; j < Q; ++j)
      lam[(size_t)j * N + n] +=
          (g0 * (L::ex(j) - ux) + g1 * (L::ey(j) - uy) + g2 * (L::ez(j) - uz)) / rho;
  }
}

// Table 1 chain alone: dJ/dX_s += sum_n dJ/deps_{n,s} r/|r| on the linear band,
// for sensitivities given per recorded slot (the order of psc_get_solid_fraction).
template <int D, bool FLAT>
__global__ void __launch_bounds__(BLOCK) k_rasterize_adjoint(Geom g, double h, int np,
                                                           const int* tile_count,
                                                           TileLists lists,
                                                           const PSnap* snap, const double* gs,
                                                           int kout, double* gX) {
  extern __shared__ double smem_d[];
  __shared__ SlotLds slot_lds;
  LdsEntry* lds = reinterpret_cast<LdsEntry*>(smem_d);
  const int tile = blockIdx.x;
  const TileList tl = load_tile_list(tile_count, lists, snap, tile, lds, nullptr, np);
  const WaveCells<FLAT> wc = wave_cells<FLAT>(g, tile);
  const LaneCell cell = lane_cell<FLAT>(g, wc);
  const int x = cell.x, y = cell.y, z = wc.z;
  const bool active = (int)(threadIdx.x & 63) <= wc.last;
  Slots s;
  s.n = 0;
  if (tl.cnt > 0) collect_slots<D, FLAT, FLAT>(g, wc, active, tl, h, s, nullptr, slot_lds);
  if (!active) return;
  const long long n = x + (long long)g.nx * (y + (long long)g.ny * z);
#pragma unroll
  for (int k = 0; k < KSLOTS; ++k) {
    if (k >= kout || k >= s.n) break;
    const double gk = gs[(size_t)n * kout + k];
    if (gk == 0.0) continue;
    const auto& P = tile_entry<FLAT>(tl, s.e[k]);
    const double rx = min_image((double)x - P.x, g.periodic[0], g.nx);
    const double ry = min_image((double)y - P.y, g.periodic[1], g.ny);
    const double rz = D == 3 ? min_image((double)z - P.z, g.periodic[2], g.nz) : 0.0;
    const double dist = sqrt(rx * rx + ry * ry + rz * rz);
    const double lin = P.cs - dist;
    if (!(dist < P.r + h && dist > P.r - h && lin > 0.0 && lin < 1.0)) continue;
    const double gd = gk / dist;
    atomicAdd(gX + 3 * P.id, gd * rx);
    atomicAdd(gX + 3 * P.id + 1, gd * ry);
    if (D == 3) atomicAdd(gX + 3 * P.id + 2, gd * rz);
  }
}

template <int Q, bool WALLS, bool FLAT>
static void launch_step_adjoint(psclbm_ctx* c, const AdjArgs& a, size_t lds) {
  if ((double)c->geom.N * sizeof(double) >= 4294967296.0) {  // (one kernel for all of them)
    k_adjoint<Q, true, FLAT, false, true><<<c->ntiles, BLOCK, lds, c->stream>>>(a);
    return;
  }
  // (rows of whole lines only: see the even steps' choice)
  if constexpr (!FLAT) {
    if ((double)c->geom.N * Q * sizeof(double) > 256.0 * 1024 * 1024) {
      k_adjoint<Q, WALLS, FLAT, true><<<c->ntiles, BLOCK, lds, c->stream>>>(a);
      return;
    }
  }
  k_adjoint<Q, WALLS, FLAT, false><<<c->ntiles, BLOCK, lds, c->stream>>>(a);
}
template <int Q>
static void launch_step_adjoint(psclbm_ctx* c, const AdjArgs& a, bool walls, size_t lds) {
  if (c->geom.flat) {
    if (walls) launch_step_adjoint<Q, true, true>(c, a, lds);
    else launch_step_adjoint<Q, false, true>(c, a, lds);
  } else {
    if (walls) launch_step_adjoint<Q, true, false>(c, a, lds);
    else launch_step_adjoint<Q, false, false>(c, a, lds);
  }
}

int launch_adjoint(psclbm_ctx* c, const double* f, const double* lam_in, double* lam_out,
                   const double* gF, const double* gT, double* gX, double* gU, double* gW,
                   double* gface) {
  AdjArgs a;
  a.g = c->geom;
  a.tau = c->cfg.tau;
  a.omega = 1.0 / c->cfg.tau;
  for (int k = 0; k < 3; ++k) a.force[k] = c->cfg.body_force[k];
  a.h = c->cfg.shell_h;
  a.np = c->np;
  a.tile_count = c->tile_count;
  a.lists = c->lists;
  a.snap = c->snap;
  a.f = f;
  a.lam_in = lam_in;
  a.lam_out = lam_out;
  a.gF = gF;
  a.gT = gT;
  a.gX = gX;
  a.gU = gU;
  a.gW = gW;
  a.gface = gface;
  a.outlet_u = c->outlet_u;
  a.outlet_g = c->outlet_g;
  a.face_stride = c->face_stride;
  a.inlet_mask = a.outlet_mask = a.moving_mask = 0;
  for (int fc = 0; fc < 6; ++fc) {
    if (c->geom.face[fc] == PSCLBM_INLET_EQ) a.inlet_mask |= 1u << fc;
    if (c->geom.face[fc] == PSCLBM_OUTLET_EQ) a.outlet_mask |= 1u << fc;
    if (c->geom.face[fc] == PSCLBM_MOVING_WALL) a.moving_mask |= 1u << fc;
  }
  a.outlet_wave = outlet_wave_mask(c->geom, a.outlet_mask);
  const unsigned edges = outlet_edges(c->geom, a.outlet_wave);
  const unsigned separate = (a.outlet_mask & ~a.outlet_wave) | edges;
  const double* F = c->cfg.body_force;
  const int fgrid = (int)((c->face_stride + 255) / 256 < 4096 ? (c->face_stride + 255) / 256 : 4096);
  int rc = launch_outlet_velocity(c, f, PSCLBM_FP64, 0, separate, edges);
  if (rc) return rc;
  const size_t lds = c->np > 0 ? (sizeof(LdsEntry) + 9 * sizeof(double)) * (size_t)c->lists.cap : 0;
  const bool walls = !(c->geom.periodic[0] && c->geom.periodic[1] && c->geom.periodic[2]);
  if (c->geom.q == 9) launch_step_adjoint<9>(c, a, walls, lds);
  else launch_step_adjoint<19>(c, a, walls, lds);
  rc = hip_ok(hipGetLastError());
  if (rc) return rc;
  for (int fc = 0; fc < 6; ++fc) {
    if (!((separate >> fc) & 1u)) continue;
    const int edge = (int)((edges >> fc) & 1u);
    if (c->geom.q == 9)
      k_outlet_adjoint<9><<<fgrid, 256, 0, c->stream>>>(c->geom, fc, edge, f, c->outlet_g, lam_out,
                                                        F[0], F[1], F[2], c->face_stride);
    else
      k_outlet_adjoint<19><<<fgrid, 256, 0, c->stream>>>(c->geom, fc, edge, f, c->outlet_g, lam_out,
                                                         F[0], F[1], F[2], c->face_stride);
  }
  return hip_ok(hipGetLastError());
}

template <int D, bool FLAT>
static int rasterize_adjoint(psclbm_ctx* c, const double* gs, int kslots, double* gX) {
  const size_t lds = (sizeof(LdsEntry) + sizeof(double)) * (size_t)c->lists.cap;
  k_rasterize_adjoint<D, FLAT><<<c->ntiles, BLOCK, lds, c->stream>>>(
      c->geom, c->cfg.shell_h, c->np, c->tile_count, c->lists, c->snap, gs,
      kslots, gX);
  return hip_ok(hipGetLastError());
}

int launch_rasterize_adjoint(psclbm_ctx* c, const double* gs, int kslots, double* gX) {
  if (c->geom.q == 9)
    return c->geom.flat ? rasterize_adjoint<2, true>(c, gs, kslots, gX)
                        : rasterize_adjoint<2, false>(c, gs, kslots, gX);
  return c->geom.flat ? rasterize_adjoint<3, true>(c, gs, kslots, gX)
                      : rasterize_adjoint<3, false>(c, gs, kslots, gX);
}

}  // namespace psclbm
