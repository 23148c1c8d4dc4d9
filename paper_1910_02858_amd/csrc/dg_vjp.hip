// Vector-Jacobian product of the split-form DGSEM operator on LGL nodes (one workgroup per
// element), for Ubar = (dL/dU)^T Utbar.
//
// The forward operator (Krais et al., FLEXI, Sec. 3.3 eq. semiDiscreteSplit with BR1 lifting,
// Sec. 3.1 eq. discreteGradient) is
//   U_t = -(1/J) acc,  acc_q = sum_dir [ sum_m 2 D_im F#(U_q, U_m) - sum_m D_im Fv_m ]
//                            + sum_faces lhat (F_face - sg F_int,q),
//   G = lift(W(U)),    W = (u, v, w, T).
// G holds the contravariant viscous fluxes Fv^dir of the lifting (LIFT_FV): the viscous flux is
// linear in the gradients, so its derivative in U needs only tau . Ja^dir, their momentum part.
// Face normals are Ja^dir at the face node of the element itself, as in the forward kernels.
// With Abar = -(1/J) Utbar (the adjoint of acc) the reverse is:
//   * each unordered pair {q, p} on a line: Fbar = 2 D_qp Abar_q + 2 D_pq Abar_p, then the
//     two-point flux's transposed Jacobian in both arguments (the partner's share goes through
//     LDS, one share per node and round, collected in a fixed order);
//   * viscous volume term: Fvbar_p = -sum_q D_qp Abar_q, then the viscous flux's transposed
//     Jacobian in U and in G;
//   * each face point: the flux enters both elements, so Fbar = lhat (Abar_master - Abar_slave),
//     and every element adds only the derivative with respect to its own trace (the neighbour's
//     Abar is read from global memory, nothing is written into another element);
//   * the lifting transposed: with H = (1/J) Gbar, Wbar = sum_dir Ja^dir . (Dhat^T H) along the
//     lines plus, on each face point, c0 Ja^dn . H (c0 = +-lhat/2) — a term that enters the
//     element's own Wbar and, the face state being the mean of both traces, the neighbour's
//     Wbar at the matching point.  The first kernel does the element's own part and leaves the
//     face terms in a face array; the second adds the neighbours' face terms and W's Jacobian
//     on the face nodes and performs the register update of the 2N scheme.
#include <hip/hip_runtime.h>

#include "dg_flux.h"
#include "dg_internal.h"
#include "dg_lines.h"

// minimum waves per SIMD of the operator's vector-Jacobian kernel (caps its registers)
#ifndef DG_VJP_MINB
#define DG_VJP_MINB 2
#endif
// stage the metric terms and kept viscous fluxes in LDS where they fit
#ifndef DG_VJP_STAGE
#define DG_VJP_STAGE 1
#endif

namespace dg {

template <int N> struct VSz {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  static constexpr int NT = ((n3 + 63) / 64) * 64;
};

template <int n> __device__ __forceinline__ int vline_node(int dn, int a, int b, int m) {
  return dn == 0 ? (m + n * (a + n * b)) : (dn == 1 ? (a + n * (m + n * b)) : (a + n * (b + n * m)));
}

// ---------------------------------------------------------------------------------- main, EC and central flux
// One node per lane; the kinetic-energy preserving flux takes k_vjp_line below.
// GEN: the mesh has face codes (faces on any side, in any orientation, symmetry planes), and
// every neighbour value is read at the neighbour's matching face point.  The face terms
// themselves need no change: with the two copies of a face flux related by the antisymmetry of
// the surface flux (same-parity sides) or equal (opposite parities), the own-trace derivative of
// both copies is lhat (Abar_own - Abar_nb) times the outward sign of this side in every case.
// A symmetry plane has one copy (Abar_nb = 0) whose outer state is the mirrored own trace: the
// outer argument's adjoint comes back mirrored, and the viscous term keeps only the normal part
// of the own momentum flux.
template <int N, bool NS, bool GEN>
__global__ void __launch_bounds__(VSz<N>::NT, DG_VJP_MINB) k_vjp_main(Geo g, Phys ph, const double *__restrict__ U,
                                                         const double *__restrict__ G,
                                                         const double *__restrict__ Utb, double *__restrict__ Ub,
                                                         double *__restrict__ Pf, double scale, int accumulate) {
  using S = VSz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = S::NT;
  constexpr int NF = NS ? 17 : 5;  // results per face point: primitive adjoint, gradient adjoint
  constexpr int NX = (NF * 6 * n2 > 9 * n3) ? NF * 6 * n2 : 9 * n3;
  __shared__ double sQ[5 * n3];  // primitive state
  __shared__ double sA[5 * n3];  // Abar = -(1/J) Utbar
  // region X: first the face-point results, then H = (1/J) Gbar (9 per node, Navier-Stokes),
  // then Ja^dir of the current direction (3 per node) and the partner shares of the pair
  // rounds (5 per node)
  static_assert(!NS || NX >= 9 * n3, "region X holds H");
  static_assert(NX >= 9 * n3, "region X holds Ja^dir and the partner shares");
  // where the LDS allows it, all metric terms (9 per node) and the momentum part of the kept
  // viscous fluxes (9 per node) are staged once at the start, so that no later phase waits on a
  // global load after a barrier
  constexpr int NST = 9 + (NS ? 9 : 0);
  constexpr bool STAGE = DG_VJP_STAGE && (10 + NST) * n3 + NX + 2 * n * n <= 160 * 1024 / 8;
  __shared__ double sX[NX];
  __shared__ double sD[n * n], sDh[n * n];
  __shared__ double sM[STAGE ? NST * n3 : 1];  // Ja^i_d at (i*3+d)*n3, then Fv^dir_c at (9+dir*3+c)*n3
  double *sF = sX, *sH = sX, *sJ = sX, *sPA = sX + 3 * n3;
  const int e = xcd_element(blockIdx.x, g.K), t = threadIdx.x;
  if (e >= g.K) return;
  const bool act = t < n3;
  const double gamma = ph.gamma, gm1 = gamma - 1.0, g1 = gamma / gm1;
  const int vf = ph.vf;
  for (int c = t; c < n * n; c += NT) { sD[c] = g.tab->D[c]; sDh[c] = g.tab->Dh[c]; }
  const double lh = g.tab->lhp[N];  // lhat at a face node (the same value at both ends)
  const double *Ue = U + (size_t)e * 5 * n3;
  const double *Ge = G + (size_t)e * 12 * n3;
  const double *Jae = g.Ja + (size_t)e * 9 * n3;
  const double *sJe = g.sJ + (size_t)e * n3;
  // this element's metric term Ja^dir_d and momentum viscous flux Fv^dir_c at a node
  auto JA = [&](int dir, int d, int node) -> double {
    if constexpr (STAGE) return sM[(dir * 3 + d) * n3 + node];
    else return Jae[(dir * 3 + d) * n3 + node];
  };
  auto FV = [&](int dir, int c, int node) -> double {
    if constexpr (STAGE) return sM[(9 + dir * 3 + c) * n3 + node];
    else return Ge[(dir * 4 + c) * n3 + node];
  };
  if (STAGE && act) {
#pragma unroll
    for (int c = 0; c < 9; ++c) sM[c * n3 + t] = Jae[c * n3 + t];
    if (NS) {
#pragma unroll
      for (int dir = 0; dir < 3; ++dir)
#pragma unroll
        for (int c = 0; c < 3; ++c) sM[(9 + dir * 3 + c) * n3 + t] = Ge[(dir * 4 + c) * n3 + t];
    }
  }
  dgf::P q;
  if (act) {
    double Uq[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = Ue[v * n3 + t];
    q = dgf::prim(Uq, gm1);
    sQ[t] = q.r; sQ[n3 + t] = q.u; sQ[2 * n3 + t] = q.v; sQ[3 * n3 + t] = q.w; sQ[4 * n3 + t] = q.p;
    const double sj = sJe[t];
#pragma unroll
    for (int v = 0; v < 5; ++v) sA[v * n3 + t] = -sj * Utb[((size_t)e * 5 + v) * n3 + t];
  }
  __syncthreads();
  // ---- faces: Fbar = lhat (Abar_master - Abar_slave); own-trace derivative only.  All six
  // faces at once, one face point per thread; the results wait in LDS per face point and every
  // node collects its (up to three) face terms in direction order.
  for (int p = t; p < 6 * n2; p += NT) {
    const int s = p / n2, ab = p % n2, a = ab % n, b = ab / n, dn = s >> 1;
    const bool plus = s & 1;
    const int qo = vline_node<n>(dn, a, b, plus ? N : 0);
    int qn, nb;
    bool bnd = false, given = false, wall = false, iso = false, outflow = false;
    if constexpr (GEN) {
      const NbFace f = nbr_face<n, true>(g, e, s, a, b);
      qn = vline_node<n>(f.dn, f.a, f.b, f.plus ? N : 0);
      bnd = f.bnd;
      outflow = bnd && f.kind == DG_BC_OUTFLOW;
      given = bnd && (f.kind == DG_BC_STATE || outflow);
      iso = bnd && f.kind == DG_BC_WALL_ISOTHERMAL;
      wall = bnd && (f.kind == DG_BC_WALL || iso);
      nb = bnd ? e : g.nbr[(size_t)e * 6 + s];  // a boundary side reads nothing of a neighbour
    } else {
      qn = vline_node<n>(dn, a, b, plus ? 0 : N);
      nb = g.nbr[(size_t)e * 6 + s];
    }
    double Uw[5], Ux[5], Aw[5], Ax[5];
    const double sjn = g.sJ[(size_t)nb * n3 + qn];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Uw[v] = Ue[v * n3 + qo];
      Ux[v] = U[((size_t)nb * 5 + v) * n3 + qn];
      Aw[v] = sA[v * n3 + qo];
      Ax[v] = bnd ? 0.0 : -sjn * Utb[((size_t)nb * 5 + v) * n3 + qn];
    }
    // normal along +xi_dn scaled by s-hat: this element's Ja^dn at the face node
    const double nt[3] = {JA(dn, 0, qo), JA(dn, 1, qo), JA(dn, 2, qo)};
    const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    const double ish = 1.0 / sh;
    const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
    if (outflow) {
      // pressure outflow: the own trace's density and velocity with p_out
      Ux[0] = Uw[0]; Ux[1] = Uw[1]; Ux[2] = Uw[2]; Ux[3] = Uw[3];
      Ux[4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
    } else if (given) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[v] = ph.ub[v];  // given outer state, independent of U
    } else if (wall) {
      // no-slip wall: the outer state is the own trace with the velocity reversed
      Ux[0] = Uw[0]; Ux[1] = -Uw[1]; Ux[2] = -Uw[2]; Ux[3] = -Uw[3]; Ux[4] = Uw[4];
    } else if (bnd) {
      // symmetry plane: the outer state is the mirrored own trace
      const double mn = 2.0 * (Uw[1] * nh[0] + Uw[2] * nh[1] + Uw[3] * nh[2]);
      Ux[0] = Uw[0]; Ux[4] = Uw[4];
      Ux[1] = Uw[1] - mn * nh[0]; Ux[2] = Uw[2] - mn * nh[1]; Ux[3] = Uw[3] - mn * nh[2];
    }
    double Fb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Fb[v] = lh * (plus ? (Aw[v] - Ax[v]) : (Ax[v] - Aw[v]));
    const double *UM = plus ? Uw : Ux, *US = plus ? Ux : Uw;
    const dgf::P PM = dgf::prim(UM, gm1), PS = dgf::prim(US, gm1);
    double Fbs[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Fbs[v] = Fb[v] * sh;
    // the primitive adjoint of the own trace (the final (dP/dU)^T map of the node applies to it)
    dgf::PA aM = dgf::zero_pa(), aS = dgf::zero_pa();
    dgf::riemann_adj_prim(ph.rs, vf, PM, PS, UM, US, nh, gamma, Fbs, aM, aS);
    dgf::PA pc = plus ? aM : aS;
    const dgf::P Po = plus ? PM : PS;
    if (outflow) {
      // the outer argument's density and velocity are the own trace's, its pressure is fixed
      const dgf::PA ao = plus ? aS : aM;
      pc.r += ao.r; pc.u += ao.u; pc.v += ao.v; pc.w += ao.w;
    } else if (wall) {
      // the outer argument is the own trace with the velocity reversed
      const dgf::PA ao = plus ? aS : aM;
      pc.r += ao.r; pc.p += ao.p;
      pc.u -= ao.u; pc.v -= ao.v; pc.w -= ao.w;
    } else if (bnd && !given) {
      // the outer argument is the mirror image of the own trace: its adjoint comes back mirrored
      const dgf::PA ao = plus ? aS : aM;
      const double an = 2.0 * (ao.u * nh[0] + ao.v * nh[1] + ao.w * nh[2]);
      pc.r += ao.r; pc.p += ao.p;
      pc.u += ao.u - an * nh[0]; pc.v += ao.v - an * nh[1]; pc.w += ao.w - an * nh[2];
    }
    if (NS) {
      // F contains -1/2 Fv(U_own, G_own) . nt; its momentum part along the face's direction is
      // the contravariant viscous flux of that direction from the lifting (G holds those)
      double gbo[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) gbo[c] = 0.0;
      const double tn[3] = {FV(dn, 0, qo), FV(dn, 1, qo), FV(dn, 2, qo)};
      double Fvb[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) Fvb[v] = -0.5 * Fb[v];
      if (given) {
        // given outer state: the term is -g, the whole own flux
#pragma unroll
        for (int v = 0; v < 5; ++v) Fvb[v] = -Fb[v];
      } else if (iso) {
        // isothermal wall: the terms are -g_m for the momentum and -(g_E - g_m . u) for the
        // energy, with u this node's velocity
        Fvb[0] = 0.0; Fvb[4] = -Fb[4];
        Fvb[1] = -Fb[1] + Fb[4] * Po.u; Fvb[2] = -Fb[2] + Fb[4] * Po.v; Fvb[3] = -Fb[3] + Fb[4] * Po.w;
        pc.u += Fb[4] * tn[0]; pc.v += Fb[4] * tn[1]; pc.w += Fb[4] * tn[2];
      } else if (wall) {
        // no-slip wall: the term is -g for the momentum, nothing for the energy
        Fvb[0] = 0.0; Fvb[4] = 0.0;
        Fvb[1] = -Fb[1]; Fvb[2] = -Fb[2]; Fvb[3] = -Fb[3];
      } else if (bnd) {
        // symmetry plane: the term is -(g.nh) nh of the own momentum flux g, no energy part
        const double fn_ = Fb[1] * nh[0] + Fb[2] * nh[1] + Fb[3] * nh[2];
        Fvb[0] = 0.0; Fvb[4] = 0.0;
        Fvb[1] = -fn_ * nh[0]; Fvb[2] = -fn_ * nh[1]; Fvb[3] = -fn_ * nh[2];
      }
      dgf::visc_flux_adj_tn(Po, tn, ph.mu, ph.kappa, nt, Fvb, pc, gbo);
#pragma unroll
      for (int c = 0; c < 12; ++c) sF[(5 + c) * 6 * n2 + p] = gbo[c];
    }
    sF[0 * 6 * n2 + p] = pc.r;
    sF[1 * 6 * n2 + p] = pc.u;
    sF[2 * 6 * n2 + p] = pc.v;
    sF[3 * 6 * n2 + p] = pc.w;
    sF[4 * 6 * n2 + p] = pc.p;
  }
  __syncthreads();
  dgf::PA pa = dgf::zero_pa();
  double gbf[12];  // gradient adjoint of the face terms at this node
#pragma unroll
  for (int c = 0; c < 12; ++c) gbf[c] = 0.0;
  const int id3[3] = {t % n, (t / n) % n, t / n2};
  if (act) {
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
      const int id = id3[dir];
      if (id != 0 && id != N) continue;
      const int s = 2 * dir + (id == N ? 1 : 0);
      const int a = dir == 0 ? id3[1] : id3[0], b = dir == 2 ? id3[1] : id3[2];
      const int p = s * n2 + a + n * b;
      pa.r += sF[p]; pa.u += sF[6 * n2 + p]; pa.v += sF[2 * 6 * n2 + p]; pa.w += sF[3 * 6 * n2 + p];
      pa.p += sF[4 * 6 * n2 + p];
      if (NS) {
#pragma unroll
        for (int c = 0; c < 12; ++c) gbf[c] += sF[(5 + c) * 6 * n2 + p];
      }
    }
  }
  double cb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  // ---- interior convective flux F_int = Fc . Ja on the faces through this node
  if (act) {
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
      const int id = id3[dir];
      if (id != 0 && id != N) continue;
      const double sg = (id == N) ? 1.0 : -1.0;
      const double nv[3] = {JA(dir, 0, t), JA(dir, 1, t), JA(dir, 2, t)};
      double Fib[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) Fib[v] = -lh * sg * sA[v * n3 + t];
      dgf::euler_flux_adj(q, nv, g1, Fib, pa);
    }
  }
  // ---- viscous part, all directions before the pair rounds: acc_m -= sum_i D_mi Fv_i gives
  // Fvbar_i = -sum_m D_mi Abar_m; the interior face term -F_int contributes +lhat sg Abar_i.
  // The gradient adjoint of this node is final afterwards.
  double hg[12];  // H = (1/J) scale Gbar of this node
  if (NS && act) {
    double gbo[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) gbo[c] = gbf[c];
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
      const int id = id3[dir];
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
      double fvb[4] = {0.0, 0.0, 0.0, 0.0};
      if (id == 0 || id == N) {
        const double sg = (id == N) ? 1.0 : -1.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) fvb[c] -= -lh * sg * sA[(1 + c) * n3 + t];
      }
      for (int m = 0; m < n; ++m) {
        const int qm = base + m * str;
        const double Dmi = sD[m * n + id];
#pragma unroll
        for (int c = 0; c < 4; ++c) fvb[c] -= Dmi * sA[(1 + c) * n3 + qm];
      }
      const double nv[3] = {JA(dir, 0, t), JA(dir, 1, t), JA(dir, 2, t)};
      const double Fvb[5] = {0.0, fvb[0], fvb[1], fvb[2], fvb[3]};
      const double tn[3] = {FV(dir, 0, t), FV(dir, 1, t), FV(dir, 2, t)};
      dgf::visc_flux_adj_tn(q, tn, ph.mu, ph.kappa, nv, Fvb, pa, gbo);
    }
    const double sj = sJe[t];
#pragma unroll
    for (int c = 0; c < 12; ++c) hg[c] = sj * (scale * gbo[c]);
  }
  // ---- lifting transposed, own part (volume and own face terms); the face terms also go to
  // the face array for the neighbours.  The velocity block of H is symmetric, H_dc = H_cd (every
  // viscous transpose adds mu (T_cd + T_dc) - 2/3 mu tr(T) delta_cd), so region X holds its six
  // distinct entries (00, 11, 22, 01, 02, 12) and the three temperature entries, 9 per node.
  dgf::PA pl = dgf::zero_pa();
  if (NS) {
    __syncthreads();  // every node has collected its face results from region X
    if (act) {
      const double h9[9] = {hg[0], hg[5], hg[10], hg[1], hg[2], hg[6], hg[3], hg[7], hg[11]};
#pragma unroll
      for (int c = 0; c < 9; ++c) sH[c * n3 + t] = h9[c];
    }
    __syncthreads();
    if (act) {
      double Wb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int dir = 0; dir < 3; ++dir) {
        const int id = id3[dir];
        const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
        const int base = t - id * str;
        const double nv[3] = {JA(dir, 0, t), JA(dir, 1, t), JA(dir, 2, t)};
        double hs[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) hs[c] = 0.0;
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
          const int qi = base + i * str;
          const double Dh = sDh[i * n + id];
#pragma unroll
          for (int c = 0; c < 9; ++c) hs[c] += Dh * sH[c * n3 + qi];
        }
        Wb[0] += nv[0] * hs[0] + nv[1] * hs[3] + nv[2] * hs[4];
        Wb[1] += nv[0] * hs[3] + nv[1] * hs[1] + nv[2] * hs[5];
        Wb[2] += nv[0] * hs[4] + nv[1] * hs[5] + nv[2] * hs[2];
        Wb[3] += nv[0] * hs[6] + nv[1] * hs[7] + nv[2] * hs[8];
        if (id == 0 || id == N) {
          const int sd = (id == N) ? 1 : 0;
          const int s = 2 * dir + sd;
          const int a = dir == 0 ? id3[1] : id3[0], b = dir == 2 ? id3[1] : id3[2];
          const double c0 = (sd ? 0.5 : -0.5) * lh;
          double *pf = Pf + ((size_t)e * 6 + s) * 4 * n2 + a + n * b;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double f = c0 * (nv[0] * hg[v] + nv[1] * hg[4 + v] + nv[2] * hg[8 + v]);
            Wb[v] += f;
            pf[v * n2] = f;
          }
        }
      }
      dgf::lift_vars_adj(q, ph.R, Wb, pl);
    }
  }
  // ---- volume: pairs and diagonal, direction by direction
  // the epilogue's loads are issued before the rounds
  double *Ube = Ub + (size_t)e * 5 * n3;
  double ub0[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (act && accumulate) {
#pragma unroll
    for (int v = 0; v < 5; ++v) ub0[v] = Ube[v * n3 + t];
  }
  for (int dir = 0; dir < 3; ++dir) {
    double nvo[3] = {0.0, 0.0, 0.0};
    const double *sJd = sJ;
    if constexpr (STAGE) {
      // the metric terms are in LDS already; every exchange round ends with a barrier, so
      // only the first direction needs one (after the last reads of region X)
      if (dir == 0) __syncthreads();
      sJd = sM + dir * 3 * n3;
      if (act) { nvo[0] = sJd[t]; nvo[1] = sJd[n3 + t]; nvo[2] = sJd[2 * n3 + t]; }
    } else {
      __syncthreads();
      if (act) {
        nvo[0] = Jae[(dir * 3) * n3 + t]; nvo[1] = Jae[(dir * 3 + 1) * n3 + t]; nvo[2] = Jae[(dir * 3 + 2) * n3 + t];
        sJ[t] = nvo[0]; sJ[n3 + t] = nvo[1]; sJ[2 * n3 + t] = nvo[2];
      }
      __syncthreads();
    }
    {
      const int id = act ? id3[dir] : 0;
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
      double Ao[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) Ao[v] = act ? sA[v * n3 + t] : 0.0;
#pragma unroll 1
      for (int sft = 1; sft <= n / 2; ++sft) {
        if (act) {
          const bool half = (2 * sft == n);  // the pair at distance n/2 is met from both ends
          int jp = id + sft;
          if (jp >= n) jp -= n;
          const int qp = base + jp * str;
          dgf::P r;
          r.r = sQ[qp]; r.u = sQ[n3 + qp]; r.v = sQ[2 * n3 + qp]; r.w = sQ[3 * n3 + qp]; r.p = sQ[4 * n3 + qp];
          const double nm[3] = {0.5 * (nvo[0] + sJd[qp]), 0.5 * (nvo[1] + sJd[n3 + qp]),
                                0.5 * (nvo[2] + sJd[2 * n3 + qp])};
          const double Dij2 = 2.0 * sD[id * n + jp], Dji2 = 2.0 * sD[jp * n + id];
          double Fb[5];
#pragma unroll
          for (int v = 0; v < 5; ++v) Fb[v] = Dij2 * Ao[v] + (half ? 0.0 : Dji2 * sA[v * n3 + qp]);
          dgf::PA pr = dgf::zero_pa();
          r.ir = 1.0 / r.r;  // the central flux's enthalpies need it
          dgf::pair_flux_adj(vf, q, r, nm, g1, Fb, pa, pr);
          // every node receives exactly one partner share per round
          sPA[qp] = pr.r; sPA[n3 + qp] = pr.u; sPA[2 * n3 + qp] = pr.v; sPA[3 * n3 + qp] = pr.w;
          sPA[4 * n3 + qp] = pr.p;
        }
        __syncthreads();
        if (act) {
          pa.r += sPA[t]; pa.u += sPA[n3 + t]; pa.v += sPA[2 * n3 + t]; pa.w += sPA[3 * n3 + t];
          pa.p += sPA[4 * n3 + t];
        }
        __syncthreads();
      }
      if (!act) continue;
      const double Dii = sD[id * n + id];
      if (Dii != 0.0) {
        double Fb[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) Fb[v] = 2.0 * Dii * Ao[v];
        dgf::euler_flux_adj(q, nvo, g1, Fb, pa);
      }
    }
  }
  if (act) {
    dgf::PA pt;
    pt.r = fma(scale, pa.r, pl.r); pt.u = fma(scale, pa.u, pl.u); pt.v = fma(scale, pa.v, pl.v);
    pt.w = fma(scale, pa.w, pl.w); pt.p = fma(scale, pa.p, pl.p);
    dgf::cons_adj(q, gm1, pt, cb);
#pragma unroll
    for (int v = 0; v < 5; ++v) Ube[v * n3 + t] = ub0[v] + cb[v];
  }
}

// ---------------------------------------------------------------------------------- main, KEP flux
// The same reverse for the kinetic-energy preserving two-point flux, one lane per line (as the split-form
// operator): the lane evaluates the adjoints of the numerical fluxes at its line's ends, of each unordered
// pair of its nodes once, and the line contractions of the viscous terms and of the transposed lifting.
// What bounds it: with one node per lane a third of the LDS accesses and 18 of 24 barriers were the exchange
// of the pairs' partner shares; vector instructions took 49 % and the LDS 46 % of the time at two waves per
// SIMD.  One product (Navier-Stokes, Roe, with its lifting and face kernels): N = 5, 24^3 curved 802 -> 580 us;
// N = 7, 16^3 curved 662 -> 485, affine 662 -> 429; N = 3, 32^3 579 -> 416; Euler N = 4, 24^3 177 -> 152.
// The pair's adjoint is the same for both of its nodes: with sums over the pair r2, u2, H2, nS = n_q + n_p,
// f = D_qp Abar_q + D_pq Abar_p, s = u2 . nS and g = 2 f_0 + f_m . u2 + f_4 H2 each node receives
// (1/8) (g s, r2 (s f_m + g nS), 4 f_m . nS, r2 s f_4) in (rho, u, p, H).  The diagonal of D and the interior
// surface flux cancel in the Euler part (2 D_ii = +-lhat on LGL nodes).
template <int N> struct VjpLds {  // doubles of one element: rho, u, v, w, H and Abar (10 per node), metric terms (9)
  static constexpr int n3 = (N + 1) * (N + 1) * (N + 1);
  // Navier-Stokes: the viscous adjoints (12 per node) take the place of the state and Abar and need two more;
  // where those cost a workgroup per CU they lie over the first two metric terms, which are then read again
  static constexpr bool TIGHT = 160 * 1024 / (21 * n3 * 8) < 160 * 1024 / (19 * n3 * 8);
};

template <int N, bool NS, bool GEN, bool AFF>
__global__ void __launch_bounds__(SplitSz<N>::NT, 2)
    k_vjp_line(Geo g, Phys ph, const double *__restrict__ U, const double *__restrict__ G,
               const double *__restrict__ Utb, double *__restrict__ Ub, double *__restrict__ Pf, double scale,
               int accumulate) {
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n, NT = SplitSz<N>::NT, IT = (n3 + NT - 1) / NT;
  constexpr bool TIGHT = NS && !AFF && VjpLds<N>::TIGHT;
  constexpr int J0 = (NS && !TIGHT) ? 12 : 10;  // first component of the metric terms
  __shared__ double sm[(AFF ? (NS ? 12 : 10) : J0 + 9) * n3];
  double *sQ = sm, *sA = sm + 5 * n3, *sJ = sm + J0 * n3;  // node slots: div_slot
  const int e = xcd_element(blockIdx.x, g.K), lane = threadIdx.x;
  if (e >= g.K) return;
  AffineConst jc = nullptr;
  if constexpr (AFF) jc = affine_const(g, e);
  const double gamma = ph.gamma, gm1 = gamma - 1.0, g1 = gamma / gm1;
  typedef const __attribute__((address_space(4))) double *Scal;
  const Scal D = (Scal)g.tab->D, Dh = (Scal)g.tab->Dh;
  const double lh = g.tab->lhp[N];  // lhat at a face node (the same value at both ends)
  const double *Ue = U + (size_t)e * 5 * n3;
  const double *Ge = G + (size_t)e * 12 * n3;
  const double *Jae = g.Ja + (size_t)e * 9 * n3;
  const int dir = n2 % 64 == 0 ? __builtin_amdgcn_readfirstlane(lane / n2) : lane / n2;
  const int ab = lane - dir * n2, a = ab % n, b = ab / n;
  const bool act = lane < 3 * n2;
  // ---- loads: the neighbours' indices, the element's arrays, both sides' face nodes
  int nb2[2] = {0, 0};
  NbFace f2[2];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd)
    if (act) {
      nb2[sd] = g.nbr[(size_t)e * 6 + 2 * dir + sd];
      f2[sd] = nbr_face<n, GEN>(g, e, 2 * dir + sd, a, b);
    }
  double U0[IT][5], Aq[IT][5], Jq[IT][9], sj[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t < n3) {
#pragma unroll
      for (int v = 0; v < 5; ++v) U0[it][v] = Ue[v * n3 + t];
#pragma unroll
      for (int v = 0; v < 5; ++v) Aq[it][v] = Utb[((size_t)e * 5 + v) * n3 + t];
      sj[it] = AFF ? jc[9] : g.sJ[(size_t)e * n3 + t];
#pragma unroll
      for (int c = 0; c < 9 && !AFF; ++c) Jq[it][c] = Jae[c * n3 + t];
    }
  }
  double Uw2[2][5], Ux2[2][5], Ax2[2][5], sx2[2];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd)
    if (act) {
      const bool bnd = GEN && f2[sd].bnd;
      const int nb = bnd ? e : nb2[sd];  // a boundary side reads nothing of a neighbour
      const int qo = vline_node<n>(dir, a, b, sd ? N : 0);
      const int qn = GEN ? vline_node<n>(f2[sd].dn, f2[sd].a, f2[sd].b, f2[sd].plus ? N : 0)
                         : vline_node<n>(dir, a, b, sd ? 0 : N);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        Uw2[sd][v] = Ue[v * n3 + qo];
        Ux2[sd][v] = U[((size_t)nb * 5 + v) * n3 + qn];
        Ax2[sd][v] = Utb[((size_t)nb * 5 + v) * n3 + qn];
      }
      sx2[sd] = AFF ? g.Jc[(size_t)nb * AFFINE_DOUBLES + 9] : g.sJ[(size_t)nb * n3 + qn];
    }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t < n3) {
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
      const dgf::P p = dgf::prim(U0[it], gm1);
      sQ[q] = p.r; sQ[n3 + q] = p.u; sQ[2 * n3 + q] = p.v; sQ[3 * n3 + q] = p.w;
      sQ[4 * n3 + q] = dgf::enthalpy(p, g1);
#pragma unroll
      for (int v = 0; v < 5; ++v) sA[v * n3 + q] = -sj[it] * Aq[it][v];
#pragma unroll
      for (int c = 0; c < 9 && !AFF; ++c) sJ[c * n3 + q] = Jq[it][c];
    }
  }
  __syncthreads();
  const LineSlots<n> slot(act ? dir : 0, act ? a : 0, act ? b : 0);
  const double *sJd = sJ + 3 * (act ? dir : 0) * n3;
  double jl[3] = {0.0, 0.0, 0.0};
  if constexpr (AFF) {
#pragma unroll
    for (int d = 0; d < 3; ++d) jl[d] = dir == 0 ? jc[d] : (dir == 1 ? jc[3 + d] : jc[6 + d]);
  }
  auto metric = [&](int d, int q) -> double {
    if constexpr (AFF) return jl[d];
    else return sJd[d * n3 + q];
  };
  double acc[n][6];          // adjoints of rho, u, v, w, p, H of the line's nodes
  double fv[NS ? n : 1][4];  // adjoints of the viscous fluxes along the line's direction
  if (act) {
    // ---- faces: Fbar = lhat (Abar_master - Abar_slave); own-trace derivative only
    double pe[2][5], fe[2][4];
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      const bool plus = sd;
      const int qo = slot(plus ? N : 0);
      const bool bnd = GEN && f2[sd].bnd;
      const bool outflow = bnd && f2[sd].kind == DG_BC_OUTFLOW;
      const bool given = bnd && (f2[sd].kind == DG_BC_STATE || outflow);
      const bool iso = bnd && f2[sd].kind == DG_BC_WALL_ISOTHERMAL;
      const bool wall = bnd && (f2[sd].kind == DG_BC_WALL || iso);
      double *Uw = Uw2[sd], *Ux = Ux2[sd];
      // normal along +xi_dir scaled by s-hat: this element's Ja^dir at the face node
      const double nt[3] = {metric(0, qo), metric(1, qo), metric(2, qo)};
      const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
      const double ish = 1.0 / sh;
      const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
      if (outflow) {
        // pressure outflow: the own trace's density and velocity with p_out
        Ux[0] = Uw[0]; Ux[1] = Uw[1]; Ux[2] = Uw[2]; Ux[3] = Uw[3];
        Ux[4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
      } else if (given) {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[v] = ph.ub[v];  // given outer state, independent of U
      } else if (wall) {
        // no-slip wall: the outer state is the own trace with the velocity reversed
        Ux[0] = Uw[0]; Ux[1] = -Uw[1]; Ux[2] = -Uw[2]; Ux[3] = -Uw[3]; Ux[4] = Uw[4];
      } else if (bnd) {
        // symmetry plane: the outer state is the mirrored own trace
        const double mn = 2.0 * (Uw[1] * nh[0] + Uw[2] * nh[1] + Uw[3] * nh[2]);
        Ux[0] = Uw[0]; Ux[4] = Uw[4];
        Ux[1] = Uw[1] - mn * nh[0]; Ux[2] = Uw[2] - mn * nh[1]; Ux[3] = Uw[3] - mn * nh[2];
      }
      double Fb[5], Fbs[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double ao = sA[v * n3 + qo], ax = bnd ? 0.0 : -sx2[sd] * Ax2[sd][v];
        Fb[v] = lh * (plus ? (ao - ax) : (ax - ao));
        Fbs[v] = Fb[v] * sh;
      }
      const double *UM = plus ? Uw : Ux, *US = plus ? Ux : Uw;
      const dgf::P PM = dgf::prim(UM, gm1), PS = dgf::prim(US, gm1);
      dgf::PA aM = dgf::zero_pa(), aS = dgf::zero_pa();
      dgf::riemann_adj_prim(ph.rs, 0, PM, PS, UM, US, nh, gamma, Fbs, aM, aS);
      dgf::PA pc = plus ? aM : aS;
      const dgf::PA ao = plus ? aS : aM;
      const dgf::P Po = plus ? PM : PS;
      if (outflow) {
        // the outer argument's density and velocity are the own trace's, its pressure is fixed
        pc.r += ao.r; pc.u += ao.u; pc.v += ao.v; pc.w += ao.w;
      } else if (wall) {
        // the outer argument is the own trace with the velocity reversed
        pc.r += ao.r; pc.p += ao.p;
        pc.u -= ao.u; pc.v -= ao.v; pc.w -= ao.w;
      } else if (bnd && !given) {
        // the outer argument is the mirror image of the own trace: its adjoint comes back mirrored
        const double an = 2.0 * (ao.u * nh[0] + ao.v * nh[1] + ao.w * nh[2]);
        pc.r += ao.r; pc.p += ao.p;
        pc.u += ao.u - an * nh[0]; pc.v += ao.v - an * nh[1]; pc.w += ao.w - an * nh[2];
      }
      if (NS) {
        // the face's own viscous flux, along the same Ja^dir as the node's: F contains -1/2 Fv . nt
#pragma unroll
        for (int c = 0; c < 4; ++c) fe[sd][c] = -0.5 * Fb[1 + c];
        if (given) {
          // given outer state: the term is -g, the whole own flux
#pragma unroll
          for (int c = 0; c < 4; ++c) fe[sd][c] = -Fb[1 + c];
        } else if (iso) {
          // isothermal wall: the terms are -g_m for the momentum and -(g_E - g_m . u) for the energy, with
          // u this node's velocity
          const int qg = vline_node<n>(dir, a, b, plus ? N : 0);
          fe[sd][0] = -Fb[1] + Fb[4] * Po.u; fe[sd][1] = -Fb[2] + Fb[4] * Po.v; fe[sd][2] = -Fb[3] + Fb[4] * Po.w;
          fe[sd][3] = -Fb[4];
          pc.u += Fb[4] * Ge[(dir * 4) * n3 + qg]; pc.v += Fb[4] * Ge[(dir * 4 + 1) * n3 + qg];
          pc.w += Fb[4] * Ge[(dir * 4 + 2) * n3 + qg];
        } else if (wall) {
          // no-slip wall: the term is -g for the momentum, nothing for the energy
          fe[sd][0] = -Fb[1]; fe[sd][1] = -Fb[2]; fe[sd][2] = -Fb[3]; fe[sd][3] = 0.0;
        } else if (bnd) {
          // symmetry plane: the term is -(g.nh) nh of the own momentum flux g, no energy part
          const double fn_ = Fb[1] * nh[0] + Fb[2] * nh[1] + Fb[3] * nh[2];
          fe[sd][0] = -fn_ * nh[0]; fe[sd][1] = -fn_ * nh[1]; fe[sd][2] = -fn_ * nh[2]; fe[sd][3] = 0.0;
        }
        // the interior face term -F_int contributes +lhat sg Abar
#pragma unroll
        for (int c = 0; c < 4; ++c) fe[sd][c] += (plus ? lh : -lh) * sA[(1 + c) * n3 + qo];
      }
      pe[sd][0] = pc.r; pe[sd][1] = pc.u; pe[sd][2] = pc.v; pe[sd][3] = pc.w; pe[sd][4] = pc.p;
      __builtin_amdgcn_sched_barrier(0);  // one end at a time: both in flight spill
    }
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 6; ++v) acc[m][v] = 0.0;
    // ---- pairs
    struct Nd { double s[5], A[5], nv[3]; };
    auto node = [&](int m) -> Nd {
      Nd x;
      const int q = slot(m);
#pragma unroll
      for (int v = 0; v < 5; ++v) { x.s[v] = sQ[v * n3 + q]; x.A[v] = sA[v * n3 + q]; }
#pragma unroll
      for (int d = 0; d < 3; ++d) x.nv[d] = metric(d, q);
      return x;
    };
#pragma unroll
    for (int i = 0; i + 1 < n; ++i) {
      const Nd X = node(i);
#pragma unroll
      for (int j = i + 1; j < n; ++j) {
        const Nd Y = node(j);
        const double Dij = D[i * n + j], Dji = D[j * n + i];
        const double r2 = X.s[0] + Y.s[0], u2 = X.s[1] + Y.s[1], v2 = X.s[2] + Y.s[2], w2 = X.s[3] + Y.s[3];
        const double H2 = X.s[4] + Y.s[4];
        const double nS[3] = {X.nv[0] + Y.nv[0], X.nv[1] + Y.nv[1], X.nv[2] + Y.nv[2]};
        double f[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) f[v] = fma(Dij, X.A[v], Dji * Y.A[v]);
        const double s = fma(u2, nS[0], fma(v2, nS[1], w2 * nS[2]));
        const double gg = fma(2.0, f[0], fma(f[1], u2, fma(f[2], v2, fma(f[3], w2, f[4] * H2))));
        const double rs = r2 * s, rg = r2 * gg;
        const double pp = fma(f[1], nS[0], fma(f[2], nS[1], f[3] * nS[2]));
        auto add = [&](double *x) {
          x[0] = fma(gg, s, x[0]);
#pragma unroll
          for (int d = 0; d < 3; ++d) x[1 + d] = fma(rs, f[1 + d], fma(rg, nS[d], x[1 + d]));
          x[4] += pp;
          x[5] = fma(rs, f[4], x[5]);
        };
        add(acc[i]);
        add(acc[j]);
        if ((j - i) % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // at most two pairs in flight
      }
      asm volatile("" ::: "memory");  // the next row's partners are read again, not kept
    }
#pragma unroll
    for (int m = 0; m < n; ++m) {
#pragma unroll
      for (int v = 0; v < 6; ++v) acc[m][v] *= v == 4 ? 0.5 : 0.125;
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) { acc[0][v] += pe[0][v]; acc[N][v] += pe[1][v]; }
    // ---- viscous volume term: acc_m -= sum_i D_mi Fv_i gives Fvbar_i = -sum_m D_mi Abar_m
    if constexpr (NS) {
#pragma unroll
      for (int m = 0; m < n; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c) fv[m][c] = m == 0 ? fe[0][c] : (m == N ? fe[1][c] : 0.0);
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const int q = slot(i);
        double A[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) A[c] = sA[(1 + c) * n3 + q];
#pragma unroll
        for (int m = 0; m < n; ++m) {
          const double d = -D[i * n + m];
#pragma unroll
          for (int c = 0; c < 4; ++c) fv[m][c] = fma(d, A[c], fv[m][c]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  double pv[IT][3];        // the viscous fluxes' adjoint in the node's velocity
  double W[NS ? n : 1][4];  // the transposed lifting's Wbar of the line's nodes
  if constexpr (NS) {
    __syncthreads();
    if (act) {
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = slot(m);
#pragma unroll
        for (int c = 0; c < 4; ++c) sm[(dir * 4 + c) * n3 + q] = fv[m][c];
      }
    }
    __syncthreads();
    // ---- node by node: the viscous fluxes' adjoint in the gradients, H = (1/J) scale Gbar.  The velocity block
    // of H is symmetric: six distinct entries (00, 11, 22, 01, 02, 12) and the three of the temperature.
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int t = lane + it * NT;
      pv[it][0] = pv[it][1] = pv[it][2] = 0.0;
      if (t < n3) {
        const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
        const double ir = 1.0 / Ue[t];
        const double u[3] = {Ue[n3 + t] * ir, Ue[2 * n3 + t] * ir, Ue[3 * n3 + t] * ir};
        const double sj = (AFF ? jc[9] : g.sJ[(size_t)e * n3 + t]) * scale;
        double T[3][3], k[3] = {0.0, 0.0, 0.0}, J01[2] = {0.0, 0.0};
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
          for (int y = 0; y < 3; ++y) T[x][y] = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          double nv[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if constexpr (AFF) nv[c] = jc[3 * d + c];
            else nv[c] = (TIGHT && 3 * d + c < 2) ? Jae[(3 * d + c) * n3 + t] : sJ[(3 * d + c) * n3 + q];
          }
          if (TIGHT && d == 0) { J01[0] = nv[0]; J01[1] = nv[1]; }
          const double F4 = sm[(d * 4 + 3) * n3 + q];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const double bm = fma(F4, u[c], sm[(d * 4 + c) * n3 + q]);
#pragma unroll
            for (int y = 0; y < 3; ++y) T[c][y] = fma(bm, nv[y], T[c][y]);
            k[c] = fma(F4, nv[c], k[c]);
            pv[it][c] = fma(F4, Ge[(d * 4 + c) * n3 + t], pv[it][c]);
          }
        }
        const double ms = ph.mu * sj, tr = (2.0 / 3.0) * (T[0][0] + T[1][1] + T[2][2]), ks = ph.kappa * sj;
        sm[q] = ms * fma(2.0, T[0][0], -tr);
        sm[n3 + q] = ms * fma(2.0, T[1][1], -tr);
        sm[2 * n3 + q] = ms * fma(2.0, T[2][2], -tr);
        sm[3 * n3 + q] = ms * (T[0][1] + T[1][0]);
        sm[4 * n3 + q] = ms * (T[0][2] + T[2][0]);
        sm[5 * n3 + q] = ms * (T[1][2] + T[2][1]);
#pragma unroll
        for (int d = 0; d < 3; ++d) sm[(6 + d) * n3 + q] = ks * k[d];
        if (TIGHT) { sJ[q] = J01[0]; sJ[n3 + q] = J01[1]; }
      }
    }
    __syncthreads();
    // ---- lifting transposed, own part: Wbar = Ja^dir . (Dhat^T H) along the line and the own face terms, which
    // also go to the face array for the neighbours
    if (act) {
#pragma unroll
      for (int m = 0; m < n; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) W[m][v] = 0.0;
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        const int m = sd ? N : 0, q = slot(m);
        const double c0 = (sd ? 0.5 : -0.5) * lh;
        const double nv[3] = {metric(0, q), metric(1, q), metric(2, q)};
        double h[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) h[c] = sm[c * n3 + q];
        const double f[4] = {c0 * (nv[0] * h[0] + nv[1] * h[3] + nv[2] * h[4]),
                             c0 * (nv[0] * h[3] + nv[1] * h[1] + nv[2] * h[5]),
                             c0 * (nv[0] * h[4] + nv[1] * h[5] + nv[2] * h[2]),
                             c0 * (nv[0] * h[6] + nv[1] * h[7] + nv[2] * h[8])};
        double *pf = Pf + ((size_t)e * 6 + 2 * dir + sd) * 4 * n2 + ab;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          W[m][v] = f[v];
          pf[v * n2] = f[v];
        }
      }
      // one entry of H after the other: (Wbar component, normal component) pairs it enters
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        constexpr int wa[9] = {0, 1, 2, 0, 0, 1, 3, 3, 3}, na[9] = {0, 1, 2, 1, 2, 2, 0, 1, 2};
        constexpr int wb[9] = {-1, -1, -1, 1, 2, 2, -1, -1, -1}, nb[9] = {0, 0, 0, 0, 0, 1, 0, 0, 0};
        double hs[n];
#pragma unroll
        for (int i = 0; i < n; ++i) {
          const double h = sm[c * n3 + slot(i)];
#pragma unroll
          for (int m = 0; m < n; ++m) hs[m] = i == 0 ? Dh[m] * h : fma(Dh[i * n + m], h, hs[m]);
        }
#pragma unroll
        for (int m = 0; m < n; ++m) {
          const int q = slot(m);
          W[m][wa[c]] = fma(metric(na[c], q), hs[m], W[m][wa[c]]);
          if (wb[c] >= 0) W[m][wb[c]] = fma(metric(nb[c], q), hs[m], W[m][wb[c]]);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);  // one entry at a time
      }
    }
  }
  // ---- the three directions' sums, in order, and the epilogue's loads
  double Uq[IT][5], ub0[IT][5];
  double *Ube = Ub + (size_t)e * 5 * n3;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Uq[it][v] = t < n3 ? Ue[v * n3 + t] : 1.0;
      ub0[it][v] = (t < n3 && accumulate) ? Ube[v * n3 + t] : 0.0;
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    __syncthreads();
    if (act && dir == d) {
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = d == 0 ? div_slot<n>(m, a, b) : (d == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
        for (int v = 0; v < 6; ++v) sm[v * n3 + q] = d == 0 ? acc[m][v] : sm[v * n3 + q] + acc[m][v];
        if constexpr (NS) {
#pragma unroll
          for (int v = 0; v < 4; ++v) sm[(6 + v) * n3 + q] = d == 0 ? W[m][v] : sm[(6 + v) * n3 + q] + W[m][v];
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t >= n3) continue;
    const int s = div_slot<n>(t % n, (t / n) % n, t / n2);
    const dgf::P q = dgf::prim(Uq[it], gm1);
    dgf::PA pa = {sm[s], sm[n3 + s], sm[2 * n3 + s], sm[3 * n3 + s], sm[4 * n3 + s]};
    dgf::PA pl = dgf::zero_pa();
    if constexpr (NS) {
      pa.u += pv[it][0]; pa.v += pv[it][1]; pa.w += pv[it][2];
      const double Wb[4] = {sm[6 * n3 + s], sm[7 * n3 + s], sm[8 * n3 + s], sm[9 * n3 + s]};
      dgf::lift_vars_adj(q, ph.R, Wb, pl);
    }
    dgf::enthalpy_adj(q, g1, sm[5 * n3 + s], pa);
    dgf::PA pt;
    pt.r = fma(scale, pa.r, pl.r); pt.u = fma(scale, pa.u, pl.u); pt.v = fma(scale, pa.v, pl.v);
    pt.w = fma(scale, pa.w, pl.w); pt.p = fma(scale, pa.p, pl.p);
    double cb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    dgf::cons_adj(q, gm1, pt, cb);
#pragma unroll
    for (int v = 0; v < 5; ++v) Ube[v * n3 + t] = ub0[it][v] + cb[v];
  }
}

// ---------------------------------------------------------------------------------- faces
// Completes Ubar on the face nodes with the neighbours' face terms of the transposed lifting
// (Wbar, then W's Jacobian at the node's state).  With upd != 0 the register of the 2N scheme
// is updated from the final Ubar of every node, Rb = ra Rb + rb Ubar (each node is read and
// written by its own thread only).
template <int N, bool GEN>
__global__ void __launch_bounds__(VSz<N>::NT) k_vjp_face(Geo g, Phys ph, const double *__restrict__ U,
                                                         const double *__restrict__ Pf, double *__restrict__ Ub,
                                                         double *__restrict__ Rb, double ra, double rb, int upd) {
  using S = VSz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3;
  const int e = xcd_element(blockIdx.x, g.K), t = threadIdx.x;
  if (e >= g.K || t >= n3) return;
  const int id3[3] = {t % n, (t / n) % n, t / n2};
  double Wb[4] = {0.0, 0.0, 0.0, 0.0};
  double tout = 0.0;  // adjoint of outflow sides' outer temperature p_out / (rho R)
  bool face = false;
#pragma unroll
  for (int dir = 0; dir < 3; ++dir) {
    const int id = id3[dir];
    if (id != 0 && id != N) continue;
    const int s = 2 * dir + (id == N ? 1 : 0);
    const int a = dir == 0 ? id3[1] : id3[0], b = dir == 2 ? id3[1] : id3[2];
    // the neighbour's term at its matching face point (structured: side s ^ 1, same index)
    if constexpr (GEN) {
      const NbFace f = nbr_face<n, true>(g, e, s, a, b);
      if (f.bnd && f.kind == DG_BC_OUTFLOW) {
        // pressure outflow: the outer W is (u, v, w, p_out / (rho R)) of this node
        const double *pf = Pf + ((size_t)e * 6 + s) * 4 * n2 + a + n * b;
        Wb[0] += pf[0]; Wb[1] += pf[n2]; Wb[2] += pf[2 * n2];
        tout += pf[3 * n2];
      } else if (f.bnd && f.kind == DG_BC_STATE) {
        // given outer state: W* depends on this element's W only through its own half
      } else if (f.bnd && f.kind == DG_BC_WALL) {
        // no-slip wall: the outer W is the own W with the velocity reversed
        const double *pf = Pf + ((size_t)e * 6 + s) * 4 * n2 + a + n * b;
        Wb[0] -= pf[0]; Wb[1] -= pf[n2]; Wb[2] -= pf[2 * n2];
        Wb[3] += pf[3 * n2];
      } else if (f.bnd && f.kind == DG_BC_WALL_ISOTHERMAL) {
        // isothermal wall: the outer W is (-u, -v, -w, 2 T_w - T)
        const double *pf = Pf + ((size_t)e * 6 + s) * 4 * n2 + a + n * b;
        Wb[0] -= pf[0]; Wb[1] -= pf[n2]; Wb[2] -= pf[2 * n2];
        Wb[3] -= pf[3 * n2];
      } else if (f.bnd) {
        // symmetry plane: the outer W is the mirrored own W, so the element's own face term
        // comes back with its velocity part mirrored
        const double *pf = Pf + ((size_t)e * 6 + s) * 4 * n2 + a + n * b;
        const double *fnp = g.fn + ((size_t)e * 6 + s) * 3 * n2 + a + n * b;
        const double nt[3] = {fnp[0], fnp[n2], fnp[2 * n2]};
        const double il = 1.0 / sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
        const double nh[3] = {nt[0] * il, nt[1] * il, nt[2] * il};
        const double w0 = pf[0], w1 = pf[n2], w2 = pf[2 * n2];
        const double wn = 2.0 * (w0 * nh[0] + w1 * nh[1] + w2 * nh[2]);
        Wb[0] += w0 - wn * nh[0]; Wb[1] += w1 - wn * nh[1]; Wb[2] += w2 - wn * nh[2];
        Wb[3] += pf[3 * n2];
      } else {
        const int nb = g.nbr[(size_t)e * 6 + s];
        const double *pf = Pf + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
#pragma unroll
        for (int v = 0; v < 4; ++v) Wb[v] += pf[v * n2];
      }
    } else {
      const int nb = g.nbr[(size_t)e * 6 + s];
      const double *pf = Pf + ((size_t)nb * 6 + (s ^ 1)) * 4 * n2 + a + n * b;
#pragma unroll
      for (int v = 0; v < 4; ++v) Wb[v] += pf[v * n2];
    }
    face = true;
  }
  if (!face && !upd) return;
  double *Ube = Ub + (size_t)e * 5 * n3 + t;
  double u[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) u[v] = Ube[v * n3];
  if (face) {
    double Uq[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = U[((size_t)e * 5 + v) * n3 + t];
    const dgf::P q = dgf::prim(Uq, ph.gamma - 1.0);
    dgf::PA pa = dgf::zero_pa();
    dgf::lift_vars_adj(q, ph.R, Wb, pa);
    pa.r -= tout * ph.pout * q.ir * q.ir / ph.R;
    double cb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    dgf::cons_adj(q, ph.gamma - 1.0, pa, cb);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      u[v] += cb[v];
      Ube[v * n3] = u[v];
    }
  }
  if (upd) {
    double *r = Rb + (size_t)e * 5 * n3 + t;
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v * n3] = ra * r[v * n3] + rb * u[v];
  }
}

// ---------------------------------------------------------------------------------- weak form
// Reverse of the weak form (Sec. 3.1, eq. semiDiscreteWeak) for the Euler equations on LG or LGL
// nodes.  The forward operator is
//   U_t,i = -(1/J_i) [ sum_dir sum_m Dhat_{id m} F^dir(U_m) + sum_faces lhat_face(i) f*_face ],
// with F^dir the contravariant Euler flux along Ja^dir_m at node m, f*_face the outward numerical
// flux times the surface element at the face point of node i's line (one value per face, the
// master's, entering the slave negated), evaluated from the two sides' traces prolonged with
// l(+-1) (LG) or read at the face nodes (LGL).  With Abar = -(1/J) Utbar:
//   * volume: Gbar^dir_m = sum_i Dhat_{id_i m} Abar_i along the line, then the flux Jacobian's
//     transpose at node m;
//   * faces: fbar = sg (sum_i lhat(i) Abar_i on this element's line - the same on the
//     neighbour's), the Riemann solver's transposed Jacobian in this element's own trace only
//     (the neighbour does the same for its trace), then the prolongation transposed onto the
//     line (LG) or the face node (LGL); a boundary side's outer state is a function of the own
//     trace and its adjoint comes back through that map.
// Nothing is written into another element.
template <int N, bool LGL, bool GEN>
__global__ void __launch_bounds__(VSz<N>::NT) k_vjp_weak(Geo g, Phys ph, const double *__restrict__ U,
                                                         const double *__restrict__ Utb, double *__restrict__ Ub,
                                                         double scale, int accumulate) {
  using S = VSz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = S::NT;
  __shared__ double sA[5 * n3];   // Abar = -(1/J) Utbar
  __shared__ double sU[5 * n3];   // the element's state
  __shared__ double sT[30 * n2];  // conservative adjoint of the own trace at every face point
  __shared__ double sDh[n * n], sl[2 * n], slh[2 * n];
  const int e = xcd_element(blockIdx.x, g.K), t = threadIdx.x;
  if (e >= g.K) return;
  const bool act = t < n3;
  const double gamma = ph.gamma, gm1 = gamma - 1.0, g1 = gamma / gm1;
  const Tab *tb = g.tab;
  for (int c = t; c < n * n; c += NT) sDh[c] = tb->Dh[c];
  if (t < n) {
    sl[t] = tb->lm[t]; sl[n + t] = tb->lp[t];
    slh[t] = tb->lhm[t]; slh[n + t] = tb->lhp[t];
  }
  const double *Ue = U + (size_t)e * 5 * n3;
  double Uo[5];
  if (act) {
    const double sj = g.sJ[(size_t)e * n3 + t];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Uo[v] = Ue[v * n3 + t];
      sU[v * n3 + t] = Uo[v];
      sA[v * n3 + t] = -sj * Utb[((size_t)e * 5 + v) * n3 + t];
    }
  }
  __syncthreads();
  for (int p = t; p < 6 * n2; p += NT) {
    const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
    const bool plus = s & 1;
    const NbFace f = nbr_face<n, GEN>(g, e, s, a, b);
    const bool bnd = GEN && f.bnd;
    const int nb = bnd ? e : g.nbr[(size_t)e * 6 + s];
    const int ns = GEN ? 2 * f.dn + (f.plus ? 1 : 0) : (s ^ 1);
    const bool nplus = ns & 1;
    // own and neighbour traces, and the weights of both sides' lines in the face adjoint
    double Uw[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, Ux[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    double Ao[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, An[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const double *lo = sl + (plus ? n : 0), *ln = sl + (nplus ? n : 0);
    const double *lho = slh + (plus ? n : 0), *lhn = slh + (nplus ? n : 0);
    const double *Un = U + (size_t)nb * 5 * n3;
    const double *Utn = Utb + (size_t)nb * 5 * n3;
    const double *sJn = g.sJ + (size_t)nb * n3;
#pragma unroll 1
    for (int m = 0; m < n; ++m) {
      if (LGL && m != (plus ? N : 0) && m != (nplus ? N : 0)) continue;
      const int q = vline_node<n>(dn, a, b, m);
      if (!LGL || m == (plus ? N : 0)) {
        const double wo = LGL ? 1.0 : lo[m], who = lho[m];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          Uw[v] += wo * sU[v * n3 + q];
          Ao[v] += who * sA[v * n3 + q];
        }
      }
      if (!bnd && (!LGL || m == (nplus ? N : 0))) {
        const int qn = vline_node<n>(f.dn, f.a, f.b, m);
        const double wn = LGL ? 1.0 : ln[m], whn = lhn[m];
        const double sjn = sJn[qn];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          Ux[v] += wn * Un[v * n3 + qn];
          An[v] += whn * (-sjn * Utn[v * n3 + qn]);
        }
      }
    }
    const double *fnp = g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
    const bool mst = GEN ? f.master : plus;
    const double sg = mst ? 1.0 : -1.0;
    const double nt[3] = {sg * fnp[0], sg * fnp[n2], sg * fnp[2 * n2]};
    const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    const double ish = 1.0 / sh;
    const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
    const bool outflow = bnd && f.kind == DG_BC_OUTFLOW;
    const bool given = bnd && (f.kind == DG_BC_STATE || outflow);
    const bool wall = bnd && (f.kind == DG_BC_WALL || f.kind == DG_BC_WALL_ISOTHERMAL);
    if (outflow) {
      Ux[0] = Uw[0]; Ux[1] = Uw[1]; Ux[2] = Uw[2]; Ux[3] = Uw[3];
      Ux[4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
    } else if (given) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[v] = ph.ub[v];
    } else if (wall) {
      Ux[0] = Uw[0]; Ux[1] = -Uw[1]; Ux[2] = -Uw[2]; Ux[3] = -Uw[3]; Ux[4] = Uw[4];
    } else if (bnd) {
      const double mn = 2.0 * (Uw[1] * nh[0] + Uw[2] * nh[1] + Uw[3] * nh[2]);
      Ux[0] = Uw[0]; Ux[4] = Uw[4];
      Ux[1] = Uw[1] - mn * nh[0]; Ux[2] = Uw[2] - mn * nh[1]; Ux[3] = Uw[3] - mn * nh[2];
    }
    // adjoint of the master's flux value (times s-hat): this element enters it with sign sg, the
    // neighbour with -sg
    double Fb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Fb[v] = sg * sh * (Ao[v] - An[v]);
    const double *UM = mst ? Uw : Ux, *US = mst ? Ux : Uw;
    const dgf::P PM = dgf::prim(UM, gm1), PS = dgf::prim(US, gm1);
    double bM[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, bS[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    dgf::riemann_adj(ph.rs, ph.vf, PM, PS, UM, US, nh, gamma, Fb, bM, bS);
    double bw[5], bx[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) { bw[v] = mst ? bM[v] : bS[v]; bx[v] = mst ? bS[v] : bM[v]; }
    if (outflow) {
      // outer state (rho, m, p_out/(gamma-1) + |m|^2/(2 rho)) of the own trace
      const double ir = 1.0 / Uw[0];
      const double k2 = (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) * ir * ir;
      bw[0] += bx[0] - 0.5 * k2 * bx[4];
      bw[1] += bx[1] + Uw[1] * ir * bx[4];
      bw[2] += bx[2] + Uw[2] * ir * bx[4];
      bw[3] += bx[3] + Uw[3] * ir * bx[4];
    } else if (wall) {
      bw[0] += bx[0]; bw[1] -= bx[1]; bw[2] -= bx[2]; bw[3] -= bx[3]; bw[4] += bx[4];
    } else if (bnd && !given) {
      // mirror image: the reflection is its own transpose
      const double mn = 2.0 * (bx[1] * nh[0] + bx[2] * nh[1] + bx[3] * nh[2]);
      bw[0] += bx[0]; bw[4] += bx[4];
      bw[1] += bx[1] - mn * nh[0]; bw[2] += bx[2] - mn * nh[1]; bw[3] += bx[3] - mn * nh[2];
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) sT[(s * 5 + v) * n2 + ab] = bw[v];
  }
  __syncthreads();
  if (act) {
    const int id3[3] = {t % n, (t / n) % n, t / n2};
    const dgf::P q = dgf::prim(Uo, gm1);
    dgf::PA pa = dgf::zero_pa();
    double ub[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const double *Jae = g.Ja + (size_t)e * 9 * n3;
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
      const int id = id3[dir];
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
      // volume: Gbar = sum over the line of Dhat_{id_i, id} Abar_i
      double Gb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      for (int m = 0; m < n; ++m) {
        const double d = sDh[m * n + id];
#pragma unroll
        for (int v = 0; v < 5; ++v) Gb[v] += d * sA[v * n3 + base + m * str];
      }
      const double nv[3] = {Jae[(dir * 3) * n3 + t], Jae[(dir * 3 + 1) * n3 + t], Jae[(dir * 3 + 2) * n3 + t]};
      dgf::euler_flux_adj(q, nv, g1, Gb, pa);
      // faces of this direction: the own trace's adjoint prolonged back onto this node
      const int fa = dir == 0 ? id3[1] : id3[0], fb = dir == 2 ? id3[1] : id3[2];
      const int ab = fa + n * fb;
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        const int s = 2 * dir + sd;
        double w;
        if (LGL) w = (id == (sd ? N : 0)) ? 1.0 : 0.0;
        else w = sl[(sd ? n : 0) + id];
        if (w == 0.0) continue;
#pragma unroll
        for (int v = 0; v < 5; ++v) ub[v] += w * sT[(s * 5 + v) * n2 + ab];
      }
    }
    dgf::cons_adj(q, gm1, pa, ub);
    double *Ube = Ub + (size_t)e * 5 * n3;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double r = scale * ub[v];
      Ube[v * n3 + t] = accumulate ? Ube[v * n3 + t] + r : r;
    }
  }
}

// ---------------------------------------------------------------------------------- launcher
template <int N>
int launch_vjp(const Geo &g, const Phys &ph, int eqn, int form, bool lgl, const double *U, const double *G, double *Pf,
               const double *Ubar_t, double *Ubar, double scale, int accumulate, double *Rb, double ra, double rb,
               hipStream_t st) {
  const bool gen = g.fc != nullptr;
  if (form == DG_FORM_WEAK) {
    if (eqn != DG_EULER) return DG_ERR_UNSUPPORTED;
    const dim3 grid(xcd_grid(g.K)), block(VSz<N>::NT);
    if (lgl && gen) hipLaunchKernelGGL((k_vjp_weak<N, true, true>), grid, block, 0, st, g, ph, U, Ubar_t, Ubar, scale, accumulate);
    else if (lgl) hipLaunchKernelGGL((k_vjp_weak<N, true, false>), grid, block, 0, st, g, ph, U, Ubar_t, Ubar, scale, accumulate);
    else if (gen) hipLaunchKernelGGL((k_vjp_weak<N, false, true>), grid, block, 0, st, g, ph, U, Ubar_t, Ubar, scale, accumulate);
    else hipLaunchKernelGGL((k_vjp_weak<N, false, false>), grid, block, 0, st, g, ph, U, Ubar_t, Ubar, scale, accumulate);
    return hipGetLastError() == hipSuccess ? DG_OK : DG_ERR_HIP;
  }
  if (form != DG_FORM_SPLIT) return DG_ERR_UNSUPPORTED;
  const dim3 grid(xcd_grid(g.K)), block(VSz<N>::NT), lines(SplitSz<N>::NT);
  const bool ns = eqn == DG_NAVIER_STOKES;
#define DG_VM(K_, B_, ...) \
  hipLaunchKernelGGL((K_<N, __VA_ARGS__>), grid, B_, 0, st, g, ph, U, G, Ubar_t, Ubar, Pf, scale, accumulate)
#define DG_VN(NS_) \
  do { \
    if (ph.vf != 0) { if (gen) DG_VM(k_vjp_main, block, NS_, true); else DG_VM(k_vjp_main, block, NS_, false); } \
    else if (g.Jc) { if (gen) DG_VM(k_vjp_line, lines, NS_, true, true); else DG_VM(k_vjp_line, lines, NS_, false, true); } \
    else { if (gen) DG_VM(k_vjp_line, lines, NS_, true, false); else DG_VM(k_vjp_line, lines, NS_, false, false); } \
  } while (0)
  if (ns) DG_VN(true); else DG_VN(false);
#undef DG_VN
#undef DG_VM
  if (hipGetLastError() != hipSuccess) return DG_ERR_HIP;
  if (ns) {
    if (gen)
      hipLaunchKernelGGL((k_vjp_face<N, true>), grid, block, 0, st, g, ph, U, Pf, Ubar, Rb, ra, rb, Rb ? 1 : 0);
    else
      hipLaunchKernelGGL((k_vjp_face<N, false>), grid, block, 0, st, g, ph, U, Pf, Ubar, Rb, ra, rb, Rb ? 1 : 0);
    if (hipGetLastError() != hipSuccess) return DG_ERR_HIP;
  }
  return DG_OK;
}

#ifdef DG_ONLY_N
template int launch_vjp<DG_ONLY_N>(const Geo &, const Phys &, int, int, bool, const double *, const double *, double *,
                                   const double *, double *, double, int, double *, double, double, hipStream_t);
#endif

}  // namespace dg
