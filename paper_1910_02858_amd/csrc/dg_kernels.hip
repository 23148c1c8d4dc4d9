// HIP kernels of the DGSEM operator for gfx950 (one workgroup per element).
//
// Paper map (Krais et al., FLEXI):
//   k_lift, k_lift_affine ... BR1 lifting of W = (u,v,w,T): Sec. 3.1, eq. discreteGradient, U* = mean of traces
//   k_split, k_line, k_main . volume integral (split flux differencing eq. semiDiscreteSplit / weak eq.
//               semiDiscrete and strong eq. semiDiscreteStrong / these for Navier-Stokes with mortars),
//               numerical surface flux (Riemann + BR1 viscous mean), surface integral, -1/J scaling, and
//               optionally the 2N-storage Runge-Kutta update of Sec. 4.4 fused into the epilogue.
//   k_reduce .. partial results for the time step (eqs. CFLCondition, DFLCondition), quadrature
//               integrals and the finiteness check, then one final pass.
//
// Layout: U[e][v][k][j][i] (i fastest), Ja[e][i*3+d][node], 1/J[e][node],
// outward normals fn[e][side][d][a + n*b].  Each workgroup stages its element's state in
// LDS; neighbour face values are read straight from global memory (for LGL nodes they are
// volume nodes of the neighbour's face layer; for LG nodes they are interpolated on the fly).
// Both elements sharing a face evaluate the same numerical flux with the master's normal and
// the master's state as the left argument, so the two contributions cancel to rounding.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dg_internal.h"
#include "dg_lines.h"

// waves per SIMD the split-form kernel is built for: 2 (256 registers: a line of 8 nodes holds 112
// doubles); at N = 8 one element's LDS fills the CU and one wave per SIMD is all there is.  Affine elements with
// the kinetic-energy preserving flux (vf 0) at N = 6, 7 need 176 registers: 168, three waves and four workgroups
// per CU instead of two, spill 44 and 60 bytes and still gain (32^3 elements: N = 7 7021 -> 6650 us a step, N = 6
// 5195 -> 4824).  Not below N = 6 (N = 5 6100 against 6090, N = 4 6940 -> 6975, N = 3 7950 -> 8900) and not for the
// entropy-conserving flux, which spills 356 bytes (N = 7 7715 -> 8795).
constexpr int split_minb(int N, int vf, bool affine) {
  return N >= 8 ? 1 : (affine && vf == 0 && N >= 6 ? 3 : 2);
}
// minimum waves per SIMD for the lifting kernel: 6 fits three 512-thread workgroups per CU
#ifndef DG_LIFT_MINB
#define DG_LIFT_MINB 6
#endif
// the lifting of meshes with non-conforming faces: at 80 registers it spills 44 bytes, at 128 (two
// workgroups per CU) none: 0.73 -> 0.65 ms at 16^3 N=7 half refined
#ifndef DG_LIFT_MORTAR_MINB
#define DG_LIFT_MORTAR_MINB 4
#endif

namespace dg {

template <int N> struct Sz {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  static constexpr int NT = ((n3 + 63) / 64) * 64;  // threads per workgroup (one node each)
};

// node of the line through face point (a,b) of direction dn at position m along dn
template <int n> __device__ __forceinline__ int line_node(int dn, int a, int b, int m) {
  return dn == 0 ? (m + n * (a + n * b)) : (dn == 1 ? (a + n * (m + n * b)) : (a + n * (b + n * m)));
}

// Symmetry-plane (slip-wall) boundary: the outer side is the mirror image of the inner one across
// the plane with unit normal nh.  mirror3 reflects a 3-vector; mirror_grad reflects gradients
// g[d*4+v] = dW_v/dx_d of W = (u, v, w, T) in the derivative direction and, for the velocity
// block, also in the component.
__device__ __forceinline__ void mirror3(double *x, const double *nh) {
  const double xn = 2.0 * (x[0] * nh[0] + x[1] * nh[1] + x[2] * nh[2]);
  x[0] -= xn * nh[0];
  x[1] -= xn * nh[1];
  x[2] -= xn * nh[2];
}
__device__ __forceinline__ void mirror_grad(double *g, const double *nh) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    double c[3] = {g[v], g[4 + v], g[8 + v]};
    mirror3(c, nh);
    g[v] = c[0]; g[4 + v] = c[1]; g[8 + v] = c[2];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) mirror3(g + 4 * d, nh);
}
// side s of element e belongs to a non-conforming face (its terms come from the mortar arrays)
__device__ __forceinline__ bool is_mortar(const Geo &g, int e, int s) {
  if (!g.fc) return false;
  const int c = g.fc[(size_t)e * 6 + s];
  return (c & 128) && (c & 7) == FACE_MORTAR;
}
__device__ __forceinline__ void unit3(const double *x, double *nh) {
  const double il = 1.0 / sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
  nh[0] = x[0] * il; nh[1] = x[1] * il; nh[2] = x[2] * il;
}

// ----------------------------------------------------------------------------- physics
// Reciprocal from v_rcp_f64 refined by two Newton steps (error well below one ulp of the
// quantities it feeds); used for the two-point fluxes, where IEEE division dominated.
__device__ __forceinline__ double frcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
struct Pr5 {
  double rho, u, v, w, p;
};

__device__ __forceinline__ Pr5 to_prim(const double *U, double gm1) {
  Pr5 P;
  P.rho = U[0];
  const double ir = frcp(U[0]);
  P.u = U[1] * ir; P.v = U[2] * ir; P.w = U[3] * ir;
  P.p = gm1 * (U[4] - 0.5 * (U[1] * P.u + U[2] * P.v + U[3] * P.w));
  return P;
}

// Euler flux along the (unnormalised) vector nv
__device__ __forceinline__ void flux_c(const double *U, const Pr5 &P, const double *nv, double *F) {
  const double un = P.u * nv[0] + P.v * nv[1] + P.w * nv[2];
  F[0] = U[0] * un;
  F[1] = U[1] * un + P.p * nv[0];
  F[2] = U[2] * un + P.p * nv[1];
  F[3] = U[3] * un + P.p * nv[2];
  F[4] = (U[4] + P.p) * un;
}

// viscous flux along nv; g[d*4+c] = dW_c/dx_d with W = (u, v, w, T)
__device__ __forceinline__ void flux_v(const Pr5 &P, const double *g, const Phys &ph, const double *nv, double *F) {
  const double mu = ph.mu;
  const double div = g[0] + g[5] + g[10];
  // tau[a][b] = mu (du_a/dx_b + du_b/dx_a) - 2/3 mu div delta_ab ; du_a/dx_b = g[b*4+a]
  const double t00 = mu * (2.0 * g[0] - (2.0 / 3.0) * div);
  const double t11 = mu * (2.0 * g[5] - (2.0 / 3.0) * div);
  const double t22 = mu * (2.0 * g[10] - (2.0 / 3.0) * div);
  const double t01 = mu * (g[4] + g[1]);
  const double t02 = mu * (g[8] + g[2]);
  const double t12 = mu * (g[9] + g[6]);
  F[0] = 0.0;
  F[1] = t00 * nv[0] + t01 * nv[1] + t02 * nv[2];
  F[2] = t01 * nv[0] + t11 * nv[1] + t12 * nv[2];
  F[3] = t02 * nv[0] + t12 * nv[1] + t22 * nv[2];
  // energy: (tau . u)_d + kappa dT/dx_d, contracted with nv
  F[4] = F[1] * P.u + F[2] * P.v + F[3] * P.w + ph.kappa * (g[3] * nv[0] + g[7] * nv[1] + g[11] * nv[2]);
}

__device__ __forceinline__ double logmean(double a, double b) {
  const double s = a + b;
  const double d = a - b;
  const double f = d / s;
  const double u = f * f;
  if (u < 1e-4) return s / (2.0 + u * (2.0 / 3.0 + u * (2.0 / 5.0 + u * (2.0 / 7.0))));
  // log(a) - log(b) as one logarithm, log1p of the difference over the smaller argument
  const double ad = fabs(d);
  return ad / log1p(ad / fmin(a, b));
}

// two-point flux along nv: vf 0 KEP (Pirozzoli), 1 EC (Chandrashekar), 2 central
__device__ __forceinline__ void flux_2pt(int vf, const double *Ua, const Pr5 &A, const double *Ub, const Pr5 &B,
                                         const double *nv, double gm1, double *F) {
  if (vf == 2) {
    double Fa[5], Fb[5];
    flux_c(Ua, A, nv, Fa);
    flux_c(Ub, B, nv, Fb);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = 0.5 * (Fa[v] + Fb[v]);
    return;
  }
  const double um = 0.5 * (A.u + B.u), vm = 0.5 * (A.v + B.v), wm = 0.5 * (A.w + B.w);
  const double umn = um * nv[0] + vm * nv[1] + wm * nv[2];
  if (vf == 0) {
    const double rhom = 0.5 * (A.rho + B.rho);
    const double pm = 0.5 * (A.p + B.p);
    const double Hm = 0.5 * ((Ua[4] + A.p) / A.rho + (Ub[4] + B.p) / B.rho);
    const double f0 = rhom * umn;
    F[0] = f0;
    F[1] = f0 * um + pm * nv[0];
    F[2] = f0 * vm + pm * nv[1];
    F[3] = f0 * wm + pm * nv[2];
    F[4] = f0 * Hm;
    return;
  }
  const double ba = 0.5 * A.rho / A.p, bb = 0.5 * B.rho / B.p;
  const double rholn = logmean(A.rho, B.rho);
  const double betaln = logmean(ba, bb);
  const double phat = 0.25 * (A.rho + B.rho) / (0.5 * (ba + bb));
  const double q2m = 0.5 * ((A.u * A.u + A.v * A.v + A.w * A.w) + (B.u * B.u + B.v * B.v + B.w * B.w));
  const double f0 = rholn * umn;
  F[0] = f0;
  F[1] = f0 * um + phat * nv[0];
  F[2] = f0 * vm + phat * nv[1];
  F[3] = f0 * wm + phat * nv[2];
  F[4] = f0 * (0.5 / (gm1 * betaln) - 0.5 * q2m) + um * F[1] + vm * F[2] + wm * F[3];
}

// Roe dissipation sum |lambda_k| alpha_k r_k, written without a rotated frame:
// shear waves act on the tangential velocity jump du - (du.n) n.
__device__ __forceinline__ void roe_diss(const double *UL, const Pr5 &L, const double *UR, const Pr5 &R,
                                         const double *nh, double gm1, double *D) {
  const double sL = sqrt(L.rho), sR = sqrt(R.rho);
  const double is = 1.0 / (sL + sR);
  const double u = (sL * L.u + sR * R.u) * is;
  const double v = (sL * L.v + sR * R.v) * is;
  const double w = (sL * L.w + sR * R.w) * is;
  const double HL = (UL[4] + L.p) / L.rho, HR = (UR[4] + R.p) / R.rho;
  const double H = (sL * HL + sR * HR) * is;
  const double q2 = u * u + v * v + w * w;
  const double c2 = gm1 * (H - 0.5 * q2);
  const double c = sqrt(c2);
  const double rt = sL * sR;
  const double un = u * nh[0] + v * nh[1] + w * nh[2];
  const double dr = R.rho - L.rho, dp = R.p - L.p;
  const double du = R.u - L.u, dv = R.v - L.v, dw = R.w - L.w;
  const double dun = du * nh[0] + dv * nh[1] + dw * nh[2];
  const double ic2 = 1.0 / c2;
  const double a1 = 0.5 * (dp - rt * c * dun) * ic2;
  const double a5 = 0.5 * (dp + rt * c * dun) * ic2;
  const double a2 = dr - dp * ic2;
  const double l1 = fabs(un - c), l2 = fabs(un), l5 = fabs(un + c);
  const double tu = du - dun * nh[0], tv = dv - dun * nh[1], tw = dw - dun * nh[2];
  const double s1 = l1 * a1, s5 = l5 * a5, s2 = l2 * a2, ss = l2 * rt;
  D[0] = s1 + s2 + s5;
  D[1] = s1 * (u - c * nh[0]) + s2 * u + ss * tu + s5 * (u + c * nh[0]);
  D[2] = s1 * (v - c * nh[1]) + s2 * v + ss * tv + s5 * (v + c * nh[1]);
  D[3] = s1 * (w - c * nh[2]) + s2 * w + ss * tw + s5 * (w + c * nh[2]);
  D[4] = s1 * (H - un * c) + s2 * 0.5 * q2 + ss * (u * tu + v * tv + w * tw) + s5 * (H + un * c);
}

// convective numerical flux f*(UL, UR, nh), nh a unit normal
__device__ __forceinline__ void riemann(const Phys &ph, const double *UL, const double *UR, const double *nh,
                                        double *F) {
  const double gm1 = ph.gamma - 1.0;
  const Pr5 L = to_prim(UL, gm1), R = to_prim(UR, gm1);
  if (ph.rs >= 2) {
    flux_2pt(ph.vf, UL, L, UR, R, nh, gm1, F);
    if (ph.rs == 3) {
      double D[5];
      roe_diss(UL, L, UR, R, nh, gm1, D);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] -= 0.5 * D[v];
    }
    return;
  }
  double FL[5], FR[5];
  flux_c(UL, L, nh, FL);
  flux_c(UR, R, nh, FR);
  if (ph.rs == 0) {
    const double cL = sqrt(ph.gamma * L.p / L.rho), cR = sqrt(ph.gamma * R.p / R.rho);
    const double unL = L.u * nh[0] + L.v * nh[1] + L.w * nh[2];
    const double unR = R.u * nh[0] + R.v * nh[1] + R.w * nh[2];
    const double lam = fmax(fabs(unL) + cL, fabs(unR) + cR);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * lam * (UR[v] - UL[v]);
    return;
  }
  double D[5];
  roe_diss(UL, L, UR, R, nh, gm1, D);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * D[v];
}

// riemann() with the solver fixed at compile time (RS = ph.rs)
template <int RS>
__device__ __forceinline__ void riemann_t(const Phys &ph, const double *UL, const double *UR, const double *nh,
                                          double *F) {
  const double gm1 = ph.gamma - 1.0;
  const Pr5 L = to_prim(UL, gm1), R = to_prim(UR, gm1);
  if (RS >= 2) {
    flux_2pt(ph.vf, UL, L, UR, R, nh, gm1, F);
    if (RS == 3) {
      double D[5];
      roe_diss(UL, L, UR, R, nh, gm1, D);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] -= 0.5 * D[v];
    }
    return;
  }
  double FL[5], FR[5];
  flux_c(UL, L, nh, FL);
  flux_c(UR, R, nh, FR);
  if (RS == 0) {
    const double cL = sqrt(ph.gamma * L.p / L.rho), cR = sqrt(ph.gamma * R.p / R.rho);
    const double unL = L.u * nh[0] + L.v * nh[1] + L.w * nh[2];
    const double unR = R.u * nh[0] + R.v * nh[1] + R.w * nh[2];
    const double lam = fmax(fabs(unL) + cL, fabs(unR) + cR);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * lam * (UR[v] - UL[v]);
    return;
  }
  double D[5];
  roe_diss(UL, L, UR, R, nh, gm1, D);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * D[v];
}

// numerical flux of the split-form kernel: as riemann(), with the two-point variants (rs 2, 3)
// evaluated by the volume flux VF of the kernel (pair2, defined below)
template <int VF>
__device__ __forceinline__ void riemann_vf(const Phys &ph, const double *UL, const double *UR, const double *nh,
                                           double *F);

__device__ __forceinline__ void grad_prim_to_W(const double *U, double gm1, double Rg, double *W) {
  const Pr5 P = to_prim(U, gm1);
  W[0] = P.u; W[1] = P.v; W[2] = P.w; W[3] = P.p / (P.rho * Rg);
}

// ----------------------------------------------------------------------------- lifting
// LDS sizes (doubles) of one element in the lifting kernel
template <int N> struct LiftLds {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  // the three regions together hold 12 values per node at the end (the staged viscous fluxes of
  // LIFT_DIV)
  static constexpr int W = 4 * n3, JA = 3 * n3, WS = (24 * n2 > 5 * n3) ? 24 * n2 : 5 * n3;
  static constexpr int AFFINE = 12 * n3;  // affine elements: no metric terms, no face means
};

// 1D tables of the lifting kernel into LDS (by the first threads of the workgroup)
template <int N>
__device__ __forceinline__ void lift_tables(const Tab *tb, int t, int nthreads, double *sDh, double *sl, double *slh) {
  constexpr int n = N + 1;
  for (int c = t; c < n * n; c += nthreads) sDh[c] = tb->Dh[c];
  if (t < n) {
    sl[t] = tb->lm[t]; sl[n + t] = tb->lp[t];
    slh[t] = tb->lhm[t]; slh[n + t] = tb->lhp[t];
  }
}

// BR1 lifting of element e by the NT threads t of one slot.  valid = false keeps the slot's
// threads in step with the workgroup barriers without touching memory.
// OUT: LIFT_G writes the gradients G[e][d*4+c][node] = dW_c/dx_d (weak and strong forms);
// LIFT_FV writes instead the momentum components c < 3 of the contravariant viscous fluxes
// Fv[e][dir*4+c][node] = (F^v . Ja^dir)_{1+c} (momentum, energy), which the reverse sweep reads (the energy's
// entries stay as they are); LIFT_DIV writes what
// the split-form operator reads, the strong-form divergence Geo::Gd (sums along the lines of D
// times Fv^dir, and the interior part of the surface term) and the face traces Geo::Gf of Fv;
// LIFT_DIVK writes both, all of Fv (the stage kept for a reverse sweep).  LIFT_GT (LG nodes) writes the
// gradients and every side's traces of them, interpolated with l(+-1) (Geo::Gtr), which the
// operator kernel reads at its faces instead of interpolating along the lines of its own and the
// neighbour's element.  On LG nodes the neighbours' traces of W come from k_prolong (Geo::Wtr).
// LIFT_WV (weak form, conforming meshes) writes what the weak-form operator reads: the volume
// term Geo::Gd (sums along the lines of D-hat times Fv^dir) and every side's viscous flux at its
// trace, F^v(U, grad W) . n with the side's own outward normal (Geo::Gf; on a boundary side
// already the BR1 mean with the outer state), and the gradients too when G is not NULL.
// LIFT_SV (strong form on LG nodes, conforming meshes) writes the face fluxes as LIFT_WV and as
// Geo::Gd the strong-form viscous term: sums along the lines of D times Fv^dir minus, for both
// faces of each line, lhat(+-1) times +- the interior viscous flux interpolated to the face (both
// in one contraction with Tab::Ds).
enum { LIFT_G = 0, LIFT_FV = 1, LIFT_DIV = 2, LIFT_DIVK = 3, LIFT_GT = 4, LIFT_WV = 5, LIFT_SV = 6 };

// The node's gradients acc[d*4+c] = dW_c/dx_d become its contravariant viscous fluxes
// acc[dir*4+c] = (F^v . Ja^dir)_{1+c} (momentum, energy): Newtonian stress with Stokes'
// hypothesis and Fourier heat flux, contracted with the metric terms jo[dir*3+d].  Every rounding
// step is spelled out (explicit fma, no contraction), so every kernel that runs the lifting
// produces the same fluxes bit for bit.
__device__ __forceinline__ void contra_visc(double *acc, const double *jo, double u, double v, double w,
                                            const Phys &ph) {
#pragma clang fp contract(off)
  const double mu = ph.mu, div = (acc[0] + acc[5]) + acc[10];
  const double t00 = mu * fma(-2.0 / 3.0, div, 2.0 * acc[0]);
  const double t11 = mu * fma(-2.0 / 3.0, div, 2.0 * acc[5]);
  const double t22 = mu * fma(-2.0 / 3.0, div, 2.0 * acc[10]);
  const double t01 = mu * (acc[4] + acc[1]);
  const double t02 = mu * (acc[8] + acc[2]);
  const double t12 = mu * (acc[9] + acc[6]);
  const double dT0 = acc[3], dT1 = acc[7], dT2 = acc[11];
#pragma unroll
  for (int dir = 0; dir < 3; ++dir) {
    const double *nv = jo + 3 * dir;
    acc[dir * 4] = fma(t02, nv[2], fma(t01, nv[1], t00 * nv[0]));
    acc[dir * 4 + 1] = fma(t12, nv[2], fma(t11, nv[1], t01 * nv[0]));
    acc[dir * 4 + 2] = fma(t22, nv[2], fma(t12, nv[1], t02 * nv[0]));
    const double q = fma(dT2, nv[2], fma(dT1, nv[1], dT0 * nv[0]));
    acc[dir * 4 + 3] = fma(ph.kappa, q, fma(acc[dir * 4 + 2], w, fma(acc[dir * 4 + 1], v, acc[dir * 4] * u)));
  }
}

// sm: the slot's LiftLds<N> regions, contiguous (W, JA, WS).
template <int N, bool LGL, int OUT, int GEN>
__device__ __forceinline__ void lift_body(const Geo &g, const Phys &ph, int e, bool valid, int t,
                                          const double *__restrict__ U, double *__restrict__ G,
                                          double *__restrict__ Fv, double *sm, const double *sDh,
                                          const double *sl, const double *slh) {
  using S = Sz<N>;
  using L = LiftLds<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = S::NT;
  constexpr bool FVO = OUT == LIFT_FV || OUT == LIFT_DIV || OUT == LIFT_DIVK;  // viscous fluxes formed
  double *sW = sm, *sJa = sm + L::W, *sWs = sm + L::W + L::JA;
  const double gm1 = ph.gamma - 1.0;
  const double *Ue = U + (size_t)e * 5 * n3;
  // the metric terms of the next direction (at most 3 per thread) and, in the last direction, the
  // node's 1/J are loaded one phase ahead
  constexpr int JPT = (3 * n3 + NT - 1) / NT;
  double jn[JPT], sjn = 0.0;
  const double *Jd0 = g.Ja + (size_t)e * 9 * n3;
#pragma unroll
  for (int r = 0; r < JPT; ++r) jn[r] = (valid && t + r * NT < 3 * n3) ? Jd0[t + r * NT] : 0.0;
  // on LGL nodes with one face point per thread, the neighbour's trace is loaded before the
  // first barrier
  constexpr bool PF = LGL && 6 * n2 <= NT;
  double Unp[5];
  if (PF && valid && t < 6 * n2) {
    const int s = t / n2, ab = t - s * n2, a = ab % n, b = ab / n;
    const int nb = g.nbr[(size_t)e * 6 + s];
    const NbFace f = nbr_face<n, (GEN > 0)>(g, e, s, a, b);
    const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(s >> 1, a, b, (s & 1) ? 0 : N);
    if (!(GEN && f.bnd)) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Unp[v] = U[((size_t)nb * 5 + v) * n3 + qn];
    }
  }
  if (valid && t < n3) {
    double Uq[5], W[4];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = Ue[v * n3 + t];
    grad_prim_to_W(Uq, gm1, ph.R, W);
#pragma unroll
    for (int v = 0; v < 4; ++v) sW[v * n3 + t] = W[v];
  }
  __syncthreads();
  // W* = mean of the two traces on every face point of the element
  for (int p = valid ? t : 6 * n2; p < 6 * n2; p += NT) {
    const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
    const bool plus = s & 1;
    const int nb = g.nbr[(size_t)e * 6 + s];
    const NbFace f = nbr_face<n, (GEN > 0)>(g, e, s, a, b);
    const double *Un = U + (size_t)(GEN && f.bnd ? e : nb) * 5 * n3;
    double WL[4], WR[4];
    if (LGL) {
      const int q = line_node<n>(dn, a, b, plus ? N : 0);
      const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(dn, a, b, plus ? 0 : N);
#pragma unroll
      for (int v = 0; v < 4; ++v) WL[v] = sW[v * n3 + q];
      if (!(GEN && f.bnd)) {
        double Uq[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) Uq[v] = PF ? Unp[v] : Un[v * n3 + qn];
        grad_prim_to_W(Uq, gm1, ph.R, WR);
      }
    } else {
      const double *lo = sl + (plus ? n : 0), *ln = GEN ? sl + (f.plus ? n : 0) : sl + (plus ? 0 : n);
#pragma unroll
      for (int v = 0; v < 4; ++v) { WL[v] = 0.0; WR[v] = 0.0; }
#pragma unroll 1
      for (int m = 0; m < n; ++m) {
        const int q = line_node<n>(dn, a, b, m);
#pragma unroll
        for (int v = 0; v < 4; ++v) WL[v] += lo[m] * sW[v * n3 + q];
      }
      if (!(GEN && f.bnd)) {
        // the neighbour's trace of W on its side of the face, from the prolongation kernel
        const double *wt = g.Wtr + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
#pragma unroll
        for (int v = 0; v < 4; ++v) WR[v] = wt[v * n2];
      }
    }
    if (GEN && f.bnd && f.kind == DG_BC_STATE) {
      // given outer state
      grad_prim_to_W(ph.ub, gm1, ph.R, WR);
    } else if (GEN && f.bnd && f.kind == DG_BC_WALL) {
      // no-slip wall: velocity reversed, temperature kept
#pragma unroll
      for (int v = 0; v < 3; ++v) WR[v] = -WL[v];
      WR[3] = WL[3];
    } else if (GEN && f.bnd && f.kind == DG_BC_WALL_ISOTHERMAL) {
      // isothermal wall: velocity reversed, mean temperature T_w
#pragma unroll
      for (int v = 0; v < 3; ++v) WR[v] = -WL[v];
      WR[3] = 2.0 * ph.tw - WL[3];
    } else if (GEN && f.bnd && f.kind == DG_BC_OUTFLOW) {
      // pressure outflow: the own trace's density and velocity with p_out (the conservative
      // trace: the face node on LGL nodes, interpolated with l(+-1) on LG nodes)
      double Uq[5];
      if (LGL) {
        const int q = line_node<n>(dn, a, b, plus ? N : 0);
#pragma unroll
        for (int v = 0; v < 5; ++v) Uq[v] = Ue[v * n3 + q];
      } else {
        const double *lo = sl + (plus ? n : 0);
#pragma unroll
        for (int v = 0; v < 5; ++v) Uq[v] = 0.0;
        for (int m = 0; m < n; ++m) {
          const int q = line_node<n>(dn, a, b, m);
#pragma unroll
          for (int v = 0; v < 5; ++v) Uq[v] += lo[m] * Ue[v * n3 + q];
        }
      }
      Uq[4] = ph.pout / gm1 + 0.5 * (Uq[1] * Uq[1] + Uq[2] * Uq[2] + Uq[3] * Uq[3]) / Uq[0];
      grad_prim_to_W(Uq, gm1, ph.R, WR);
    } else if (GEN == 2 && f.bnd && f.kind == FACE_MORTAR) {
      // non-conforming face: the surface term comes from the mortar face array
#pragma unroll
      for (int v = 0; v < 4; ++v) WR[v] = WL[v];
    } else if (GEN && f.bnd) {
      // symmetry plane: the outer W is the inner one with the velocity reflected
      const double *fnp = g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
      const double nt[3] = {fnp[0], fnp[n2], fnp[2 * n2]};
      double nh[3];
      unit3(nt, nh);
#pragma unroll
      for (int v = 0; v < 4; ++v) WR[v] = WL[v];
      mirror3(WR, nh);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) sWs[(s * 4 + v) * n2 + ab] = 0.5 * (WL[v] + WR[v]);
  }
  double acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = 0.0;
  const int i = t % n, j = (t / n) % n, k = t / n2;
  double jo[9];  // this node's metric terms, kept for the viscous fluxes
  double gd[4] = {0.0, 0.0, 0.0, 0.0};  // the viscous divergence (LIFT_DIV, LIFT_DIVK)
#pragma unroll
  for (int dir = 0; dir < 3; ++dir) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < JPT; ++r)
      if (valid && t + r * NT < 3 * n3) sJa[t + r * NT] = jn[r];
    if (dir < 2) {
      const double *Jd = g.Ja + ((size_t)e * 9 + (dir + 1) * 3) * n3;
#pragma unroll
      for (int r = 0; r < JPT; ++r) jn[r] = (valid && t + r * NT < 3 * n3) ? Jd[t + r * NT] : 0.0;
    }
    if (dir == 2 && valid && t < n3) sjn = g.sJ[(size_t)e * n3 + t];  // for the epilogue
    __syncthreads();
    if ((FVO || OUT == LIFT_WV || OUT == LIFT_SV) && valid && t < n3) {
#pragma unroll
      for (int d = 0; d < 3; ++d) jo[dir * 3 + d] = sJa[d * n3 + t];
    }
    if (valid && t < n3) {
      const int id = dir == 0 ? i : (dir == 1 ? j : k);
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
      // not unrolled: with all of a line's loads in flight the kernel exceeds its register budget
#pragma unroll 1
      for (int m = 0; m < n; ++m) {
        const int qm = base + m * str;
        const double Dh = sDh[id * n + m];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double c1 = Dh * sJa[d * n3 + qm];
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[d * 4 + v] += c1 * sW[v * n3 + qm];
        }
      }
      if (LGL && (id == 0 || id == N)) {
        // surface on the face of this direction through the node: on LGL nodes the outward
        // normal times s-hat is +-Ja^dir at the node itself
        const bool plus = id == N;
        const int s = 2 * dir + (plus ? 1 : 0);
        const double lh = slh[(plus ? n : 0) + id];
        const int a = dir == 0 ? j : i, b = dir == 2 ? j : k;
        const int ab = a + n * b;
        const double sl_ = plus ? lh : -lh;
        if (GEN == 2 && is_mortar(g, e, s)) {
          // non-conforming face: W* s n_d (outward) from the mortar face array
          const double *ml = g.mlift + (size_t)g.mslot[(size_t)e * 6 + s] * 12 * n2 + ab;
#pragma unroll
          for (int c = 0; c < 12; ++c) acc[c] += lh * ml[c * n2];
        } else {
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            const double c1 = sl_ * sJa[d * n3 + t];
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[d * 4 + v] += c1 * sWs[(s * 4 + v) * n2 + ab];
          }
        }
      }
    }
  }
  if (!LGL && valid && t < n3) {
    // surface: lhat(+-1) [W* nt_d] on each side
    for (int s = 0; s < 6; ++s) {
      const int dn = s >> 1;
      const bool plus = s & 1;
      const int id = dn == 0 ? i : (dn == 1 ? j : k);
      const double lh = slh[(plus ? n : 0) + id];
      if (LGL && lh == 0.0) continue;
      const int a = dn == 0 ? j : i, b = dn == 2 ? j : k;
      const int ab = a + n * b;
      if (GEN == 2 && is_mortar(g, e, s)) {
        const double *ml = g.mlift + (size_t)g.mslot[(size_t)e * 6 + s] * 12 * n2 + ab;
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] += lh * ml[c * n2];
        continue;
      }
      const double *nt = g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double c1 = lh * nt[d * n2];
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[d * 4 + v] += c1 * sWs[(s * 4 + v) * n2 + ab];
      }
    }
  }
  if (valid && t < n3) {
    const double sj = sjn;
    {
      // the gradients are rounded once, whatever is computed from them (so the three output
      // variants give the same bits)
#pragma clang fp contract(off)
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] *= sj;
    }
    if (GEN == 2 && LGL) {
      // face nodes of non-conforming sides keep their gradients for the mortar flux kernel
#pragma unroll
      for (int dir = 0; dir < 3; ++dir) {
        const int id = dir == 0 ? i : (dir == 1 ? j : k);
        if (id != 0 && id != N) continue;
        const int s = 2 * dir + (id == N ? 1 : 0);
        const int slot = g.mslot[(size_t)e * 6 + s];
        if (slot < 0) continue;
        const int ab = (dir == 0 ? j : i) + n * (dir == 2 ? j : k);
        double *mg = g.mg + (size_t)slot * 12 * n2 + ab;
#pragma unroll
        for (int c = 0; c < 12; ++c) mg[c * n2] = acc[c];
      }
    }
    if (OUT == LIFT_G || OUT == LIFT_GT || ((OUT == LIFT_WV || OUT == LIFT_SV || OUT == LIFT_DIV) && G)) {
      double *Ge = G + (size_t)e * 12 * n3;
#pragma unroll
      for (int c = 0; c < 12; ++c) Ge[c * n3 + t] = acc[c];
    }
    if (FVO) {
      contra_visc(acc, jo, sW[t], sW[n3 + t], sW[2 * n3 + t], ph);
      if (OUT == LIFT_FV || OUT == LIFT_DIVK) {
        double *Fe = Fv + (size_t)e * 12 * n3;
#pragma unroll
        for (int c = 0; c < 12; ++c)
          if (OUT == LIFT_DIVK || c % 4 != 3) Fe[c * n3 + t] = acc[c];
      }
      if (OUT == LIFT_DIV || OUT == LIFT_DIVK) {
        // the traces Fv^dir on the element's faces through this node, and their interior part
        // -+lhat(+-1) Fv^dir of the surface term
#pragma unroll
        for (int dir = 0; dir < 3; ++dir) {
          const int id = dir == 0 ? i : (dir == 1 ? j : k);
          if (id != 0 && id != N) continue;
          const bool plus = id == N;
          const int s = 2 * dir + (plus ? 1 : 0);
          const int ab = (dir == 0 ? j : i) + n * (dir == 2 ? j : k);
          double *gf = g.Gf + ((size_t)e * 6 + s) * 4 * n2 + ab;
          const double lh = slh[(plus ? n : 0) + id];
          const double sl_ = plus ? -lh : lh;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            gf[c * n2] = acc[dir * 4 + c];
            gd[c] = fma(sl_, acc[dir * 4 + c], gd[c]);
          }
        }
      }
    }
  }
  if constexpr (OUT == LIFT_WV || OUT == LIFT_SV) {
    // weak form (and strong form on LG nodes): every side's viscous flux at its trace (LG:
    // gradients interpolated from LDS, U from the prolongation; LGL: the face node's), with the
    // side's own outward normal; on a boundary side the BR1 mean with the outer state as the
    // operator would form it (this side is the master).  The node's contravariant fluxes for the
    // volume term below are formed first.
    double u = 0.0, v = 0.0, w = 0.0;
    if (valid && t < n3) { u = sW[t]; v = sW[n3 + t]; w = sW[2 * n3 + t]; }
    __syncthreads();
    if (valid && t < n3) {
      const int q = div_slot<n>(i, j, k);
#pragma unroll
      for (int c = 0; c < 12; ++c) sm[c * n3 + q] = acc[c];
      // the node's contravariant fluxes now: 12 values held across the face loop instead of the
      // gradients and the metric terms
      contra_visc(acc, jo, u, v, w, ph);
    }
    __syncthreads();
    for (int p = valid ? t : 6 * n2; p < 6 * n2; p += NT) {
      const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
      const bool plus = s & 1;
      double gq[12], Uq[5];
      if (LGL) {
        const int m = plus ? N : 0;
        const int q = dn == 0 ? div_slot<n>(m, a, b) : (dn == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
        for (int c = 0; c < 12; ++c) gq[c] = sm[c * n3 + q];
        const int qn = line_node<n>(dn, a, b, m);
#pragma unroll
        for (int c = 0; c < 5; ++c) Uq[c] = Ue[c * n3 + qn];
      } else {
        const double *lo = sl + (plus ? n : 0);
#pragma unroll
        for (int c = 0; c < 12; ++c) gq[c] = 0.0;
#pragma unroll 1
        for (int m = 0; m < n; ++m) {
          const int q = dn == 0 ? div_slot<n>(m, a, b) : (dn == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
          for (int c = 0; c < 12; ++c) gq[c] += lo[m] * sm[c * n3 + q];
        }
        const double *ut = g.Utr + ((size_t)e * 6 + s) * 5 * n2 + ab;
#pragma unroll
        for (int c = 0; c < 5; ++c) Uq[c] = ut[c * n2];
      }
      const double *fnp = g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
      const double nt[3] = {fnp[0], fnp[n2], fnp[2 * n2]};
      double Fo[5];
      flux_v(to_prim(Uq, gm1), gq, ph, nt, Fo);
      const NbFace f = nbr_face<n, (GEN > 0)>(g, e, s, a, b);
      if (GEN && f.bnd && f.kind != DG_BC_STATE && f.kind != DG_BC_OUTFLOW) {
        // walls and symmetry planes: the outer state and gradients; a given outer state or
        // outflow takes the outer viscous flux equal to the inner one (the mean is Fo itself)
        const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
        const double ish = 1.0 / sh;
        const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
        double Ux[5], gx[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) gx[c] = gq[c];
        if (f.kind == DG_BC_WALL_ISOTHERMAL || f.kind == DG_BC_WALL) {
          // no-slip wall: velocity reversed; at an adiabatic wall the temperature gradient mirrored
          Ux[0] = Uq[0]; Ux[1] = -Uq[1]; Ux[2] = -Uq[2]; Ux[3] = -Uq[3]; Ux[4] = Uq[4];
          if (f.kind == DG_BC_WALL) {
            double tg[3] = {gq[3], gq[7], gq[11]};
            mirror3(tg, nh);
            gx[3] = tg[0]; gx[7] = tg[1]; gx[11] = tg[2];
          }
        } else {
          // symmetry plane: mirror image of the inner state and gradients
#pragma unroll
          for (int c = 0; c < 5; ++c) Ux[c] = Uq[c];
          mirror3(Ux + 1, nh);
          mirror_grad(gx, nh);
        }
        double Fx[5];
        flux_v(to_prim(Ux, gm1), gx, ph, nt, Fx);
#pragma unroll
        for (int c = 1; c < 5; ++c) Fo[c] = 0.5 * (Fo[c] + Fx[c]);
      } else if (GEN && f.bnd) {
#pragma unroll
        for (int c = 1; c < 5; ++c) Fo[c] = 0.5 * (Fo[c] + Fo[c]);
      }
      double *pv = g.Gf + ((size_t)e * 6 + s) * 4 * n2 + ab;
#pragma unroll
      for (int c = 0; c < 4; ++c) pv[c * n2] = Fo[1 + c];
    }
  }
  if constexpr (OUT == LIFT_DIV || OUT == LIFT_DIVK || OUT == LIFT_WV || OUT == LIFT_SV) {
    // strong-form divergence of the viscous fluxes for the split-form operator:
    // Gd_c = sum_dir (sum_m D_{id,m} Fv^dir_c(m on the line) + [face node] -+lhat(+-1) Fv^dir_c),
    // the interior part of the surface term taken with the volume term; for the weak form
    // (LIFT_WV) Gd_c = sum_dir sum_m Dhat_{id,m} Fv^dir_c(m on the line), for the strong form on LG
    // nodes (LIFT_SV) the same with Tab::Ds.  The three regions are
    // free once every thread is past its last read of them.
    __syncthreads();
    if (valid && t < n3) {
      const int q = div_slot<n>(i, j, k);
#pragma unroll
      for (int c = 0; c < 12; ++c) sm[c * n3 + q] = acc[c];
    }
    __syncthreads();
    // one line, one direction and two components per task: the line's values are read once and
    // its n results written back in place (each LDS value is read once, not n times); the
    // matrix comes from the table through the scalar cache, the same for every lane
    // (LIFT_SV: Tab::Ds, the strong-form derivative with the interior fluxes interpolated to the
    // line's two faces and lifted back, -lhat(+1) l(+1) + lhat(-1) l(-1))
    const __attribute__((address_space(4))) double *Dg = (const __attribute__((address_space(4))) double *)(
        OUT == LIFT_WV ? g.tab->Dh : (OUT == LIFT_SV ? g.tab->Ds : g.tab->D));
    // TPD task slots per direction: 2 n^2 rounded up to whole waves where the three directions
    // then still fit the workgroup in one pass (n = 7: 98 -> 128, 384 lanes), so that every wave
    // works on one direction
    constexpr int TPW = (2 * n2 + 63) / 64 * 64;
    constexpr int TPD = (2 * n2) % 64 != 0 && 3 * TPW <= NT ? TPW : 2 * n2;
    for (int task = valid ? t : 3 * TPD; task < 3 * TPD; task += NT) {
      const int dir = TPD % 64 == 0 ? __builtin_amdgcn_readfirstlane(task / TPD) : task / TPD;
      const int r = task - dir * TPD, cp = r / n2, ln = r - cp * n2;
      if (TPD != 2 * n2 && r >= 2 * n2) continue;  // a padding slot
      const int a = ln % n, b = ln / n;
      double *s0 = sm + (dir * 4 + 2 * cp) * n3, *s1 = s0 + n3;
      double f0[n], f1[n];
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = dir == 0 ? div_slot<n>(m, a, b) : (dir == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
        f0[m] = s0[q];
        f1[m] = s1[q];
      }
#pragma unroll 2
      for (int id = 0; id < n; ++id) {
        double o0 = 0.0, o1 = 0.0;
#pragma unroll
        for (int m = 0; m < n; ++m) {
          const double D = Dg[id * n + m];
          o0 = fma(D, f0[m], o0);
          o1 = fma(D, f1[m], o1);
        }
        const int q = dir == 0 ? div_slot<n>(id, a, b) : (dir == 1 ? div_slot<n>(a, id, b) : div_slot<n>(a, b, id));
        s0[q] = o0;
        s1[q] = o1;
      }
    }
    __syncthreads();
    if (valid && t < n3) {
      const int q = div_slot<n>(i, j, k);
#pragma unroll
      for (int dir = 0; dir < 3; ++dir) {
#pragma unroll
        for (int c = 0; c < 4; ++c) gd[c] += sm[(dir * 4 + c) * n3 + q];
      }
      double *Gde = g.Gd + (size_t)e * 4 * n3 + t;
#pragma unroll
      for (int c = 0; c < 4; ++c) Gde[c * n3] = gd[c];
    }
  }
  if constexpr (OUT == LIFT_GT) {
    // LG face traces, each face point by one thread: the gradients (staged once the three
    // regions are free), then the conservative state, each summed along the face-normal line
    // with l(+-1) in the order the operator kernel would
    __syncthreads();
    if (valid && t < n3) {
      const int q = div_slot<n>(i, j, k);
#pragma unroll
      for (int c = 0; c < 12; ++c) sm[c * n3 + q] = acc[c];
    }
    __syncthreads();
    for (int p = valid ? t : 6 * n2; p < 6 * n2; p += NT) {
      const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
      const double *lo = sl + ((s & 1) ? n : 0);
      double gq[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) gq[c] = 0.0;
#pragma unroll 1
      for (int m = 0; m < n; ++m) {
        const int q = dn == 0 ? div_slot<n>(m, a, b) : (dn == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
        for (int c = 0; c < 12; ++c) gq[c] += lo[m] * sm[c * n3 + q];
      }
      double *gt = g.Gtr + ((size_t)e * 6 + s) * 12 * n2 + ab;
#pragma unroll
      for (int c = 0; c < 12; ++c) gt[c * n2] = gq[c];
    }
  }
}

// BR1 lifting of an affine element e by NT lanes, outputs as lift_body (dir-direction Fv along the element's
// constant Ja^dir).  The reference derivatives and the divergence are line tasks: a lane holds its line's four
// values of W in registers, forms the surface means at its two ends, and writes its n results to LDS, where
// every node collects its three directions' values.
// What bounds it: with one node per lane each value was read n times, 120 of the 190 LDS accesses of a node at
// N = 7; the LDS was busy 75 % of the time.  Here 40 of 60: weak form on LG nodes (N = 7, 16^3) 136 -> 87 us a launch,
// split form (N = 7, 32^3) 557 -> 505; a step of the 32-member ensemble 3115 -> 2933 us.
// Every rounding step is spelled out (explicit fma, no contraction): the same bits from every launch shape.
// sm: 12 values per node (slots: div_slot).  valid = false keeps the lanes in step with the barriers.
template <int N, bool LGL, int OUT, int GEN, int NT>
__device__ __forceinline__ void lift_affine(const Geo &g, const Phys &ph, const Tab *tab, int e, bool valid, int lane,
                                            const double *__restrict__ U, double *__restrict__ G,
                                            double *__restrict__ Fv, double *sm) {
#pragma clang fp contract(off)
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n, IT = (n3 + NT - 1) / NT;
  const double gm1 = ph.gamma - 1.0;
  const double *Ue = U + (size_t)e * 5 * n3;
  const AffineConst jc = affine_const(g, e);
  const Scalars tb(tab);
  const int dir = (n2 % 64 == 0 && NT % 64 == 0) ? __builtin_amdgcn_readfirstlane(lane / n2) : lane / n2;
  const int ab = lane - dir * n2, a = ab % n, b = ab / n;
  const bool act = valid && lane < 3 * n2;
  // loads: the neighbours' indices, the element's state, the traces beyond the line's two ends
  int nb2[2] = {0, 0};
  NbFace f2[2];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd)
    if (act) {
      nb2[sd] = g.nbr[(size_t)e * 6 + 2 * dir + sd];
      f2[sd] = nbr_face<n, (GEN > 0)>(g, e, 2 * dir + sd, a, b);
    }
  double Uq[IT][5];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Uq[it][v] = Ue[v * n3 + t];
    }
  }
  constexpr int NX = LGL ? 5 : 4;  // the other side's conservative state, on LG nodes its trace of W (k_prolong)
  double Ux[2][NX];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd)
    if (act && !(GEN && f2[sd].bnd)) {
      const NbFace f = f2[sd];
      const double *x;
      int st;
      if (LGL) {
        x = U + (size_t)nb2[sd] * 5 * n3 + (GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(dir, a, b, sd ? 0 : N));
        st = n3;
      } else {
        x = g.Wtr + ((size_t)nb2[sd] * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
        st = n2;
      }
#pragma unroll
      for (int v = 0; v < NX; ++v) Ux[sd][v] = x[v * st];
    }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
      double W[4];
      grad_prim_to_W(Uq[it], gm1, ph.R, W);
#pragma unroll
      for (int v = 0; v < 4; ++v) sm[v * n3 + q] = W[v];
    }
  }
  __syncthreads();
  const LineSlots<n> slot(act ? dir : 0, act ? a : 0, act ? b : 0);
  double f[4][n];      // W of the line's nodes; the velocities are kept for the viscous work
  double ws[2][4];     // surface means at its ends
  double nd[3] = {0.0, 0.0, 0.0};  // Ja^dir, +- the outward normal of the line's two faces times s-hat
  if (act) {
#pragma unroll
    for (int d = 0; d < 3; ++d) nd[d] = dir == 0 ? jc[d] : (dir == 1 ? jc[3 + d] : jc[6 + d]);
#pragma unroll
    for (int m = 0; m < n; ++m) {
      const int q = slot(m);
#pragma unroll
      for (int v = 0; v < 4; ++v) f[v][m] = sm[v * n3 + q];
    }
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      double WL[4], WR[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (LGL) {
          WL[v] = f[v][sd ? N : 0];
        } else {
          WL[v] = 0.0;
#pragma unroll
          for (int m = 0; m < n; ++m) WL[v] = fma(sd ? tb.lp[m] : tb.lm[m], f[v][m], WL[v]);
        }
        WR[v] = WL[v];
      }
      const bool bnd = GEN && f2[sd].bnd;
      const int kind = f2[sd].kind;
      if (!bnd) {
        if constexpr (LGL) {
          grad_prim_to_W(Ux[sd], gm1, ph.R, WR);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) WR[v] = Ux[sd][v];
        }
      } else if (kind == DG_BC_STATE) {
        grad_prim_to_W(ph.ub, gm1, ph.R, WR);  // given outer state
      } else if (kind == DG_BC_WALL || kind == DG_BC_WALL_ISOTHERMAL) {
        // no-slip wall: velocity reversed, temperature kept; isothermal: mean temperature T_w
#pragma unroll
        for (int v = 0; v < 3; ++v) WR[v] = -WL[v];
        if (kind == DG_BC_WALL_ISOTHERMAL) WR[3] = 2.0 * ph.tw - WL[3];
      } else if (kind == DG_BC_OUTFLOW) {
        // pressure outflow: the own trace's density and velocity with p_out (the conservative trace: the
        // face node on LGL nodes, interpolated with l(+-1) on LG nodes)
        double Ut[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        for (int m = LGL ? (sd ? N : 0) : 0; m < (LGL && !sd ? 1 : n); ++m) {
          const double l = LGL ? 1.0 : (sd ? tb.lp[m] : tb.lm[m]);
#pragma unroll
          for (int v = 0; v < 5; ++v) Ut[v] = fma(l, Ue[v * n3 + line_node<n>(dir, a, b, m)], Ut[v]);
        }
        Ut[4] = ph.pout / gm1 + 0.5 * (Ut[1] * Ut[1] + Ut[2] * Ut[2] + Ut[3] * Ut[3]) / Ut[0];
        grad_prim_to_W(Ut, gm1, ph.R, WR);
      } else if (kind != FACE_MORTAR) {
        // symmetry plane: the outer W is the inner one with the velocity reflected
        double nh[3];
        unit3(nd, nh);
        mirror3(WR, nh);
      }
      // a non-conforming face's surface term comes from the mortar face array (below)
#pragma unroll
      for (int v = 0; v < 4; ++v) ws[sd][v] = GEN == 2 && bnd && kind == FACE_MORTAR ? 0.0 : 0.5 * (WL[v] + WR[v]);
    }
  }
  __syncthreads();  // every line has read its values
  if (act) {
#pragma unroll
    for (int id = 0; id < n; ++id) {
      double o[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const double d = tb.Dh[id * n + m];
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = fma(d, f[v][m], o[v]);
      }
      // surface: +-lhat(+-1) W*
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (!LGL || id == 0) o[v] = fma(-tb.lhm[id], ws[0][v], o[v]);
        if (!LGL || id == N) o[v] = fma(tb.lhp[id], ws[1][v], o[v]);
      }
      const int q = slot(id);
#pragma unroll
      for (int v = 0; v < 4; ++v) sm[(dir * 4 + v) * n3 + q] = o[v];
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);  // one result at a time
    }
  }
  __syncthreads();
  // ---- node by node: gradients, then the contravariant viscous fluxes
  constexpr bool DIVO = OUT == LIFT_DIV || OUT == LIFT_DIVK || OUT == LIFT_WV || OUT == LIFT_SV;
#pragma unroll(IT <= 2 ? IT : 1)
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (!valid || t >= n3) continue;
    const int i = t % n, j = (t / n) % n, k = t / n2, q = div_slot<n>(i, j, k);
    double acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = 0.0;
#pragma unroll
    for (int dr = 0; dr < 3; ++dr) {
      if (GEN == 2) {
        // non-conforming faces: W* s n_d (outward) from the mortar face array
        const int id = dr == 0 ? i : (dr == 1 ? j : k), fab = (dr == 0 ? j : i) + n * (dr == 2 ? j : k);
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
          if (!is_mortar(g, e, 2 * dr + sd) || (LGL && id != (sd ? N : 0))) continue;
          const double lh = sd ? tab->lhp[id] : tab->lhm[id];
          const double *ml = g.mlift + (size_t)g.mslot[(size_t)e * 6 + 2 * dr + sd] * 12 * n2 + fab;
#pragma unroll
          for (int c = 0; c < 12; ++c) acc[c] = fma(lh, ml[c * n2], acc[c]);
        }
      }
      double dw[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) dw[v] = sm[(dr * 4 + v) * n3 + q];
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[d * 4 + v] = fma(jc[dr * 3 + d], dw[v], acc[d * 4 + v]);
    }
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] *= jc[9];
    if (GEN == 2 && LGL) {
      // face nodes of non-conforming sides keep their gradients for the mortar flux kernel
#pragma unroll
      for (int dr = 0; dr < 3; ++dr) {
        const int id = dr == 0 ? i : (dr == 1 ? j : k);
        if (id != 0 && id != N) continue;
        const int ms = g.mslot[(size_t)e * 6 + 2 * dr + (id == N ? 1 : 0)];
        if (ms < 0) continue;
        double *mg = g.mg + (size_t)ms * 12 * n2 + (dr == 0 ? j : i) + n * (dr == 2 ? j : k);
#pragma unroll
        for (int c = 0; c < 12; ++c) mg[c * n2] = acc[c];
      }
    }
    if (OUT == LIFT_G || OUT == LIFT_GT || ((OUT == LIFT_WV || OUT == LIFT_SV || OUT == LIFT_DIV) && G)) {
      double *Ge = G + (size_t)e * 12 * n3;
#pragma unroll
      for (int c = 0; c < 12; ++c) Ge[c * n3 + t] = acc[c];
    }
    if constexpr (OUT == LIFT_GT) {
#pragma unroll
      for (int c = 0; c < 12; ++c) sm[c * n3 + q] = acc[c];
    }
    if constexpr (DIVO || OUT == LIFT_FV) {
      const double div = acc[0] + acc[5] + acc[10];
      const double t00 = ph.mu * fma(-2.0 / 3.0, div, 2.0 * acc[0]);
      const double t11 = ph.mu * fma(-2.0 / 3.0, div, 2.0 * acc[5]);
      const double t22 = ph.mu * fma(-2.0 / 3.0, div, 2.0 * acc[10]);
      const double t01 = ph.mu * (acc[4] + acc[1]);
      const double t02 = ph.mu * (acc[8] + acc[2]);
      const double t12 = ph.mu * (acc[9] + acc[6]);
      double W[4];
      if (OUT == LIFT_DIVK) {
        double Un[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) Un[v] = Ue[v * n3 + t];
        grad_prim_to_W(Un, gm1, ph.R, W);
      }
#pragma unroll
      for (int dr = 0; dr < 3; ++dr) {
        const double n0 = jc[3 * dr], n1 = jc[3 * dr + 1], n2_ = jc[3 * dr + 2];
        // momentum fluxes and the temperature gradient along Ja^dr
        const double F0 = fma(t02, n2_, fma(t01, n1, t00 * n0));
        const double F1 = fma(t12, n2_, fma(t11, n1, t01 * n0));
        const double F2 = fma(t22, n2_, fma(t12, n1, t02 * n0));
        const double qn = fma(acc[11], n2_, fma(acc[7], n1, acc[3] * n0));
        if (OUT == LIFT_FV || OUT == LIFT_DIVK) {
          double *Fe = Fv + ((size_t)e * 12 + dr * 4) * n3 + t;
          Fe[0] = F0; Fe[n3] = F1; Fe[2 * n3] = F2;
          if (OUT == LIFT_DIVK) Fe[3 * n3] = fma(ph.kappa, qn, fma(F2, W[2], fma(F1, W[1], F0 * W[0])));
        }
        if constexpr (DIVO) {
          sm[(dr * 4) * n3 + q] = F0;
          sm[(dr * 4 + 1) * n3 + q] = F1;
          sm[(dr * 4 + 2) * n3 + q] = F2;
          sm[(dr * 4 + 3) * n3 + q] = qn;
        }
      }
    }
  }
  if constexpr (DIVO) {
    __syncthreads();
    if (act) {
      // the line's fluxes along its direction: momentum, energy
      double F[4][n];
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = slot(m);
#pragma unroll
        for (int c = 0; c < 4; ++c) F[c][m] = sm[(dir * 4 + c) * n3 + q];
      }
      if constexpr (OUT == LIFT_WV || OUT == LIFT_SV) {
        // every side's viscous flux at its trace along its own outward normal (both linear in the gradients:
        // interpolated after the contraction with the constant normal); on a boundary side the BR1 mean with
        // the outer state, in closed form
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
          double T[4] = {0.0, 0.0, 0.0, 0.0}, ut[3];
          if (LGL) {
#pragma unroll
            for (int c = 0; c < 4; ++c) T[c] = F[c][sd ? N : 0];
#pragma unroll
            for (int c = 0; c < 3; ++c) ut[c] = f[c][sd ? N : 0];
          } else {
#pragma unroll
            for (int m = 0; m < n; ++m)
#pragma unroll
              for (int c = 0; c < 4; ++c) T[c] = fma(sd ? tb.lp[m] : tb.lm[m], F[c][m], T[c]);
            const double *utr = g.Utr + ((size_t)e * 6 + 2 * dir + sd) * 5 * n2 + ab;
            const double ir = 1.0 / utr[0];
#pragma unroll
            for (int c = 0; c < 3; ++c) ut[c] = utr[(1 + c) * n2] * ir;
          }
          T[3] *= ph.kappa;
          const bool bnd = GEN && f2[sd].bnd && f2[sd].kind != DG_BC_STATE && f2[sd].kind != DG_BC_OUTFLOW;
          if (!bnd) {
            T[3] = fma(T[2], ut[2], fma(T[1], ut[1], fma(T[0], ut[0], T[3])));
          } else if (f2[sd].kind == DG_BC_WALL) {
            T[3] = 0.0;  // no-slip wall: reversed velocity and mirrored heat flux
          } else if (f2[sd].kind != DG_BC_WALL_ISOTHERMAL) {
            // symmetry plane: the normal part of the momentum flux (an isothermal wall keeps the heat flux)
            double nh[3];
            unit3(nd, nh);
            const double gm = T[0] * nh[0] + T[1] * nh[1] + T[2] * nh[2];
#pragma unroll
            for (int c = 0; c < 3; ++c) T[c] = gm * nh[c];
            T[3] = 0.0;
          }
          double *pv = g.Gf + ((size_t)e * 6 + 2 * dir + sd) * 4 * n2 + ab;
#pragma unroll
          for (int c = 0; c < 4; ++c) pv[c * n2] = sd ? T[c] : -T[c];
        }
      }
#pragma unroll
      for (int m = 0; m < n; ++m)
        F[3][m] = fma(ph.kappa, F[3][m], fma(F[2][m], f[2][m], fma(F[1][m], f[1][m], F[0][m] * f[0][m])));
      if constexpr (OUT == LIFT_DIV || OUT == LIFT_DIVK) {
        // the traces on the line's two faces
#pragma unroll
        for (int sd = 0; sd < 2; ++sd) {
          double *gf = g.Gf + ((size_t)e * 6 + 2 * dir + sd) * 4 * n2 + ab;
#pragma unroll
          for (int c = 0; c < 4; ++c) gf[c * n2] = F[c][sd ? N : 0];
        }
      }
      const Scalar M = OUT == LIFT_WV ? tb.Dh : (OUT == LIFT_SV ? tb.Ds : tb.D);
#pragma unroll
      for (int id = 0; id < n; ++id) {
        double o[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int m = 0; m < n; ++m) {
          double d = M[id * n + m];
          // the interior part of the surface term: -+lhat(+-1) Fv at the face nodes
          if ((OUT == LIFT_DIV || OUT == LIFT_DIVK) && m == id && id == 0) d += tb.lhm[0];
          if ((OUT == LIFT_DIV || OUT == LIFT_DIVK) && m == id && id == N) d -= tb.lhp[N];
#pragma unroll
          for (int c = 0; c < 4; ++c) o[c] = fma(d, F[c][m], o[c]);
        }
        const int q = slot(id);
#pragma unroll
        for (int c = 0; c < 4; ++c) sm[(dir * 4 + c) * n3 + q] = o[c];
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int t = lane + it * NT;
      if (!valid || t >= n3) continue;
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
      double *Gde = g.Gd + (size_t)e * 4 * n3 + t;
#pragma unroll
      for (int c = 0; c < 4; ++c) Gde[c * n3] = (sm[c * n3 + q] + sm[(4 + c) * n3 + q]) + sm[(8 + c) * n3 + q];
    }
  }
  if constexpr (OUT == LIFT_GT) {
    // the gradients' traces on the line's two faces
    __syncthreads();
    if (act) {
#pragma unroll 1
      for (int c = 0; c < 12; ++c) {
        double x0 = 0.0, x1 = 0.0;
#pragma unroll
        for (int m = 0; m < n; ++m) {
          const double v = sm[c * n3 + slot(m)];
          x0 = fma(tb.lm[m], v, x0);
          x1 = fma(tb.lp[m], v, x1);
        }
        double *gt = g.Gtr + (((size_t)e * 6 + 2 * dir) * 12 + c) * n2 + ab;
        gt[0] = x0;
        gt[12 * n2] = x1;
      }
    }
  }
}

// Prolongation on LG nodes (Navier-Stokes): every side's traces of the conservative state and of
// W = (u, v, w, T), each interpolated with l(+-1) along the face-normal lines of the element
// (Utr, Wtr of Geo), so that the lifting and operator kernels read their neighbours' traces
// contiguously instead of the neighbours' whole lines.
template <int N>
__global__ void __launch_bounds__(Sz<N>::NT) k_prolong(Geo g, Phys ph, const double *__restrict__ U) {
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n, NT = Sz<N>::NT;
  __shared__ double sm[9 * n3];
  __shared__ double sl[2 * n];
  const int t = threadIdx.x;
  if (t < n) { sl[t] = g.tab->lm[t]; sl[n + t] = g.tab->lp[t]; }
  const int e = xcd_element(blockIdx.x, g.K);
  if (e >= g.K) return;
  if (t < n3) {
    const double *Ue = U + (size_t)e * 5 * n3;
    const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
    double Uq[5], W[4];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Uq[v] = Ue[v * n3 + t];
      sm[v * n3 + q] = Uq[v];
    }
    grad_prim_to_W(Uq, ph.gamma - 1.0, ph.R, W);
#pragma unroll
    for (int v = 0; v < 4; ++v) sm[(5 + v) * n3 + q] = W[v];
  }
  __syncthreads();
  for (int p = t; p < 6 * n2; p += NT) {
    const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
    const double *lo = sl + ((s & 1) ? n : 0);
    double x[9];
#pragma unroll
    for (int v = 0; v < 9; ++v) x[v] = 0.0;
#pragma unroll 1
    for (int m = 0; m < n; ++m) {
      const int q = dn == 0 ? div_slot<n>(m, a, b) : (dn == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
      for (int v = 0; v < 9; ++v) x[v] += lo[m] * sm[v * n3 + q];
    }
    double *ut = g.Utr + ((size_t)e * 6 + s) * 5 * n2 + ab;
    double *wt = g.Wtr + ((size_t)e * 6 + s) * 4 * n2 + ab;
#pragma unroll
    for (int v = 0; v < 5; ++v) ut[v * n2] = x[v];
#pragma unroll
    for (int v = 0; v < 4; ++v) wt[v * n2] = x[5 + v];
  }
}

// waves per SIMD each lifting instantiation is built for (caps its registers)
template <bool LGL, int OUT, int GEN> constexpr int lift_minb() {
  if ((OUT == LIFT_WV || OUT == LIFT_SV) && GEN > 0) return 4;  // boundary code: 128 registers
  if (GEN == 2 && LGL) return DG_LIFT_MORTAR_MINB;
  return (LGL || GEN == 0) ? DG_LIFT_MINB : 2;
}

template <int N, bool LGL, int OUT, int GEN>
__global__ void __launch_bounds__(Sz<N>::NT, (lift_minb<LGL, OUT, GEN>()))
    k_lift(Geo g, Phys ph, const double *__restrict__ U, double *__restrict__ G, double *__restrict__ Fv) {
  using L = LiftLds<N>;
  constexpr int n = L::n;
  __shared__ double sm[L::W + L::JA + L::WS];
  __shared__ double sDh[n * n], sl[2 * n], slh[2 * n];
  lift_tables<N>(g.tab, threadIdx.x, Sz<N>::NT, sDh, sl, slh);
  const int e = xcd_element(blockIdx.x, g.K);
  if (e >= g.K) return;
  lift_body<N, LGL, OUT, GEN>(g, ph, e, true, threadIdx.x, U, G, Fv, sm, sDh, sl, slh);
}

// waves per SIMD the affine lifting is built for
template <int N> constexpr int lift_affine_minb() { return N <= 5 ? 4 : 3; }

template <int N, bool LGL, int OUT, int GEN>
__global__ void __launch_bounds__(SplitSz<N>::NT, lift_affine_minb<N>())
    k_lift_affine(Geo g, Phys ph, const double *__restrict__ U, double *__restrict__ G, double *__restrict__ Fv) {
  __shared__ double sm[LiftLds<N>::AFFINE];
  const int e = xcd_element(blockIdx.x, g.K);
  if (e >= g.K) return;
  lift_affine<N, LGL, OUT, GEN, SplitSz<N>::NT>(g, ph, g.tab, e, true, threadIdx.x, U, G, Fv, sm);
}

// ----------------------------------------------------------------------------- operator, weak/strong
// Weak- and strong-form operator (eqs. semiDiscrete, semiDiscreteStrong): k_line, and k_main for
// Navier-Stokes on meshes with non-conforming faces, whose lifting leaves the gradients.

// Navier-Stokes, non-conforming faces: one node per lane, face fluxes first, then per direction the node's
// contravariant flux into LDS and the contraction along its line.  FORM: 0 weak, 2 strong.
// mode 0: write U_t, 1: fused RK stage.  AFF: the metric terms are the element's constants (Geo::Jc).
template <int N, bool LGL, int FORM, bool AFF>
__global__ void __launch_bounds__(Sz<N>::NT)
    k_main(Geo g, Phys ph, const double *__restrict__ U, const double *__restrict__ G, double *__restrict__ out,
           double *__restrict__ R, double ca, double cb, double dt, int mode) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = S::NT;
  __shared__ double sU[5 * n3];
  __shared__ double sX[5 * n3];
  __shared__ double sF[6 * 5 * n2];
  __shared__ double sD[n * n], sl[2 * n], slh[2 * n];
  const int e = xcd_element(blockIdx.x, g.K);
  const int t = threadIdx.x;
  if (e >= g.K) return;
  AffineConst jc = nullptr;
  if constexpr (AFF) jc = affine_const(g, e);
  const double gm1 = ph.gamma - 1.0;
  const Tab *tb = g.tab;
  // strong form on LG nodes: the derivative matrix carries the interior flux's interpolation
  // to the line's two faces (Tab::Ds), so the surface terms add the numerical flux alone
  for (int c = t; c < n * n; c += NT) sD[c] = (FORM == 0) ? tb->Dh[c] : (LGL ? tb->D[c] : tb->Ds[c]);
  if (t < n) {
    sl[t] = tb->lm[t]; sl[n + t] = tb->lp[t];
    slh[t] = tb->lhm[t]; slh[n + t] = tb->lhp[t];
  }
  const double *Ue = U + (size_t)e * 5 * n3;
  const double *Ge = G + (size_t)e * 12 * n3;
  double Uo[5];
  if (t < n3) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Uo[v] = Ue[v * n3 + t];
      sU[v * n3 + t] = Uo[v];
    }
  }
  __syncthreads();
  // numerical surface flux on the six faces, stored outward for this element
  for (int p = t; p < 6 * n2; p += NT) {
    const int s = p / n2, ab = p - s * n2, a = ab % n, b = ab / n, dn = s >> 1;
    const bool plus = s & 1;
    const int nb = g.nbr[(size_t)e * 6 + s];
    const NbFace f = nbr_face<n, true>(g, e, s, a, b);
    const bool bnd = f.bnd;
    if (bnd && f.kind == FACE_MORTAR) {
      // non-conforming face: the outward flux from the mortar face array
      const double *mf = g.mflux + (size_t)g.mslot[(size_t)e * 6 + s] * 5 * n2 + ab;
#pragma unroll
      for (int v = 0; v < 5; ++v) sF[(s * 5 + v) * n2 + ab] = mf[v * n2];
      continue;
    }
    const double *Un = U + (size_t)(bnd ? e : nb) * 5 * n3;
    const double *Gn = G + (size_t)(bnd ? e : nb) * 12 * n3;
    double Uw[5], Ux[5], gw[12], gx[12];  // w: this element's trace, x: neighbour's trace
    if (LGL) {
      const int q = line_node<n>(dn, a, b, plus ? N : 0);
      const int qn = line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0);
#pragma unroll
      for (int v = 0; v < 5; ++v) { Uw[v] = sU[v * n3 + q]; Ux[v] = bnd ? 0.0 : Un[v * n3 + qn]; }
#pragma unroll
      for (int c = 0; c < 12; ++c) { gw[c] = Ge[c * n3 + q]; gx[c] = bnd ? 0.0 : Gn[c * n3 + qn]; }
    } else {
      // the lifting kernel has interpolated every side's traces of U and of the gradients; this side's
      // U trace from LDS, the rest read contiguously
      const double *lo = sl + (plus ? n : 0);
      const double *gt = g.Gtr + ((size_t)e * 6 + s) * 12 * n2 + ab;
      const size_t sn = (size_t)(bnd ? e : nb) * 6 + 2 * f.dn + (f.plus ? 1 : 0);
      const double *utn = g.Utr + sn * 5 * n2 + f.a + n * f.b;
      const double *gtn = g.Gtr + sn * 12 * n2 + f.a + n * f.b;
#pragma unroll
      for (int v = 0; v < 5; ++v) { Uw[v] = 0.0; Ux[v] = 0.0; }
#pragma unroll 1
      for (int m = 0; m < n; ++m) {
        const int q = line_node<n>(dn, a, b, m);
#pragma unroll
        for (int v = 0; v < 5; ++v) Uw[v] += lo[m] * sU[v * n3 + q];
      }
#pragma unroll
      for (int c = 0; c < 12; ++c) { gw[c] = gt[c * n2]; gx[c] = 0.0; }
      if (!bnd) {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[v] = utn[v * n2];
#pragma unroll
        for (int c = 0; c < 12; ++c) gx[c] = gtn[c * n2];
      }
    }
    // the master's normal and state go first (fn holds the outward normal, the master's
    // negated on the slave side)
    const double *fnp = AFF ? g.Jc + (size_t)e * AFFINE_DOUBLES + 10 + 3 * s : g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
    const int fst = AFF ? 1 : n2;
    const bool mst = f.master;
    const double sg = mst ? 1.0 : -1.0;
    const double nt[3] = {sg * fnp[0], sg * fnp[fst], sg * fnp[2 * fst]};
    const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    const double ish = 1.0 / sh;
    const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
    const bool given = bnd && (f.kind == DG_BC_STATE || f.kind == DG_BC_OUTFLOW);
    if (given) {
      // given outer state, or the pressure outflow's (inner density and velocity, p_out); the
      // outer viscous flux is taken equal to the inner one below
      if (f.kind == DG_BC_OUTFLOW) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Ux[v] = Uw[v];
        Ux[4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
      } else {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[v] = ph.ub[v];
      }
    } else if (bnd) {
#pragma unroll
      for (int c = 0; c < 12; ++c) gx[c] = gw[c];
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[v] = Uw[v];
      if (f.kind == DG_BC_WALL_ISOTHERMAL || f.kind == DG_BC_WALL) {
        // no-slip wall: velocity reversed, velocity gradient kept; the temperature gradient kept at an
        // isothermal wall, mirrored at an adiabatic one
        Ux[1] = -Uw[1]; Ux[2] = -Uw[2]; Ux[3] = -Uw[3];
        if (f.kind == DG_BC_WALL) {
          double tg[3] = {gw[3], gw[7], gw[11]};
          mirror3(tg, nh);
          gx[3] = tg[0]; gx[7] = tg[1]; gx[11] = tg[2];
        }
      } else {
        // symmetry plane: mirror image of the inner state and gradients
        mirror3(Ux + 1, nh);
        mirror_grad(gx, nh);
      }
    }
    const double *UM = mst ? Uw : Ux, *US = mst ? Ux : Uw;
    double F[5];
    riemann(ph, UM, US, nh, F);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] *= sh;
    const double *gM = mst ? gw : gx, *gS = mst ? gx : gw;
    double FvM[5], FvS[5];
    const Pr5 PM = to_prim(UM, gm1), PS = to_prim(US, gm1);
    flux_v(PM, gM, ph, nt, FvM);
    if (given) {
#pragma unroll
      for (int v = 0; v < 5; ++v) FvS[v] = FvM[v];
    } else {
      flux_v(PS, gS, ph, nt, FvS);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) sF[(s * 5 + v) * n2 + ab] = sg * (F[v] - 0.5 * (FvM[v] + FvS[v]));
  }
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int i = t % n, j = (t / n) % n, k = t / n2;
  Pr5 Po;
  double go[12];  // the node's lifted gradients, loaded after the face phase
  if (t < n3) {
    Po = to_prim(Uo, gm1);
#pragma unroll
    for (int c = 0; c < 12; ++c) go[c] = Ge[c * n3 + t];
  }
  for (int dir = 0; dir < 3; ++dir) {
    double Fint[5], nv[3];
    __syncthreads();
    if (t < n3) {
      if constexpr (AFF) {
        nv[0] = jc[3 * dir]; nv[1] = jc[3 * dir + 1]; nv[2] = jc[3 * dir + 2];
      } else {
        const double *Jd = g.Ja + ((size_t)e * 9 + dir * 3) * n3 + t;
        nv[0] = Jd[0]; nv[1] = Jd[n3]; nv[2] = Jd[2 * n3];
      }
      double Fc[5], Fv[5];
      flux_c(Uo, Po, nv, Fc);
      flux_v(Po, go, ph, nv, Fv);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        Fint[v] = Fc[v] - Fv[v];
        sX[v * n3 + t] = Fint[v];
      }
    }
    __syncthreads();
    if (t < n3) {
      const int id = dir == 0 ? i : (dir == 1 ? j : k);
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
#pragma unroll 4
      for (int m = 0; m < n; ++m) {
        const double Dm = sD[id * n + m];
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[v] += Dm * sX[v * n3 + base + m * str];
      }
      // surface integral of the two faces of this direction
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        const int s = 2 * dir + sd;
        const double lh = slh[(sd ? n : 0) + id];
        if (LGL && lh == 0.0) continue;
        const int a = dir == 0 ? j : i, b = dir == 2 ? j : k;
        const int ab = a + n * b;
        const double sg = sd ? 1.0 : -1.0;
        // strong form on LGL nodes: minus the face node's own interior flux (on LG nodes its
        // interpolation is part of Tab::Ds)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          double pen = sF[(s * 5 + v) * n2 + ab];
          if (FORM != 0 && LGL) pen -= sg * Fint[v];
          acc[v] += lh * pen;
        }
      }
    }
  }
  if (t < n3) {
    const double sj = AFF ? jc[9] : g.sJ[(size_t)e * n3 + t];
    double *Oe = out + (size_t)e * 5 * n3;
    double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double ut = -acc[v] * sj;
      if (mode == 0) {
        Oe[v * n3 + t] = ut;
      } else {
        // a = 0 (first stage) does not read R, so R may hold anything on entry
        const double r = (ca != 0.0 ? ca * Re[v * n3 + t] : 0.0) + dt * ut;
        Re[v * n3 + t] = r;
        Oe[v * n3 + t] = sU[v * n3 + t] + cb * r;  // the node's state from LDS: not held in registers
      }
    }
  }
}

// ----------------------------------------------------------------------------- split form, LGL
// one Newton step: for ratios that only enter through a correction of relative size < 1e-4
__device__ __forceinline__ double frcp1(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// per-node state of the two-point fluxes: rho, u, v, w, and
//   EC:  b = beta = rho/(2p), q = |u|^2
//   KEP, central: b = p, q = H = (E+p)/rho
struct PS {
  double r, u, v, w, b, q;
};

// Coefficients of f/artanh(f) = 1 + C1 u + C2 u^2 + C3 u^3 + O(u^4), u = f^2 (inverse of the
// series artanh(f)/f = 1 + u/3 + u^2/5 + u^3/7 + ...); the truncation error is below 3e-18
// relative for u < 1e-4.
#define DG_LM_C1 (-1.0 / 3.0)
#define DG_LM_C2 (-4.0 / 45.0)
#define DG_LM_C3 (-44.0 / 945.0)

// Twice the two-point flux of the pair (A, B) contracted with the mean metric, given the
// metric sum nS = Ja(A) + Ja(B) (eq. semiDiscreteSplit: the volume term is 2 D_ij F#(i,j)).
// VF 0: kinetic-energy preserving (Pirozzoli); 1: entropy conserving (Chandrashekar) with the
// logarithmic means f (a+b)/(2 artanh f), f = (a-b)/(a+b), by series for f^2 < 1e-4 and by
// logarithms otherwise; 2: mean of the two Euler fluxes.  kg = 1/(gamma-1).
// SER: both ratios are known to lie in the series' range (no logarithms compiled in).
template <int VF, bool SER = false>
__device__ __forceinline__ void pair2(const PS &A, const PS &B, const double *nS, double kg, double *F) {
  const double su = A.u + B.u, sv = A.v + B.v, sw = A.w + B.w;
  if (VF == 2) {
    const double una = A.u * nS[0] + A.v * nS[1] + A.w * nS[2];
    const double unb = B.u * nS[0] + B.v * nS[1] + B.w * nS[2];
    const double ma = 0.5 * A.r * una, mb = 0.5 * B.r * unb, ps = 0.5 * (A.b + B.b);
    F[0] = ma + mb;
    F[1] = fma(ma, A.u, fma(mb, B.u, ps * nS[0]));
    F[2] = fma(ma, A.v, fma(mb, B.v, ps * nS[1]));
    F[3] = fma(ma, A.w, fma(mb, B.w, ps * nS[2]));
    F[4] = fma(ma, A.q, mb * B.q);
    return;
  }
  const double un = su * nS[0] + sv * nS[1] + sw * nS[2];  // 4 {u}.{Ja}
  const double sr = A.r + B.r;
  double f0, pp, e4;
  if (VF == 0) {
    // {rho}{u.Ja}, {u} F_rho + {p}{Ja}, F_rho {H}
    f0 = 0.25 * sr * un;
    pp = 0.5 * (A.b + B.b);
    e4 = 0.5 * (A.q + B.q);
  } else {
    const double dr = A.r - B.r;
    const double fr = dr * frcp1(sr);
    const double ur = fr * fr;
    double rl;  // rho^ln / 2
    // beyond the series, log(a) - log(b) as one logarithm of the larger over the smaller
    // argument (the same bits from either end of the pair)
    if (SER || ur < 1e-4) {
      rl = 0.25 * sr * fma(ur, fma(ur, fma(ur, DG_LM_C3, DG_LM_C2), DG_LM_C1), 1.0);
    } else {
      rl = 0.5 * fabs(dr) / log(fmax(A.r, B.r) * frcp(fmin(A.r, B.r)));
    }
    const double sb = A.b + B.b, db = A.b - B.b;
    const double rb = frcp(sb);
    const double fb = db * rb, ub = fb * fb;
    double eb;  // 1 / (2 (gamma-1) beta^ln)
    if (SER || ub < 1e-4) {
      eb = kg * rb * fma(ub, fma(ub, fma(ub, 1.0 / 7.0, 1.0 / 5.0), 1.0 / 3.0), 1.0);
    } else {
      eb = 0.5 * kg * log(fmax(A.b, B.b) * frcp(fmin(A.b, B.b))) / fabs(db);
    }
    f0 = rl * un;                // 2 rho^ln {u}.{Ja}
    pp = 0.5 * sr * rb;          // {rho} / (2 {beta})
    e4 = eb - 0.25 * (A.q + B.q);
  }
  const double hg = 0.5 * f0;
  F[0] = f0;
  F[1] = fma(hg, su, pp * nS[0]);
  F[2] = fma(hg, sv, pp * nS[1]);
  F[3] = fma(hg, sw, pp * nS[2]);
  if (VF == 0)
    F[4] = f0 * e4;
  else
    F[4] = fma(0.5, su * F[1] + sv * F[2] + sw * F[3], f0 * e4);
}

// partner state from the LDS copy (rho, u, v, w, beta|H); the sixth field is derived:
// |u|^2 for EC, p = ((gamma-1)/gamma) rho (H - |u|^2/2) for KEP and central (gg = (gamma-1)/gamma)
template <int VF>
__device__ __forceinline__ PS load_ps(const double *sS, int n3, int q, double gg) {
  PS s;
  s.r = sS[q]; s.u = sS[n3 + q]; s.v = sS[2 * n3 + q]; s.w = sS[3 * n3 + q];
  const double q2 = s.u * s.u + s.v * s.v + s.w * s.w;
  if (VF == 1) {
    s.b = sS[4 * n3 + q];
    s.q = q2;
  } else {
    s.q = sS[4 * n3 + q];
    s.b = gg * s.r * (s.q - 0.5 * q2);
  }
  return s;
}

template <int VF>
__device__ __forceinline__ void riemann_vf(const Phys &ph, const double *UL, const double *UR, const double *nh,
                                           double *F) {
  if (ph.rs < 2) {
    riemann(ph, UL, UR, nh, F);
    return;
  }
  const double gm1 = ph.gamma - 1.0;
  const Pr5 L = to_prim(UL, gm1), R = to_prim(UR, gm1);
  PS a, b;
  a.r = L.rho; a.u = L.u; a.v = L.v; a.w = L.w;
  b.r = R.rho; b.u = R.u; b.v = R.v; b.w = R.w;
  if (VF == 1) {
    a.b = 0.5 * L.rho / L.p; a.q = L.u * L.u + L.v * L.v + L.w * L.w;
    b.b = 0.5 * R.rho / R.p; b.q = R.u * R.u + R.v * R.v + R.w * R.w;
  } else {
    a.b = L.p; a.q = (UL[4] + L.p) / L.rho;
    b.b = R.p; b.q = (UR[4] + R.p) / R.rho;
  }
  // pair2 along the metric sum nh + nh returns twice the flux along nh
  const double n2[3] = {2.0 * nh[0], 2.0 * nh[1], 2.0 * nh[2]};
  pair2<VF>(a, b, n2, 1.0 / gm1, F);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] *= 0.5;
  if (ph.rs == 3) {
    double D[5];
    roe_diss(UL, L, UR, R, nh, gm1, D);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] -= 0.5 * D[v];
  }
}

// LDS sizes (doubles) of one element in the split-form kernel: the conservative state (5 per node), the
// two-point state rho, u, v, w, beta|H (5 per node) and the metric terms Ja^i_d (9 per node; none on
// affine elements); the accumulated result takes the place of the metric terms (affine: of the two-point
// state) once every line has read them.
// ENDS: whether the far ends' lanes also take the sums of their half of the line.  Pairs across the middle are then
// evaluated twice (44 instead of 28 at N = 7, 22 by each lane), which pays for the short fluxes; with the logarithmic
// means (VF 1) it does not (64 elements, curved: N = 7 125.7 us a step against 123.7, N = 8 161.7 against 154.9).  Where
// both halves lie in one wave it cannot.
template <int N, int VF> constexpr bool split_halves() { return EndsSz<N>::HALF % 64 == 0 && VF != 1; }

template <int N> struct SplitLds {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  static constexpr int A = 19 * n3, AFFINE = 10 * n3;
  template <bool AFF, bool ENDS> static constexpr int nodes() { return line_apart<N, ENDS>() ? 20 * n3 : (AFF ? AFFINE : A); }
  // ENDS without split sums: and the far ends' fluxes
  template <int VF, bool AFF, bool ENDS> static constexpr int size() {
    return nodes<AFF, ENDS>() + (ENDS && !split_halves<N, VF>() ? 15 * n2 : 0);
  }
};

struct LineNode {  // a node of a line: its two-point state and the line direction's metric terms
  PS s;
  double nv[3];
};

// Split-form operator on LGL nodes (eq. semiDiscreteSplit) for element e by the NT lanes of one slot.
// A lane owns one line: it holds the line's n states and metric terms in registers, evaluates each
// unordered pair of its nodes once and adds the pair to both nodes' sums in registers, and evaluates the
// numerical fluxes of the two faces at the line's ends.  The three directions' sums meet in LDS in a
// fixed order.
// What bounds it: with one node per lane and the partner's share of each pair passed through LDS the
// kernel issued 1686 vector instructions per node (VALU busy 71 %) and 20 LDS accesses per pair; a line
// per lane has no exchange, no redundant half round (28 pairs for 8 nodes, not 32) and five barriers per
// element, at 2 waves per SIMD.
// valid = false keeps the slot's lanes in step with the workgroup barriers without touching memory.
// AFF: every element is affine, its metric terms and 1/J are the element's constants (Geo::Jc): 10 of the
// 43 doubles per node are not read, and of the 41 KB of LDS at N = 7 instead of 78 four workgroups fit a CU; by
// registers two do with the EC and central fluxes, four with the KEP flux (split_minb).
// mode 0 writes U_t, 1 the fused RK stage.  FVM: the sides that meet a finite-volume element take their
// flux from Geo::fvFx.
template <int N, bool NS, int VF, int GEN, bool FVM, bool AFF>
__device__ __forceinline__ void split_body(const Geo &g, const Phys &ph, const Tab *tab, int e, bool valid, int lane,
                                           const double *__restrict__ U, double *__restrict__ out,
                                           double *__restrict__ R, double ca, double cb, double dt, int mode,
                                           double *sm) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = SplitSz<N>::NT;
  constexpr int IT = (n3 + NT - 1) / NT;  // nodes per lane in the node loops
  const double gm1 = ph.gamma - 1.0, kg = 1.0 / gm1, gg = gm1 / ph.gamma;
  const double *Ue = U + (size_t)e * 5 * n3;
  const double *Jae = g.Ja + (size_t)e * 9 * n3;
  double *sU = sm, *sS = sm + 5 * n3, *sJ = sm + 10 * n3;  // node slots: div_slot
  double *sAcc = AFF ? sS : sJ;
  AffineConst jc = nullptr;
  if constexpr (AFF) jc = affine_const(g, e);
  // the 1D tables through the scalar cache
  const __attribute__((address_space(4))) double *D = (const __attribute__((address_space(4))) double *)tab->D;
  const double lh0 = tab->lhm[0], lhN = tab->lhp[N];
  // this lane's line: direction, and its position (a, b) among the direction's lines, which is also the
  // face point of its two ends
  const int dir = n2 % 64 == 0 ? __builtin_amdgcn_readfirstlane(lane / n2) : lane / n2;
  const int ab = lane - dir * n2, a = ab % n, b = ab / n;
  const bool act = valid && lane < 3 * n2;
  // the two end faces' neighbours first (loads return in order: behind the others, the neighbours' traces
  // would wait for all of them), then the state and metric terms for LDS and the faces' other sides
  int nb2[2] = {0, 0};
  NbFace f2[2];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd)
    if (act) {
      nb2[sd] = g.nbr[(size_t)e * 6 + 2 * dir + sd];
      f2[sd] = nbr_face<n, (GEN > 0)>(g, e, 2 * dir + sd, a, b);
    }
  double Uq[IT][5];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Uq[it][v] = Ue[v * n3 + t];
    }
  }
  double Jq[IT][9];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (!AFF && valid && t < n3) {
#pragma unroll
      for (int c = 0; c < 9; ++c) Jq[it][c] = Jae[c * n3 + t];
    }
  }
  double Ux[2][5], Vo[2][4], Vn[2][4];  // the end faces: the other side's state, both sides' viscous fluxes
  int kind[2];                // -1 inner face, else the boundary kind; -2 a face whose flux is given (Ux)
#pragma unroll
  for (int sd = 0; sd < 2; ++sd) {
    kind[sd] = -1;
    if (!act) continue;
    const int s = 2 * dir + sd;
    const bool plus = sd;
    const int nb = nb2[sd];
    const NbFace f = f2[sd];
    const bool bnd = GEN && f.bnd;
    if (GEN == 2 && bnd && f.kind == FACE_MORTAR) {
      // non-conforming face: the outward flux from the mortar face array
      const double *mf = g.mflux + (size_t)g.mslot[(size_t)e * 6 + s] * 5 * n2 + ab;
      kind[sd] = -2;
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[sd][v] = mf[v * n2];
      continue;
    }
    if (FVM && g.fvflag[nb]) {
      // face shared with a finite-volume element: the outward flux at the face nodes
      const double *fx = g.fvFx + ((size_t)e * 6 + s) * 5 * n2 + ab;
      kind[sd] = -2;
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[sd][v] = fx[v * n2];
      continue;
    }
    if (bnd) kind[sd] = f.kind;
    if (!bnd) {
      const double *Un = U + (size_t)nb * 5 * n3;
      const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(dir, a, b, plus ? 0 : N);
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[sd][v] = Un[v * n3 + qn];
    }
    if (NS) {
      // both sides' contravariant viscous flux of the face's direction from the lifting (a boundary side:
      // the own trace); only loaded here, so that both faces' loads are in flight at once
      const double *fo = g.Gf + ((size_t)e * 6 + s) * 4 * n2 + ab;
      const double *fnb = bnd ? fo : g.Gf + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
#pragma unroll
      for (int c = 0; c < 4; ++c) { Vo[sd][c] = fo[c * n2]; Vn[sd][c] = fnb[c * n2]; }
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
      const Pr5 P = to_prim(Uq[it], gm1);
#pragma unroll
      for (int v = 0; v < 5; ++v) sU[v * n3 + q] = Uq[it][v];
      sS[q] = P.rho; sS[n3 + q] = P.u; sS[2 * n3 + q] = P.v; sS[3 * n3 + q] = P.w;
      // beta = rho / (2 p) for EC, the total enthalpy otherwise
      sS[4 * n3 + q] = (VF == 1) ? 0.5 * P.rho / P.p : (Uq[it][4] + P.p) / P.rho;
#pragma unroll
      for (int c = 0; c < 9 && !AFF; ++c) sJ[c * n3 + q] = Jq[it][c];
    }
  }
  __syncthreads();
  double acc[n][5];
  if (act) {
    const LineSlots<n> slot(dir, a, b);
    // the line direction's metric terms at a node
    const double *sJd = sJ + 3 * dir * n3;
    double jl[3] = {0.0, 0.0, 0.0};
    if constexpr (AFF) {
#pragma unroll
      for (int d = 0; d < 3; ++d) jl[d] = dir == 0 ? jc[d] : (dir == 1 ? jc[3 + d] : jc[6 + d]);
    }
    auto metric = [&](int d, int q) -> double {
      if constexpr (AFF) return jl[d];
      else return sJd[d * n3 + q];
    };
    // numerical surface fluxes at the line's ends, lifted (outward times lhat), and the interior
    // convective part: 2 D_ii F(U_i) (D_ii is non-zero only at the ends of LGL lines) -+ lhat F_int
    double fe[2][5];
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      const bool plus = sd;
      const int qo = slot(plus ? N : 0);
      const double sg = plus ? 1.0 : -1.0, lh = plus ? lhN : lh0;
      double Uw[5], Fo[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) Uw[v] = sU[v * n3 + qo];
      // normal along +xi scaled by s-hat: Ja^dir at the face node, the master's on the master side and
      // (up to rounding, the metric terms being continuous across the face) on the slave
      const double nt[3] = {metric(0, qo), metric(1, qo), metric(2, qo)};
      const Pr5 Pw = {Uw[0], sS[n3 + qo], sS[2 * n3 + qo], sS[3 * n3 + qo],
                      gm1 * (Uw[4] - 0.5 * (Uw[1] * sS[n3 + qo] + Uw[2] * sS[2 * n3 + qo] + Uw[3] * sS[3 * n3 + qo]))};
      flux_c(Uw, Pw, nt, Fo);
      const double cd = 2.0 * D[plus ? N * n + N : 0] - sg * lh;
      double F[5];
      if ((GEN == 2 || FVM) && kind[sd] == -2) {
#pragma unroll
        for (int v = 0; v < 5; ++v) F[v] = sg * Ux[sd][v];
      } else {
        const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
        const double ish = 1.0 / sh;
        const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
        const bool bnd = GEN && kind[sd] >= 0;
        const bool outflow = bnd && kind[sd] == DG_BC_OUTFLOW;
        const bool given = bnd && (kind[sd] == DG_BC_STATE || outflow);
        const bool iso = bnd && kind[sd] == DG_BC_WALL_ISOTHERMAL;
        const bool wall = bnd && (kind[sd] == DG_BC_WALL || iso);
        if (bnd) {
#pragma unroll
          for (int v = 0; v < 5; ++v) Ux[sd][v] = Uw[v];
          if (outflow) {
            // pressure outflow: the own trace's density and velocity with p_out
            Ux[sd][4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
          } else if (given) {
#pragma unroll
            for (int v = 0; v < 5; ++v) Ux[sd][v] = ph.ub[v];  // given outer state
          } else if (wall) {
            Ux[sd][1] = -Uw[1]; Ux[sd][2] = -Uw[2]; Ux[sd][3] = -Uw[3];  // no-slip wall: velocity reversed
          } else {
            mirror3(Ux[sd] + 1, nh);  // symmetry plane: mirror image of the inner state
          }
        }
        riemann_vf<VF>(ph, plus ? Uw : Ux[sd], plus ? Ux[sd] : Uw, nh, F);
#pragma unroll
        for (int v = 0; v < 5; ++v) F[v] *= sh;
        if (NS) {
          // BR1 mean of the viscous fluxes along this side's +xi normal Ja^dir (the normal metric of a
          // conforming face is continuous: the neighbour's Ja of its face direction is +-Ja^dir, + where
          // one side is a +xi side and the other a -xi side)
          double V[4];
          const double sn = (GEN && f2[sd].plus == plus) ? -1.0 : 1.0;
#pragma unroll
          for (int c = 0; c < 4; ++c) V[c] = bnd ? Vo[sd][c] : 0.5 * (Vo[sd][c] + sn * Vn[sd][c]);
          if (!bnd || given) {
            // given outer state: the outer viscous flux equals the inner one
#pragma unroll
            for (int c = 0; c < 4; ++c) F[1 + c] -= V[c];
          } else if (wall) {
            // no-slip wall: the outer momentum flux equals the inner one, the outer energy flux is its
            // negative (reversed velocity, mirrored heat flux), so the mean keeps the momentum; at an
            // isothermal wall the outer gradient is the inner one, so the mean energy flux is the inner
            // heat flux: the inner energy flux minus the work (tau Ja^dir) . u
#pragma unroll
            for (int c = 0; c < 3; ++c) F[1 + c] -= V[c];
            if (iso) F[4] -= V[3] - (V[0] * Uw[1] + V[1] * Uw[2] + V[2] * Uw[3]) * (1.0 / Uw[0]);
          } else {
            // symmetry plane: the mirrored outer flux cancels the inner shear and heat flux, the mean
            // keeps the normal part of the momentum flux
            const double gm = V[0] * nh[0] + V[1] * nh[1] + V[2] * nh[2];
#pragma unroll
            for (int c = 0; c < 3; ++c) F[1 + c] -= gm * nh[c];
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) fe[sd][v] = fma(cd, Fo[v], (sg * lh) * F[v]);
    }
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[m][v] = m == 0 ? fe[0][v] : (m == N ? fe[1][v] : 0.0);
    // EC: where every pair of every line of this wave lies in the series' range (the largest ratio of a
    // line is that of its largest and smallest value) the unrolled loop below needs no logarithm
    bool series = true;
    if constexpr (VF == 1) {
      double r0 = sS[slot(0)], r1 = r0, b0 = sS[4 * n3 + slot(0)], b1 = b0;
#pragma unroll
      for (int m = 1; m < n; ++m) {
        const double r = sS[slot(m)], bt = sS[4 * n3 + slot(m)];
        r0 = fmin(r0, r); r1 = fmax(r1, r);
        b0 = fmin(b0, bt); b1 = fmax(b1, bt);
      }
      const double dr = r1 - r0, sr = r1 + r0, db = b1 - b0, sb = b1 + b0;
      series = dr * dr < 0.99e-4 * (sr * sr) && db * db < 0.99e-4 * (sb * sb);
      series = __all(series);
    }
    if (VF != 1 || series) {
      // node i in registers, its partners read from LDS one pair ahead of their use (a whole line in
      // registers spills 500 bytes at n = 8); the first partner is the next row's node
      auto node = [&](int m) -> LineNode {
        LineNode x;
        const int q = slot(m);
        x.s = load_ps<VF>(sS, n3, q, gg);
#pragma unroll
        for (int d = 0; d < 3; ++d) x.nv[d] = metric(d, q);
        return x;
      };
      LineNode A = node(0), B = node(1), An = B, Bn = B;
#pragma unroll
      for (int i = 0; i + 1 < n; ++i) {
#pragma unroll
        for (int j = i + 1; j < n; ++j) {
          if (j == i + 1) An = B;
          if (j + 1 < n) Bn = node(j + 1);
          else if (i + 2 < n) Bn = node(i + 2);
          const double nS[3] = {A.nv[0] + B.nv[0], A.nv[1] + B.nv[1], A.nv[2] + B.nv[2]};
          double F[5];
          pair2<VF, true>(A.s, B.s, nS, kg, F);
          const double Dij = D[i * n + j], Dji = D[j * n + i];
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            acc[i][v] = fma(Dij, F[v], acc[i][v]);
            acc[j][v] = fma(Dji, F[v], acc[j][v]);
          }
          B = Bn;
          // at most two pairs in flight: more spill (n <= 6 fits as scheduled)
          if (n > 6 && (j - i) % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        }
        A = An;
        asm volatile("" ::: "memory");  // the next row's partners are read again, not kept
      }
    } else {
      // the same pairs (i, i + s mod n) with logarithms, the states read from LDS as they are met; a
      // rolled loop over i whose sums move down one place per turn, so that node i's is always the first
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        const int qi = slot(i);
        const PS A = load_ps<VF>(sS, n3, qi, gg);
        const double na[3] = {metric(0, qi), metric(1, qi), metric(2, qi)};
#pragma unroll
        for (int sft = 1; sft <= n / 2; ++sft) {
          if (2 * sft == n && 2 * i >= n) continue;  // met from the other end
          const int j = i + sft < n ? i + sft : i + sft - n;
          const int qj = slot(j);
          const PS B = load_ps<VF>(sS, n3, qj, gg);
          const double nS[3] = {na[0] + metric(0, qj), na[1] + metric(1, qj), na[2] + metric(2, qj)};
          double F[5];
          pair2<VF>(A, B, nS, kg, F);
          const double Dij = D[i * n + j], Dji = D[j * n + i];
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            acc[0][v] = fma(Dij, F[v], acc[0][v]);
            acc[sft][v] = fma(Dji, F[v], acc[sft][v]);
          }
        }
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double x = acc[0][v];
#pragma unroll
          for (int m = 0; m + 1 < n; ++m) acc[m][v] = acc[m + 1][v];
          acc[N][v] = x;
        }
      }
    }
  }
  // the epilogue's loads are issued before the directions' sums meet
  double Rq[IT][5], gd[IT][4], sjq[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
      sjq[it] = AFF ? jc[9] : g.sJ[(size_t)e * n3 + t];
      if (NS) {
        // viscous part in strong form, formed by the lifting kernel
#pragma unroll
        for (int c = 0; c < 4; ++c) gd[it][c] = g.Gd[((size_t)e * 4 + c) * n3 + t];
      }
      if (mode == 1 && ca != 0.0) {
        const double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
        for (int v = 0; v < 5; ++v) Rq[it][v] = Re[v * n3 + t];
      }
    }
  }
  // the three directions' sums, in order
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    __syncthreads();
    if (act && dir == d) {
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = d == 0 ? div_slot<n>(m, a, b) : (d == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m));
#pragma unroll
        for (int v = 0; v < 5; ++v) sAcc[v * n3 + q] = d == 0 ? acc[m][v] : sAcc[v * n3 + q] + acc[m][v];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (!(valid && t < n3)) continue;
    const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
    double r[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] = sAcc[v * n3 + q];
    if (NS) {
#pragma unroll
      for (int c = 0; c < 4; ++c) r[1 + c] -= gd[it][c];
    }
    double *Oe = out + (size_t)e * 5 * n3;
    if (mode == 0) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Oe[v * n3 + t] = -r[v] * sjq[it];
    } else {
      double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        // a = 0 (first stage) does not read R, so R may hold anything on entry
        const double x = (ca != 0.0 ? ca * Rq[it][v] : 0.0) + dt * (-r[v] * sjq[it]);
        Re[v * n3 + t] = x;
        Oe[v * n3 + t] = sU[v * n3 + q] + cb * x;
      }
    }
  }
}

template <int N, bool NS, int VF, int GEN, bool FVM, bool AFF>
__global__ void __launch_bounds__(SplitSz<N>::NT, split_minb(N, VF, AFF)) k_split(Geo g, Phys ph, const double *__restrict__ U,
                                                     double *__restrict__ out, double *__restrict__ R, double ca,
                                                     double cb, double dt, int mode) {
  __shared__ double sm[AFF ? SplitLds<N>::AFFINE : SplitLds<N>::A];
  const int e = xcd_element(blockIdx.x, g.K);
  if (e >= g.K) return;
  if (FVM && g.fvflag[e]) return;  // a finite-volume element
  split_body<N, NS, VF, GEN, FVM, AFF>(g, ph, g.tab, e, true, threadIdx.x, U, out, R, ca, cb, dt, mode, sm);
}

// The same with a lane per end of every line (see EndsSz): the fluxes at the two ends are evaluated at once, and with
// the short pair fluxes each lane sums one half of the line's nodes.  For degrees 1 and 2, where both ends' lanes fit
// the one wave (1 M nodes, curved, KEP: N = 1 2570 -> 1797 us a step, N = 2 913 -> 756), and for small meshes (small_mesh).
// The bits are those of split_body.  (One body for both took 64 us instead of 62 at N = 5, curved, 16^3, from another
// schedule alone.)
template <int N, bool NS, int VF, int GEN, bool FVM, bool AFF>
__device__ __forceinline__ void split_ends(const Geo &g, const Phys &ph, const Tab *tab, int e, bool valid, int lane,
                                           const double *__restrict__ U, double *__restrict__ out,
                                           double *__restrict__ R, double ca, double cb, double dt, int mode,
                                           double *sm) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = EndsSz<N>::NT, NL = 3 * n2;
  constexpr bool WU = split_halves<N, VF>();
  constexpr bool SEP = !ends_always(N);  // the directions' sums in LDS of their own
  constexpr int IT = (n3 + NT - 1) / NT;  // nodes per lane in the node loops
  const double gm1 = ph.gamma - 1.0, kg = 1.0 / gm1, gg = gm1 / ph.gamma;
  const double *Ue = U + (size_t)e * 5 * n3;
  const double *Jae = g.Ja + (size_t)e * 9 * n3;
  double *sU = sm, *sS = sm + 5 * n3, *sJ = sm + 10 * n3;  // node slots: div_slot
  double *sAcc = AFF || !ends_always(N) ? sS : sJ;
  AffineConst jc = nullptr;
  if constexpr (AFF) jc = affine_const(g, e);
  // the 1D tables through the scalar cache
  const __attribute__((address_space(4))) double *D = (const __attribute__((address_space(4))) double *)tab->D;
  const double lh0 = tab->lhm[0], lhN = tab->lhp[N];
  // this lane's line: direction, and its position (a, b) among the direction's lines, which is also the
  // face point of its two ends, and the end whose flux it evaluates
  const int end = line_end<N, true>(lane), line = lane - end * EndsSz<N>::HALF;
  const int dir = n2 % 64 == 0 ? __builtin_amdgcn_readfirstlane(line / n2) : line / n2;
  const int ab = line - dir * n2, a = ab % n, b = ab / n;
  const bool act = valid && line < NL && end < 2;
  // the two end faces' neighbours first (loads return in order: behind the others, the neighbours' traces
  // would wait for all of them), then the state and metric terms for LDS and the faces' other sides
  const int s = 2 * dir + end;
  const bool plus = end;
  int nb = 0;
  NbFace f;
  if (act) {
    nb = g.nbr[(size_t)e * 6 + s];
    f = nbr_face<n, (GEN > 0)>(g, e, s, a, b);
  }
  double Uq[IT][5];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Uq[it][v] = Ue[v * n3 + t];
    }
  }
  double Jq[IT][9];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (!AFF && valid && t < n3) {
#pragma unroll
      for (int c = 0; c < 9; ++c) Jq[it][c] = Jae[c * n3 + t];
    }
  }
  double Ux[5], Vo[4], Vn[4];  // the end face: the other side's state, both sides' viscous fluxes
  int kind = -1;               // -1 inner face, else the boundary kind; -2 a face whose flux is given (Ux)
  if (act) {
    const bool bnd = GEN && f.bnd;
    // the outward flux of a non-conforming face, or of one shared with a finite-volume element
    const double *gx = nullptr;
    if (GEN == 2 && bnd && f.kind == FACE_MORTAR) gx = g.mflux + (size_t)g.mslot[(size_t)e * 6 + s] * 5 * n2 + ab;
    if (FVM && g.fvflag[nb]) gx = g.fvFx + ((size_t)e * 6 + s) * 5 * n2 + ab;
    if ((GEN == 2 || FVM) && gx) {
      kind = -2;
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[v] = gx[v * n2];
    } else {
      if (bnd) kind = f.kind;
      if (!bnd) {
        const double *Un = U + (size_t)nb * 5 * n3;
        const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(dir, a, b, plus ? 0 : N);
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[v] = Un[v * n3 + qn];
      }
      if (NS) {
        // both sides' contravariant viscous flux of the face's direction from the lifting (a boundary side:
        // the own trace)
        const double *fo = g.Gf + ((size_t)e * 6 + s) * 4 * n2 + ab;
        const double *fnb = bnd ? fo : g.Gf + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
#pragma unroll
        for (int c = 0; c < 4; ++c) { Vo[c] = fo[c * n2]; Vn[c] = fnb[c * n2]; }
      }
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
      const Pr5 P = to_prim(Uq[it], gm1);
#pragma unroll
      for (int v = 0; v < 5; ++v) sU[v * n3 + q] = Uq[it][v];
      sS[q] = P.rho; sS[n3 + q] = P.u; sS[2 * n3 + q] = P.v; sS[3 * n3 + q] = P.w;
      // beta = rho / (2 p) for EC, the total enthalpy otherwise
      sS[4 * n3 + q] = (VF == 1) ? 0.5 * P.rho / P.p : (Uq[it][4] + P.p) / P.rho;
#pragma unroll
      for (int c = 0; c < 9 && !AFF; ++c) sJ[c * n3 + q] = Jq[it][c];
    }
  }
  __syncthreads();
  double acc[n][5];
  constexpr int NF = WU ? 1 : 2;
  double fe[NF][5];  // this lane's end (without split sums: then the line's two ends)
  // the line direction's metric terms at a node
  const double *sJd = sJ + 3 * dir * n3;
  double jl[3] = {0.0, 0.0, 0.0};
  auto metric = [&](int d, int q) -> double {
    if constexpr (AFF) return jl[d];
    else return sJd[d * n3 + q];
  };
  auto faces = [&](const LineSlots<n> &slot) {
    if constexpr (AFF) {
#pragma unroll
      for (int d = 0; d < 3; ++d) jl[d] = dir == 0 ? jc[d] : (dir == 1 ? jc[3 + d] : jc[6 + d]);
    }
    // numerical surface fluxes at the line's ends, lifted (outward times lhat), and the interior
    // convective part: 2 D_ii F(U_i) (D_ii is non-zero only at the ends of LGL lines) -+ lhat F_int
    const int qo = slot(plus ? N : 0);
    const double sg = plus ? 1.0 : -1.0, lh = plus ? lhN : lh0;
    double Uw[5], Fo[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uw[v] = sU[v * n3 + qo];
    // normal along +xi scaled by s-hat: Ja^dir at the face node, the master's on the master side and
    // (up to rounding, the metric terms being continuous across the face) on the slave
    const double nt[3] = {metric(0, qo), metric(1, qo), metric(2, qo)};
    const Pr5 Pw = {Uw[0], sS[n3 + qo], sS[2 * n3 + qo], sS[3 * n3 + qo],
                    gm1 * (Uw[4] - 0.5 * (Uw[1] * sS[n3 + qo] + Uw[2] * sS[2 * n3 + qo] + Uw[3] * sS[3 * n3 + qo]))};
    flux_c(Uw, Pw, nt, Fo);
    const double cd = 2.0 * (plus ? D[N * n + N] : D[0]) - sg * lh;
    double F[5];
    if ((GEN == 2 || FVM) && kind == -2) {
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] = sg * Ux[v];
    } else {
      const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
      const double ish = 1.0 / sh;
      const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
      const bool bnd = GEN && kind >= 0;
      const bool outflow = bnd && kind == DG_BC_OUTFLOW;
      const bool given = bnd && (kind == DG_BC_STATE || outflow);
      const bool iso = bnd && kind == DG_BC_WALL_ISOTHERMAL;
      const bool wall = bnd && (kind == DG_BC_WALL || iso);
      if (bnd) {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[v] = Uw[v];
        if (outflow) {
          // pressure outflow: the own trace's density and velocity with p_out
          Ux[4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
        } else if (given) {
#pragma unroll
          for (int v = 0; v < 5; ++v) Ux[v] = ph.ub[v];  // given outer state
        } else if (wall) {
          Ux[1] = -Uw[1]; Ux[2] = -Uw[2]; Ux[3] = -Uw[3];  // no-slip wall: velocity reversed
        } else {
          mirror3(Ux + 1, nh);  // symmetry plane: mirror image of the inner state
        }
      }
      double UM[5], US[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) { UM[v] = plus ? Uw[v] : Ux[v]; US[v] = plus ? Ux[v] : Uw[v]; }
      riemann_vf<VF>(ph, UM, US, nh, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] *= sh;
      if (NS) {
        // BR1 mean of the viscous fluxes along this side's +xi normal Ja^dir (the normal metric of a
        // conforming face is continuous: the neighbour's Ja of its face direction is +-Ja^dir, + where
        // one side is a +xi side and the other a -xi side)
        double V[4];
        const double sn = (GEN && f.plus == plus) ? -1.0 : 1.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) V[c] = bnd ? Vo[c] : 0.5 * (Vo[c] + sn * Vn[c]);
        if (!bnd || given) {
          // given outer state: the outer viscous flux equals the inner one
#pragma unroll
          for (int c = 0; c < 4; ++c) F[1 + c] -= V[c];
        } else if (wall) {
          // no-slip wall: the outer momentum flux equals the inner one, the outer energy flux is its
          // negative (reversed velocity, mirrored heat flux), so the mean keeps the momentum; at an
          // isothermal wall the outer gradient is the inner one, so the mean energy flux is the inner
          // heat flux: the inner energy flux minus the work (tau Ja^dir) . u
#pragma unroll
          for (int c = 0; c < 3; ++c) F[1 + c] -= V[c];
          if (iso) F[4] -= V[3] - (V[0] * Uw[1] + V[1] * Uw[2] + V[2] * Uw[3]) * (1.0 / Uw[0]);
        } else {
          // symmetry plane: the mirrored outer flux cancels the inner shear and heat flux, the mean
          // keeps the normal part of the momentum flux
          const double gm = V[0] * nh[0] + V[1] * nh[1] + V[2] * nh[2];
#pragma unroll
          for (int c = 0; c < 3; ++c) F[1 + c] -= gm * nh[c];
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) fe[0][v] = fma(cd, Fo[v], (sg * lh) * F[v]);
  };
  // the sums of the nodes M0 <= m < M1 (all, or the near or the far half of the line): each node meets its partners
  // in the same order whoever sums it, so the bits do not depend on the split
  auto pairs = [&](const LineSlots<n> &slot, auto m0, auto m1) {
    constexpr int M0 = decltype(m0)::value, M1 = decltype(m1)::value;
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[m][v] = m == 0 ? fe[0][v] : (m == N ? fe[M0 > 0 ? 0 : NF - 1][v] : 0.0);
    // EC: where every pair of every line of this wave lies in the series' range (the largest ratio of a
    // line is that of its largest and smallest value) the unrolled loop below needs no logarithm
    bool series = true;
    if constexpr (VF == 1) {
      double r0 = sS[slot(0)], r1 = r0, b0 = sS[4 * n3 + slot(0)], b1 = b0;
#pragma unroll
      for (int m = 1; m < n; ++m) {
        const double r = sS[slot(m)], bt = sS[4 * n3 + slot(m)];
        r0 = fmin(r0, r); r1 = fmax(r1, r);
        b0 = fmin(b0, bt); b1 = fmax(b1, bt);
      }
      const double dr = r1 - r0, sr = r1 + r0, db = b1 - b0, sb = b1 + b0;
      series = dr * dr < 0.99e-4 * (sr * sr) && db * db < 0.99e-4 * (sb * sb);
      series = __all(series);
    }
    if (VF != 1 || series) {
      // node i in registers, its partners read from LDS one pair ahead of their use (a whole line in
      // registers spills 500 bytes at n = 8); the first partner is the next row's node
      auto node = [&](int m) -> LineNode {
        LineNode x;
        const int q = slot(m);
        x.s = load_ps<VF>(sS, n3, q, gg);
#pragma unroll
        for (int d = 0; d < 3; ++d) x.nv[d] = metric(d, q);
        return x;
      };
      LineNode A = node(0), B = node(1), An = B, Bn = B;
#pragma unroll
      for (int i = 0; i + 1 < n; ++i) {
#pragma unroll
        for (int j = i + 1; j < n; ++j) {
          if (j == i + 1) An = B;
          if (j + 1 < n) Bn = node(j + 1);
          else if (i + 2 < n) Bn = node(i + 2);
          const bool si = i >= M0 && i < M1, sj = j >= M0 && j < M1;  // whose sums are taken here
          if (!si && !sj) {
            B = Bn;
            continue;
          }
          const double nS[3] = {A.nv[0] + B.nv[0], A.nv[1] + B.nv[1], A.nv[2] + B.nv[2]};
          double F[5];
          pair2<VF, true>(A.s, B.s, nS, kg, F);
          const double Dij = D[i * n + j], Dji = D[j * n + i];
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            if (si) acc[i][v] = fma(Dij, F[v], acc[i][v]);
            if (sj) acc[j][v] = fma(Dji, F[v], acc[j][v]);
          }
          B = Bn;
          // at most two pairs in flight: more spill (n <= 6 fits as scheduled)
          if (n > 6 && (j - i) % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        }
        A = An;
        asm volatile("" ::: "memory");  // the next row's partners are read again, not kept
      }
    } else {
      // the same pairs (i, i + s mod n) with logarithms, the states read from LDS as they are met; a
      // rolled loop over i whose sums move down one place per turn, so that node i's is always the first
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        const int qi = slot(i);
        const PS A = load_ps<VF>(sS, n3, qi, gg);
        const double na[3] = {metric(0, qi), metric(1, qi), metric(2, qi)};
#pragma unroll
        for (int sft = 1; sft <= n / 2; ++sft) {
          if (2 * sft == n && 2 * i >= n) continue;  // met from the other end
          const int j = i + sft < n ? i + sft : i + sft - n;
          const int qj = slot(j);
          const PS B = load_ps<VF>(sS, n3, qj, gg);
          const double nS[3] = {na[0] + metric(0, qj), na[1] + metric(1, qj), na[2] + metric(2, qj)};
          double F[5];
          pair2<VF>(A, B, nS, kg, F);
          const double Dij = D[i * n + j], Dji = D[j * n + i];
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            acc[0][v] = fma(Dij, F[v], acc[0][v]);
            acc[sft][v] = fma(Dji, F[v], acc[sft][v]);
          }
        }
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double x = acc[0][v];
#pragma unroll
          for (int m = 0; m + 1 < n; ++m) acc[m][v] = acc[m + 1][v];
          acc[N][v] = x;
        }
      }
    }
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, n / 2> IH;
  typedef std::integral_constant<int, n> IN;
  if constexpr (WU) {
    if (act) {
      const LineSlots<n> slot(dir, a, b);
      faces(slot);
      if (end) pairs(slot, IH(), IN());
      else pairs(slot, I0(), IH());
    }
  } else {
    // the far end's flux to the line's own lane
    double *sF = sm + SplitLds<N>::template nodes<AFF, true>();
    const LineSlots<n> slot(act ? dir : 0, act ? a : 0, act ? b : 0);
    if (act) faces(slot);
    if (act && end) {
#pragma unroll
      for (int v = 0; v < 5; ++v) sF[v * NL + line] = fe[0][v];
    }
    __syncthreads();
    if (act && !end) {
#pragma unroll
      for (int v = 0; v < 5; ++v) fe[1][v] = sF[v * NL + line];
      pairs(slot, I0(), IN());
    }
  }
  // the epilogue's loads are issued before the directions' sums meet
  double Rq[IT][5], gd[IT][4], sjq[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (valid && t < n3) {
      sjq[it] = AFF ? jc[9] : g.sJ[(size_t)e * n3 + t];
      if (NS) {
        // viscous part in strong form, formed by the lifting kernel
#pragma unroll
        for (int c = 0; c < 4; ++c) gd[it][c] = g.Gd[((size_t)e * 4 + c) * n3 + t];
      }
      if (mode == 1 && ca != 0.0) {
        const double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
        for (int v = 0; v < 5; ++v) Rq[it][v] = Re[v * n3 + t];
      }
    }
  }
  // the three directions' sums, in order (SEP: put down at once, added below in that order)
#pragma unroll
  for (int d = 0; d < (SEP ? 1 : 3); ++d) {
    __syncthreads();
    if (act && (WU || !end) && (SEP || dir == d)) {
      const LineSlots<n> slot(dir, a, b);
      double *sD = sAcc + (SEP ? dir * 5 * n3 : 0);
#pragma unroll
      for (int m = 0; m < n; ++m) {
        if (WU && (m >= n / 2) != (end != 0)) continue;
        const int q = SEP ? slot(m) : (d == 0 ? div_slot<n>(m, a, b) : (d == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m)));
#pragma unroll
        for (int v = 0; v < 5; ++v) sD[v * n3 + q] = SEP || d == 0 ? acc[m][v] : sD[v * n3 + q] + acc[m][v];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (!(valid && t < n3)) continue;
    const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
    double r[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      r[v] = sAcc[v * n3 + q];
      if (SEP) r[v] = (r[v] + sAcc[(5 + v) * n3 + q]) + sAcc[(10 + v) * n3 + q];
    }
    if (NS) {
#pragma unroll
      for (int c = 0; c < 4; ++c) r[1 + c] -= gd[it][c];
    }
    double *Oe = out + (size_t)e * 5 * n3;
    if (mode == 0) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Oe[v * n3 + t] = -r[v] * sjq[it];
    } else {
      double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        // a = 0 (first stage) does not read R, so R may hold anything on entry
        const double x = (ca != 0.0 ? ca * Rq[it][v] : 0.0) + dt * (-r[v] * sjq[it]);
        Re[v * n3 + t] = x;
        Oe[v * n3 + t] = sU[v * n3 + q] + cb * x;
      }
    }
  }
}

template <int N, bool NS, int VF, int GEN, bool FVM, bool AFF>
__global__ void __launch_bounds__(EndsSz<N>::NT, (split_minb(N, VF, AFF))) k_split_ends(Geo g, Phys ph, const double *__restrict__ U,
                                                     double *__restrict__ out, double *__restrict__ R, double ca,
                                                     double cb, double dt, int mode) {
  __shared__ double sm[SplitLds<N>::template size<VF, AFF, true>()];
  const int e = xcd_element(blockIdx.x, g.K);
  if (e >= g.K) return;
  if (FVM && g.fvflag[e]) return;  // a finite-volume element
  split_ends<N, NS, VF, GEN, FVM, AFF>(g, ph, g.tab, e, true, threadIdx.x, U, out, R, ca, cb, dt, mode, sm);
}

// ----------------------------------------------------------------------------- weak/strong form, by lines
// Waves per SIMD k_line is built for: at three no instance spills but those of boundary meshes with a two-point
// flux (36 bytes); four (128 registers) spill in the Euler operator at N = 3 and take 2122 us a step of 48^3
// elements instead of 2026.
template <int N> constexpr int line_minb() { return N >= 8 ? 2 : 3; }

// Weak- and strong-form operator of conforming meshes (Euler: also with non-conforming faces), one lane per
// line as the split operator: the lane evaluates the numerical fluxes of the faces at its line's ends, adds
// every node's flux along the line, times the matrix's column, to the line's n sums, and the two fluxes times
// lhat(+-1).  FORM 0 weak (D-hat), 2 strong (D; on LG nodes Tab::Ds, whose surface term is the numerical flux
// alone).  Navier-Stokes: the lifting has formed the viscous volume term (Geo::Gd) and the faces' viscous
// fluxes (Geo::Gf): contravariant traces for the strong form on LGL nodes, else each side's flux along its
// own outward normal.
// What bounds it: with one node per lane the Euler operator on LG nodes at N = 3 waited for memory 70 % of
// its wavefronts' time (seven dependent trips: a neighbour's index, then its lines two nodes at a time, for
// each of two rounds of face points, and the register at the end).  Here every load of an element is issued
// before the first barrier.  A step of 48^3 elements (Euler, LG, N = 3) 2408 -> 2026 us; of 16^3 (Navier-Stokes,
// weak form, LG, N = 7: half the LDS accesses) 1433 -> 1247 us; strong form, LGL, N = 4, curved 467 -> 456 us.
// AFF, FVM, mode as for the split operator.  ENDS too, each lane taking one half of the line's nodes' fluxes (Euler
// on LG nodes, 64 elements, curved: N = 5 54.8 -> 44.7 us a step, N = 7 76.2 -> 67.8).  TP: two-point surface flux (riemann 2, 3): its logarithmic means
// cost 60 registers more, so LLF and Roe take the instance without them.
template <int N, bool LGL, bool NS, int FORM, int GEN, bool FVM, bool AFF, bool TP, bool ENDS>
__global__ void __launch_bounds__((line_lanes<N, ENDS>()), (line_minb<N>()))
    k_line(Geo g, Phys ph, const double *__restrict__ U, double *__restrict__ out, double *__restrict__ R, double ca,
           double cb, double dt, int mode) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3, NT = line_lanes<N, ENDS>(), IT = (n3 + NT - 1) / NT;
  constexpr int NL = 3 * n2, NE = ENDS ? 1 : 2;
  constexpr bool WU = EndsSz<N>::HALF % 64 == 0;  // an end's lanes fill whole waves
  constexpr bool SEP = line_apart<N, ENDS>();  // the directions' sums in LDS of their own
  static_assert(SEP == (ENDS && WU));
  constexpr bool PFM = NS && !(FORM == 2 && LGL);  // face viscous fluxes along each side's own normal
  // state, metric terms (none on affine elements); the result takes the metric terms' place; ENDS with both
  // halves in one wave: the far ends' fluxes
  __shared__ double sm[SEP ? 20 * n3 : (AFF ? 10 : 14) * n3 + (ENDS ? 5 * NL : 0)];
  double *sU = sm, *sJ = sm + 5 * n3, *sAcc = sJ;
  const int e = xcd_element(blockIdx.x, g.K), lane = threadIdx.x;
  if (e >= g.K) return;
  if (FVM && g.fvflag[e]) return;  // a finite-volume element
  AffineConst jc = nullptr;
  if constexpr (AFF) jc = affine_const(g, e);
  const double gm1 = ph.gamma - 1.0;
  const double *Ue = U + (size_t)e * 5 * n3;
  const Tab *tab = g.tab;
  typedef const __attribute__((address_space(4))) double *Scal;
  const Scal M = (Scal)(FORM == 0 ? tab->Dh : (LGL ? tab->D : tab->Ds));
  const Scal lm = (Scal)tab->lm, lp = (Scal)tab->lp, lhm = (Scal)tab->lhm, lhp = (Scal)tab->lhp;
  const int end = line_end<N, ENDS>(lane), line = lane - end * EndsSz<N>::HALF;
  const int dir = n2 % 64 == 0 ? __builtin_amdgcn_readfirstlane(line / n2) : line / n2;
  const int ab = line - dir * n2, a = ab % n, b = ab / n;
  const bool act = line < NL && end < 2;
  // the neighbours' indices first (loads return in order), then everything else the element reads
  int nb2[NE] = {};
  NbFace f2[NE];
#pragma unroll
  for (int x = 0; x < NE; ++x)
    if (act) {
      const int sd = ENDS ? end : x;
      nb2[x] = g.nbr[(size_t)e * 6 + 2 * dir + sd];
      f2[x] = nbr_face<n, (GEN > 0)>(g, e, 2 * dir + sd, a, b);
    }
  double Uq[IT][5], Rq[IT][5];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t < n3) {
#pragma unroll
      for (int v = 0; v < 5; ++v) Uq[it][v] = Ue[v * n3 + t];
    }
  }
  double Jq[IT][9];
  if constexpr (!AFF) {
    const double *Jae = g.Ja + (size_t)e * 9 * n3;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int t = lane + it * NT;
      if (t < n3) {
#pragma unroll
        for (int c = 0; c < 9; ++c) Jq[it][c] = Jae[c * n3 + t];
      }
    }
  }
  constexpr bool LINES = !LGL && !NS;     // the neighbours' traces are interpolated here from their lines
  constexpr int CH = n <= 4 || ENDS ? n : 2;  // nodes of the neighbours' lines in flight
  double Ux[NE][5], Vo[NE][4], Vn[NE][4], nt2[NE][3];
  int kind[NE];  // -1 inner face, else the boundary kind; -2 a face whose outward flux is given (Ux)
#pragma unroll
  for (int x = 0; x < NE; ++x) {
    kind[x] = -1;
    if (!act) continue;
    const int sd = ENDS ? end : x, s = 2 * dir + sd;
    const int nb = nb2[x];
    const NbFace f = f2[x];
    const bool bnd = GEN && f.bnd;
    const double *fnp = AFF ? g.Jc + (size_t)e * AFFINE_DOUBLES + 10 + 3 * s : g.fn + ((size_t)e * 6 + s) * 3 * n2 + ab;
    const int fst = AFF ? 1 : n2;
#pragma unroll
    for (int d = 0; d < 3; ++d) nt2[x][d] = fnp[d * fst];
    const double *gx = nullptr;
    if (GEN == 2 && bnd && f.kind == FACE_MORTAR) gx = g.mflux + (size_t)g.mslot[(size_t)e * 6 + s] * 5 * n2 + ab;
    if (FVM && !bnd && g.fvflag[nb]) gx = g.fvFx + ((size_t)e * 6 + s) * 5 * n2 + ab;
    if ((GEN == 2 || FVM) && gx) {
      // the outward flux from the mortar face array, or of a face shared with a finite-volume element
      kind[x] = -2;
#pragma unroll
      for (int v = 0; v < 5; ++v) Ux[x][v] = gx[v * n2];
      continue;
    }
    if (bnd) kind[x] = f.kind;
    if (!bnd && !LINES) {
      if (LGL) {
        const double *Un = U + (size_t)nb * 5 * n3;
        const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, f.plus ? N : 0) : line_node<n>(dir, a, b, sd ? 0 : N);
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[x][v] = Un[v * n3 + qn];
      } else {
        const double *ut = g.Utr + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 5 * n2 + f.a + n * f.b;
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[x][v] = ut[v * n2];
      }
    }
    if (NS) {
      const double *fo = g.Gf + ((size_t)e * 6 + s) * 4 * n2 + ab;
      const double *fnb = bnd ? fo : g.Gf + ((size_t)nb * 6 + 2 * f.dn + (f.plus ? 1 : 0)) * 4 * n2 + f.a + n * f.b;
#pragma unroll
      for (int c = 0; c < 4; ++c) { Vo[x][c] = fo[c * n2]; Vn[x][c] = fnb[c * n2]; }
    }
  }
  // the epilogue's loads: the register here where they are few, the rest below
  constexpr bool PRE = IT == 1 && !NS;
  double gd[IT][4], sjq[IT];
  auto load_epilogue = [&]() {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int t = lane + it * NT;
      if (t < n3) {
        sjq[it] = AFF ? jc[9] : g.sJ[(size_t)e * n3 + t];
        if (NS) {
#pragma unroll
          for (int c = 0; c < 4; ++c) gd[it][c] = g.Gd[((size_t)e * 4 + c) * n3 + t];
        }
        if (mode == 1 && ca != 0.0) {
          const double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
          for (int v = 0; v < 5; ++v) Rq[it][v] = Re[v * n3 + t];
        }
      }
    }
  };
  if constexpr (PRE) load_epilogue();
  if constexpr (LINES) {
    if (act) {
#pragma unroll
      for (int x = 0; x < NE; ++x)
#pragma unroll
        for (int v = 0; v < 5; ++v)
          if (kind[x] != -2) Ux[x][v] = 0.0;
#pragma unroll(CH == n ? n : 1)
      for (int c = 0; c < n; c += CH) {
        double y[NE][CH][5];
#pragma unroll
        for (int x = 0; x < NE; ++x) {
          if (kind[x] != -1) continue;
          const NbFace f = f2[x];
          const double *Un = U + (size_t)nb2[x] * 5 * n3;
#pragma unroll
          for (int m = 0; m < CH; ++m)
            if (c + m < n) {
              const int qn = GEN ? line_node<n>(f.dn, f.a, f.b, c + m) : line_node<n>(dir, a, b, c + m);
#pragma unroll
              for (int v = 0; v < 5; ++v) y[x][m][v] = Un[v * n3 + qn];
            }
        }
#pragma unroll
        for (int x = 0; x < NE; ++x) {
          if (kind[x] != -1) continue;
          const bool np = GEN ? f2[x].plus : !(ENDS ? end : x);
#pragma unroll
          for (int m = 0; m < CH; ++m)
            if (c + m < n) {
              const double l = np ? lp[c + m] : lm[c + m];
#pragma unroll
              for (int v = 0; v < 5; ++v) Ux[x][v] = fma(l, y[x][m][v], Ux[x][v]);
            }
        }
      }
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t < n3) {
      const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
#pragma unroll
      for (int v = 0; v < 5; ++v) sU[v * n3 + q] = Uq[it][v];
#pragma unroll
      for (int c = 0; c < 9 && !AFF; ++c) sJ[c * n3 + q] = Jq[it][c];
    }
  }
  __syncthreads();
  double acc[n][5];
  constexpr int NF = ENDS && WU ? 1 : 2;
  double F2[NF][5];  // numerical fluxes at the line's ends, outward
  auto faces = [&](const LineSlots<n> &slot) {
#pragma unroll
    for (int x = 0; x < NE; ++x) {
      const bool plus = ENDS ? end : x;
      if ((GEN == 2 || FVM) && kind[x] == -2) {
#pragma unroll
        for (int v = 0; v < 5; ++v) F2[x][v] = Ux[x][v];
        continue;
      }
      double Uw[5];
      if (LGL) {
        const int qo = slot(plus ? N : 0);
#pragma unroll
        for (int v = 0; v < 5; ++v) Uw[v] = sU[v * n3 + qo];
      } else {
#pragma unroll
        for (int v = 0; v < 5; ++v) Uw[v] = 0.0;
#pragma unroll 4
        for (int m = 0; m < n; ++m) {
          const int q = slot(m);
          const double l = plus ? lp[m] : lm[m];
#pragma unroll
          for (int v = 0; v < 5; ++v) Uw[v] = fma(l, sU[v * n3 + q], Uw[v]);
        }
      }
      // the master's normal and state go first (the stored normal is outward, the master's negated on
      // the slave side)
      const bool mst = GEN ? f2[x].master : plus;
      const double sg = mst ? 1.0 : -1.0;
      const double nt[3] = {sg * nt2[x][0], sg * nt2[x][1], sg * nt2[x][2]};
      const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
      const double ish = 1.0 / sh;
      const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
      const bool bnd = GEN && kind[x] >= 0;
      const bool outflow = bnd && kind[x] == DG_BC_OUTFLOW;
      const bool given = bnd && (kind[x] == DG_BC_STATE || outflow);
      const bool iso = bnd && kind[x] == DG_BC_WALL_ISOTHERMAL;
      const bool wall = bnd && (kind[x] == DG_BC_WALL || iso);
      if (bnd) {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ux[x][v] = Uw[v];
        if (outflow) {
          // pressure outflow: the own trace's density and velocity with p_out
          Ux[x][4] = ph.pout / gm1 + 0.5 * (Uw[1] * Uw[1] + Uw[2] * Uw[2] + Uw[3] * Uw[3]) / Uw[0];
        } else if (given) {
#pragma unroll
          for (int v = 0; v < 5; ++v) Ux[x][v] = ph.ub[v];  // given outer state
        } else if (wall) {
          Ux[x][1] = -Uw[1]; Ux[x][2] = -Uw[2]; Ux[x][3] = -Uw[3];  // no-slip wall: velocity reversed
        } else {
          mirror3(Ux[x] + 1, nh);  // symmetry plane: mirror image of the inner state
        }
      }
      double UM[5], US[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) { UM[v] = mst ? Uw[v] : Ux[x][v]; US[v] = mst ? Ux[x][v] : Uw[v]; }
      double F[5];
      if constexpr (TP) riemann(ph, UM, US, nh, F);
      else if (ph.rs == DG_RS_LLF) riemann_t<DG_RS_LLF>(ph, UM, US, nh, F);
      else riemann_t<DG_RS_ROE>(ph, UM, US, nh, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) F2[x][v] = (sg * sh) * F[v];
      if (PFM) {
        // minus the outward BR1 mean of the viscous flux: each side's flux carries its own outward normal
        // (the two normals of a face are negatives of each other), a boundary side's is the mean itself
#pragma unroll
        for (int c = 0; c < 4; ++c) F2[x][1 + c] -= bnd ? Vo[x][c] : 0.5 * (Vo[x][c] - Vn[x][c]);
      } else if (NS) {
        // minus the BR1 mean of the viscous flux along this side's +xi direction (the split form's reading
        // of the traces and boundary kinds), applied outward
        const double sp = plus ? 1.0 : -1.0;
        const double sn = (GEN && f2[x].plus == plus) ? -1.0 : 1.0;
        double V[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) V[c] = bnd ? Vo[x][c] : 0.5 * (Vo[x][c] + sn * Vn[x][c]);
        if (wall) {
          // the momentum part of the inner flux; at an isothermal wall the inner heat flux (the energy flux
          // minus the work of the stress)
          V[3] = iso ? V[3] - (V[0] * Uw[1] + V[1] * Uw[2] + V[2] * Uw[3]) * (1.0 / Uw[0]) : 0.0;
        } else if (bnd && !given) {
          // symmetry plane: the normal part of the momentum flux
          const double gm = V[0] * nh[0] + V[1] * nh[1] + V[2] * nh[2];
          V[0] = gm * nh[0]; V[1] = gm * nh[1]; V[2] = gm * nh[2];
          V[3] = 0.0;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) F2[x][1 + c] -= sp * V[c];
      }
      if (!ENDS) __builtin_amdgcn_sched_barrier(0);  // one end at a time: both in flight spill
    }
  };
  // the sums over the nodes M0 <= m < M1 and over the line's ends that lie among them
  auto contract = [&](const LineSlots<n> &slot, auto m0, auto m1) {
    constexpr int M0 = decltype(m0)::value, M1 = decltype(m1)::value;
    // surface integral (on LGL nodes lhat is non-zero at the ends only)
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        if (LGL) acc[m][v] = m == 0 && M0 == 0 ? lhm[0] * F2[0][v] : (m == N && M1 == n ? lhp[N] * F2[M0 > 0 ? 0 : NF - 1][v] : 0.0);
        else if (M0 > 0) acc[m][v] = lhp[m] * F2[0][v];
        else if (M1 < n) acc[m][v] = lhm[m] * F2[0][v];
        else acc[m][v] = fma(lhm[m], F2[0][v], lhp[m] * F2[NF - 1][v]);
      }
    double jl[3] = {0.0, 0.0, 0.0};
    if constexpr (AFF) {
#pragma unroll
      for (int d = 0; d < 3; ++d) jl[d] = dir == 0 ? jc[d] : (dir == 1 ? jc[3 + d] : jc[6 + d]);
    }
    const double *sJd = sJ + 3 * dir * n3;
    // volume integral: node by node, its flux times the matrix's column into the line's sums
#pragma unroll
    for (int m = M0; m < M1; ++m) {
      const int q = slot(m);
      double Uo[5], Fc[5], nv[3];
#pragma unroll
      for (int v = 0; v < 5; ++v) Uo[v] = sU[v * n3 + q];
#pragma unroll
      for (int d = 0; d < 3; ++d) nv[d] = AFF ? jl[d] : sJd[d * n3 + q];
      flux_c(Uo, to_prim(Uo, gm1), nv, Fc);
#pragma unroll
      for (int i = 0; i < n; ++i) {
        double c = M[i * n + m];
        // strong form on LGL nodes: minus the face node's own interior flux (on LG nodes part of Tab::Ds)
        if (FORM != 0 && LGL && i == m && m == 0) c += lhm[0];
        if (FORM != 0 && LGL && i == m && m == N) c -= lhp[N];
#pragma unroll
        for (int v = 0; v < 5; ++v) acc[i][v] = fma(c, Fc[v], acc[i][v]);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);  // one node's flux at a time: more in flight spill
    }
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, (n + 1) / 2> IH;
  typedef std::integral_constant<int, n> IN;
  if constexpr (!ENDS) {
    if (act) {
      const LineSlots<n> slot(dir, a, b);
      faces(slot);
      contract(slot, I0(), IN());
    }
  } else if constexpr (WU) {
    if (act) {
      const LineSlots<n> slot(dir, a, b);
      faces(slot);
      if (end) contract(slot, IH(), IN());
      else contract(slot, I0(), IH());
    }
  } else {
    // both halves in one wave: the far end's flux to the line's own lane
    double *sF = sm + (AFF ? 10 : 14) * n3;
    const LineSlots<n> slot(act ? dir : 0, act ? a : 0, act ? b : 0);
    if (act) faces(slot);
    if (act && end) {
#pragma unroll
      for (int v = 0; v < 5; ++v) sF[v * NL + line] = F2[0][v];
    }
    __syncthreads();
    if (act && !end) {
#pragma unroll
      for (int v = 0; v < 5; ++v) F2[1][v] = sF[v * NL + line];
      contract(slot, I0(), IN());
    }
  }
  if constexpr (!PRE) load_epilogue();
  // the three directions' sums, in order (SEP: apart, first the near ends' halves, then the far ends' on top)
#pragma unroll
  for (int d = 0; d < (SEP ? 2 : 3); ++d) {
    __syncthreads();
    if (act && (SEP ? end == d : !(ENDS && end) && dir == d)) {
      const LineSlots<n> slot(dir, a, b);
      double *sD = sAcc + (SEP ? dir * 5 * n3 : 0);
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const int q = SEP ? slot(m) : (d == 0 ? div_slot<n>(m, a, b) : (d == 1 ? div_slot<n>(a, m, b) : div_slot<n>(a, b, m)));
#pragma unroll
        for (int v = 0; v < 5; ++v) sD[v * n3 + q] = d == 0 ? acc[m][v] : sD[v * n3 + q] + acc[m][v];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int t = lane + it * NT;
    if (t >= n3) continue;
    const int q = div_slot<n>(t % n, (t / n) % n, t / n2);
    double *Oe = out + (size_t)e * 5 * n3;
    double *Re = R + (size_t)e * 5 * n3;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double r = sAcc[v * n3 + q];
      if (SEP) r = (r + sAcc[(5 + v) * n3 + q]) + sAcc[(10 + v) * n3 + q];
      if (NS && v > 0) r -= gd[it][v - 1];  // the viscous volume term, formed by the lifting kernel
      const double ut = -r * sjq[it];
      if (mode == 0) {
        Oe[v * n3 + t] = ut;
      } else {
        // a = 0 (first stage) does not read R, so R may hold anything on entry
        const double x = (ca != 0.0 ? ca * Rq[it][v] : 0.0) + dt * ut;
        Re[v * n3 + t] = x;
        Oe[v * n3 + t] = sU[v * n3 + q] + cb * x;
      }
    }
  }
}

// ----------------------------------------------------------------------------- ensemble batch
// Workgroups of the batched kernels walk the concatenated element list of all members of one
// degree; EPB elements share a workgroup (one slot of Sz<N>::NT threads each, line_lanes in
// the split-form kernel, wave aligned).
// Each slot finds its member by bisection of the element prefix sums.
// AFF: no, every or some member's elements are affine.  AFF_MIXED takes each member's own path, so that a member's
// result has the bits of its one-mesh launch whatever its neighbours in the batch; one launch for both kinds, at the
// registers and LDS of the larger: a launch each took 201 us a step instead of 163 (16 members of degree 3 with 4^3 to
// 7^3 elements).
enum { AFF_NONE = 0, AFF_ALL = 1, AFF_MIXED = 2 };
__device__ __forceinline__ int member_of(const int *first, int count, int item) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int N, int AFF> constexpr int lift_b_lanes() { return AFF == AFF_ALL ? SplitSz<N>::NT : Sz<N>::NT; }
template <int N, int AFF> constexpr int lift_b_minb() {
  return AFF == AFF_NONE ? DG_LIFT_MINB : (AFF == AFF_ALL ? lift_affine_minb<N>() : 4);
}

template <int N, int EPB, bool GEN, int AFF>
__global__ void __launch_bounds__((lift_b_lanes<N, AFF>()) * EPB, (lift_b_minb<N, AFF>())) k_lift_b(BatchView bv) {
  using L = LiftLds<N>;
  constexpr int n = L::n, NT = lift_b_lanes<N, AFF>(), SM = AFF == AFF_ALL ? L::AFFINE : L::W + L::JA + L::WS;
  constexpr bool TAB = AFF != AFF_ALL;
  __shared__ double sm[EPB * SM];
  __shared__ double sDh[TAB ? n * n : 1], sl[TAB ? 2 * n : 1], slh[TAB ? 2 * n : 1];
  if constexpr (TAB) lift_tables<N>(bv.tab, threadIdx.x, NT * EPB, sDh, sl, slh);
  const BatchBlock B = batch_block(bv, EPB, blockIdx.x);
  if (B.item >= B.end) return;
  const int slot = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  const int t = threadIdx.x - slot * NT;
  const int item = B.item + slot;
  const bool valid = item < B.end;
  const int mi = member_of(bv.first, bv.count, valid ? item : B.end - 1);
  const Member &M = bv.m[mi];
  const int e = valid ? item - bv.first[mi] : 0;
  if (AFF == AFF_ALL || (AFF == AFF_MIXED && B.affine)) {
    lift_affine<N, true, LIFT_DIV, GEN, NT>(M.g, M.ph, bv.tab, e, valid, t, M.U, nullptr, nullptr, sm + slot * SM);
  } else {
    if constexpr (TAB) lift_body<N, true, LIFT_DIV, GEN>(M.g, M.ph, e, valid, t, M.U, nullptr, nullptr, sm + slot * SM, sDh, sl, slh);
  }
}

// one element of a member, one RK stage
template <int N, bool NS, int VF, int GEN, bool AFF>
__device__ __forceinline__ void split_member(const Member &M, const Tab *tab, int e, bool valid, int t, double *sm) {
  if constexpr (ends_always(N)) split_ends<N, NS, VF, GEN, false, AFF>(M.g, M.ph, tab, e, valid, t, M.U, M.out, M.R, M.a, M.b, M.dt, 1, sm);
  else split_body<N, NS, VF, GEN, false, AFF>(M.g, M.ph, tab, e, valid, t, M.U, M.out, M.R, M.a, M.b, M.dt, 1, sm);
}

template <int N, bool NS, int VF, int EPB, bool GEN, int AFF>
__global__ void __launch_bounds__((line_lanes<N, ends_always(N)>()) * EPB, (split_minb(N, VF, AFF == AFF_ALL))) k_split_b(BatchView bv) {
  constexpr bool ENDS = ends_always(N);
  constexpr int NT = line_lanes<N, ENDS>(), L = SplitLds<N>::template size<VF, AFF == AFF_ALL, ENDS>();
  __shared__ double sm[EPB * L];
  const BatchBlock B = batch_block(bv, EPB, blockIdx.x);
  if (B.item >= B.end) return;
  const int slot = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  const int t = threadIdx.x - slot * NT;
  const int item = B.item + slot;
  const bool valid = item < B.end;
  const int mi = member_of(bv.first, bv.count, valid ? item : B.end - 1);
  const Member &M = bv.m[mi];
  const int e = valid ? item - bv.first[mi] : 0;
  if (AFF == AFF_ALL || (AFF == AFF_MIXED && B.affine))
    split_member<N, NS, VF, GEN, true>(M, bv.tab, e, valid, t, sm + slot * L);
  else
    split_member<N, NS, VF, GEN, false>(M, bv.tab, e, valid, t, sm + slot * L);
}

// ----------------------------------------------------------------------------- reductions
// WHAT RED_TIMESTEP -> {max sum lambda_c, max sum lambda_v}; RED_INTEGRALS -> {rho, m1, m2, m3, E, KE,
// entropy, min J}; RED_FINITE -> {count of non-finite}
template <int WHAT> struct Red {
  static constexpr int NC = WHAT == RED_TIMESTEP ? 2 : (WHAT == RED_INTEGRALS ? 8 : 1);
  static __device__ __forceinline__ double init(int c) { return WHAT == RED_INTEGRALS && c == 7 ? 1e300 : 0.0; }
  static __device__ __forceinline__ double join(int c, double x, double y) {
    if (WHAT == RED_TIMESTEP) return fmax(x, y);
    if (WHAT == RED_INTEGRALS && c == 7) return fmin(x, y);
    return x + y;
  }
  // every lane's val joined over the workgroup of NT lanes (a fixed butterfly per wave, then the waves in
  // order); the result in lane 0.  sm: NC NT / 64 doubles.
  template <int NT> static __device__ __forceinline__ void workgroup(double *val, double *sm) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) val[c] = join(c, val[c], __shfl_xor(val[c], off, 64));
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) sm[w * NC + c] = val[c];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int v = 1; v < NT / 64; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c) val[c] = join(c, val[c], sm[v * NC + c]);
    }
  }
};

// A fixed number of workgroups walk the nodes of the whole mesh and leave one row of partial results each.
// One workgroup per element, its eight components folded through LDS, took 17 us for 885 k nodes (N = 5,
// 42 MB of state) and left 4096 rows to the last kernel, 12 us more; now 6 (finiteness), 16 (integrals) and 19
// (time step, which reads the metric terms), and 3 to 8 for the last kernel.
template <int N, int WHAT>
__global__ void __launch_bounds__(256) k_reduce(Geo g, Phys ph, const double *__restrict__ U,
                                                double *__restrict__ partial) {
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n, NC = Red<WHAT>::NC;
  __shared__ double sm[4 * NC];
  const double gm1 = ph.gamma - 1.0;
  double val[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) val[c] = Red<WHAT>::init(c);
  const unsigned total = (unsigned)g.K * n3, step = gridDim.x * 256u;  // fewer than 2^31 nodes
  for (unsigned q = blockIdx.x * 256u + threadIdx.x; q < total; q += step) {
    const int e = q / n3, t = q - e * n3;
    double Uq[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = U[((size_t)e * 5 + v) * n3 + t];
    if constexpr (WHAT == RED_FINITE) {
      double bad = 0.0;
#pragma unroll
      for (int v = 0; v < 5; ++v) bad += isfinite(Uq[v]) ? 0.0 : 1.0;
      val[0] += bad;
    } else if constexpr (WHAT == RED_TIMESTEP) {
      // the metric terms per node, or the element's constants
      const double *Jd = g.Jc ? g.Jc + (size_t)e * AFFINE_DOUBLES : g.Ja + (size_t)e * 9 * n3 + t;
      const int js = g.Jc ? 1 : n3;
      const double sj = g.Jc ? Jd[9] : g.sJ[(size_t)e * n3 + t];
      const Pr5 P = to_prim(Uq, gm1);
      const double c = sqrt(ph.gamma * P.p / P.rho);
      double sc = 0.0, sv = 0.0;
#pragma unroll
      for (int dir = 0; dir < 3; ++dir) {
        const double a0 = Jd[(3 * dir) * js], a1 = Jd[(3 * dir + 1) * js], a2 = Jd[(3 * dir + 2) * js];
        const double nn = a0 * a0 + a1 * a1 + a2 * a2;
        sc += (fabs(P.u * a0 + P.v * a1 + P.w * a2) + c * sqrt(nn)) * sj;
        sv += fmax(4.0 / 3.0, ph.gamma / ph.Pr) * (ph.mu / P.rho) * nn * sj * sj;
      }
      val[0] = fmax(val[0], sc);
      val[1] = fmax(val[1], sv);
    } else {
      const double sj = g.sJ[(size_t)e * n3 + t];
      const Pr5 P = to_prim(Uq, gm1);
      const int i = t % n, j = (t / n) % n, k = t / n2;
      const double wq = g.tab->w[i] * g.tab->w[j] * g.tab->w[k] / sj;
#pragma unroll
      for (int v = 0; v < 5; ++v) val[v] += wq * Uq[v];
      val[5] += wq * 0.5 * (Uq[1] * P.u + Uq[2] * P.v + Uq[3] * P.w);
      const double s = log(P.p) - ph.gamma * log(P.rho);
      val[6] += wq * (-P.rho * s / gm1);
      val[7] = fmin(val[7], 1.0 / sj);
    }
  }
  Red<WHAT>::template workgroup<256>(val, sm);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) partial[(size_t)blockIdx.x * NC + c] = val[c];
  }
}

// ----------------------------------------------------------------------------- mortars
// Non-conforming faces (Sec. 3.2), one workgroup per face: the big side's traces are
// interpolated to every small side's points (I^L or I^U along each cut face direction), the
// small side's term is evaluated there with the small element's own outward normal and written to
// its face-array slot, and projected back to the big side (P^L, P^U; negated: outward of the big
// element).  The element kernels read these slots for the sides their face codes mark.

// value of the nv-component field X ([e][nv][n^3]) at face point (a,b) of side s of element e:
// the face node on LGL nodes, interpolated along the face normal with l(+-1) on LG nodes
template <int n, bool LGL, int NV>
__device__ __forceinline__ void face_trace(const double *__restrict__ X, int e, int s, int a, int b,
                                           const double *lm, const double *lp, double *out) {
  constexpr int n3 = n * n * n;
  const int dn = s >> 1;
  const bool plus = s & 1;
  const double *Xe = X + (size_t)e * NV * n3;
  if (LGL) {
    const int q = line_node<n>(dn, a, b, plus ? n - 1 : 0);
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = Xe[v * n3 + q];
  } else {
    const double *l = plus ? lp : lm;
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = 0.0;
#pragma unroll 1
    for (int m = 0; m < n; ++m) {
      const int q = line_node<n>(dn, a, b, m);
#pragma unroll
      for (int v = 0; v < NV; ++v) out[v] += l[m] * Xe[v * n3 + q];
    }
  }
}

// lifted variables W = (u, v, w, T) at face point (a,b) of side s of element e: W of the face
// node on LGL nodes; on LG nodes W at every node of the line, interpolated with l(+-1) (as the
// conforming lifting does)
template <int n, bool LGL>
__device__ __forceinline__ void face_trace_W(const double *__restrict__ U, int e, int s, int a, int b,
                                             const double *lm, const double *lp, double gm1, double Rg, double *W) {
  constexpr int n3 = n * n * n;
  const int dn = s >> 1;
  const bool plus = s & 1;
  const double *Ue = U + (size_t)e * 5 * n3;
  double Uq[5];
  if (LGL) {
    const int q = line_node<n>(dn, a, b, plus ? n - 1 : 0);
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = Ue[v * n3 + q];
    grad_prim_to_W(Uq, gm1, Rg, W);
    return;
  }
  const double *l = plus ? lp : lm;
#pragma unroll
  for (int v = 0; v < 4; ++v) W[v] = 0.0;
  for (int m = 0; m < n; ++m) {
    const int q = line_node<n>(dn, a, b, m);
    double Wq[4];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = Ue[v * n3 + q];
    grad_prim_to_W(Uq, gm1, Rg, Wq);
#pragma unroll
    for (int v = 0; v < 4; ++v) W[v] += l[m] * Wq[v];
  }
}

// face point of the big side's sub-face that small-side point (a,b) meets (orientation code o:
// swap if o & 4, then reverse the first index if o & 1, the second if o & 2)
template <int n> __device__ __forceinline__ void sub_point(int o, int a, int b, int &a2, int &b2) {
  const int p = (o & 4) ? b : a, q = (o & 4) ? a : b;
  a2 = (o & 1) ? n - 1 - p : p;
  b2 = (o & 2) ? n - 1 - q : q;
}

// Lanes of one mortar's workgroup: one per point of up to four small sides.
template <int N> struct MortarSz {
  static constexpr int n2 = (N + 1) * (N + 1), NT = (4 * n2 + 63) / 64 * 64;
};

// A mortar's big side is cut into na parts along its first face direction and nb along its second; small
// side pos = p1 + na p2.  Interpolation to the small sides and projection back are applied one face
// direction at a time (n products a value instead of n^2), all components of all points spread over the
// lanes: a mesh has few such faces, so the chain of one workgroup's steps is what the kernels wait on.  One
// rolled n^2 sum per point and lane (64 lanes for the projection) took 72 us (fluxes) and 64 us (lifting) a
// launch for 128 faces at N = 7; now 11 and 10 us.
// sM = [IL | IU | PL | PU].

// first direction of the interpolation: T[(p1 NV + v) n^2 + i + n l] = sum_m I_p1[i][m] X[v][m + n l]
template <int n, int NV>
__device__ __forceinline__ void mortar_interp_a(const double *sM, int type, int na, const double *X, double *T, int t,
                                                int nth) {
  constexpr int n2 = n * n;
  for (int q = t; q < na * NV * n2; q += nth) {
    const int p1 = q / (NV * n2), r = q - p1 * NV * n2, pt = r % n2, i = pt % n, l = pt / n;
    if (type & 1) {
      const double *M = sM + p1 * n2 + i * n, *x = X + (r - pt) + n * l;
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < n; ++m) s += M[m] * x[m];
      T[q] = s;
    } else {
      T[q] = X[r];
    }
  }
}
// second direction, at the sub-face point (a2, b2) of small side pos: out[v], v < NV
template <int n, int NV>
__device__ __forceinline__ void mortar_interp_b(const double *sM, int type, int na, int pos, int a2, int b2,
                                                const double *T, double *out) {
  constexpr int n2 = n * n;
  const int p1 = pos % na, p2 = pos / na;
  const double *x = T + p1 * NV * n2 + a2, *M = sM + p2 * n2 + b2 * n;
#pragma unroll
  for (int v = 0; v < NV; ++v) out[v] = 0.0;
  if (type & 2) {
#pragma unroll 4
    for (int l = 0; l < n; ++l) {
#pragma unroll
      for (int v = 0; v < NV; ++v) out[v] += M[l] * x[v * n2 + n * l];
    }
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = x[v * n2 + n * b2];
  }
}
// projection of the small sides' NC values X[(pos NC + c) n^2 + a2 + n b2] onto the big side, negated
// (outward of the big element), into out[c n^2 + i + n j]; Y: 2 NC n^2 doubles of scratch
template <int n, int NC>
__device__ __forceinline__ void mortar_project(const double *sM, int type, int na, int nb, const double *X, double *Y,
                                               double *__restrict__ out, int t, int nth) {
  constexpr int n2 = n * n;
  for (int q = t; q < nb * NC * n2; q += nth) {
    const int p2 = q / (NC * n2), r = q - p2 * NC * n2, pt = r % n2, i = pt % n, l = pt / n;
    double s = 0.0;
    if (type & 1) {
#pragma unroll
      for (int p1 = 0; p1 < 2; ++p1) {
        const double *M = sM + (2 + p1) * n2 + i * n, *x = X + (p1 + 2 * p2) * NC * n2 + (r - pt) + n * l;
#pragma unroll
        for (int m = 0; m < n; ++m) s += M[m] * x[m];
      }
    } else {
      s = X[p2 * NC * n2 + r];
    }
    Y[q] = s;
  }
  __syncthreads();
  for (int q = t; q < NC * n2; q += nth) {
    const int pt = q % n2, i = pt % n, j = pt / n;
    double s = 0.0;
    if (type & 2) {
#pragma unroll
      for (int p2 = 0; p2 < 2; ++p2) {
        const double *M = sM + (2 + p2) * n2 + j * n, *y = Y + p2 * NC * n2 + (q - pt) + i;
#pragma unroll
        for (int l = 0; l < n; ++l) s += M[l] * y[n * l];
      }
    } else {
      s = Y[q];
    }
    out[q] = -s;
  }
}

template <int N, bool LGL>
__global__ void __launch_bounds__(MortarSz<N>::NT) k_mortar_lift(Geo g, Phys ph, const MortarDesc *__restrict__ md,
                                                                 const double *__restrict__ U) {
  constexpr int n = N + 1, n2 = n * n, NT = MortarSz<N>::NT;
  __shared__ double sM[4 * n2];       // IL, IU, PL, PU
  __shared__ double sWB[4 * n2];      // W = (u, v, w, T) of the big side's trace
  __shared__ double sTa[2 * 12 * n2]; // interpolated along the first direction; then the projection's scratch
  __shared__ double sT[4 * 12 * n2];  // the small sides' surface terms at their sub-face points
  const int t = threadIdx.x;
  const Tab *tb = g.tab;
  const MortarDesc &m = md[blockIdx.x];  // read in place: its arrays are indexed by sub-face
  const int type = m.type, na = (type & 1) ? 2 : 1, nb = (type & 2) ? 2 : 1, cnt = na * nb;
  const double gm1 = ph.gamma - 1.0;
  // this lane's point of a small side: its trace and normal are loaded before the first barrier
  const bool act = t < cnt * n2;
  const int pos = act ? t / n2 : 0, ab = t - pos * n2, a = ab % n, b = ab / n;
  const int es = m.es[pos], ss = m.ss[pos];
  double Ws[4], nt[3];
  if (act) {
    face_trace_W<n, LGL>(U, es, ss, a, b, tb->lm, tb->lp, gm1, ph.R, Ws);
    const double *fnp = g.fn + ((size_t)es * 6 + ss) * 3 * n2 + ab;
    nt[0] = fnp[0]; nt[1] = fnp[n2]; nt[2] = fnp[2 * n2];
  }
  for (int c = t; c < n2; c += NT) {
    sM[c] = tb->IL[c]; sM[n2 + c] = tb->IU[c]; sM[2 * n2 + c] = tb->PL[c]; sM[3 * n2 + c] = tb->PU[c];
  }
  if (t < n2) {
    double W[4];
    face_trace_W<n, LGL>(U, m.eb, m.sb, t % n, t / n, tb->lm, tb->lp, gm1, ph.R, W);
#pragma unroll
    for (int v = 0; v < 4; ++v) sWB[v * n2 + t] = W[v];
  }
  __syncthreads();
  mortar_interp_a<n, 4>(sM, type, na, sWB, sTa, t, NT);
  __syncthreads();
  if (act) {
    int a2, b2;
    sub_point<n>(m.o[pos], a, b, a2, b2);
    double WB[4];
    mortar_interp_b<n, 4>(sM, type, na, pos, a2, b2, sTa, WB);
    double *ml = g.mlift + (size_t)m.sl[pos] * 12 * n2 + ab;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double tv = nt[d] * (0.5 * (Ws[v] + WB[v]));
        ml[(d * 4 + v) * n2] = tv;
        sT[(pos * 12 + d * 4 + v) * n2 + a2 + n * b2] = tv;
      }
  }
  __syncthreads();
  mortar_project<n, 12>(sM, type, na, nb, sT, sTa, g.mlift + (size_t)m.slot * 12 * n2, t, NT);
}

// G: the lifted gradients [K][12][n^3] (read on LG nodes); on LGL nodes the gradients at the
// mortar sides' points come from Geo::mg, written by the lifting kernel
template <int N, bool LGL, bool NS>
__global__ void __launch_bounds__(MortarSz<N>::NT) k_mortar_flux(Geo g, Phys ph, const MortarDesc *__restrict__ md,
                                                                 const double *__restrict__ U,
                                                                 const double *__restrict__ G) {
  constexpr int n = N + 1, n2 = n * n, NT = MortarSz<N>::NT, NV = NS ? 17 : 5;
  __shared__ double sM[4 * n2];
  __shared__ double sB[NV * n2];       // the big side's trace: U (5), for Navier-Stokes the gradients (12)
  __shared__ double sTa[2 * NV * n2];  // interpolated along the first direction; then the projection's scratch
  __shared__ double sF[4 * 5 * n2];    // the small sides' fluxes at their sub-face points
  const int t = threadIdx.x;
  const Tab *tb = g.tab;
  const MortarDesc &m = md[blockIdx.x];  // read in place: its arrays are indexed by sub-face
  const int type = m.type, na = (type & 1) ? 2 : 1, nb = (type & 2) ? 2 : 1, cnt = na * nb;
  const double gm1 = ph.gamma - 1.0;
  // this lane's point of a small side, the master of its part of the face: its own trace and normal are
  // loaded before the first barrier
  const bool act = t < cnt * n2;
  const int pos = act ? t / n2 : 0, ab = t - pos * n2, a = ab % n, b = ab / n;
  const int es = m.es[pos], ss = m.ss[pos];
  double UM[5], gM[12], nt[3];
  if (act) {
    face_trace<n, LGL, 5>(U, es, ss, a, b, tb->lm, tb->lp, UM);
    if (NS && LGL) {
      const double *mg = g.mg + (size_t)m.sl[pos] * 12 * n2 + ab;
#pragma unroll
      for (int c = 0; c < 12; ++c) gM[c] = mg[c * n2];
    } else if (NS) {
      face_trace<n, false, 12>(G, es, ss, a, b, tb->lm, tb->lp, gM);
    }
    const double *fnp = g.fn + ((size_t)es * 6 + ss) * 3 * n2 + ab;
    nt[0] = fnp[0]; nt[1] = fnp[n2]; nt[2] = fnp[2 * n2];
  }
  for (int c = t; c < n2; c += NT) {
    sM[c] = tb->IL[c]; sM[n2 + c] = tb->IU[c]; sM[2 * n2 + c] = tb->PL[c]; sM[3 * n2 + c] = tb->PU[c];
  }
  if (t < n2) {
    double Uq[5];
    face_trace<n, LGL, 5>(U, m.eb, m.sb, t % n, t / n, tb->lm, tb->lp, Uq);
#pragma unroll
    for (int v = 0; v < 5; ++v) sB[v * n2 + t] = Uq[v];
    if (NS) {
      double gq[12];
      if (LGL) {
        const double *mg = g.mg + (size_t)m.slot * 12 * n2 + t;
#pragma unroll
        for (int c = 0; c < 12; ++c) gq[c] = mg[c * n2];
      } else {
        face_trace<n, false, 12>(G, m.eb, m.sb, t % n, t / n, tb->lm, tb->lp, gq);
      }
#pragma unroll
      for (int c = 0; c < 12; ++c) sB[(5 + c) * n2 + t] = gq[c];
    }
  }
  __syncthreads();
  mortar_interp_a<n, NV>(sM, type, na, sB, sTa, t, NT);
  __syncthreads();
  if (act) {
    int a2, b2;
    sub_point<n>(m.o[pos], a, b, a2, b2);
    double XS[NV];  // the big side's state (and gradients) at this point
    mortar_interp_b<n, NV>(sM, type, na, pos, a2, b2, sTa, XS);
    const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    const double ish = 1.0 / sh;
    const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
    double F[5];
    riemann(ph, UM, XS, nh, F);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] *= sh;
    if constexpr (NS) {
      // BR1: mean of the two sides' viscous fluxes, the big side's state and gradients interpolated
      double FvM[5], FvS[5];
      flux_v(to_prim(UM, gm1), gM, ph, nt, FvM);
      flux_v(to_prim(XS, gm1), XS + 5, ph, nt, FvS);
#pragma unroll
      for (int v = 0; v < 5; ++v) F[v] -= 0.5 * (FvM[v] + FvS[v]);
    }
    double *mf = g.mflux + (size_t)m.sl[pos] * 5 * n2 + ab;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      mf[v * n2] = F[v];
      sF[(pos * 5 + v) * n2 + a2 + n * b2] = F[v];
    }
  }
  __syncthreads();
  mortar_project<n, 5>(sM, type, na, nb, sF, sTa, g.mflux + (size_t)m.slot * 5 * n2, t, NT);
}

// ----------------------------------------------------------------------------- FV subcells
// Shock capturing with finite volumes on (N+1)^3 equal subcells of each troubled element (Sec. 4):
// the element's U then holds subcell means; V = V_DG=>FV converts (eq. FVvdm, dg2fv).  Euler
// equations, conforming meshes without boundary sides.

__device__ __forceinline__ double fv_limit(int lim, double a, double b) {
  if (lim == 0 || a * b <= 0.0) return 0.0;
  if (lim == 1) return fabs(a) < fabs(b) ? a : b;  // minmod
  return 2.0 * a * b / (a + b);                   // van Leer
}
__device__ __forceinline__ void fv_prim(const double *U, double gm1, double *W) {
  const double ir = 1.0 / U[0];
  W[0] = U[0]; W[1] = U[1] * ir; W[2] = U[2] * ir; W[3] = U[3] * ir;
  W[4] = gm1 * (U[4] - 0.5 * U[0] * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]));
}
__device__ __forceinline__ void fv_cons(const double *W, double gm1, double *U) {
  U[0] = W[0]; U[1] = W[0] * W[1]; U[2] = W[0] * W[2]; U[3] = W[0] * W[3];
  U[4] = W[4] / gm1 + 0.5 * W[0] * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]);
}

// reconstructed state of finite-volume element e at its boundary subface (a,b) of side s: the
// limited slope of the adjacent subcell from the next inner subcell and the outer datum Do
template <int n>
__device__ __forceinline__ void fv_recon(const double *__restrict__ U, const FvGeo &f, double gm1, int e, int s, int a,
                                         int b, const double *Do, double *Uf) {
  constexpr int n3 = n * n * n;
  const int dn = s >> 1;
  const bool plus = s & 1;
  const double *Ue = U + (size_t)e * 5 * n3;
  const int q0 = line_node<n>(dn, a, b, plus ? n - 1 : 0), q1 = line_node<n>(dn, a, b, plus ? n - 2 : 1);
  double U0[5], U1[5], W0[5], W1[5], Wo[5], Wf[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) { U0[v] = Ue[v * n3 + q0]; U1[v] = Ue[v * n3 + q1]; }
  fv_prim(U0, gm1, W0);
  fv_prim(U1, gm1, W1);
  fv_prim(Do, gm1, Wo);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double sm = plus ? W0[v] - W1[v] : W0[v] - Wo[v];
    const double sp = plus ? Wo[v] - W0[v] : W1[v] - W0[v];
    const double sg = fv_limit(f.limiter, sm, sp);
    Wf[v] = plus ? W0[v] + 0.5 * sg : W0[v] - 0.5 * sg;
  }
  fv_cons(Wf, gm1, Uf);
}

// (M x M) applied at face point (a,b) of a face field T[v][ia + n jb] (5 fields): sum over jb of
// M[b][jb] (sum over ia of M[a][ia] T[ia + n jb])
template <int n>
__device__ __forceinline__ void face_mm(const double *M, int a, int b, const double *T, double *out) {
  constexpr int n2 = n * n;
  double r[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int jb = 0; jb < n; ++jb) {
    double c[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ia = 0; ia < n; ++ia) {
      const double m = M[a * n + ia];
#pragma unroll
      for (int v = 0; v < 5; ++v) c[v] += m * T[v * n2 + ia + n * jb];
    }
    const double m2 = M[b * n + jb];
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] += m2 * c[v];
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) out[v] = r[v];
}

// Work lists of the hybrid operator, rebuilt whenever the element types change: the finite-volume
// elements (count[0] of them in list) and the master sides e*6+s of the faces that touch one
// (count[1] in faces).  The order of either list is arbitrary: every item writes only its own
// outputs.
template <int N> __global__ void k_fv_lists_zero(FvGeo f) {
  if (threadIdx.x == 0) { f.count[0] = 0; f.count[1] = 0; }
}

template <int N, bool GEN>
__global__ void __launch_bounds__(256) k_fv_lists(Geo g, FvGeo f) {
  constexpr int n = N + 1;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (q >= 6 * g.K) return;
  const int e = q / 6, s = q - 6 * e;
  if (s == 0 && f.flag[e]) f.list[atomicAdd(&f.count[0], 1)] = e;
  const int nb = g.nbr[q];
  if (nb < 0) return;
  const NbFace f0 = nbr_face<n, (GEN > 0)>(g, e, s, 0, 0);
  if (f0.master && (f.flag[e] || f.flag[nb])) f.faces[atomicAdd(&f.count[1], 1)] = q;
}

template <int N> struct FvFaceSz {
  static constexpr int NT = ((N + 1) * (N + 1) + 63) / 64 * 64;  // threads: one face point each
};

// Faces that touch a finite-volume element, one workgroup per face of the work list (looping over
// it): the numerical flux at the (N+1)^2 subfaces from both sides' face data (the DG side's trace
// taken to subface means with V in both face directions, the FV side reconstructed); writes both
// sides' outward fluxes (a DG side's back to its face nodes with V^-1) and both sides' view of the
// other's face datum.
template <int N, bool LGL, bool GEN>
__global__ void __launch_bounds__(FvFaceSz<N>::NT) k_fv_face(Geo g, Phys ph, FvGeo f, const double *__restrict__ U) {
  constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  __shared__ double sV[n * n], sVi[n * n];
  __shared__ double sTe[5 * n2], sTn[5 * n2];  // DG traces (own / neighbour face coordinates)
  __shared__ double sFe[5 * n2], sFn[5 * n2];  // outward subface fluxes of both sides
  const int t = threadIdx.x;
  for (int c = t; c < n * n; c += blockDim.x) { sV[c] = f.V[c]; sVi[c] = f.Vi[c]; }
  const int nf = f.count[1];
  const double gm1 = ph.gamma - 1.0;
  const Tab *tb = g.tab;
  const bool pt = t < n2;
  const int a = pt ? t % n : 0, b = pt ? t / n : 0;
  for (int it = blockIdx.x; it < nf; it += gridDim.x) {
    const int q = f.faces[it], e = q / 6, s = q - 6 * e;
    const int nb = g.nbr[q];
    const NbFace fm = nbr_face<n, (GEN > 0)>(g, e, s, a, b);
    const int ns = GEN ? 2 * fm.dn + (fm.plus ? 1 : 0) : (s ^ 1);
    const int a2 = fm.a, b2 = fm.b;
    const bool fe = f.flag[e], fn = f.flag[nb];
    __syncthreads();  // the previous face's reads of the LDS fields are done
    if (pt) {
      double tr[5];
      if (!fe) {
        face_trace<n, LGL, 5>(U, e, s, a, b, tb->lm, tb->lp, tr);
#pragma unroll
        for (int v = 0; v < 5; ++v) sTe[v * n2 + t] = tr[v];
      }
      if (!fn) {
        face_trace<n, LGL, 5>(U, nb, ns, a2, b2, tb->lm, tb->lp, tr);
#pragma unroll
        for (int v = 0; v < 5; ++v) sTn[v * n2 + a2 + n * b2] = tr[v];
      }
    }
    __syncthreads();
    if (pt) {
      // face data: the adjacent subcell (FV) or the subface mean of the trace (DG)
      double De[5], Dn[5], Ue[5], Un[5];
      if (fe) {
        const int qe = line_node<n>(s >> 1, a, b, (s & 1) ? n - 1 : 0);
#pragma unroll
        for (int v = 0; v < 5; ++v) De[v] = U[((size_t)e * 5 + v) * n3 + qe];
      } else {
        face_mm<n>(sV, a, b, sTe, De);
      }
      if (fn) {
        const int qn = line_node<n>(ns >> 1, a2, b2, (ns & 1) ? n - 1 : 0);
#pragma unroll
        for (int v = 0; v < 5; ++v) Dn[v] = U[((size_t)nb * 5 + v) * n3 + qn];
      } else {
        face_mm<n>(sV, a2, b2, sTn, Dn);
      }
      double *dxe = f.Dx + ((size_t)e * 6 + s) * 5 * n2 + t;
      double *dxn = f.Dx + ((size_t)nb * 6 + ns) * 5 * n2 + a2 + n * b2;
#pragma unroll
      for (int v = 0; v < 5; ++v) { dxe[v * n2] = Dn[v]; dxn[v * n2] = De[v]; }
      if (fe) {
        fv_recon<n>(U, f, gm1, e, s, a, b, Dn, Ue);
      } else {
#pragma unroll
        for (int v = 0; v < 5; ++v) Ue[v] = De[v];
      }
      if (fn) {
        fv_recon<n>(U, f, gm1, nb, ns, a2, b2, De, Un);
      } else {
#pragma unroll
        for (int v = 0; v < 5; ++v) Un[v] = Dn[v];
      }
      // the master's (this side's) face-mean metric, outward
      const bool plus = s & 1;
      const double *Nm = f.Nf + ((((size_t)e * 3 + (s >> 1)) * (n + 1) + (plus ? n : 0)) * n2 + t) * 3;
      const double sgn = plus ? 1.0 : -1.0;
      const double nt[3] = {sgn * Nm[0], sgn * Nm[1], sgn * Nm[2]};
      const double sh = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
      const double ish = 1.0 / sh;
      const double nh[3] = {nt[0] * ish, nt[1] * ish, nt[2] * ish};
      double F[5];
      riemann(ph, Ue, Un, nh, F);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        sFe[v * n2 + t] = sh * F[v];
        sFn[v * n2 + a2 + n * b2] = -(sh * F[v]);
      }
    }
    __syncthreads();
    if (pt) {
      // thread t writes point t of either side (in that side's own face coordinates)
      double o[5];
      double *fx = f.Fx + ((size_t)e * 6 + s) * 5 * n2 + t;
      if (fe) {
#pragma unroll
        for (int v = 0; v < 5; ++v) o[v] = sFe[v * n2 + t];
      } else {
        face_mm<n>(sVi, a, b, sFe, o);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) fx[v * n2] = o[v];
      fx = f.Fx + ((size_t)nb * 6 + ns) * 5 * n2 + t;
      if (fn) {
#pragma unroll
        for (int v = 0; v < 5; ++v) o[v] = sFn[v * n2 + t];
      } else {
        face_mm<n>(sVi, a, b, sFn, o);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) fx[v * n2] = o[v];
    }
  }
}

// Finite-volume elements of the work list, one workgroup per element (looping over the list):
// second-order subcell update, eq. fv_dof_time_derivative.
template <int N, int MODE, int RS>
__global__ void __launch_bounds__(Sz<N>::NT, 4) k_fv_volume(Geo g, Phys ph, FvGeo f, const double *__restrict__ U,
                                                         double *__restrict__ out, double *__restrict__ R, double ca,
                                                         double cb, double dt) {
  using S = Sz<N>;
  constexpr int n = S::n, n2 = S::n2, n3 = S::n3;
  __shared__ double sW[5 * n3];  // primitive subcell means
  __shared__ double sF[5 * n3];  // flux through each subcell's + face (inner faces)
  const int t = threadIdx.x;
  const bool act = t < n3;
  const double gm1 = ph.gamma - 1.0;
  const int nfv = f.count[0];
  for (int it = blockIdx.x; it < nfv; it += gridDim.x) {
    const int e = f.list[it];
    __syncthreads();  // the previous element's reads of the LDS fields are done
    if (act) {
      double Uo[5], W[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) Uo[v] = U[((size_t)e * 5 + v) * n3 + t];
      fv_prim(Uo, gm1, W);
#pragma unroll
      for (int v = 0; v < 5; ++v) sW[v * n3 + t] = W[v];
    }
    const int id3[3] = {t % n, (t / n) % n, t / n2};
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int dir = 0; dir < 3; ++dir) {
      __syncthreads();  // sW is complete; the previous direction's reads of sF are done
      const int id = act ? id3[dir] : 0;
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int a = dir == 0 ? id3[1] : id3[0], b = dir == 2 ? id3[1] : id3[2];
      const int ab = a + n * b;
      if (act && id < N) {
        // inner face id + 1/2 between subcells c0 = id and c1 = id + 1 along dir: the two
        // reconstructed states from the stencil c0 - 1 .. c1 + 1, whose ends beyond the element
        // are the outer face data of its sides
        double Wm[5], Wp[5];
        if (id > 0) {
#pragma unroll
          for (int v = 0; v < 5; ++v) Wm[v] = sW[v * n3 + t - str];
        } else {
          double Do[5];
          const double *dx = f.Dx + ((size_t)e * 6 + 2 * dir) * 5 * n2 + ab;
#pragma unroll
          for (int v = 0; v < 5; ++v) Do[v] = dx[v * n2];
          fv_prim(Do, gm1, Wm);
        }
        if (id + 1 < N) {
#pragma unroll
          for (int v = 0; v < 5; ++v) Wp[v] = sW[v * n3 + t + 2 * str];
        } else {
          double Do[5];
          const double *dx = f.Dx + ((size_t)e * 6 + 2 * dir + 1) * 5 * n2 + ab;
#pragma unroll
          for (int v = 0; v < 5; ++v) Do[v] = dx[v * n2];
          fv_prim(Do, gm1, Wp);
        }
        double UL[5], UR[5];
        {
          double WL[5], WR[5];
#pragma unroll
          for (int v = 0; v < 5; ++v) {
            const double w0 = sW[v * n3 + t], w1 = sW[v * n3 + t + str];
            WL[v] = w0 + 0.5 * fv_limit(f.limiter, w0 - Wm[v], w1 - w0);
            WR[v] = w1 - 0.5 * fv_limit(f.limiter, w1 - w0, Wp[v] - w1);
          }
          fv_cons(WL, gm1, UL);
          fv_cons(WR, gm1, UR);
        }
        const double *Nm = f.Nf + ((((size_t)e * 3 + dir) * (n + 1) + id + 1) * n2 + ab) * 3;
        const double sh = sqrt(Nm[0] * Nm[0] + Nm[1] * Nm[1] + Nm[2] * Nm[2]);
        const double ish = 1.0 / sh;
        const double nh[3] = {Nm[0] * ish, Nm[1] * ish, Nm[2] * ish};
        double F[5];
        riemann_t<RS>(ph, UL, UR, nh, F);
        // the subcell's outward flux on its + face; the next subcell's - face reads it from sF
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double fp = sh * F[v];
          sF[v * n3 + t] = fp;
          acc[v] += fp;
        }
      }
      __syncthreads();
      if (act) {
        const double *fx0 = f.Fx + ((size_t)e * 6 + 2 * dir) * 5 * n2 + ab;
        const double *fx1 = f.Fx + ((size_t)e * 6 + 2 * dir + 1) * 5 * n2 + ab;
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          // outward fluxes of the subcell: + face (above for inner faces), then - face
          if (id == N) acc[v] += fx1[v * n2];
          acc[v] += (id > 0) ? -sF[v * n3 + t - str] : fx0[v * n2];
        }
      }
    }
    if (act) {
      const double iwj = 1.0 / (f.w * f.Jbar[(size_t)e * n3 + t]);
      double *Oe = out + (size_t)e * 5 * n3;
      if (MODE == 0) {
#pragma unroll
        for (int v = 0; v < 5; ++v) Oe[v * n3 + t] = -acc[v] * iwj;
      } else {
        double *Re = R + (size_t)e * 5 * n3;
        const double *Ue = U + (size_t)e * 5 * n3;  // read again (from L2) rather than held
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const double r = (ca != 0.0 ? ca * Re[v * n3 + t] : 0.0) + dt * (-acc[v] * iwj);
          Re[v * n3 + t] = r;
          Oe[v * n3 + t] = Ue[v * n3 + t] + cb * r;
        }
      }
    }
  }
}

// apply the n x n matrix A along all three directions to the 5 fields of sX (in place through sY)
template <int n, int NV = 5>
__device__ __forceinline__ void fv_tensor3(const double *A, double *sX, int t, bool act) {
  constexpr int n2 = n * n, n3 = n2 * n;
  const int i = t % n, j = (t / n) % n, k = t / n2;
  for (int dir = 0; dir < 3; ++dir) {
    double r[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) r[v] = 0.0;
    if (act) {
      const int id = dir == 0 ? i : (dir == 1 ? j : k);
      const int str = dir == 0 ? 1 : (dir == 1 ? n : n2);
      const int base = t - id * str;
      for (int m = 0; m < n; ++m) {
        const double c = A[id * n + m];
#pragma unroll
        for (int v = 0; v < NV; ++v) r[v] += c * sX[v * n3 + base + m * str];
      }
    }
    __syncthreads();  // every line is read before any node is overwritten
    if (act) {
#pragma unroll
      for (int v = 0; v < NV; ++v) sX[v * n3 + t] = r[v];
    }
    __syncthreads();
  }
}

// troubled-cell indicator (modal decay of rho p) and, with do_switch, the switch with hysteresis in
// place (U <- V U to finite volume above hi, U <- V^-1 U back to DG below lo)
template <int N>
__global__ void __launch_bounds__(Sz<N>::NT) k_fv_switch(Geo g, Phys ph, FvGeo f, double *__restrict__ U,
                                                         int do_switch) {
  using S = Sz<N>;
  constexpr int n = S::n, n3 = S::n3;
  __shared__ double sX[5 * n3], sU[5 * n3];
  __shared__ double sA[3 * n * n];  // V, Vi, Li
  __shared__ double sE[3 * (Sz<N>::NT / 64)];
  __shared__ int sNew;
  const int e = blockIdx.x, t = threadIdx.x;
  const bool act = t < n3;
  for (int c = t; c < n * n; c += blockDim.x) { sA[c] = f.V[c]; sA[n * n + c] = f.Vi[c]; sA[2 * n * n + c] = f.Li[c]; }
  const bool isfv = f.flag[e];
  if (act) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double u = U[((size_t)e * 5 + v) * n3 + t];
      sU[v * n3 + t] = u;
      sX[v * n3 + t] = u;
    }
  }
  __syncthreads();
  if (isfv) fv_tensor3<n>(sA + n * n, sX, t, act);  // nodal values of the element's DG reading
  if (act) {
    double W[5], Uq[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Uq[v] = sX[v * n3 + t];
    fv_prim(Uq, ph.gamma - 1.0, W);
    sX[t] = W[0] * W[4];  // q = rho p in field 0
  }
  __syncthreads();
  fv_tensor3<n, 1>(sA + 2 * n * n, sX, t, act);  // modal coefficients (field 0)
  {
    // energies: of all modes, of those whose largest index is N, of those whose largest index is
    // N-1; summed per wave by a fixed butterfly, then over the waves in order
    double E3[3] = {0.0, 0.0, 0.0};
    if (act) {
      const int i = t % n, j = (t / n) % n, k = t / (n * n);
      const int m = i > j ? (i > k ? i : k) : (j > k ? j : k);
      const double c2 = sX[t] * sX[t];
      E3[0] = c2;
      E3[1] = m == N ? c2 : 0.0;
      E3[2] = m == N - 1 ? c2 : 0.0;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) E3[c] += __shfl_xor(E3[c], off, 64);
    if ((t & 63) == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) sE[3 * (t >> 6) + c] = E3[c];
    }
  }
  __syncthreads();
  if (t == 0) {
    double tot = 0.0, eN = 0.0, eN1 = 0.0;
    for (int w = 0; w < Sz<N>::NT / 64; ++w) { tot += sE[3 * w]; eN += sE[3 * w + 1]; eN1 += sE[3 * w + 2]; }
    const double r1 = eN / fmax(tot, 1e-300);
    const double r2 = eN1 / fmax(tot - eN, 1e-300);
    const double ind = log10(fmax(fmax(r1, r2), 1e-300));
    f.ind[e] = ind;
    int nw = isfv ? 1 : 0;
    if (do_switch) {
      if (!isfv && ind > f.hi) nw = 1;
      if (isfv && ind < f.lo) nw = 0;
    }
    sNew = nw;
  }
  __syncthreads();
  const int nw = sNew;
  if (nw == (isfv ? 1 : 0)) return;  // uniform across the workgroup
  fv_tensor3<n>(nw ? sA : sA + n * n, sU, t, act);
  if (act) {
#pragma unroll
    for (int v = 0; v < 5; ++v) U[((size_t)e * 5 + v) * n3 + t] = sU[v * n3 + t];
  }
  if (t == 0) f.flag[e] = (uint8_t)nw;
}

// ----------------------------------------------------------------------------- launchers
#define DG_CHECK_LAUNCH()                                   \
  do {                                                      \
    hipError_t _e = hipGetLastError();                      \
    if (_e != hipSuccess) return DG_ERR_HIP;                \
  } while (0)

// The kernels that take an element's metric terms as constants (AFF) run on meshes whose every element is
// affine (Geo::Jc is set up by dg_init exactly there); any other mesh reads them per node.
// Whether a mesh takes the kernels with a lane per end of every line: where its workgroups run in one round (one per CU
// from N = 6 on, two below), so that the chain of one lane's steps is the time.  A step of 343 and 512 elements takes
// 0.81 to 0.97 of the other kernels' time at N = 4, 5 and 1.03 to 1.22 at N = 6, 7; of 216 elements 0.82 to 0.97 at
// N = 4 to 8; of 1000 elements 0.93 to 1.13 at N = 4, 5.  Against one node per lane, 64 elements, curved: split EC N = 7
// 122.0 -> 118.3 us a step, weak form on LG nodes N = 5 120.0 -> 111.4 (without this rule 126.5 and 124.2).
static bool small_mesh(int N, int K) { return K <= (N >= 6 ? 256 : 512); }

template <int N, bool LGL, bool NS, int FORM>
static int launch_main_t(const Geo &g, const Phys &ph, const double *U, const double *G, double *out, double *R,
                         double a, double b, double dt, int mode, hipStream_t st) {
  const dim3 grid(xcd_grid(g.K));
  // GEN: 0 structured, 1 face codes, 2 face codes and non-conforming faces
  const int lev = g.fc == nullptr ? 0 : (g.mslot ? 2 : 1);
  if constexpr (NS) {
    if (lev == 2) {
      const dim3 block(Sz<N>::NT);
      if (g.Jc) hipLaunchKernelGGL((k_main<N, LGL, FORM, true>), grid, block, 0, st, g, ph, U, G, out, R, a, b, dt, mode);
      else hipLaunchKernelGGL((k_main<N, LGL, FORM, false>), grid, block, 0, st, g, ph, U, G, out, R, a, b, dt, mode);
      DG_CHECK_LAUNCH();
      return DG_OK;
    }
  }
  const bool tp = ph.rs >= DG_RS_VOLFLUX;
#define DG_KM(G_, F_, A_, T_, E_) \
  hipLaunchKernelGGL((k_line<N, LGL, NS, FORM, G_, F_, A_, T_, E_>), grid, dim3(line_lanes<N, E_>()), 0, st, g, ph, U, out, R, a, b, dt, mode)
#define DG_KMT(G_, F_) \
  do { \
    constexpr bool E = ends_always(N); \
    if (g.Jc) { if (tp) DG_KM(G_, F_, true, true, E); else DG_KM(G_, F_, true, false, E); } \
    else { if (tp) DG_KM(G_, F_, false, true, E); else DG_KM(G_, F_, false, false, E); } \
  } while (0)
#define DG_KMS(G_, F_) \
  do { if (g.Jc) DG_KM(G_, F_, true, true, true); else DG_KM(G_, F_, false, true, true); } while (0)
  if (!ends_always(N) && small_mesh(N, g.K)) {
    // one instance for every mesh and surface flux
    if constexpr (!NS) {
      if (g.fvflag) DG_KMS(1, true); else DG_KMS(2, false);
    } else {
      DG_KMS(2, false);
    }
  } else if constexpr (!NS) {
    if (g.fvflag) DG_KMT(1, true);
    else if (lev == 2) DG_KMT(2, false);
    else if (lev == 1) DG_KMT(1, false);
    else DG_KMT(0, false);
  } else {
    if (lev == 1) DG_KMT(1, false); else DG_KMT(0, false);
  }
#undef DG_KMS
#undef DG_KMT
#undef DG_KM
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N, bool NS, int VF>
static int launch_split_t(const Geo &g, const Phys &ph, const double *U, double *out, double *R, double a, double b,
                          double dt, int mode, hipStream_t st) {
  const dim3 grid(xcd_grid(g.K));
#define DG_KSE(G_, F_, A_, E_) \
  do { \
    if constexpr (E_) hipLaunchKernelGGL((k_split_ends<N, NS, VF, G_, F_, A_>), grid, dim3(EndsSz<N>::NT), 0, st, g, ph, U, out, R, a, b, dt, mode); \
    else hipLaunchKernelGGL((k_split<N, NS, VF, G_, F_, A_>), grid, dim3(SplitSz<N>::NT), 0, st, g, ph, U, out, R, a, b, dt, mode); \
  } while (0)
#define DG_KS(G_, F_, E_) \
  do { if (g.Jc) DG_KSE(G_, F_, true, E_); else DG_KSE(G_, F_, false, E_); } while (0)
  // GEN: 0 structured, 1 face codes, 2 face codes and non-conforming faces
  const int lev = g.fc == nullptr ? 0 : (g.mslot ? 2 : 1);
  constexpr bool E = ends_always(N);
  const bool small = !E && small_mesh(N, g.K);  // one instance for every mesh
  if constexpr (!NS) {
    if (g.fvflag) {
      if (small) DG_KS(1, true, true); else DG_KS(1, true, E);
      DG_CHECK_LAUNCH();
      return DG_OK;
    }
  }
  if (small) DG_KS(2, false, true);
  else if (lev == 0) DG_KS(0, false, E);
  else if (lev == 1) DG_KS(1, false, E);
  else DG_KS(2, false, E);
#undef DG_KS
#undef DG_KSE
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N, bool LGL, bool NS>
static int launch_form(const Geo &g, const Phys &ph, int form, const double *U, const double *G, double *out,
                       double *R, double a, double b, double dt, int mode, hipStream_t st) {
  if (form == DG_FORM_WEAK) return launch_main_t<N, LGL, NS, 0>(g, ph, U, G, out, R, a, b, dt, mode, st);
  if (form == DG_FORM_STRONG) return launch_main_t<N, LGL, NS, 2>(g, ph, U, G, out, R, a, b, dt, mode, st);
  if (!LGL) return DG_ERR_UNSUPPORTED;
  if (form == DG_FORM_SPLIT) {
    if (ph.vf == DG_VF_EC) return launch_split_t<N, NS, 1>(g, ph, U, out, R, a, b, dt, mode, st);
    if (ph.vf == DG_VF_KEP) return launch_split_t<N, NS, 0>(g, ph, U, out, R, a, b, dt, mode, st);
    return launch_split_t<N, NS, 2>(g, ph, U, out, R, a, b, dt, mode, st);
  }
  return DG_ERR_UNSUPPORTED;
}

template <int N>
int launch_prolong(const Geo &g, const Phys &ph, const double *U, hipStream_t st) {
  hipLaunchKernelGGL((k_prolong<N>), dim3(xcd_grid(g.K)), dim3(Sz<N>::NT), 0, st, g, ph, U);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_lift(const Geo &g, const Phys &ph, bool lgl, int out, const double *U, double *G, double *Fv,
                hipStream_t st) {
  const dim3 grid(xcd_grid(g.K)), block(Sz<N>::NT), lines(SplitSz<N>::NT);
  // GEN: 0 structured, 1 face codes, 2 face codes and non-conforming faces
  const int lev = g.fc == nullptr ? 0 : (g.mslot ? 2 : 1);
#define DG_KLG(L_, O_, G_) \
  do { \
    if (g.Jc) hipLaunchKernelGGL((k_lift_affine<N, L_, O_, G_>), grid, lines, 0, st, g, ph, U, G, Fv); \
    else hipLaunchKernelGGL((k_lift<N, L_, O_, G_>), grid, block, 0, st, g, ph, U, G, Fv); \
  } while (0)
#define DG_KL(L_, O_) \
  do { if (lev == 0) DG_KLG(L_, O_, 0); else DG_KLG(L_, O_, 1); } while (0)
  // only what rhs_dispatch and the reverse ask for: gradients on meshes with non-conforming faces (weak and strong
  // form), the fluxes for the reverse and the weak and strong forms' viscous terms on conforming ones
  if (out == LIFT_G && lgl && lev == 2) DG_KLG(true, LIFT_G, 2);
  else if (out == LIFT_GT && !lgl && lev == 2) DG_KLG(false, LIFT_GT, 2);
  else if (out == LIFT_SV && !lgl && lev < 2) DG_KL(false, LIFT_SV);
  else if (out == LIFT_WV && lgl && lev < 2) DG_KL(true, LIFT_WV);
  else if (out == LIFT_WV && !lgl && lev < 2) DG_KL(false, LIFT_WV);
  else if (out == LIFT_FV && lgl && lev < 2) DG_KL(true, LIFT_FV);
  else if (out == LIFT_DIV && lgl && lev < 2) DG_KL(true, LIFT_DIV);
  else if (out == LIFT_DIV && lgl) DG_KLG(true, LIFT_DIV, 2);
  else if (out == LIFT_DIVK && lgl && lev < 2) DG_KL(true, LIFT_DIVK);
  else if (out == LIFT_DIVK && lgl) DG_KLG(true, LIFT_DIVK, 2);
  else return DG_ERR_UNSUPPORTED;
#undef DG_KLG
#undef DG_KL
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_main(const Geo &g, const Phys &ph, bool lgl, int eqn, int form, const double *U, const double *G,
                double *out, double *R, double a, double b, double dt, int mode, hipStream_t st) {
  const bool ns = (eqn == DG_NAVIER_STOKES);
  if (lgl) {
    if (ns) return launch_form<N, true, true>(g, ph, form, U, G, out, R, a, b, dt, mode, st);
    return launch_form<N, true, false>(g, ph, form, U, G, out, R, a, b, dt, mode, st);
  }
  if (ns) return launch_form<N, false, true>(g, ph, form, U, G, out, R, a, b, dt, mode, st);
  return launch_form<N, false, false>(g, ph, form, U, G, out, R, a, b, dt, mode, st);
}

template <int N, int EPB, int AFF>
static int launch_batch_lift_t(const BatchView &bv, hipStream_t st) {
  const dim3 grid(batch_grid(bv, EPB)), block(lift_b_lanes<N, AFF>() * EPB);
  if (bv.general) hipLaunchKernelGGL((k_lift_b<N, EPB, true, AFF>), grid, block, 0, st, bv);
  else hipLaunchKernelGGL((k_lift_b<N, EPB, false, AFF>), grid, block, 0, st, bv);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N, int EPB> static int launch_batch_lift_a(const BatchView &bv, hipStream_t st) {
  if (bv.n_affine == 0) return launch_batch_lift_t<N, EPB, AFF_NONE>(bv, st);
  if (bv.n_affine == bv.total) return launch_batch_lift_t<N, EPB, AFF_ALL>(bv, st);
  return launch_batch_lift_t<N, EPB, AFF_MIXED>(bv, st);
}

template <int N, bool NS, int VF, int EPB, int AFF>
static int launch_batch_split_t(const BatchView &bv, hipStream_t st) {
  const dim3 grid(batch_grid(bv, EPB)), block(line_lanes<N, ends_always(N)>() * EPB);
  if (bv.general) hipLaunchKernelGGL((k_split_b<N, NS, VF, EPB, true, AFF>), grid, block, 0, st, bv);
  else hipLaunchKernelGGL((k_split_b<N, NS, VF, EPB, false, AFF>), grid, block, 0, st, bv);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N, bool NS, int VF, int EPB> static int launch_batch_split_a(const BatchView &bv, hipStream_t st) {
  if (bv.n_affine == 0) return launch_batch_split_t<N, NS, VF, EPB, AFF_NONE>(bv, st);
  if (bv.n_affine == bv.total) return launch_batch_split_t<N, NS, VF, EPB, AFF_ALL>(bv, st);
  return launch_batch_split_t<N, NS, VF, EPB, AFF_MIXED>(bv, st);
}

template <int N, bool NS, int EPB>
static int launch_batch_split_vf(const BatchView &bv, int vf, hipStream_t st) {
  if (vf == DG_VF_EC) return launch_batch_split_a<N, NS, 1, EPB>(bv, st);
  if (vf == DG_VF_KEP) return launch_batch_split_a<N, NS, 0, EPB>(bv, st);
  return launch_batch_split_a<N, NS, 2, EPB>(bv, st);
}

template <int N>
int launch_batch_lift(const BatchView &bv, int epb, hipStream_t st) {
  if (bv.total <= 0) return DG_OK;
  if (epb == 1) return launch_batch_lift_a<N, 1>(bv, st);
  if constexpr (batch_max_epb(N) >= 2)
    if (epb == 2) return launch_batch_lift_a<N, 2>(bv, st);
  if constexpr (batch_max_epb(N) >= 4)
    if (epb == 4) return launch_batch_lift_a<N, 4>(bv, st);
  return DG_ERR_UNSUPPORTED;
}

template <int N>
int launch_batch_split(const BatchView &bv, bool ns, int vf, int epb, hipStream_t st) {
  if (bv.total <= 0) return DG_OK;
  if (epb == 1) return ns ? launch_batch_split_vf<N, true, 1>(bv, vf, st) : launch_batch_split_vf<N, false, 1>(bv, vf, st);
  if constexpr (batch_max_epb(N) >= 2)
    if (epb == 2)
      return ns ? launch_batch_split_vf<N, true, 2>(bv, vf, st) : launch_batch_split_vf<N, false, 2>(bv, vf, st);
  if constexpr (batch_max_epb(N) >= 4)
    if (epb == 4)
      return ns ? launch_batch_split_vf<N, true, 4>(bv, vf, st) : launch_batch_split_vf<N, false, 4>(bv, vf, st);
  return DG_ERR_UNSUPPORTED;
}

template <int N>
int launch_fv_face(const Geo &g, const Phys &ph, const FvGeo &f, bool lgl, const double *U, hipStream_t st) {
  const dim3 grid(std::min(3 * g.K, 4096)), block(FvFaceSz<N>::NT);
  const bool gen = g.fc != nullptr;
  if (lgl && gen) hipLaunchKernelGGL((k_fv_face<N, true, true>), grid, block, 0, st, g, ph, f, U);
  else if (lgl) hipLaunchKernelGGL((k_fv_face<N, true, false>), grid, block, 0, st, g, ph, f, U);
  else if (gen) hipLaunchKernelGGL((k_fv_face<N, false, true>), grid, block, 0, st, g, ph, f, U);
  else hipLaunchKernelGGL((k_fv_face<N, false, false>), grid, block, 0, st, g, ph, f, U);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_fv_volume(const Geo &g, const Phys &ph, const FvGeo &f, const double *U, double *out, double *R, double a,
                     double b, double dt, int mode, hipStream_t st) {
  const dim3 grid(std::min(g.K, 1024)), block(Sz<N>::NT);
#define DG_FVV(RS)                                                                                       \
  if (ph.rs == RS) {                                                                                     \
    if (mode == 0) hipLaunchKernelGGL((k_fv_volume<N, 0, RS>), grid, block, 0, st, g, ph, f, U, out, R, a, b, dt); \
    else hipLaunchKernelGGL((k_fv_volume<N, 1, RS>), grid, block, 0, st, g, ph, f, U, out, R, a, b, dt);           \
  }
  DG_FVV(0) DG_FVV(1) DG_FVV(2) DG_FVV(3)
#undef DG_FVV
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_fv_lists(const Geo &g, const FvGeo &f, hipStream_t st) {
  hipLaunchKernelGGL(k_fv_lists_zero<N>, dim3(1), dim3(64), 0, st, f);
  const dim3 grid((6 * g.K + 255) / 256);
  if (g.fc) hipLaunchKernelGGL((k_fv_lists<N, true>), grid, dim3(256), 0, st, g, f);
  else hipLaunchKernelGGL((k_fv_lists<N, false>), grid, dim3(256), 0, st, g, f);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_fv_switch(const Geo &g, const Phys &ph, const FvGeo &f, double *U, int do_switch, hipStream_t st) {
  hipLaunchKernelGGL((k_fv_switch<N>), dim3(g.K), dim3(Sz<N>::NT), 0, st, g, ph, f, U, do_switch);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_mortar_lift(const Geo &g, const Phys &ph, bool lgl, const MortarDesc *md, int nm, const double *U,
                       hipStream_t st) {
  if (nm <= 0) return DG_OK;
  if (lgl) hipLaunchKernelGGL((k_mortar_lift<N, true>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U);
  else hipLaunchKernelGGL((k_mortar_lift<N, false>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_mortar_flux(const Geo &g, const Phys &ph, bool lgl, int eqn, const MortarDesc *md, int nm,
                       const double *U, const double *G, hipStream_t st) {
  if (nm <= 0) return DG_OK;
  const bool ns = eqn == DG_NAVIER_STOKES;
  if (lgl && ns) hipLaunchKernelGGL((k_mortar_flux<N, true, true>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U, G);
  else if (lgl) hipLaunchKernelGGL((k_mortar_flux<N, true, false>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U, G);
  else if (ns) hipLaunchKernelGGL((k_mortar_flux<N, false, true>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U, G);
  else hipLaunchKernelGGL((k_mortar_flux<N, false, false>), dim3(nm), dim3(MortarSz<N>::NT), 0, st, g, ph, md, U, G);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

template <int N>
int launch_reduce(const Geo &g, const Phys &ph, int what, const double *U, double *partial, hipStream_t st) {
  const dim3 grid(reduce_rows(g.K, (N + 1) * (N + 1) * (N + 1))), block(256);
  if (what == RED_TIMESTEP) hipLaunchKernelGGL((k_reduce<N, RED_TIMESTEP>), grid, block, 0, st, g, ph, U, partial);
  else if (what == RED_INTEGRALS) hipLaunchKernelGGL((k_reduce<N, RED_INTEGRALS>), grid, block, 0, st, g, ph, U, partial);
  else hipLaunchKernelGGL((k_reduce<N, RED_FINITE>), grid, block, 0, st, g, ph, U, partial);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

#if !defined(DG_ONLY_N) && !defined(DG_FUSED_BATCH)
// one workgroup folds the rows of partial results in a fixed order; the components beyond WHAT's are zero
template <int WHAT>
__global__ void __launch_bounds__(1024) k_final_reduce(const double *__restrict__ partial, int rows,
                                                       double *__restrict__ out) {
  constexpr int NC = Red<WHAT>::NC;
  __shared__ double sm[16 * NC];
  double val[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) val[c] = Red<WHAT>::init(c);
  for (int r = threadIdx.x; r < rows; r += 1024) {
#pragma unroll
    for (int c = 0; c < NC; ++c) val[c] = Red<WHAT>::join(c, val[c], partial[(size_t)r * NC + c]);
  }
  Red<WHAT>::template workgroup<1024>(val, sm);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int c = 0; c < 8; ++c) out[c] = c < NC ? val[c < NC ? c : 0] : 0.0;
  }
}

// quadrature weight of every node: J w_i w_j w_k
__global__ void k_mass(const double *__restrict__ sJ, const double *__restrict__ w, int n, size_t total,
                       double *__restrict__ out) {
  size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const int n3 = n * n * n;
  for (; q < total; q += stride) {
    const int node = (int)(q % n3);
    const int i = node % n, j = (node / n) % n, k = node / (n * n);
    out[q] = w[i] * w[j] * w[k] / sJ[q];
  }
}

// y = alpha y + beta x; x may be y
__global__ void k_axpby(double *y, const double *x, double alpha, double beta, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) y[i] = alpha * y[i] + beta * x[i];
}

int launch_final_reduce(int what, const double *partial, int rows, double *out, hipStream_t st) {
  const dim3 one(1), block(1024);
  if (what == RED_TIMESTEP) hipLaunchKernelGGL(k_final_reduce<RED_TIMESTEP>, one, block, 0, st, partial, rows, out);
  else if (what == RED_INTEGRALS) hipLaunchKernelGGL(k_final_reduce<RED_INTEGRALS>, one, block, 0, st, partial, rows, out);
  else hipLaunchKernelGGL(k_final_reduce<RED_FINITE>, one, block, 0, st, partial, rows, out);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

int launch_mass(const double *sJ, const double *w, int n, size_t total, double *out, hipStream_t st) {
  size_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_mass, dim3((unsigned)blocks), dim3(256), 0, st, sJ, w, n, total, out);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

int launch_axpby(double *y, const double *x, double alpha, double beta, size_t n, hipStream_t st) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)blocks), dim3(256), 0, st, y, x, alpha, beta, n);
  DG_CHECK_LAUNCH();
  return DG_OK;
}
#endif

#ifdef DG_FUSED_BATCH
// ----------------------------------------------------------------------------- fused ensemble
// One lifting and one operator launch per stage for the members of every degree (structured
// members): group g of the work takes the workgroups [start[g], start[g+1]) of the grid, each
// workgroup of 512 lanes holds fused_epb elements of its group's degree in slots of the degree's
// own lane count, and the static LDS is the largest degree's, carved per slot.  Lanes past the
// last slot run the per-element code as invalid slots (no memory access, every barrier).
constexpr int FUSED_SPLIT_LDS = 2 * SplitLds<7>::A;  // 152 KB: one workgroup per CU
template <int N> constexpr int fused_epb_split() {
  constexpr bool ENDS = ends_always(N);
  constexpr int by_lanes = 512 / line_lanes<N, ENDS>();
  constexpr int by_lds = FUSED_SPLIT_LDS / SplitLds<N>::template size<0, false, ENDS>();
  return by_lanes < by_lds ? by_lanes : by_lds;
}
template <int N> constexpr int fused_epb_lift() {
  constexpr int by_lanes = 512 / Sz<N>::NT;
  constexpr int by_lds = (LiftLds<7>::W + LiftLds<7>::JA + LiftLds<7>::WS) /
                         (LiftLds<N>::W + LiftLds<N>::JA + LiftLds<N>::WS);
  return by_lanes < by_lds ? by_lanes : by_lds;
}

__device__ __forceinline__ int fused_group(const FusedView &fv, int b) {
  int gi = 0;
  while (gi + 1 < fv.ng && b >= fv.start[gi + 1]) ++gi;
  return gi;
}

// workgroup blk of group bv: its affine members' elements, then the others'
__device__ __forceinline__ BatchBlock fused_block(const BatchView &bv, int epb, int blk) {
  const int na = affine_blocks(bv, epb);
  if (blk < na) return {blk * epb, bv.n_affine, true};
  return {bv.n_affine + (blk - na) * epb, bv.total, false};
}

template <int N, bool NS, int VF>
__device__ __forceinline__ void fused_split_group(const BatchView &bv, int blk, double *smem) {
  constexpr bool ENDS = ends_always(N);
  constexpr int NT = line_lanes<N, ENDS>(), EPB = fused_epb_split<N>(), L = SplitLds<N>::template size<VF, false, ENDS>();
  const BatchBlock B = fused_block(bv, EPB, blk);
  const int raw = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  const int slot = raw < EPB ? raw : EPB - 1;
  const int t = threadIdx.x - raw * NT;
  const int item = B.item + slot;
  const bool valid = raw < EPB && item < B.end;
  const int mi = member_of(bv.first, bv.count, valid ? item : B.end - 1);
  const Member &M = bv.m[mi];
  const int e = valid ? item - bv.first[mi] : 0;
  double *sm = smem + slot * L;
  if (B.affine)
    split_member<N, NS, VF, 0, true>(M, bv.tab, e, valid, t, sm);
  else
    split_member<N, NS, VF, 0, false>(M, bv.tab, e, valid, t, sm);
}

template <bool NS, int VF>
__global__ void __launch_bounds__(512, 2) k_split_f(FusedView fv) {
  __shared__ double smem[FUSED_SPLIT_LDS];
  const int nb = fv.start[fv.ng];
  const int b = xcd_element(blockIdx.x, nb);
  if (b >= nb) return;
  const int gi = fused_group(fv, b);
  const int lb = b - fv.start[gi];
  switch (fv.N[gi]) {
    case 1: fused_split_group<1, NS, VF>(fv.v[gi], lb, smem); break;
    case 2: fused_split_group<2, NS, VF>(fv.v[gi], lb, smem); break;
    case 3: fused_split_group<3, NS, VF>(fv.v[gi], lb, smem); break;
    case 4: fused_split_group<4, NS, VF>(fv.v[gi], lb, smem); break;
    case 5: fused_split_group<5, NS, VF>(fv.v[gi], lb, smem); break;
    case 6: fused_split_group<6, NS, VF>(fv.v[gi], lb, smem); break;
    default: fused_split_group<7, NS, VF>(fv.v[gi], lb, smem); break;
  }
}

template <int N>
__device__ __forceinline__ void fused_lift_group(const BatchView &bv, int blk, double *smem, double *sDh, double *sl,
                                                 double *slh) {
  using L = LiftLds<N>;
  constexpr int NT = Sz<N>::NT, EPB = fused_epb_lift<N>();
  lift_tables<N>(bv.tab, threadIdx.x, 512, sDh, sl, slh);
  const BatchBlock B = fused_block(bv, EPB, blk);
  const int raw = __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  const int slot = raw < EPB ? raw : EPB - 1;
  const int t = threadIdx.x - raw * NT;
  const int item = B.item + slot;
  const bool valid = raw < EPB && item < B.end;
  const int mi = member_of(bv.first, bv.count, valid ? item : B.end - 1);
  const Member &M = bv.m[mi];
  const int e = valid ? item - bv.first[mi] : 0;
  double *sm = smem + slot * (L::W + L::JA + L::WS);
  if (B.affine)
    lift_affine<N, true, LIFT_DIV, 0, NT>(M.g, M.ph, bv.tab, e, valid, t, M.U, nullptr, nullptr, sm);
  else
    lift_body<N, true, LIFT_DIV, 0>(M.g, M.ph, e, valid, t, M.U, nullptr, nullptr, sm, sDh, sl, slh);
}

__global__ void __launch_bounds__(512, 4) k_lift_f(FusedView fv) {
  __shared__ double smem[LiftLds<7>::W + LiftLds<7>::JA + LiftLds<7>::WS];
  __shared__ double sDh[64], sl[16], slh[16];
  const int nb = fv.start[fv.ng];
  const int b = xcd_element(blockIdx.x, nb);
  if (b >= nb) return;
  const int gi = fused_group(fv, b);
  const int lb = b - fv.start[gi];
  switch (fv.N[gi]) {
    case 1: fused_lift_group<1>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    case 2: fused_lift_group<2>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    case 3: fused_lift_group<3>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    case 4: fused_lift_group<4>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    case 5: fused_lift_group<5>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    case 6: fused_lift_group<6>(fv.v[gi], lb, smem, sDh, sl, slh); break;
    default: fused_lift_group<7>(fv.v[gi], lb, smem, sDh, sl, slh); break;
  }
}

int fused_epb(int N, bool lift) {
  switch (N) {
#define DG_CASE(NN) \
  case NN: return lift ? fused_epb_lift<NN>() : fused_epb_split<NN>();
    DG_CASE(1) DG_CASE(2) DG_CASE(3) DG_CASE(4) DG_CASE(5) DG_CASE(6) DG_CASE(7)
#undef DG_CASE
    default: return 0;
  }
}

int launch_fused_lift(const FusedView &fv, hipStream_t st) {
  hipLaunchKernelGGL(k_lift_f, dim3(xcd_grid(fv.start[fv.ng])), dim3(512), 0, st, fv);
  DG_CHECK_LAUNCH();
  return DG_OK;
}

int launch_fused_split(const FusedView &fv, bool ns, int vf, hipStream_t st) {
  const dim3 grid(xcd_grid(fv.start[fv.ng])), block(512);
#define DG_FS(NS_, VF_) hipLaunchKernelGGL((k_split_f<NS_, VF_>), grid, block, 0, st, fv)
  if (ns) {
    if (vf == DG_VF_EC) DG_FS(true, 1);
    else if (vf == DG_VF_KEP) DG_FS(true, 0);
    else DG_FS(true, 2);
  } else {
    if (vf == DG_VF_EC) DG_FS(false, 1);
    else if (vf == DG_VF_KEP) DG_FS(false, 0);
    else DG_FS(false, 2);
  }
#undef DG_FS
  DG_CHECK_LAUNCH();
  return DG_OK;
}
#endif

#ifdef DG_ONLY_N
template int launch_prolong<DG_ONLY_N>(const Geo &, const Phys &, const double *, hipStream_t);
template int launch_lift<DG_ONLY_N>(const Geo &, const Phys &, bool, int, const double *, double *, double *,
                                    hipStream_t);
template int launch_main<DG_ONLY_N>(const Geo &, const Phys &, bool, int, int, const double *, const double *,
                                    double *, double *, double, double, double, int, hipStream_t);
template int launch_reduce<DG_ONLY_N>(const Geo &, const Phys &, int, const double *, double *, hipStream_t);
template int launch_mortar_lift<DG_ONLY_N>(const Geo &, const Phys &, bool, const MortarDesc *, int, const double *,
                                           hipStream_t);
template int launch_fv_face<DG_ONLY_N>(const Geo &, const Phys &, const FvGeo &, bool, const double *, hipStream_t);
template int launch_fv_volume<DG_ONLY_N>(const Geo &, const Phys &, const FvGeo &, const double *, double *, double *,
                                         double, double, double, int, hipStream_t);
template int launch_fv_switch<DG_ONLY_N>(const Geo &, const Phys &, const FvGeo &, double *, int, hipStream_t);
template int launch_fv_lists<DG_ONLY_N>(const Geo &, const FvGeo &, hipStream_t);
template int launch_mortar_flux<DG_ONLY_N>(const Geo &, const Phys &, bool, int, const MortarDesc *, int,
                                           const double *, const double *, hipStream_t);
template int launch_batch_lift<DG_ONLY_N>(const BatchView &, int, hipStream_t);
template int launch_batch_split<DG_ONLY_N>(const BatchView &, bool, int, int, hipStream_t);
#endif

}  // namespace dg
