// Meshes whose every element is affine: which they are, and the constant metric terms of their elements.
// Host code without HIP.
#pragma once
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <limits>
#include <thread>
#include <vector>

namespace dg {

// Constant metric terms of an affine element: Ja^i_d at i*3+d, 1/J at 9, and the outward scaled normal of
// every side (the master's, negated on slaves) at 10 + 3*side + d.
constexpr int AFFINE_DOUBLES = 28;

inline bool is_mortar_side(const int8_t *mort, int q) { return mort && mort[q] != 0; }

// Deviation of an element's nodes from its affine map that counts as rounding of the coordinates: 4 ulp of the
// mesh's largest coordinate (a shift or a rotation rounds at the size of the mesh, not of the element; lattices of
// 4 to 160 elements per direction, at the origin, centred, rotated and sheared, deviate by at most 2), but in no
// reference direction more than 1.6e-13 / ng of the element's extent (ng nodes: 2e-14 at degree 7).  What the
// constants leave out, the derivatives of the per-node terms carry into the operator amplified by about the degree:
// 7e-13 of the whole vector on a rotated lattice of 48^3 elements at N = 7 (1.4e-14 of the extent), 2e-13 at N = 3.
// A mesh a thousand element sizes away from the origin lies beyond, and keeps its metric terms per node.
// Where it holds it pays: 32^3 elements centred at 0, N = 7, split form, 10265 -> 7765 us a step; 48^3, N = 3, Euler
// on LG nodes, 2730 -> 2179.
constexpr double AFFINE_ULP = 4.0 * 2.220446049250313e-16, AFFINE_EXTENT = 1.6e-13;

// The constants of every element [K][AFFINE_DOUBLES], or empty if some element is not affine.  xgeo [K][3][ng^3]
// at the ng LGL nodes x; nbr, side, mort [K][6] as in dg_mesh (validated).
// Ja^dir of two elements that share a face is the same vector (to a sign): it depends on the face's edges alone.
// Taken from each element's own corners, it would differ across the face by the rounding of the coordinates, and
// the two sides' fluxes would cancel only to that.  So all elements that follow each other through opposite faces
// share one value, the middle of the range of their own (independent of the elements' numbering).
inline std::vector<double> affine_constants(int K, int ng, const long double *x, const double *xgeo, const int32_t *nbr,
                                            const int8_t *side, const int8_t *mort) {
  typedef long double xf;
  const int ng3 = ng * ng * ng;
  const xf extent = 2.0L * (xf)AFFINE_EXTENT / ng;  // an element spans 2 in every reference direction
  std::vector<double> C((size_t)K * AFFINE_DOUBLES, 0.0);
  std::vector<xf> Ja((size_t)K * 9);       // the elements' own
  std::vector<xf> slack((size_t)K * 3);    // what the deviation allowed to the nodes can move Ja^dir by
  auto element = [&](int e, double rounding) -> bool {
    const double *X = xgeo + (size_t)e * 3 * ng3;
    xf A[3][3], c[3];  // about the first corner: x = c + sum_d A[d] xi_d
    for (int m = 0; m < 3; ++m) {
      const double *Xm = X + m * ng3;
      c[m] = A[0][m] = A[1][m] = A[2][m] = 0.0L;
      for (int k = 0; k < 8; ++k) {
        const int i = (k & 1) ? ng - 1 : 0, j = (k & 2) ? ng - 1 : 0, l = (k & 4) ? ng - 1 : 0;
        const xf v = ((xf)Xm[i + ng * (j + ng * l)] - (xf)Xm[0]) / 8.0L;
        c[m] += v;
        A[0][m] += (k & 1) ? v : -v; A[1][m] += (k & 2) ? v : -v; A[2][m] += (k & 4) ? v : -v;
      }
    }
    xf *J3 = Ja.data() + (size_t)e * 9, J = 0.0L, len[3], eps[3];
    for (int i = 0; i < 3; ++i) {
      const xf *p = A[(i + 1) % 3], *q = A[(i + 2) % 3];
      for (int d = 0; d < 3; ++d) {
        const int d1 = (d + 1) % 3, d2 = (d + 2) % 3;
        J3[i * 3 + d] = p[d1] * q[d2] - p[d2] * q[d1];
        if (i == 0) J += A[0][d] * J3[d];
      }
      len[i] = std::sqrt(J3[i * 3] * J3[i * 3] + J3[i * 3 + 1] * J3[i * 3 + 1] + J3[i * 3 + 2] * J3[i * 3 + 2]);
    }
    if (!(J > 0.0L) || !std::isfinite((double)(1.0L / J))) return false;
    // a deviation v of a node is Ja^i . v / J in reference direction i
    for (int i = 0; i < 3; ++i) eps[i] = std::min(extent, rounding * len[i] / J);
    // the largest deviations of the three coordinates together decide, for all but turned elements near the limit
    double most[3];
    for (int m = 0; m < 3; ++m) {
      const double *Xm = X + m * ng3;
      double big = 0.0;
      for (int l = 0; l < ng; ++l)
        for (int j = 0; j < ng; ++j) {
          const xf at = (xf)Xm[0] + c[m] + A[1][m] * x[j] + A[2][m] * x[l];
          for (int i = 0; i < ng; ++i) {
            const double v = std::fabs((double)((xf)Xm[i + ng * (j + ng * l)] - at - A[0][m] * x[i]));
            if (!(v <= rounding)) return false;
            big = std::max(big, v);
          }
        }
      most[m] = big;
    }
    bool near = true;
    for (int d = 0; d < 3; ++d)
      near = near && std::fabs(J3[d * 3]) * most[0] + std::fabs(J3[d * 3 + 1]) * most[1] + std::fabs(J3[d * 3 + 2]) * most[2] <= extent * J;
    for (int q = 0; !near && q < ng3; ++q) {
      const int i = q % ng, j = q / ng % ng, l = q / (ng * ng);
      xf v[3];
      for (int m = 0; m < 3; ++m)
        v[m] = ((xf)X[m * ng3 + q] - (xf)X[m * ng3]) - (c[m] + A[0][m] * x[i] + A[1][m] * x[j] + A[2][m] * x[l]);
      for (int d = 0; d < 3; ++d)
        if (!(std::fabs(J3[d * 3] * v[0] + J3[d * 3 + 1] * v[1] + J3[d * 3 + 2] * v[2]) <= extent * J)) return false;
    }
    for (int i = 0; i < 3; ++i) {
      const int p = (i + 1) % 3, q = (i + 2) % 3;
      slack[(size_t)e * 3 + i] = 4.0L * ((eps[p] + eps[q]) * len[i] + eps[i] * (len[p] + len[q]));
    }
    C[(size_t)e * AFFINE_DOUBLES + 9] = (double)(1.0L / J);
    return true;
  };
  // a curved mesh ends here, before the other elements are read and threads are started
  if (!element(0, std::numeric_limits<double>::infinity())) return {};
  double big = 0.0;
  // an affine element is widest at its corners (32^3 elements of 8^3 nodes, eight threads: 185 ms of setup with all
  // nodes searched and every node's deviation taken into the reference directions, 45 so)
  for (size_t b = 0; b < (size_t)K * 3; ++b)
    for (int k = 0; k < 8; ++k)
      big = std::max(big, std::fabs(xgeo[b * ng3 + (size_t)(ng - 1) * ((k & 1) + ng * ((k >> 1 & 1) + ng * (k >> 2)))]));
  // elements are independent: split them over host threads, which all stop at the first that is not affine
  std::atomic<bool> affine{true};
  unsigned nthr = std::thread::hardware_concurrency();
  if (const char *env = std::getenv("OMP_NUM_THREADS")) nthr = (unsigned)std::max(1, std::atoi(env));
  nthr = std::max(1u, std::min(nthr, 32u));
  if ((size_t)K < 64 * (size_t)nthr) nthr = 1;
  auto work = [&](unsigned tid) {
    const int e0 = (int)((size_t)K * tid / nthr), e1 = (int)((size_t)K * (tid + 1) / nthr);
    for (int e = e0; e < e1 && affine.load(std::memory_order_relaxed); ++e)
      if (!element(e, AFFINE_ULP * big)) affine = false;
  };
  if (nthr == 1) {
    work(0);
  } else {
    std::vector<std::thread> pool;
    for (unsigned t = 0; t < nthr; ++t) pool.emplace_back(work, t);
    for (auto &th : pool) th.join();
  }
  if (!affine) return {};
  // one value of Ja^dir along every chain of opposite faces: sets of (element, direction), each with the sign of
  // its vector against its set's root (+ where a +xi side meets a -xi side)
  std::vector<int> up((size_t)K * 3);
  std::vector<signed char> sg((size_t)K * 3, 1);
  for (int q = 0; q < 3 * K; ++q) up[q] = q;
  auto root = [&](int q, signed char &s) {  // paths are halved as they are walked
    s = 1;
    while (up[q] != q) {
      sg[q] = (signed char)(sg[q] * sg[up[q]]);
      up[q] = up[up[q]];
      s = (signed char)(s * sg[q]);
      q = up[q];
    }
    return q;
  };
  for (int e = 0; e < K; ++e)
    for (int s = 0; s < 6; ++s) {
      const int nb = nbr[e * 6 + s], ns = side[e * 6 + s];
      if (nb < 0 || is_mortar_side(mort, e * 6 + s)) continue;
      signed char s1, s2;
      const int r1 = root(3 * e + (s >> 1), s1), r2 = root(3 * nb + (ns >> 1), s2);
      const signed char f = (signed char)(((s & 1) != (ns & 1) ? 1 : -1) * s1 * s2);
      if (r1 == r2) {
        if (f < 0) return {};  // a chain that comes back reversed
      } else {
        up[std::max(r1, r2)] = std::min(r1, r2);
        sg[std::max(r1, r2)] = f;
      }
    }
  std::vector<xf> lo((size_t)K * 9, std::numeric_limits<xf>::infinity()), hi((size_t)K * 9, -std::numeric_limits<xf>::infinity());
  for (int q = 0; q < 3 * K; ++q) {
    signed char s;
    const int r = root(q, s);
    for (int d = 0; d < 3; ++d) {
      const xf v = s * Ja[(size_t)q * 3 + d];
      lo[(size_t)r * 3 + d] = std::min(lo[(size_t)r * 3 + d], v);
      hi[(size_t)r * 3 + d] = std::max(hi[(size_t)r * 3 + d], v);
    }
  }
  for (int q = 0; q < 3 * K; ++q) {
    signed char s;
    const int r = root(q, s), e = q / 3, i = q % 3;
    double *o = C.data() + (size_t)e * AFFINE_DOUBLES;
    for (int d = 0; d < 3; ++d) {
      const xf v = s * (0.5L * (lo[(size_t)r * 3 + d] + hi[(size_t)r * 3 + d]));
      // a slow taper, each element's share of it within the rounding
      if (!(std::fabs(v - Ja[(size_t)q * 3 + d]) <= slack[q])) return {};
      o[i * 3 + d] = (double)v;
      o[10 + 3 * (2 * i) + d] = -(double)v;
      o[10 + 3 * (2 * i + 1) + d] = (double)v;
    }
  }
  return C;
}

}  // namespace dg
