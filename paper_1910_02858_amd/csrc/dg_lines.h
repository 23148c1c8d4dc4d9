// Device helpers of the kernels that take one lane per line of an element: LDS slots, lanes per element, the
// constants of affine elements.
#pragma once
#include "dg_internal.h"

namespace dg {

// LDS slot of node (i, j, k) in one component array.  For n = 8 the index bits are swizzled so that the 64
// lanes that read the m-th node of 64 different lines hit distinct banks in each direction (and in node order):
// i is XORed with two bits of j and k, j with the low bits of k.  For n = 4 likewise the 16 lanes of each
// direction: without it 40 % of the LDS time of the N = 3 kernels were bank conflicts (Euler on LG nodes, 48^3
// 2028 -> 2009 us a step; reverse of the split form, 32^3 curved 417 -> 394; split EC 32^3 1128 -> 1100).
template <int n> __device__ __forceinline__ int div_slot(int i, int j, int k) {
  if constexpr (n == 4) return (i ^ k) + 4 * (j ^ k) + 16 * k;
  else if constexpr (n == 8) return (i ^ ((j >> 2) | ((k & 3) << 1))) + 8 * (j ^ (k & 3)) + 64 * k;
  else return i + n * (j + n * k);
}

// Constant metric terms of an affine element (Geo::Jc) through the scalar cache.
typedef const __attribute__((address_space(4))) double *AffineConst;
__device__ __forceinline__ AffineConst affine_const(const Geo &g, int e) {
  return (AffineConst)(g.Jc + (size_t)__builtin_amdgcn_readfirstlane(e) * AFFINE_DOUBLES);
}

// LDS slots (div_slot) of the nodes of one line, without a branch on its direction: the swizzles
// of n = 4 and 8 are linear over the index bits, slot = base ^ (contribution of the position's bits); else
// base + m stride.
template <int n> struct LineSlots {
  int base, s1, s2, s4;
  __device__ __forceinline__ LineSlots(int dir, int a, int b) {
    const int i = dir == 0 ? 0 : a, j = dir == 0 ? a : (dir == 1 ? 0 : b), k = dir == 2 ? 0 : b;
    base = div_slot<n>(i, j, k);
    if constexpr (n == 8) {
      s1 = dir == 0 ? 1 : (dir == 1 ? 8 : 74);
      s2 = dir == 0 ? 2 : (dir == 1 ? 16 : 148);
      s4 = dir == 0 ? 4 : (dir == 1 ? 33 : 256);
    } else if constexpr (n == 4) {
      s1 = dir == 0 ? 1 : (dir == 1 ? 4 : 21);
      s2 = dir == 0 ? 2 : (dir == 1 ? 8 : 42);
      s4 = 0;
    } else {
      s1 = dir == 0 ? 1 : (dir == 1 ? n : n * n);
      s2 = s4 = 0;
    }
  }
  __device__ __forceinline__ int operator()(int m) const {
    if constexpr (n == 8 || n == 4) return base ^ ((m & 1 ? s1 : 0) ^ (m & 2 ? s2 : 0) ^ (m & 4 ? s4 : 0));
    else return base + m * s1;
  }
};

// Lanes of one element in the kernels that take one lane per line: the lines of the three directions, 3 n^2.
template <int N> struct SplitSz {
  static constexpr int n = N + 1, NL = 3 * n * n;
  static constexpr int NT = (NL + 63) / 64 * 64;
};

// With a lane per end of every line (ENDS): the first HALF lanes take the lines and the fluxes at their near ends,
// the next HALF the fluxes at the far ends; wave aligned where the two halves do not fit one wave.
template <int N> struct EndsSz {
  static constexpr int NL = SplitSz<N>::NL, HALF = 2 * NL <= 64 ? NL : (NL + 63) / 64 * 64;
  static constexpr int NT = (2 * HALF + 63) / 64 * 64;
};
template <int N, bool ENDS> constexpr int line_lanes() { return ENDS ? EndsSz<N>::NT : SplitSz<N>::NT; }
template <int N, bool ENDS> __device__ __forceinline__ int line_end(int lane) {
  if constexpr (!ENDS) return 0;
  else if constexpr (EndsSz<N>::HALF % 64 == 0) return __builtin_amdgcn_readfirstlane(lane / EndsSz<N>::HALF);
  else return lane / EndsSz<N>::HALF;
}
// one wave holds both ends of every line of degrees 1 and 2: a second lane costs nothing there
constexpr bool ends_always(int N) { return N <= 2; }
// the kernels of small meshes: one workgroup per CU, so the three directions' sums may lie in LDS side by side, put
// down after one barrier instead of one after the other
template <int N, bool ENDS> constexpr bool line_apart() { return ENDS && !ends_always(N); }

// The 1D tables through the scalar cache.
typedef const __attribute__((address_space(4))) double *Scalar;
struct Scalars {
  Scalar D, Dh, Ds, lm, lp, lhm, lhp;
  __device__ __forceinline__ Scalars(const Tab *t)
      : D((Scalar)t->D), Dh((Scalar)t->Dh), Ds((Scalar)t->Ds), lm((Scalar)t->lm), lp((Scalar)t->lp),
        lhm((Scalar)t->lhm), lhp((Scalar)t->lhp) {}
};

}  // namespace dg
