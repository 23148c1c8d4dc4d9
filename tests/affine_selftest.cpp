// The library's affine test and constants (dg_affine.h) behind one C function for the host test.
#include "../paper_1910_02858_amd/csrc/dg_affine.h"

extern "C" int affine(int K, int ng, const double *x, const double *xgeo, const int32_t *nbr, const int8_t *side,
                      const int8_t *mort, double *out) {
  const std::vector<long double> xl(x, x + ng);
  const std::vector<double> C = dg::affine_constants(K, ng, xl.data(), xgeo, nbr, side, mort);
  std::copy(C.begin(), C.end(), out);
  return C.empty() ? 0 : 1;
}
