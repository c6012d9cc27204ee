// Pieces shared by the two shape-function kernels.
#pragma once

#include "launch.h"
#include "otm_common.h"

namespace otm {

// exp(x) for the shifted exponents of the LME weights (x <= 0 up to
// rounding): Cody-Waite reduction x = k ln2 + r with ln2 split in a 32-bit
// head and its remainder (k ln2_hi is exact), |r| <= ln2/2, then the Taylor
// polynomial of degree 12 in Horner form (truncation below 2e-16 relative on
// that range) and a scale by 2^k; 0 below -745.  The coefficients 1 / i! come
// from an array `taylor` in constant memory that each unit defines for itself,
// visible outside it, so that they reach the FMAs from scalar registers (a
// static array's values would be folded into vector registers).
#define OTM_EXP_TAYLOR                                                                       \
  {1.0, 1.0, 0.5, 0.16666666666666666, 0.041666666666666664, 0.008333333333333333,           \
   0.001388888888888889, 0.0001984126984126984, 2.48015873015873e-05, 2.7557319223985893e-06, \
   2.755731922398589e-07, 2.505210838544172e-08, 2.08767569878681e-09}
OTM_DEV double lme_exp(const double* taylor, double x) {
  const double k = rint(x * 1.4426950408889634);
  double r = fma(k, -0.6931471803691238, x);
  r = fma(k, -1.9082149292705877e-10, r);
  double p = taylor[12];
#pragma unroll
  for (int i = 11; i >= 0; --i) p = fma(p, r, taylor[i]);
  const double e = ldexp(p, (int)k);
  return x < -745.0 ? 0.0 : e;
}

// Totals of pairs (none with lo > hi).
struct PairWindow {
  int64_t lo, hi;
  OTM_DEV bool holds(int64_t pairs) const { return pairs >= lo && pairs <= hi; }
};

// The pipelined kernel (lme_pipelined.hip), OTM_FP64: it works on lists of `mine`
// pairs in all and leaves others untouched.
void launch_lme_pipelined(int64_t n_nodes, const double* x_nodes, int64_t n_mp,
                          const double* x_mp, const int64_t* nbr_offsets, const int32_t* nbr_idx,
                          int64_t pair_capacity, double beta, double tol, int32_t max_iter,
                          double* lam, double* N, double* dN, const double4* packed,
                          otm_diag* diag, PairWindow mine, hipStream_t s, const AsmIn* fused,
                          const SegIn* seg);

}  // namespace otm
