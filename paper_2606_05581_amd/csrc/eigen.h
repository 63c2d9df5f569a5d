// Timing record of the eigen step's dense products and the small triangular
// inverse it shares with the mesh Laplacian basis (eigen.hip).
#pragma once
#include "msk_internal.h"

namespace msk {

// Summed kernel time and algorithmic flops of the eigen step's dense
// products, by precision (FP32: the products with C; FP64: the basis
// products and the final Rayleigh quotients).
struct EigGemmTimes {
  int64_t fp32_products = 0, fp64_products = 0;
  double fp32_ms = 0, fp32_flops = 0, fp64_ms = 0, fp64_flops = 0;
};

// R and Ri = R^-1 of the Cholesky factor G = R^T R of the symmetric n x n G
// (n <= kCholMax, row-major, on the device); *ok = 0 and R and Ri unwritten
// where a pivot is not above rel_tol times the largest diagonal entry, else 1.
// R or Ri may be G.
constexpr int kCholMax = 128;  // the factor, a square of doubles, stands in one workgroup's LDS
hipError_t launch_chol_inverse(const double* G, int n, double rel_tol, double* R, double* Ri, unsigned long long* ok,
                               hipStream_t s);

}  // namespace msk
