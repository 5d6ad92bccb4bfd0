// Separable banded solves of the direct B-spline transform (host-callable).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tbs {

constexpr int kBandTab = 32;  // rows after which the factor of a truncated band has reached its limit

// L D L^T of a symmetric Toeplitz band b_0..b_W (W <= 2), truncated at the low end: row i has the
// entries l1, l2 left of the diagonal and 1 / D in dinv; rows from kBandTab - 1 on are alike.
struct BandFactor {
  double l1[kBandTab], l2[kBandTab], dinv[kBandTab];
};
BandFactor band_factor(const double* b, int W);

// v <- (E^-1 along each of the three axes) v for v[z][y][x], E the Toeplitz band of half-width W
// (truncated at both ends, or circulant); the last axis adds its result to dst instead of storing it
// in v, which is left with intermediate values.  tmp: an array like v.  One launch per axis, two where its
// lines are cut into segments.
hipError_t launch_band_solve(double* v, double* tmp, double* dst, const int dims[3], int W, int periodic,
                             const BandFactor& f, hipStream_t st);

}  // namespace tbs
