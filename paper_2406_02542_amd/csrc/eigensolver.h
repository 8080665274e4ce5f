// Host-side interface of the eigensolver (eigensolver.hip) to the calibration (calibrate.hip).
#pragma once

#include "common.h"

namespace loki {

constexpr size_t kEigReflBytes = (size_t)(kD - 1) * (kD / 2) * 2 * sizeof(double);  // a head's share of EigRegions::refl

// Device memory the solver works in, for n heads.
struct EigRegions {
  double* cov;       // [n][128][128] the symmetric matrices; overwritten
  double* mat;       // [n][128][128]
  char* refl;        // [n][kEigReflBytes]
  int* state;        // [n]
  char* spare;       // [n * spare_halves] blocks of 64 KiB, 16-byte aligned
  int spare_halves;  // per head, at least 1; more let a launch run several Jacobi sweeps
};

// P [n][128][128]: column j the eigenvector of the j-th largest eigenvalue, its largest entry
// positive; eigenvalues [n][128] decreasing.
hipError_t launch_eigensolver(int Hkv, const EigRegions& r, float* P, float* eigenvalues, hipStream_t st);

}  // namespace loki
