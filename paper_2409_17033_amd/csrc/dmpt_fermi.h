// Internal launchers of the finite-temperature path (dmpt_fermi.hip).
// Matrices are n_pad x n_pad FP32, zero padded, row-major or (tiled) in the
// small-size kernels' layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "dmpt_internal.h"

namespace dmpt {

// FP64 partials of (Tr M, ||M||_F^2) of nmat matrices (`stride` floats apart):
// part[2 (k nblk + b)], part[2 (k nblk + b) + 1] for block b of matrix k.
hipError_t launch_trace_sq(const float* m, size_t stride, int nmat, int n, int n_pad, int tiled, double* part, int nblk,
                           hipStream_t s);
// Shift of each observable: chi'_k = Y_k + g_k (I/4 - E^2).
struct FermiShift {
  float g[kMaxObs];
};
// D = I/2 + E, chi_k = scale chi'_k (n x n, row-major; either may be NULL) and the
// FP64 partials of Tr[A_k D] (nblk per observable).
hipError_t launch_fermi_output(const float* e, const float* e2, const float* y, size_t ystride, const float* a, int n,
                               int n_pad, int nobs, int tiled, FermiShift shift, double scale, float* d_out,
                               float* chi_out, double* a0_part, int nblk, hipStream_t s);

}  // namespace dmpt
