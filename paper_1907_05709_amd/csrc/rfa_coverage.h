// rfa_coverage.h -- coverage loss of a damage integral (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rfa {

constexpr int kCoverageBlocks = 512;  // work-groups of the sums: two per compute unit

// Loss of omega[n] over the classes tumour and liver of labels[n] into
// loss[0], 1 / max(tumour voxels, 1) into per_tumour[0]; codes[n] (nullable)
// receives the classes for the gradient; partial: 3 kCoverageBlocks doubles.
hipError_t launch_coverage(const float* omega, const uint8_t* labels, long long n, int tumour,
                           int liver, double voxel_cm3, double weight, uint8_t* codes,
                           double* partial, double* loss, double* per_tumour, hipStream_t st);

// out[n] = grad[0] dloss/domega.
hipError_t launch_coverage_grad(const float* omega, const uint8_t* codes, long long n,
                                double voxel_cm3, double weight, const double* per_tumour,
                                const double* grad, float* out, hipStream_t st);

}  // namespace rfa
