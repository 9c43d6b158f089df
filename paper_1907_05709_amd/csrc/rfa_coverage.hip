// rfa_coverage.hip -- coverage loss of a damage integral and its gradient.
//
// d = Omega^4 / (1 + Omega^4) is the damaged fraction of a voxel (0 where
// Omega is not positive, NaN among it),
//   loss = sum_tumour (1 - d) / max(N_tumour, 1) + weight sum_liver d,
// with weight the healthy weight times the voxel volume in cm^3, all in
// double.  One pass reads the integral (4 bytes a voxel) and the labels (1)
// and, where a gradient will follow, leaves a code byte of the two classes;
// the gradient's pass reads integral and code and writes 4 bytes.  Partial
// sums are formed over a fixed partition, so that the value does not change
// from call to call.
//
// What bounds it: launches (128^3: the sums 8 us, the gradient 7, at 10 and 19
// MB).  The same loss as tensor operations is some 45 launches of 8-byte
// passes and their host work: 100 steps and their gradients on 128^3 3.57 ->
// 3.17 ms without them, 60 steps on 88x80x75 1.26 -> 0.94 ms.
#include <hip/hip_runtime.h>

#include "rfa_coverage.h"

namespace rfa {
namespace {

constexpr int kThreads = 256;
constexpr unsigned kTumour = 1u, kLiver = 2u;

// Four consecutive values of a tensor that may start anywhere.
typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u4 __attribute__((aligned(1)));

// Omega^-4 of a positive Omega (0 for inf).
__device__ __forceinline__ double inverse4(double om) {
  const double s = om * om;
  return 1.0 / (s * s);
}

__device__ __forceinline__ void add_voxel(float omega, unsigned code, double& undertreated,
                                          double& tumour, double& liver) {
  if (code == 0u) return;
  const double om = (double)omega;
  const double d = om > 0.0 ? 1.0 / (1.0 + inverse4(om)) : 0.0;
  if (code & kTumour) {
    undertreated += 1.0 - d;
    tumour += 1.0;
  }
  if (code & kLiver) liver += d;
}

__device__ __forceinline__ unsigned code_of(unsigned label, unsigned tumour, unsigned liver) {
  return (label == tumour ? kTumour : 0u) | (label == liver ? kLiver : 0u);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Sums of kCoverageBlocks work-groups: partial[3][kCoverageBlocks].
__global__ __launch_bounds__(kThreads) void k_coverage_sums(const float* __restrict__ omega,
                                                            const uint8_t* __restrict__ labels,
                                                            long long n, unsigned tumour,
                                                            unsigned liver,
                                                            uint8_t* __restrict__ codes,
                                                            double* __restrict__ partial) {
  double s[3] = {0.0, 0.0, 0.0};
  const long long quads = n / 4, stride = (long long)kCoverageBlocks * kThreads;
  const long long first = (long long)blockIdx.x * kThreads + threadIdx.x;
  for (long long q = first; q < quads; q += stride) {
    const f4 om = *(const f4*)(omega + 4 * q);
    const unsigned lb = *(const u4*)(labels + 4 * q);
    unsigned packed = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned c = code_of((lb >> (8 * j)) & 0xffu, tumour, liver);
      packed |= c << (8 * j);
      add_voxel(om[j], c, s[0], s[1], s[2]);
    }
    if (codes) *(u4*)(codes + 4 * q) = packed;
  }
  const long long tail = 4 * quads + first;
  if (tail < n) {
    const unsigned c = code_of(labels[tail], tumour, liver);
    add_voxel(omega[tail], c, s[0], s[1], s[2]);
    if (codes) codes[tail] = (uint8_t)c;
  }
  __shared__ double sums[3][kThreads / 64];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s[k] = wave_sum(s[k]);
    if ((threadIdx.x & 63) == 0) sums[k][threadIdx.x >> 6] = s[k];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) t += sums[threadIdx.x][w];
    partial[threadIdx.x * kCoverageBlocks + blockIdx.x] = t;
  }
}

// loss[0] and per_tumour[0] = 1 / max(N_tumour, 1) from the partial sums, one
// wave for each of the three.
__global__ __launch_bounds__(192) void k_coverage_finish(const double* __restrict__ partial,
                                                         double voxel_cm3, double weight,
                                                         double* __restrict__ loss,
                                                         double* __restrict__ per_tumour) {
  static_assert(kCoverageBlocks % 64 == 0, "whole waves of partial sums");
  const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double v[kCoverageBlocks / 64];
#pragma unroll
  for (int i = 0; i < kCoverageBlocks / 64; ++i)
    v[i] = partial[k * kCoverageBlocks + 64 * i + lane];
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < kCoverageBlocks / 64; ++i) t += v[i];
  t = wave_sum(t);
  __shared__ double s[3];
  if (lane == 0) s[k] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double voxels = s[1] > 1.0 ? s[1] : 1.0;
    loss[0] = s[0] / voxels + weight * (s[2] * voxel_cm3);
    per_tumour[0] = 1.0 / voxels;
  }
}

// dL/dOmega = grad[0] (weight_liver - 1 / N on the tumour) 4 d^2 Omega^-5.  The
// classes multiply rather than select, so that a factor that is not finite
// shows on every voxel with damage, as it does in the tensor operations.
__device__ __forceinline__ float slope(float omega, unsigned code, double in_tumour,
                                       double in_liver) {
  const double om = (double)omega;
  if (!(om > 0.0)) return 0.0f;
  const double w = in_tumour * ((code & kTumour) ? 1.0 : 0.0) +
                   in_liver * ((code & kLiver) ? 1.0 : 0.0);
  const double p = inverse4(om), d = 1.0 / (1.0 + p);
  return (float)(w * (4.0 * (d * d) * (p / om)));
}

__global__ __launch_bounds__(kThreads) void k_coverage_grad(
    const float* __restrict__ omega, const uint8_t* __restrict__ codes, long long n,
    double voxel_cm3, double weight, const double* __restrict__ per_tumour,
    const double* __restrict__ grad, float* __restrict__ out) {
  const double g = grad[0];
  const double in_tumour = -(g * per_tumour[0]), in_liver = g * (weight * voxel_cm3);
  const long long q = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (4 * q + 4 <= n) {
    const f4 om = *(const f4*)(omega + 4 * q);
    const unsigned c = *(const u4*)(codes + 4 * q);
    f4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = slope(om[j], (c >> (8 * j)) & 0xffu, in_tumour, in_liver);
    *(f4*)(out + 4 * q) = r;
  } else {
    for (long long i = 4 * q; i < n; ++i) out[i] = slope(omega[i], codes[i], in_tumour, in_liver);
  }
}

}  // namespace

hipError_t launch_coverage(const float* omega, const uint8_t* labels, long long n, int tumour,
                           int liver, double voxel_cm3, double weight, uint8_t* codes,
                           double* partial, double* loss, double* per_tumour, hipStream_t st) {
  hipLaunchKernelGGL(k_coverage_sums, dim3(kCoverageBlocks), dim3(kThreads), 0, st, omega, labels,
                     n, (unsigned)tumour, (unsigned)liver, codes, partial);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL(k_coverage_finish, dim3(1), dim3(192), 0, st, partial, voxel_cm3, weight, loss,
                     per_tumour);
  return hipGetLastError();
}

hipError_t launch_coverage_grad(const float* omega, const uint8_t* codes, long long n,
                                double voxel_cm3, double weight, const double* per_tumour,
                                const double* grad, float* out, hipStream_t st) {
  const long long blocks = (n + 4ll * kThreads - 1) / (4ll * kThreads);
  if (blocks > 0x7fffffffll) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_coverage_grad, dim3((unsigned)blocks), dim3(kThreads), 0, st, omega, codes,
                     n, voxel_cm3, weight, per_tumour, grad, out);
  return hipGetLastError();
}

}  // namespace rfa
