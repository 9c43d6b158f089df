// rfa_adjoint_device.h -- the adjoint update of one voxel, shared by the adjoint
// kernels (internal).
#pragma once

#include <hip/hip_runtime.h>

#include "rfa_device.h"

namespace rfa {

// The face coefficients of one class pair along one axis, each float-float
// table entry rounded to float: x = C(q, p) (q's own row), y = C(p, q).
// Table entries in bytes: row of a class = its masked label << 4, entry =
// the other class's masked label (the label keeps the class times 8).
__device__ __forceinline__ float2 pair_from_table(const float2* __restrict__ cf, int axis,
                                                  unsigned cq, unsigned cp) {
  const char* t = reinterpret_cast<const char*>(cf + axis * kMaxClasses * kMaxClasses);
  const float2 a = *reinterpret_cast<const float2*>(t + ((cq << 4) | cp));
  const float2 b = *reinterpret_cast<const float2*>(t + ((cp << 4) | cq));
  return make_float2(a.x + a.y, b.x + b.y);
}

// Pair table: pc[axis][a][c] = pair_from_table(cf, axis, a, c), built once
// per work-group so the per-voxel update reads one entry per face.
__device__ __forceinline__ void stage_pairs(float2* pc, float4* cls, const Tables* tab,
                                            int nthreads) {
  constexpr int per_axis = kMaxClasses * kMaxClasses;
  for (int t = threadIdx.x; t < 3 * per_axis; t += nthreads) {
    const int ax = t / per_axis, r = t - ax * per_axis;
    const unsigned a = (unsigned)(r / kMaxClasses), c = (unsigned)(r % kMaxClasses);
    pc[t] = pair_from_table(&tab->cf[0][0], ax, a << kClassShift, c << kClassShift);
  }
  if ((int)threadIdx.x < kMaxClasses) cls[threadIdx.x] = tab->cls[threadIdx.x];
}

// Pair-table lookup in the same byte-offset form.
__device__ __forceinline__ float2 pair_from_pairs(const float2* __restrict__ pc, int axis,
                                                  unsigned cq, unsigned cp) {
  const char* t = reinterpret_cast<const char*>(pc + axis * kMaxClasses * kMaxClasses);
  return *reinterpret_cast<const float2*>(t + ((cq << 4) | cp));
}

// Adjoint update of one voxel q: lam_out = (M^T lam_in)_q + w_q dt rate'(theta^n_q),
// and the accumulations sacc += lam_in_q, facc += lam_in_q (-B theta^n_q), for
// a free voxel; a held voxel gets lam_out = 0 and accumulates nothing
// (returns false).  Neighbours in the order x-, x+, y-, y+, z-, z+; pair(axis,
// cq, cp) gives {C(q, p), C(p, q)} for masked labels, from the forward's
// tables or from the pair table (the same floats either way); cls points at
// the class table.  Branch-free: a held voxel's neighbour values may be
// arbitrary (the tiled kernel leaves halo cells outside the grid unwritten)
// and reach nothing but selects on the held flags.
template <class Pair>
__device__ __forceinline__ bool adjoint_voxel(float lam, float th, unsigned lq, float pf,
                                              float w, const float (&nlam)[6],
                                              const unsigned (&nlab)[6], Pair pair,
                                              const float4* __restrict__ cls,
                                              const StepConst& K, float& lam_out,
                                              float& sacc, float& facc) {
  const bool held = (lq & kHeld) != 0u;
  const float4 cl = cls[class_of(lq)];
  const float B = (cl.x + cl.y) * pf;
  const unsigned cq = lq & kClassMask;
  float diag = 1.0f - B;
  float off = 0.0f;
#pragma unroll
  for (int f = 0; f < 6; ++f) {
    const unsigned lp = nlab[f];
    const float2 c = pair(f >> 1, cq, lp & kClassMask);
    diag -= c.x;                                        // C(q, p): q's own row
    const float o = __builtin_fmaf(c.y, nlam[f], off);  // C(p, q)
    off = (lp & kHeld) ? off : o;
  }
  // damage-rate derivative at theta^n, the rate evaluated as the forward
  // step evaluates it (zero off tissue and where the exponent is capped)
  const float r = __builtin_amdgcn_rcpf(K.tak + th);
  const float x = K.c2 * th * r;
  const float rate = K.dtka * __builtin_amdgcn_exp2f(fminf(x, K.clamp2));
  const float dr0 = rate * (K.c2 * 0.69314718f) * K.tak * (r * r);
  const float dr = ((lq & kTissue) != 0u && x < K.clamp2) ? dr0 : 0.0f;
  const float lo = __builtin_fmaf(diag, lam, off) + w * dr;
  lam_out = held ? 0.0f : lo;
  sacc = held ? sacc : sacc + lam;
  facc = held ? facc : __builtin_fmaf(-cl.x - cl.y, th * lam, facc);
  return !held;
}

}  // namespace rfa
