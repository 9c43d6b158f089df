// rfa_pair.h -- launcher of the two-step kernel (internal).
#pragma once

#include <hip/hip_runtime.h>

#include "rfa_kernels.h"
#include "rfa_tiled.h"

namespace rfa {

// Footprint of a work-group of the two-step kernel: waves * 64 * v
// consecutive voxels of a (y, z) plane, starting at a multiple of seg, v
// consecutive ones a lane.  Its segment, seg voxels, starts pair_lead()
// voxels later (a row, rounded up so that a lane owns all its voxels or
// none), and at least nz voxels on either side are its halo.  The plane's
// first and last rows, which are held, lie in the halo of the first and the
// last segment and are stored by them.
__host__ __device__ __forceinline__ int pair_lead(int nz, int v) { return (nz + v - 1) / v * v; }

// First voxel of the footprint's lane i, f = base + v i.  Where the plane's
// voxels are odd in number, two a lane would run over its end: that lane
// starts one voxel earlier and shares it with its neighbour, to the same bits.
__device__ __forceinline__ int pair_first(int f, int v, int np) {
  return v == 2 && f == np - 1 ? f - 1 : f;
}

struct PairShape {
  int waves = 0;   // wavefronts per work-group
  int v = 0;       // voxels per lane
  int xc = 0;      // x planes per work-group
  int seg = 0;     // owned voxels per segment
  int segs = 0;    // segments per plane
  int chunks = 0;  // chunks along x
  int nwg = 0;     // work-groups per launch
};

// Wave code: class in bits 0-3, which of the wave's voxels are tissue in bits
// 4-5; kPairIrregular if its coefficients differ from voxel to voxel.
constexpr unsigned kPairIrregular = 255u;
constexpr unsigned kPairTissueFree = 0x10u;  // the free voxels
constexpr unsigned kPairTissueAll = 0x20u;   // every voxel inside the plane

// What a launch moves besides the state of StepBuffers.
enum PairMode {
  kPairFull = 0,  // both steps' damage and latches
  kPairKeep = 1,  // the same, and the hi image between the steps is kept
  kPairTemp = 2   // temperature only, the hi image between the steps kept
};

// Whether the kernel exists for this work-group and grid.
bool pair_fits(Grid3 g, int waves, int v, int xc);
PairShape pair_shape(Grid3 g, int waves, int v, int xc);
// Bytes of a shape's wave codes, and the kernel that fills them (after every
// change of the labels or the class table).
size_t pair_code_bytes(Grid3 g, const PairShape& s);
hipError_t launch_pair_codes(Grid3 g, const PairShape& s, const uint8_t* lab,
                             const ClassParams& cp, uint8_t* codes, hipStream_t st);
// The same for many grids of one kind of work-group in one launch: a table of
// jobs on the device (first: the work-groups of the jobs before it), n_wg
// work-groups in all.
struct AlikeClasses {
  unsigned short held[kMaxClasses];  // of each class: those of the same conductivity
  unsigned short open[kMaxClasses];  // and of the same heat capacity
};
struct PairCodeJob {
  const uint8_t* lab;
  uint8_t* codes;
  int ny, nz, seg, segs;
  unsigned n_codes, first;
  AlikeClasses alike;
};
PairCodeJob pair_code_job(Grid3 g, const PairShape& s, const uint8_t* lab, const ClassParams& cp,
                          uint8_t* codes);
unsigned pair_code_wg(const PairCodeJob& job);
hipError_t launch_pair_code_jobs(int waves, int v, const PairCodeJob* jobs, int n_jobs,
                                 unsigned n_wg, hipStream_t st);
// Two steps, with the step constants of b.tab.  b.codes: the shape's wave
// codes; hi_mid: the image between the steps (kPairKeep, kPairTemp).
hipError_t launch_step_pair(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode,
                            float* hi_mid, int store, hipStream_t st);

// One grid of a batch: its arrays, its shape's segments and chunk length.
// Image 0 is the current image at batch parity 0; a launch at parity p reads
// image p and writes image 1 - p.  No damage-coupled perfusion.
struct PairInstance {
  float* hi[2];
  float* lo[2];
  uint8_t* lab;
  const float* src;
  float* om;
  const float* perf;
  const Tables* tab;
  const uint8_t* codes;
  int n_classes;
  int nx, ny, nz;
  int xc, seg, segs;
  int pad;
};

// One work item: segment sg over chunk `chunk` of an instance.
struct PairItem {
  int inst, sg, chunk, pad;
};

// Two steps of the items [first_item, first_item + n_items), all of instances
// with (perf) or without a perfusion field, with work-groups of waves x v.
// partials (nullable) receives 3 floats per item, indexed by item.
hipError_t launch_pair_batch(int waves, int v, const PairInstance* inst, const PairItem* items,
                             int first_item, int n_items, bool perf, int parity, float* partials,
                             hipStream_t st);

// Estimated time (us) of a launch of nwg work-groups that march xc planes,
// and the kinds of work-group it knows (false: no kind `index`).
bool pair_kind(int index, int* waves, int* v);
double pair_estimate(int waves, int v, int nwg, int xc);
// The same for nwg work-groups of different lengths: `planes` iterations in
// all, `longest` in one of them.
double pair_estimate_uneven(int waves, int v, int nwg, long long planes, int longest);

// The kinds of work-group (waves x voxels per lane), for launch_step_pair().
#define RFA_PAIR_LAUNCH(name)                                                             \
  hipError_t name(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode, \
                  float* hi_mid, int store, hipStream_t st)
RFA_PAIR_LAUNCH(launch_pair_16x2);
RFA_PAIR_LAUNCH(launch_pair_8x2);
RFA_PAIR_LAUNCH(launch_pair_8x1);
RFA_PAIR_LAUNCH(launch_pair_4x1);
#define RFA_PAIR_BATCH(name)                                                              \
  hipError_t name(const PairInstance* inst, const PairItem* items, int first_item,       \
                  int n_items, bool perf, int parity, float* partials, hipStream_t st)
RFA_PAIR_BATCH(launch_batch_16x2);
RFA_PAIR_BATCH(launch_batch_8x2);
RFA_PAIR_BATCH(launch_batch_8x1);
RFA_PAIR_BATCH(launch_batch_4x1);

}  // namespace rfa
