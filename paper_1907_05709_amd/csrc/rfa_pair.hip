// rfa_pair.hip -- shapes, wave codes and launches of the two-step kernel
// (rfa_pair_kernel.h; each work-group size is compiled by its own source).
#include "rfa_pair.h"

namespace rfa {

// Wave codes: for plane x, segment and wave of the footprint, the class that
// all its free voxels share if every neighbour has that class's conductivity
// and every free one its heat capacity (0 without free voxels), and which of
// its voxels are tissue; kPairIrregular otherwise.  The coefficients of such a
// wave's free voxels are all C(c, c), the harmonic mean of equal
// conductivities over equal heat capacities: those of their own rows, and
// (for the adjoint) those of their free neighbours'.  The host compares the
// classes, so that a voxel's test is a bit of a mask rather than 12 reads of
// their values, and a voxel's six neighbours are read at once (128^3 31.2 ->
// 12.7 us; bound by the latency of two rounds of byte reads).
__device__ __forceinline__ void pair_codes(const PairCodeJob& job, unsigned wg, int nt, int v) {
  __shared__ unsigned held_like[kMaxClasses], open_like[kMaxClasses];
  if (threadIdx.x < kMaxClasses) {
    held_like[threadIdx.x] = job.alike.held[threadIdx.x];
    open_like[threadIdx.x] = job.alike.open[threadIdx.x];
  }
  __syncthreads();
  const uint8_t* lab = job.lab;
  const int nz = job.nz, seg = job.seg, segs = job.segs;
  const int lane = threadIdx.x & 63;
  const int nw = nt / 64, np = job.ny * nz;
  const unsigned id = wg * 4 + (threadIdx.x >> 6);
  if (id >= job.n_codes) return;
  const unsigned line = id / nw;
  const int wave = (int)(id % nw);
  const int sg = (int)(line % segs);
  const size_t plane = (line / segs) * (size_t)np;
  unsigned code = 0u;
  bool found = false, regular = true;
  bool none = true, only_free = true, all = true;  // which voxels are tissue
  for (int j = 0; j < v; ++j) {
    const int f = pair_first(sg * seg + v * (wave * 64 + lane), v, np) + j;  // the kernel's
    const bool valid = f < np;
    bool free = false, ok = true, tissue = false;
    unsigned c = 0u;
    if (valid) {
      const uint8_t* p = lab + plane + f;
      tissue = (p[0] & kTissue) != 0u;
      if (!(p[0] & kHeld)) {  // free voxels are never on the outer layer
        free = true;
        c = class_of(p[0]);
        const unsigned held = held_like[c], open = open_like[c];
        auto same = [&](ptrdiff_t o) {
          const unsigned q = p[o];
          return (((q & kHeld) ? held : open) >> class_of(q) & 1u) != 0u;
        };
        // all six reads in flight at once
        ok = same(-1) & same(1) & same(-nz) & same(nz) & same(-(ptrdiff_t)np) & same(np);
      }
    }
    none = none && __ballot(tissue) == 0ull;
    only_free = only_free && __ballot(tissue != free) == 0ull;
    all = all && __ballot(valid && !tissue) == 0ull;
    const unsigned long long m = __ballot(free);
    if (m == 0ull) continue;
    if (!found) code = (unsigned)__builtin_amdgcn_readlane((int)c, __ffsll(m) - 1);
    found = true;
    regular = regular && __ballot(free && (!ok || c != code)) == 0ull;
  }
  regular = regular && (none || only_free || all);
  code |= none ? 0u : (only_free ? kPairTissueFree : kPairTissueAll);
  if (lane == 0) job.codes[id] = (uint8_t)(regular ? code : kPairIrregular);
}

__global__ __launch_bounds__(256) void k_pair_codes(PairCodeJob job, int nt, int v) {
  pair_codes(job, blockIdx.x, nt, v);
}

// One launch for the grids of a batch (64 of 24^3 to 30^3: one kernel of 14 us
// in place of 64 of 2.7, one after another).
__global__ __launch_bounds__(256) void k_pair_code_jobs(const PairCodeJob* jobs, int n_jobs,
                                                        int nt, int v) {
  int j = 0;  // the last job that starts at or before this work-group
  for (int above = n_jobs; above - j > 1;) {
    const int mid = (j + above) / 2;
    if (jobs[mid].first <= blockIdx.x)
      j = mid;
    else
      above = mid;
  }
  pair_codes(jobs[j], blockIdx.x - jobs[j].first, nt, v);
}

namespace {

// Work-groups built, and what a launch of them takes.  A launch costs about
// 3 us plus, per round of resident work-groups, xc + 2 plane iterations (the
// first step runs on one plane more at either end of a chunk).  An
// iteration's time grows with the work-groups m that share a compute unit,
// a + b m; a and b fitted to runs of 19 grids from 32^3 to 256^3, every kind
// and up to 22 chunk lengths.  Over those grids the pick is within 1 % of
// the fastest (geometric mean; 4.6 % at worst).
struct PairKind {
  int waves, v, max_nz;
  int per_cu;   // work-groups a compute unit holds
  double a, b;  // us per iteration
};
constexpr PairKind kPairKinds[] = {{16, 2, 256, 1, 1.2, 1.15},
                                   {8, 2, 128, 2, 0.98, 0.57},
                                   {8, 1, 128, 2, 0.64, 0.34},
                                   {4, 1, 96, 5, 0.7, 0.155}};
constexpr double kLaunchUs = 2.8;
constexpr int kCu = 256;

}  // namespace

bool pair_kind(int index, int* waves, int* v) {
  if (index < 0 || index >= (int)(sizeof kPairKinds / sizeof kPairKinds[0])) return false;
  *waves = kPairKinds[index].waves;
  *v = kPairKinds[index].v;
  return true;
}

double pair_estimate(int waves, int v, int nwg, int xc) {
  for (const PairKind& k : kPairKinds) {
    if (k.waves != waves || k.v != v) continue;
    const int slots = kCu * k.per_cu, rest = nwg % slots;
    double us = kLaunchUs + (nwg / slots) * (xc + 2) * (k.a + k.b * k.per_cu);
    if (rest) us += (xc + 2) * (k.a + k.b * ((rest + kCu - 1) / kCu));
    return us;
  }
  return 1e300;
}

double pair_estimate_uneven(int waves, int v, int nwg, long long planes, int longest) {
  for (const PairKind& k : kPairKinds) {
    if (k.waves != waves || k.v != v) continue;
    const int slots = kCu * k.per_cu;
    // one round: the longest; more: the slots share the work and, on average,
    // wait for half of a last work-group
    if (nwg <= slots) return kLaunchUs + longest * (k.a + k.b * ((nwg + kCu - 1) / kCu));
    return kLaunchUs + ((double)planes / slots + 0.5 * longest) * (k.a + k.b * k.per_cu);
  }
  return 1e300;
}

bool pair_fits(Grid3 g, int waves, int v, int xc) {
  for (const PairKind& k : kPairKinds)
    if (k.waves == waves && k.v == v)
      return g.nz <= k.max_nz && 2 * g.nz <= 64 * waves &&
             64 * waves * v - pair_lead(g.nz, v) - g.nz >= 64 &&
             (double)(xc + 6) * g.ny * g.nz * 4.0 < 2147483647.0;
  return false;
}

PairShape pair_shape(Grid3 g, int waves, int v, int xc) {
  PairShape s;
  s.waves = waves;
  s.v = v;
  s.xc = xc;
  const int np = g.ny * g.nz;
  const int lead = pair_lead(g.nz, v);
  const int most = (64 * waves * v - lead - g.nz) / 32 * 32;
  // the plane's first and last rows are held and go along as halo
  const int inner = np - lead - g.nz;
  s.segs = (inner + most - 1) / most;
  s.seg = ((inner + s.segs - 1) / s.segs + 31) / 32 * 32;
  s.segs = (inner + s.seg - 1) / s.seg;
  s.chunks = (g.nx + xc - 1) / xc;
  s.nwg = s.segs * s.chunks;
  return s;
}

size_t pair_code_bytes(Grid3 g, const PairShape& s) {
  return (size_t)g.nx * s.segs * s.waves;
}

PairCodeJob pair_code_job(Grid3 g, const PairShape& s, const uint8_t* lab, const ClassParams& cp,
                          uint8_t* codes) {
  PairCodeJob job{lab, codes, g.ny, g.nz, s.seg, s.segs, (unsigned)pair_code_bytes(g, s), 0, {}};
  for (int a = 0; a < cp.n; ++a)
    for (int b = 0; b < cp.n; ++b) {
      if (cp.k[a] != cp.k[b]) continue;
      job.alike.held[a] |= 1u << b;
      if (cp.rc[a] == cp.rc[b]) job.alike.open[a] |= 1u << b;
    }
  return job;
}

unsigned pair_code_wg(const PairCodeJob& job) { return (job.n_codes + 3) / 4; }

hipError_t launch_pair_codes(Grid3 g, const PairShape& s, const uint8_t* lab,
                             const ClassParams& cp, uint8_t* codes, hipStream_t st) {
  const PairCodeJob job = pair_code_job(g, s, lab, cp, codes);
  hipLaunchKernelGGL(k_pair_codes, dim3(pair_code_wg(job)), dim3(256), 0, st, job, 64 * s.waves,
                     s.v);
  return hipGetLastError();
}

hipError_t launch_pair_code_jobs(int waves, int v, const PairCodeJob* jobs, int n_jobs,
                                 unsigned n_wg, hipStream_t st) {
  hipLaunchKernelGGL(k_pair_code_jobs, dim3(n_wg), dim3(256), 0, st, jobs, n_jobs, 64 * waves, v);
  return hipGetLastError();
}

hipError_t launch_step_pair(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode,
                            float* hi_mid, int store, hipStream_t st) {
  if (!pair_fits(g, s.waves, s.v, s.xc) || !b.codes || (mode != kPairFull && !hi_mid))
    return hipErrorInvalidValue;
  if (s.waves == 16 && s.v == 2) return launch_pair_16x2(s, g, b, mode, hi_mid, store, st);
  if (s.waves == 8 && s.v == 2) return launch_pair_8x2(s, g, b, mode, hi_mid, store, st);
  if (s.waves == 8 && s.v == 1) return launch_pair_8x1(s, g, b, mode, hi_mid, store, st);
  if (s.waves == 4 && s.v == 1) return launch_pair_4x1(s, g, b, mode, hi_mid, store, st);
  return hipErrorInvalidValue;
}

hipError_t launch_pair_batch(int waves, int v, const PairInstance* inst, const PairItem* items,
                             int first_item, int n_items, bool perf, int parity, float* partials,
                             hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  auto launch = [&](auto f) {
    return f(inst, items, first_item, n_items, perf, parity, partials, st);
  };
  if (waves == 16 && v == 2) return launch(launch_batch_16x2);
  if (waves == 8 && v == 2) return launch(launch_batch_8x2);
  if (waves == 8 && v == 1) return launch(launch_batch_8x1);
  if (waves == 4 && v == 1) return launch(launch_batch_4x1);
  return hipErrorInvalidValue;
}

}  // namespace rfa
