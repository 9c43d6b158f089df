// rfa_step.hip -- step scheduling (kernel choice, launch shapes, launch loop).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rfa_step.h"

namespace rfa {

namespace {
constexpr int kTargetWg = 1024;  // ~4 work-groups per CU on 256 CUs

// Stepping working set (two state images, class bytes, source, damage:
// ~29 B per voxel) beyond ~3/4 of the 256 MB last-level cache: stream the
// stores instead of writing them through.
int store_for(Grid3 g) {
  return (double)g.n() * 29.0 > 192.0 * (1 << 20) ? kPolicyStream : kPolicyThrough;
}
}

namespace {
StepPlan with_one(StepPlan p, const StepPlan& one) {
  p.one_kind = one.kind;
  p.one_ty = one.ty;
  p.one_xc = one.xc;
  p.one_nwg = one.nwg;
  p.one_zv = one.zv;
  return p;
}

StepPlan with_store(StepPlan p, Grid3 g) {
  p.store = store_for(g);
  return p;
}

// x chunk giving about `target` work-groups for `tiles` tiles per plane,
// rounded up to the kernels' four-plane unroll
int default_xc(Grid3 g, int tiles, int target = kTargetWg) {
  const int chunks = std::max(1, (target + tiles - 1) / tiles);
  const int xc = (g.nx + chunks - 1) / chunks;
  return std::min(g.nx, std::max(4, (xc + 3) / 4 * 4));
}

// Work-groups that fit the chip at once with the wide kernel (4-wave
// work-groups, 2 resident waves per SIMD with 4 voxels per lane, 4 with 2).
int wide_target_wg(int zv) { return zv == 4 ? 512 : 1024; }
}  // namespace

StepPlan plan_naive(Grid3 g) {
  StepPlan p;
  p.kind = kStepNaive;
  p.depth = 1;
  p.ty = 4;
  p.xc = 1;
  p.nwg = naive_wg_count(g);
  p.zv = 1;
  p.store = kPolicyBack;
  return with_one(p, p);
}

StepPlan plan_tiled(Grid3 g, int ty, int xc) {
  const TiledShape s = tiled_shape(g, ty, xc);
  StepPlan p;
  p.kind = kStepTiled;
  p.depth = 1;
  p.ty = ty;
  p.xc = xc;
  p.nwg = s.nwg;
  p.zv = 1;
  return with_one(with_store(p, g), p);
}

StepPlan plan_wide(Grid3 g, int zv, int ty, int xc) {
  const TiledShape s = wide_shape(g, zv, ty, xc);
  StepPlan p;
  p.kind = kStepTiled;
  p.depth = 1;
  p.ty = ty;
  p.xc = xc;
  p.nwg = s.nwg;
  p.zv = zv;
  return with_one(with_store(p, g), p);
}

StepPlan plan_tiled2(Grid3 g, int ty, int xc) {
  const TiledShape s = tiled2_shape(g, ty, xc);
  StepPlan p;
  p.kind = kStepTiled;
  p.depth = 2;
  p.ty = ty;
  p.xc = xc;
  p.nwg = s.nwg;
  p.zv = 1;
  return with_one(with_store(p, g), plan_default(g, kStepTiled, 1, 0, 0, 0));
}

StepPlan plan_pair(Grid3 g, int waves, int v, int xc) {
  const PairShape s = pair_shape(g, waves, v, xc);
  StepPlan p;
  p.kind = kStepTiled;
  p.depth = 2;
  p.ty = waves;
  p.xc = xc;
  p.nwg = s.nwg;
  p.pv = v;
  return with_one(with_store(p, g), plan_default(g, kStepTiled, 1, 0, 0, 0));
}

StepPlan plan_one(const StepPlan& p) {
  StepPlan o = p;
  o.kind = p.one_kind;
  o.depth = 1;
  o.ty = p.one_ty;
  o.xc = p.one_xc;
  o.nwg = p.one_nwg;
  o.zv = p.one_zv;
  o.pv = 0;
  return o;
}

namespace {

// Two-step plan with the least estimated time, waves / tile_x as asked (0:
// any); false if no work-group fits the grid.  It picks e.g. 4 waves x 1
// voxel at 32^3 (3.3 us a step; one-step kernel 6.0), 8 x 1 at 64^3 (4.9;
// 6.4), 16 x 2 at 128^3 (10.8; 13.3) and 256^3 (57.0; 80).
bool best_pair(Grid3 g, int waves, int tile_x, StepPlan* out) {
  double best = 1e300;
  int w, v;
  for (int kind = 0; pair_kind(kind, &w, &v); ++kind) {
    if (waves && waves != w) continue;
    const int lo = tile_x ? std::min(tile_x, g.nx) : 1;
    const int hi = tile_x ? lo : std::min(g.nx, 64);
    for (int xc = lo; xc <= hi; ++xc) {
      if (!pair_fits(g, w, v, xc)) continue;
      const double us = pair_estimate(w, v, pair_shape(g, w, v, xc).nwg, xc);
      if (us < best) {
        best = us;
        *out = plan_pair(g, w, v, xc);
      }
    }
  }
  return best < 1e300;
}

StepPlan default_shape(Grid3 g, int kernel, int depth, int tile_y, int tile_x, int zv) {
  if (kernel == kStepNaive || !tiled_fits(g, 4)) return plan_naive(g);
  // two steps per launch wherever a work-group holds the rows (nz <= 256),
  // unless the options ask for one step or for a shape of its kernels
  StepPlan pair;
  if (depth == 2 && best_pair(g, tile_y, tile_x, &pair)) return pair;
  if (depth == 0 && !tile_y && !tile_x && !zv && best_pair(g, 0, 0, &pair)) {
    pair.time_rest = true;
    return pair;
  }
  // automatic: four z voxels per lane once a tile row spans 256 voxels, two
  // (with 8-row tiles) from 96
  if (zv == 0 && depth != 2 && g.nz >= 256 && g.nz % 4 == 0) zv = 4;
  if (zv == 0 && depth != 2 && g.nz >= 96 && g.nz % 2 == 0) zv = 2;
  if (depth != 2 && (zv == 2 || zv == 4) && wide_fits(g, zv, 4) && tile_y != 16) {
    const int ty = tile_y ? tile_y : (zv == 2 ? 8 : 4);
    const int tiles = ((g.nz + 64 * zv - 1) / (64 * zv)) * ((g.ny + ty - 1) / ty);
    int xc = tile_x ? std::min(tile_x, g.nx) : default_xc(g, tiles, wide_target_wg(zv));
    while (xc > 4 && !wide_fits(g, zv, xc)) xc /= 2;
    return plan_wide(g, zv, ty, xc);
  }
  if (depth == 2 && tiled2_fits(g, 4)) {
    const int ty = tile_y == 16 ? 16 : 8;
    const int tiles = ((g.nz + 61) / 62) * ((g.ny + ty - 3) / (ty - 2));
    // the x-march runs planes x0 - 1 .. x0 + xc four at a time: xc = 2 mod 4
    // leaves no pass over planes outside the chunk
    int xc = tile_x ? std::min(tile_x, g.nx) : std::min(g.nx, default_xc(g, tiles) + 2);
    while (xc > 4 && !tiled2_fits(g, xc)) xc /= 2;
    return plan_tiled2(g, ty, xc);
  }
  int ty = tile_y;
  if (ty == 0) ty = g.ny >= 192 ? 8 : 4;
  const int tiles = ((g.nz + 63) / 64) * ((g.ny + ty - 1) / ty);
  int xc = tile_x ? std::min(tile_x, g.nx) : default_xc(g, tiles);
  while (xc > 4 && !tiled_fits(g, xc)) xc /= 2;
  return plan_tiled(g, ty, xc);
}
}  // namespace

StepPlan plan_default(Grid3 g, int kernel, int depth, int tile_y, int tile_x, int zv,
                      int store) {
  StepPlan p = default_shape(g, kernel, depth, tile_y, tile_x, zv);
  if (store > 0 && p.kind != kStepNaive) p.store = store - 1;
  return p;
}

int plan_candidates(Grid3 g, int max_depth, StepPlan* out, int max_out) {
  int n = 0;
  const int xcs[] = {4, 8, 16, 32, 64};
  const int tys[] = {4, 8, 16};
  for (int ty : tys)
    for (int xc : xcs) {
      if (n >= max_out) return n;
      if ((xc > g.nx && xc != 4) || !tiled_fits(g, std::min(xc, g.nx))) continue;
      out[n++] = plan_tiled(g, ty, std::min(xc, g.nx));
    }
  const int zvs[] = {2, 4};
  const int tysw[] = {4, 8};
  const int xcsw[] = {4, 8, 16, 32, 64};
  for (int zv : zvs)
    for (int ty : tysw)
      for (int xc : xcsw) {
        if (n >= max_out) return n;
        if ((xc > g.nx && xc != 4) || !wide_fits(g, zv, std::min(xc, g.nx))) continue;
        out[n++] = plan_wide(g, zv, ty, std::min(xc, g.nx));
      }
  if (max_depth < 2) return n;
  for (int waves : {16, 8, 4})
    for (int v : {2, 1})
      for (int xc : {2, 4, 6, 8, 12, 20, 43}) {
        if (n >= max_out) return n;
        if (xc <= g.nx && pair_fits(g, waves, v, xc)) out[n++] = plan_pair(g, waves, v, xc);
      }
  StepPlan pair;
  if (n < max_out && best_pair(g, 0, 0, &pair)) {
    out[n++] = pair;
    return n;
  }
  // grids without a pair plan: the 2.5-D two-step kernel
  const int tys2[] = {8, 16};
  const int xcs2[] = {6, 14, 30, 62};  // 2 mod 4: no pass outside the chunk
  for (int ty : tys2)
    for (int xc : xcs2) {
      if (n >= max_out) return n;
      if ((xc > g.nx && xc != 4) || !tiled2_fits(g, std::min(xc, g.nx))) continue;
      out[n++] = plan_tiled2(g, ty, std::min(xc, g.nx));
    }
  return n;
}

int plan_max_wg(Grid3 g) {
  int m = naive_wg_count(g);
  const int tys[] = {4, 8, 16};
  for (int ty : tys) m = std::max(m, tiled_shape(g, ty, 1).nwg);
  m = std::max(m, tiled2_shape(g, 8, 1).nwg);
  return m;
}

hipError_t launch_plan(Grid3 g, const StepPlan& plan, const StepBuffers& b, const StepConst& K,
                       hipStream_t st) {
  if (plan.kind == kStepNaive) return launch_step_naive(g, b, K, st);
  if (plan.pv)
    return launch_step_pair(pair_shape(g, plan.ty, plan.pv, plan.xc), g, b, kPairFull, nullptr,
                            plan.store, st);
  if (plan.depth == 2)
    return launch_step_tiled2(tiled2_shape(g, plan.ty, plan.xc), g, b, K, plan.store, st);
  if (plan.zv > 1)
    return launch_step_wide(plan.zv, wide_shape(g, plan.zv, plan.ty, plan.xc), g, b, K,
                            plan.store, st);
  return launch_step_tiled(tiled_shape(g, plan.ty, plan.xc), g, b, K, plan.store, st);
}

hipError_t launch_plan_temperature(Grid3 g, const StepPlan& plan, const StepBuffers& b,
                                   float* hi_mid, const StepConst& K, hipStream_t st) {
  if (plan.pv)
    return launch_step_pair(pair_shape(g, plan.ty, plan.pv, plan.xc), g, b, kPairTemp, hi_mid,
                            plan.store, st);
  if (plan.kind != kStepNaive && plan.depth == 1 && plan.zv > 1)
    return launch_step_wide_temperature(plan.zv, wide_shape(g, plan.zv, plan.ty, plan.xc), g, b,
                                        K, plan.store, st);
  return launch_plan(g, plan, b, K, st);
}

rfa_status run_steps(Grid3 g, const StepPlan& plan, StepState& s, const StepConst& K,
                     int n_steps, float* partials, int slots, double* dacc, hipEvent_t* events,
                     int period, int* n_timed, int* n_launches, int* n_timed_steps,
                     hipStream_t st) {
  if (s.traj && plan.depth != 1 && !plan.pv) return RFA_ERR_ARG;
  // one launch of p with the current images, which it then swaps
  auto launch = [&](const StepPlan& p, float* part) -> hipError_t {
    StepBuffers b{};
    b.hi_in = s.hi[*s.cur];
    b.lo_in = s.lo[*s.cur];
    b.hi_out = s.hi[1 - *s.cur];
    b.lo_out = s.lo[1 - *s.cur];
    float* mid = nullptr;
    if (s.traj) {
      float* h = s.traj + (size_t)*s.traj_t * s.traj_n;
      mid = h + s.traj_n;
      b.hi_in = h;
      b.hi_out = h + p.depth * s.traj_n;
    }
    b.lab = s.lab;
    b.src = s.src;
    b.omega = *s.om;
    const bool swap_om = p.pv && s.om_alt;
    b.omega_out = swap_om ? *s.om_alt : *s.om;
    b.perf = s.perf;
    b.tab = s.tab;
    b.n_classes = s.n_classes;
    b.codes = s.codes;
    b.partials = part;
    const hipError_t e =
        p.pv && s.traj ? launch_step_pair(pair_shape(g, p.ty, p.pv, p.xc), g, b, kPairKeep, mid,
                                          p.store, st)
                       : launch_plan(g, p, b, K, st);
    if (e != hipSuccess) return e;
    if (s.traj) *s.traj_t += p.depth;
    *s.cur = 1 - *s.cur;
    if (swap_om) std::swap(*s.om, *s.om_alt);
    return hipSuccess;
  };
  int n_main = n_steps / plan.depth;
  if (s.even && plan.depth == 2) n_main &= ~1;
  const int n_rest = n_steps - n_main * plan.depth;
  int pending = 0;
  int timed = 0;
  for (int n = 0; n < n_main; ++n) {
    // Blocks of `period` consecutive launches are bracketed by one event pair
    // (the diagnostic reductions fall between blocks, never inside one).
    const bool open = events && (n % period) == 0;
    const bool close = events && ((n % period) == period - 1 || n == n_main - 1);
    if (open && hipEventRecord(events[2 * timed], st) != hipSuccess) return RFA_ERR_HIP;
    if (launch(plan, partials ? partials + (size_t)pending * plan.nwg * 3 : nullptr) != hipSuccess)
      return RFA_ERR_HIP;
    if (close) {
      if (hipEventRecord(events[2 * timed + 1], st) != hipSuccess) return RFA_ERR_HIP;
      ++timed;
    }
    if (partials && ++pending == slots) {
      if (launch_reduce_partials(partials, pending, plan.nwg, dacc, st) != hipSuccess)
        return RFA_ERR_HIP;
      pending = 0;
    }
  }
  if (partials && pending > 0)
    if (launch_reduce_partials(partials, pending, plan.nwg, dacc, st) != hipSuccess)
      return RFA_ERR_HIP;
  const StepPlan one = plan_one(plan);
  const bool time_rest = events && plan.time_rest;
  for (int r = 0; r < n_rest; ++r) {
    if (time_rest && hipEventRecord(events[2 * timed], st) != hipSuccess) return RFA_ERR_HIP;
    if (launch(one, partials) != hipSuccess) return RFA_ERR_HIP;
    if (time_rest && hipEventRecord(events[2 * timed++ + 1], st) != hipSuccess) return RFA_ERR_HIP;
    if (partials && launch_reduce_partials(partials, 1, one.nwg, dacc, st) != hipSuccess)
      return RFA_ERR_HIP;
  }
  if (n_timed) *n_timed = timed;
  const int rest = time_rest ? n_rest : 0;
  if (n_launches) *n_launches = events ? n_main + rest : 0;
  if (n_timed_steps) *n_timed_steps = events ? n_main * plan.depth + rest : 0;
  return RFA_OK;
}

}  // namespace rfa
