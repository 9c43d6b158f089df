// rfa_pair_kernel.h -- two time steps per pass over memory (temporal blocking).
//
// A work-group owns a flat segment of a (y, z) plane (seg consecutive voxels;
// whole rows need no z halo and no lanes are lost to rows that are not a
// multiple of 64) and marches it along x.  Its footprint is the segment and
// the nz voxels before and after it: the first step is computed on the
// footprint, the second on the segment, one plane behind:
//   iteration x: barrier; loads of plane x + 2 issued;
//                first step of plane x (x neighbours from registers), its
//                result and input plane x + 1 (own voxels and nz halo voxels
//                on either side) go to the LDS buffers last read before
//                the barrier;
//                second step of plane x - 1 (its x + 1 neighbour is the plane
//                just computed), stored.
// One barrier per plane for two steps; every pass issues the same memory
// instructions (stores that must not happen get an out-of-range offset), so
// the compiler's wait counts stay exact.
//
// Arithmetic.  Each step is voxel_thermal() / damage_increment() of
// rfa_device.h with the operands of the one-step kernels, so the states are
// bitwise theirs.  Two things cost fewer instructions:
//  * the difference to the x + 1 neighbour is the next plane's difference to
//    x - 1, negated (exact), so it is formed once;
//  * most waves lie in one tissue: where all free voxels of a wave's plane
//    have one class and every neighbour that class's conductivity (its wave
//    code, made once per tissue by k_pair_codes), the coefficients are
//    scalars: no neighbour class bytes, no table reads.  Where such a wave
//    is also cold (|theta| below K.cold everywhere, so that the damage
//    exponent rounds to 2^0), the transcendentals are skipped.
//
// What bounds it: on large grids memory and issue alike (256^3 with sums 57.0
// us a step: 452 MB a launch below the L2, 1.08 times the 25 bytes a voxel, is
// 4.0 TB/s; vector instructions issue in 0.80 of a busy compute unit's cycles,
// 224 a wave and plane for two steps of two voxels), on small ones the planes
// computed twice and the latency of a plane (128^3: 0.71 of the cycles, 2.1
// waves a SIMD, 44 % of their time spent waiting; 63 MB a launch, 1.19 times).
// A vector memory instruction costs as much as 16 arithmetic ones, so a lane's
// two voxels are consecutive and move as one access (11 a wave and plane; 22
// with single ones); uniform branches cost as much as the few instructions
// they skip, so there are few.  The first step on halo rows and planes is
// computed twice, so the footprint is trimmed to what the second step reads:
// held rows at a plane's ends belong to nobody's segment, and halo voxels pass
// on a temperature but no damage, latch or sum.  Against one step a pass (us a
// step, with sums): 32^3 6.0 -> 3.3, 48^3 6.4 -> 3.9, 64^3
// 6.4 -> 4.9, 96^3 12.0 -> 7.1, 128^3 13.3 -> 10.8, 161x149x117 without sums
// 20.6 -> 12.5, 160x152x144 coupled 35.7 -> 16.6, 256x256x234 91 -> 52.4,
// 256^3 80 -> 57.0.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "rfa_pair.h"
#include "rfa_tile_common.h"

namespace rfa {

namespace {

using namespace tile;

constexpr int kPairRing = 4;  // register sets: planes x - 1 .. x + 2

template <int NT, int V, int MAXNZ>
struct PairSmem {
  static constexpr int P = NT * V;            // footprint
  static constexpr int CELLS = P + 2 * MAXNZ;
  float2 cf[3 * kMaxClasses * kMaxClasses];
  float4 cls[kMaxClasses];
  uint8_t lab[kPairRing][CELLS];
  alignas(16) float2 in[2][CELLS];    // input planes: footprint q at pair_lead + q
  alignas(16) float2 mid[2][CELLS];   // first-step planes, likewise (halo cells unused)
  float red[3 * NT / 64];
};

template <int V>
struct PairPlane {
  float h[V], l[V], om[V], s[V], pf[V];
  unsigned b[V];
  float hh, hl;  // halo element
  unsigned hb;
};

// Coefficients of one class, read through the scalar cache (uniform class
// and constant memory: the tables are written before the launch).
struct ClassCoef {
  float2 k[3];
  float4 c;
};
typedef const __attribute__((address_space(4))) float ConstF;

__device__ __forceinline__ ClassCoef class_coef(const Tables* tab, unsigned c) {
  ConstF* t = (ConstF*)(uintptr_t)tab;
  ClassCoef r;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ConstF* k = t + 2 * (a * kMaxClasses * kMaxClasses + c * (kMaxClasses + 1));
    r.k[a] = make_float2(k[0], k[1]);
  }
  ConstF* q = t + offsetof(Tables, cls) / 4 + 4 * c;
  r.c = make_float4(q[0], q[1], q[2], q[3]);
  return r;
}

// The step constants, read where they are used: as kernel arguments they
// would occupy eight scalar registers through the plane loop, which spills.
__device__ __forceinline__ PairConst step_constants(const Tables* tab) {
  uintptr_t p = (uintptr_t)tab;
  asm volatile("" : "+s"(p));  // keeps the loads here
  ConstF* q = (ConstF*)p + offsetof(Tables, K) / 4;
  PairConst K;
  K.dtka = q[0];
  K.c2 = q[1];
  K.tak = q[2];
  K.clamp2 = q[3];
  K.cap = q[4];
  K.thr = q[5];
  K.decay2 = q[6];
  K.cold = q[7];
  return K;
}

// min(v, m) for a wave-uniform bound m, without the canonicalisation
// fminf() adds to each operand; v_min_f32 has fminf's NaN rule.
__device__ __forceinline__ float min_uniform(float v, float m) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "s"(m), "v"(v));
  return r;
}

__device__ __forceinline__ bool lane_of(unsigned long long m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

}  // namespace

namespace {

// The march of one work-group: segment sg of planes [x0, x1).  out: its
// partial sums (DIAG).
// EVEN: rows of an even number of voxels and two voxels a lane, whose LDS cells
// are then 16-byte aligned in every row and move as one access.  As two of 8
// bytes, 16 apart from lane to lane, they meet in the same banks (128^3: 41 %
// of the LDS cycles; 11.5 us a step against 10.7).
template <int NT, int V, int MAXNZ, bool PERF, bool DIAG, int AUX, int MODE, bool EVEN>
__device__ __forceinline__ void pair_march(PairSmem<NT, V, MAXNZ>& sm, const StepBuffers& b,
                                           float* hi_mid, int nx, int ny, int nz, int x0, int x1,
                                           int seg, int segs, int sg, float* out) {
  using S = PairSmem<NT, V, MAXNZ>;
  constexpr bool TEMP = MODE == kPairTemp;
  constexpr bool KEEP = MODE != kPairFull;
  constexpr int P = S::P;
  constexpr int NW = NT / 64;
  const int xb = max(x0 - 2, 0);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int np = ny * nz;
  const unsigned psz = (unsigned)np;
  const int lead = pair_lead(nz, V);
  const int fp = sg * seg;  // first voxel of the footprint; the segment starts lead later

  __amdgpu_buffer_rsrc_t r_hi, r_lo, r_lab, r_src, r_om, r_omo, r_pf, r_hio, r_loo, r_mid;
  {
    const size_t off = (size_t)xb * psz;
    const size_t rest = (size_t)(nx - xb) * psz;
    r_hi = make_rsrc(b.hi_in + off, rest * 4);
    r_lo = make_rsrc(b.lo_in + off, rest * 4);
    r_lab = make_rsrc(b.lab + off, rest);
    r_src = make_rsrc(b.src + off, rest * 4);
    r_om = make_rsrc(b.omega + off, rest * 4);
    r_omo = PERF ? make_rsrc(b.omega_out + off, rest * 4) : r_om;
    r_pf = PERF ? make_rsrc(b.perf + off, rest * 4) : r_src;
    r_hio = make_rsrc(b.hi_out + off, rest * 4);
    r_loo = make_rsrc(b.lo_out + off, rest * 4);
    r_mid = KEEP ? make_rsrc(hi_mid + off, rest * 4) : r_hio;
  }

  // Own voxels, V consecutive ones: the first's column in the plane (0, a
  // held corner, outside the grid) and store offset (out of range unless
  // owned)
  const int first = pair_first(fp + V * tid, V, np);
  const int cell = lead + first - fp;  // LDS cell of the first
  const unsigned col = first < np ? (unsigned)first : 0u;
  unsigned long long ownm[V];  // lanes whose voxel is owned
  bool owns = false;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int f = first + v, q = f - fp;
    // the plane's first and last rows are held (outer layer): they belong to
    // the first and last segment, as part of their halo; a voxel shared by
    // two lanes is the first one's
    const bool owned = f < np && (q >= lead || sg == 0) && (q < lead + seg || sg == segs - 1) &&
                       q >= V * tid;
    ownm[v] = __ballot(owned);
    owns = owns || owned;
  }
  const unsigned col4 = col * 4u, own4 = owns ? col4 : kOob;
  const bool wave_valid = first < np, wave_owns = owns;
  const bool do_mid = __ballot(wave_valid) != 0ull;  // uniform
  const unsigned long long out_lanes = __ballot(wave_owns);  // 0: the wave stores nothing

  // Halo element: the nz voxels before and after the footprint.  Elements
  // outside the plane stand next to held voxels only: any finite value.
  const bool has_halo = tid < 2 * nz;
  int hcell = 0;
  unsigned hoff = kOob;
  if (has_halo) {
    const int f = tid < nz ? fp - nz + tid : fp - nz + P + tid;
    hcell = lead - nz + (tid < nz ? tid : P + tid);
    if (f >= 0 && f < np) hoff = (unsigned)f;
  }
  const unsigned hoff4 = hoff == kOob ? kOob : hoff * 4u;

  auto plane_of = [&](int x) { return min(max(x, 0), nx - 1) - xb; };  // uniform
  auto load = [&](int x, PairPlane<V>& q) {
    const int so1 = plane_of(x) * (int)psz, so4 = so1 * 4;
    ld_u8v<V>(q.b, r_lab, col, so1);
    ld_f32v<V>(q.h, r_hi, col4, so4);
    ld_f32v<V>(q.l, r_lo, col4, so4);
    q.hh = ld_f32(r_hi, hoff4, so4);
    q.hl = ld_f32(r_lo, hoff4, so4);
    q.hb = ld_u8(r_lab, hoff, so1);
  };
  // what only the own step of plane x needs: source increments of lanes with
  // a flagged voxel (its class bytes are there; 0 on others), damage
  // integral, perfusion factor
  auto load_s = [&](int x, PairPlane<V>& q) {
    const int so4 = plane_of(x) * (int)psz * 4;
    unsigned any = 0u;
#pragma unroll
    for (int v = 0; v < V; ++v) any |= q.b[v];
    ld_f32v<V>(q.s, r_src, (any & kSource) ? col4 : kOob, so4);
    // the damage integral enters the temperature only through the coupling:
    // without a field it is read on owned voxels alone
    if constexpr (!TEMP) ld_f32v<V>(q.om, r_om, PERF ? col4 : own4, so4);
#pragma unroll
    for (int v = 0; v < V; ++v)
      if constexpr (TEMP) q.om[v] = 0.0f;
    if constexpr (PERF) ld_f32v<V>(q.pf, r_pf, col4, so4);
  };

  PairPlane<V> ring[kPairRing];
  const int xs = x0 - 1;  // first plane of the first step
  float din[V], dmid[V];  // difference to the x + 1 neighbour of the plane before
  {
    float ph[V], pl[V];
    unsigned pb[V];
    const int so4 = plane_of(xs - 1) * (int)psz * 4;
    ld_f32v<V>(ph, r_hi, col4, so4);
    ld_f32v<V>(pl, r_lo, col4, so4);
    ld_u8v<V>(pb, r_lab, col, so4 / 4);  // plane xs - 1
#pragma unroll
    for (int v = 0; v < V; ++v) sm.lab[3][cell + v] = (uint8_t)pb[v];
    load(xs, ring[0]);
    load(xs + 1, ring[1]);
    stage_tables(sm.cf, sm.cls, b.tab, b.n_classes, NT);
    load_s(xs, ring[0]);
#pragma unroll
    for (int v = 0; v < V; ++v) din[v] = ff_diff(ring[0].h[v], ring[0].l[v], ph[v], pl[v]);
  }
  unsigned long long mheld[V];  // held lanes of the plane before
#pragma unroll
  for (int v = 0; v < V; ++v) {
    dmid[v] = 0.0f;
    mheld[v] = 0ull;
    ring[3].h[v] = ring[3].l[v] = ring[3].om[v] = ring[3].s[v] = 0.0f;
    ring[3].pf[v] = 1.0f;
    ring[3].b[v] = 0u;
  }

  Partial acc{0.0f, 0.0f, 0u};
  unsigned mono = 0u;  // cooling voxels of the wave (scalar)
  // halo cells of the first-step planes are never written: they enter only
  // lanes whose results are dropped, but must be finite
  for (int c = tid; c < 2 * nz; c += NT) {
    const int e = lead - nz + (c < nz ? c : P + c);
    sm.mid[0][e] = sm.mid[1][e] = make_float2(0.0f, 0.0f);
  }
  // nor does a lane write the cell after a shared voxel
  if (first != fp + V * tid) {
    const float2 zero = make_float2(0.0f, 0.0f);
    sm.in[0][cell + V] = sm.in[1][cell + V] = zero;
    sm.mid[0][cell + V] = sm.mid[1][cell + V] = zero;
#pragma unroll
    for (int k = 0; k < kPairRing; ++k) sm.lab[k][cell + V] = 0;
  }

  // One step of this lane's V voxels, in place in q.  t: plane in LDS, dn:
  // difference to x + 1, dp: difference of x - 1 to the plane (both from
  // registers), tl / tp: class bytes of the plane and of x - 1 in LDS, bn: of
  // x + 1 (latch bits of either step; they are not read), heldm: lanes whose
  // voxel is held, own: not 0 where damage, latches and sums are wanted.
  // That is where the plane and some of the wave's voxels are the
  // work-group's own; halo voxels pass on their temperature alone.
  // Results are formed first and selected by lane masks: a branch costs more
  // than the few instructions it would save.
  auto step = [&](const float2* t, const uint8_t* tl, const uint8_t* tp, unsigned code,
                  PairPlane<V>& q, const float (&dn)[V], const float (&dp)[V],
                  const unsigned (&bn)[V], const unsigned long long (&heldm)[V],
                  unsigned long long own) {
    const PairConst K = step_constants(b.tab);
    auto cntm = [&](int v) { return ownm[v] & ~heldm[v]; };
    float f[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      f[v] = 1.0f;
      if constexpr (PERF) f[v] = q.pf[v] * __builtin_amdgcn_exp2f(-q.om[v] * K.decay2);
    }
    float nh[V], nl[V];
    // rows y - 1 and y + 1 (EVEN: both voxels in one 16-byte read)
    float4 rm, rp;
    if constexpr (EVEN) {
      rm = *reinterpret_cast<const float4*>(t + (cell - nz));
      rp = *reinterpret_cast<const float4*>(t + (cell + nz));
    }
    auto row = [&](int v, int o, const float4& r) {
      if constexpr (EVEN) return v == 0 ? make_float2(r.x, r.y) : make_float2(r.z, r.w);
      return t[cell + v + o];
    };
    // differences along z, each formed once: to the voxel before the lane's,
    // between them, to the one after (a difference reversed is its negative)
    float dz[V + 1];
    {
      const float2 zm = t[cell - 1], zp = t[cell + V];
      dz[0] = -ff_diff(zm.x, zm.y, q.h[0], q.l[0]);
#pragma unroll
      for (int v = 1; v < V; ++v) dz[v] = ff_diff(q.h[v], q.l[v], q.h[v - 1], q.l[v - 1]);
      dz[V] = ff_diff(zp.x, zp.y, q.h[V - 1], q.l[V - 1]);
    }
    if (code != kPairIrregular) {
      const ClassCoef coef = class_coef(b.tab, code & (kMaxClasses - 1));
      const float2 k[6] = {coef.k[0], coef.k[0], coef.k[1], coef.k[1], coef.k[2], coef.k[2]};
      unsigned long long warm = 0ull, falls = 0ull;
      float incs[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float h = q.h[v], l = q.l[v];
        const float2 ym = row(v, -nz, rm), yp = row(v, nz, rp);
        const float d[6] = {-dp[v], dn[v], ff_diff(ym.x, ym.y, h, l), ff_diff(yp.x, yp.y, h, l),
                            -dz[v], dz[v + 1]};
        float h2, l2, cond, perf;
        thermal_update(h, l, k, coef.c, d, q.s[v], f[v], h2, l2, cond, perf, incs[v]);
        nh[v] = lane_of(heldm[v]) ? h : h2;
        nl[v] = lane_of(heldm[v]) ? l : l2;
        if (DIAG && own != 0ull) {
          // lanes that do not count add 0 times a finite term
          const float w = lane_of(cntm(v)) ? coef.c.w : 0.0f;
          acc.perf = __builtin_fmaf(w, perf, acc.perf);
          acc.bnd = __builtin_fmaf(w, cond, acc.bnd);
          falls |= __ballot(incs[v] < 0.0f);
        }
        warm |= __ballot(!(fabsf(h) < K.cold));
      }
      if (DIAG && own != 0ull && falls != 0ull) {
#pragma unroll
        for (int v = 0; v < V; ++v) mono += __popcll(__ballot(cools(q.h[v], incs[v])) & cntm(v));
      }
      if (!TEMP && own != 0ull) {
        auto add = [&](int v, float rate) {
          const float o = min_uniform(q.om[v] + rate, K.cap);
          const unsigned long long tism =
              (code & kPairTissueAll) ? ~0ull : ((code & kPairTissueFree) ? ~heldm[v] : 0ull);
          q.om[v] = lane_of(tism) ? o : q.om[v];
        };
        if (warm != 0ull) {
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const float x = K.c2 * q.h[v] * __builtin_amdgcn_rcpf(K.tak + q.h[v]);
            add(v, K.dtka * __builtin_amdgcn_exp2f(min_uniform(x, K.clamp2)));
          }
        } else {
#pragma unroll
          for (int v = 0; v < V; ++v) add(v, K.dtka);
        }
        unsigned long long hot = 0ull;
#pragma unroll
        for (int v = 0; v < V; ++v) hot |= __ballot(nh[v] >= K.thr);
        if (hot != 0ull) {
#pragma unroll
          for (int v = 0; v < V; ++v) q.b[v] = latch(q.b[v], nh[v], nl[v], K);
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float h = q.h[v], l = q.l[v];
        const unsigned lb = q.b[v];
        const int c = cell + v;
        const float2 ym = row(v, -nz, rm), yp = row(v, nz, rp);
        const float d[6] = {-dp[v], dn[v], ff_diff(ym.x, ym.y, h, l), ff_diff(yp.x, yp.y, h, l),
                            -dz[v], dz[v + 1]};
        const float2 k[6] = {table_entry(sm.cf, 0, lb, tp[c]),
                             table_entry(sm.cf, 0, lb, bn[v]),
                             table_entry(sm.cf, 1, lb, tl[c - nz]),
                             table_entry(sm.cf, 1, lb, tl[c + nz]),
                             table_entry(sm.cf, 2, lb, tl[c - 1]),
                             table_entry(sm.cf, 2, lb, tl[c + 1])};
        const float4 c4 = sm.cls[class_of(lb)];
        float h2, l2, cond, perf, inc;
        thermal_update(h, l, k, c4, d, q.s[v], f[v], h2, l2, cond, perf, inc);
        nh[v] = lane_of(heldm[v]) ? h : h2;
        nl[v] = lane_of(heldm[v]) ? l : l2;
        if (DIAG && own != 0ull) {
          const float w = lane_of(cntm(v)) ? c4.w : 0.0f;
          acc.perf = __builtin_fmaf(w, perf, acc.perf);
          acc.bnd = __builtin_fmaf(w, cond, acc.bnd);
          mono += __popcll(__ballot(cools(h, inc)) & cntm(v));
        }
        if (!TEMP && own != 0ull) {
          q.om[v] = damage_add<true>(q.om[v], damage_increment(h, K), (lb & kTissue) != 0u, K);
          q.b[v] = latch(lb, nh[v], nl[v], K);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      q.h[v] = nh[v];
      q.l[v] = nl[v];
    }
  };

  // a lane's temperatures to LDS
  auto put = [&](float2* p, const PairPlane<V>& q) {
    if constexpr (EVEN) {
      *reinterpret_cast<float4*>(p) = make_float4(q.h[0], q.l[0], q.h[1], q.l[1]);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) p[v] = make_float2(q.h[v], q.l[v]);
    }
  };

  // input plane q (of ring slot SL) to LDS
  auto publish = [&](auto SL_, const PairPlane<V>& q) {
    constexpr int SL = decltype(SL_)::value;
    put(sm.in[SL & 1] + cell, q);
#pragma unroll
    for (int v = 0; v < V; ++v) sm.lab[SL][cell + v] = (uint8_t)q.b[v];
    if (has_halo) {
      sm.in[SL & 1][hcell] = make_float2(q.hh, q.hl);
      sm.lab[SL][hcell] = (uint8_t)q.hb;
    }
  };

  unsigned code = 0u, code_next, code_shift;
  auto fetch_code = [&](int x) {
    code_next = code_word(b.codes, ((size_t)(plane_of(x) + xb) * segs + sg) * NW + wave,
                          code_shift);
  };
  auto next_code = [&]() { return (code_next >> code_shift) & 0xffu; };
  fetch_code(xs);

  auto iterate = [&](auto SL_, int x) {
    constexpr int SL = decltype(SL_)::value;   // plane x
    constexpr int SP = (SL + 3) % kPairRing;   // plane x - 1
    constexpr int SN = (SL + 1) % kPairRing;   // plane x + 1
    constexpr int SA = (SL + 2) % kPairRing;   // receives plane x + 2; in LDS still plane x - 2
    constexpr int BUF = SL & 1;
    PairPlane<V>& C = ring[SL];
    PairPlane<V>& N = ring[SN];
    PairPlane<V>& B = ring[SP];  // after its first step
    __syncthreads();
    load(x + 2, ring[SA]);
    // wave codes of planes x - 1 and x; that of x + 1 is under way
    const unsigned pcode = code;
    code = next_code();
    fetch_code(x + 1);
    // first step of plane x
    float dn[V];
    unsigned long long held[V];
    const bool in_chunk = x >= x0 && x < x1;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      dn[v] = ff_diff(N.h[v], N.l[v], C.h[v], C.l[v]);
      held[v] = __ballot((C.b[v] & kHeld) != 0u);
    }
    unsigned long long own = in_chunk ? out_lanes : 0ull;
    // a scalar, tested where it is used (with sums it would be spilled)
    if constexpr (!DIAG) asm("" : "+s"(own));
    if (do_mid)
      step(sm.in[BUF], sm.lab[SL], sm.lab[SP], code, C, dn, din, N.b, held, own);
    put(sm.mid[BUF] + cell, C);
#pragma unroll
    for (int v = 0; v < V; ++v) din[v] = dn[v];
    publish(std::integral_constant<int, SN>{}, N);
    load_s(x + 1, N);
    if constexpr (KEEP) {
      const int so = plane_of(x) * (int)psz * 4;
      st_f32v<AUX, V>(C.h, r_mid, in_chunk ? own4 : kOob, so);
    }
    // second step of plane x - 1
    {
      float dm[V];
      const bool out = x > x0;  // uniform: plane x - 1 is in the chunk
#pragma unroll
      for (int v = 0; v < V; ++v) {
        dm[v] = ff_diff(C.h[v], C.l[v], B.h[v], B.l[v]);
      }
      if (out_lanes != 0ull && out) {
        step(sm.mid[BUF ^ 1], sm.lab[SP], sm.lab[SA], pcode, B, dm, dmid, C.b, mheld, out_lanes);
        if constexpr (!TEMP) {
          // class bytes are stored where a latch flipped in either step: a
          // branch, as few waves hold a latched voxel
          unsigned long long latched = 0ull;
#pragma unroll
          for (int v = 0; v < V; ++v) latched |= __ballot((B.b[v] & kLatch) != 0u);
          if (latched != 0ull) {
#pragma unroll
            for (int v = 0; v < V; ++v)
              st_u8<AUX>(B.b[v], r_lab,
                         lane_of(ownm[v]) && B.b[v] != sm.lab[SP][cell + v] ? col + v : kOob,
                         plane_of(x - 1) * (int)psz);
          }
        }
      }
      const int so = plane_of(x - 1) * (int)psz;
      const unsigned v4 = out ? own4 : kOob;
      st_f32v<AUX, V>(B.h, r_hio, v4, so * 4);
      st_f32v<AUX, V>(B.l, r_loo, v4, so * 4);
      if constexpr (!TEMP) st_f32v<AUX, V>(B.om, r_omo, v4, so * 4);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        dmid[v] = dm[v];
        mheld[v] = held[v];
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  static_assert(kPairRing == 4, "unrolled for a ring of four planes");
  publish(I0{}, ring[0]);
  for (int x = xs;; x += kPairRing) {
    iterate(I0{}, x);
    if (x + 1 > x1) break;
    iterate(I1{}, x + 1);
    if (x + 2 > x1) break;
    iterate(I2{}, x + 2);
    if (x + 3 > x1) break;
    iterate(I3{}, x + 3);
    if (x + 4 > x1) break;
  }
  if (DIAG && (tid & 63) == 0) acc.mono += mono;
  if constexpr (DIAG) write_partials(acc, sm.red, NW, out);
}

}  // namespace

template <int NT, int V, int MAXNZ, bool PERF, bool DIAG, int AUX, int MODE, bool EVEN>
__global__ __launch_bounds__(NT, 4) void k_step_pair(StepBuffers b, float* hi_mid, int nx, int ny,
                                                     int nz, int xc, int seg, int segs,
                                                     int nwg) {
  __shared__ PairSmem<NT, V, MAXNZ> sm;
  const int wg = remap_xcd(blockIdx.x, nwg);
  const int x0 = (wg / segs) * xc;
  pair_march<NT, V, MAXNZ, PERF, DIAG, AUX, MODE, EVEN>(
      sm, b, hi_mid, nx, ny, nz, x0, min(x0 + xc, nx), seg, segs, wg % segs,
      DIAG ? b.partials + (size_t)wg * 3 : nullptr);
}

// The same over the work items of a batch group (one work-group per item, in
// XCD-aware order).  Items and instances are read through the scalar cache;
// stores are written back as the caches will.  Bound by issue: the 64-grid
// sweep runs at 292 GVox/s, 200 with one step a launch.
template <int NT, int V, int MAXNZ, bool PERF, bool DIAG>
__global__ __launch_bounds__(NT, 4) void k_step_pair_batch(const PairInstance* inst,
                                                           const PairItem* items, int first_item,
                                                           int n_items, int parity,
                                                           float* partials) {
  __shared__ PairSmem<NT, V, MAXNZ> sm;
  typedef const __attribute__((address_space(4))) PairInstance ConstInstance;
  typedef const __attribute__((address_space(4))) PairItem ConstItem;
  const int it = first_item + remap_xcd(blockIdx.x, n_items);
  ConstItem* w = (ConstItem*)(uintptr_t)items + it;
  ConstInstance* I = (ConstInstance*)(uintptr_t)inst + w->inst;
  StepBuffers b;
  b.hi_in = parity ? I->hi[1] : I->hi[0];
  b.lo_in = parity ? I->lo[1] : I->lo[0];
  b.hi_out = parity ? I->hi[0] : I->hi[1];
  b.lo_out = parity ? I->lo[0] : I->lo[1];
  b.lab = I->lab;
  b.src = I->src;
  b.omega = I->om;
  b.omega_out = I->om;
  b.perf = I->perf;
  b.tab = I->tab;
  b.n_classes = I->n_classes;
  b.codes = I->codes;
  b.partials = nullptr;
  const int nx = I->nx, xc = I->xc;
  const int x0 = w->chunk * xc;
  float* out = DIAG ? partials + (size_t)it * 3 : nullptr;
  // a batch mixes even and odd rows; both forms in one kernel spill scalar
  // registers (24 grids of 64 .. 160, with sums: 177 us a step against 171)
  pair_march<NT, V, MAXNZ, PERF, DIAG, kStoreBack, kPairFull, false>(
      sm, b, nullptr, nx, I->ny, I->nz, x0, min(x0 + xc, nx), I->seg, I->segs, w->sg, out);
}


namespace {

template <int NT, int V, int MAXNZ, bool PERF, bool DIAG, int AUX, int MODE>
hipError_t launch_rows(const PairShape& s, Grid3 g, const StepBuffers& b, float* hi_mid,
                       hipStream_t st) {
  const dim3 grid(s.nwg), block(NT);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, b, hi_mid, g.nx, g.ny, g.nz, s.xc, s.seg,
                       s.segs, s.nwg);
    return hipGetLastError();
  };
  if constexpr (V == 2)
    if (g.nz % 2 == 0) return go(k_step_pair<NT, V, MAXNZ, PERF, DIAG, AUX, MODE, true>);
  return go(k_step_pair<NT, V, MAXNZ, PERF, DIAG, AUX, MODE, false>);
}

template <int NT, int V, int MAXNZ, bool PERF, bool DIAG, int AUX>
hipError_t launch_mode(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode,
                       float* hi_mid, hipStream_t st) {
  if (mode == kPairFull)
    return launch_rows<NT, V, MAXNZ, PERF, DIAG, AUX, kPairFull>(s, g, b, hi_mid, st);
  if constexpr (!DIAG) {
    if (mode == kPairKeep)
      return launch_rows<NT, V, MAXNZ, PERF, false, AUX, kPairKeep>(s, g, b, hi_mid, st);
    if (mode == kPairTemp)
      return launch_rows<NT, V, MAXNZ, PERF, false, AUX, kPairTemp>(s, g, b, hi_mid, st);
  }
  return hipErrorInvalidValue;
}

template <int NT, int V, int MAXNZ, int AUX>
hipError_t launch_kind(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode,
                       float* hi_mid, hipStream_t st) {
  if (b.perf)
    return b.partials
               ? launch_mode<NT, V, MAXNZ, true, true, AUX>(s, g, b, mode, hi_mid, st)
               : launch_mode<NT, V, MAXNZ, true, false, AUX>(s, g, b, mode, hi_mid, st);
  return b.partials ? launch_mode<NT, V, MAXNZ, false, true, AUX>(s, g, b, mode, hi_mid, st)
                    : launch_mode<NT, V, MAXNZ, false, false, AUX>(s, g, b, mode, hi_mid, st);
}

template <int NT, int V, int MAXNZ>
hipError_t launch_store(const PairShape& s, Grid3 g, const StepBuffers& b, PairMode mode,
                        float* hi_mid, int store, hipStream_t st) {
  switch (store) {
    case kPolicyThrough:
      return launch_kind<NT, V, MAXNZ, kStoreThrough>(s, g, b, mode, hi_mid, st);
    case kPolicyStream:
      return launch_kind<NT, V, MAXNZ, kStoreStream>(s, g, b, mode, hi_mid, st);
    default:
      return launch_kind<NT, V, MAXNZ, kStoreBack>(s, g, b, mode, hi_mid, st);
  }
}

template <int NT, int V, int MAXNZ>
hipError_t launch_batch(const PairInstance* inst, const PairItem* items, int first_item,
                        int n_items, bool perf, int parity, float* partials, hipStream_t st) {
  const dim3 grid(n_items), block(NT);
  if (perf && partials)
    hipLaunchKernelGGL((k_step_pair_batch<NT, V, MAXNZ, true, true>), grid, block, 0, st, inst,
                       items, first_item, n_items, parity, partials);
  else if (perf)
    hipLaunchKernelGGL((k_step_pair_batch<NT, V, MAXNZ, true, false>), grid, block, 0, st, inst,
                       items, first_item, n_items, parity, partials);
  else if (partials)
    hipLaunchKernelGGL((k_step_pair_batch<NT, V, MAXNZ, false, true>), grid, block, 0, st, inst,
                       items, first_item, n_items, parity, partials);
  else
    hipLaunchKernelGGL((k_step_pair_batch<NT, V, MAXNZ, false, false>), grid, block, 0, st, inst,
                       items, first_item, n_items, parity, partials);
  return hipGetLastError();
}

}  // namespace

}  // namespace rfa
