// rfa_adjoint_pair.hip -- two adjoint steps per pass over memory.
//
// The schedule of the two-step forward kernel (rfa_pair_kernel.h): a
// work-group owns a flat segment of a (y, z) plane with nz halo voxels on
// either side and marches along x; the first adjoint step (lambda^{n+1} ->
// lambda^n) is computed on the footprint one plane ahead of the second
// (lambda^n -> lambda^{n-1}) on the segment, with one barrier per plane.  It moves
// lambda, the weight, the class byte, the perfusion factor and the
// accumulators once for two steps (about 18 bytes per voxel-step instead of
// 29).  Waves whose code gives one class use scalar coefficients: there a
// held neighbour needs no test, since lambda is 0 on held voxels and adds
// nothing.  Where such a wave is cold (|theta| below K.cold, so that T_aK +
// theta = T_aK and 2^x = 1) the damage-rate derivative is one constant.
//
// What bounds it: the latency of a plane and the planes computed twice (128^3,
// 5 planes a work-group: 105 MB a launch below the L2, 1.49 times the 33 bytes
// a voxel, since the planes at a chunk's ends are read by both sides: 5.2 TB/s
// from the last-level cache; vector instructions issue in 0.55 of the cycles).
// Half the vector memory instructions (two voxels a lane in one access, 25 -> 13
// a wave and plane) left 128^3 at 10.1 us a step, aligned LDS accesses on even
// rows 9.95.  Against one step a launch: 128^3 16.5 -> 9.95 us a step, 88x80x75
// 13.0 -> 5.0, 64^3 6.35 -> 3.85.
//
// The per-voxel operations and their order are those of adjoint_voxel(), so
// two steps are bitwise two launches of the one-step kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "rfa_adjoint.h"
#include "rfa_adjoint_device.h"
#include "rfa_tile_common.h"

namespace rfa {

namespace {

using namespace tile;

constexpr int kRing = 4;  // register sets: planes x - 1 .. x + 2

template <int NT, int V, int MAXNZ>
struct AdjPairSmem {
  static constexpr int P = NT * V;
  static constexpr int CELLS = P + 2 * MAXNZ;
  float2 pc[3 * kMaxClasses * kMaxClasses];  // pair table
  float4 cls[kMaxClasses];
  alignas(8) float in[2][CELLS];   // lambda^{n+1}: footprint q at pair_lead + q
  alignas(8) float mid[2][CELLS];  // lambda^n
  uint8_t lab[kRing][CELLS];
};

template <int V>
struct AdjPairPlane {
  float lam[V], th[V], w[V], pf[V], fa[V], sa[V];
  unsigned b[V];
  float hl;
  unsigned hb;
};

typedef const __attribute__((address_space(4))) float ConstF;

}  // namespace

// EVEN: rows of an even number of voxels and two voxels a lane, whose cells are
// then one aligned access in every row (as in the forward kernel).
template <int NT, int V, int MAXNZ, bool PERF, bool EVEN>
__global__ __launch_bounds__(NT, 4) void k_adjoint_pair(AdjointBuffers a, int nx, int ny, int nz,
                                                        int xc, int seg, int segs, int nwg) {
  using S = AdjPairSmem<NT, V, MAXNZ>;
  constexpr int P = S::P;
  constexpr int NW = NT / 64;
  __shared__ S sm;
  const int wg = remap_xcd(blockIdx.x, nwg);
  const int sg = wg % segs;
  const int x0 = (wg / segs) * xc;
  const int x1 = min(x0 + xc, nx);
  const int xb = max(x0 - 2, 0);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int np = ny * nz;
  const int lead = pair_lead(nz, V);
  const int fp = sg * seg;  // first voxel of the footprint; the segment starts lead later

  __amdgpu_buffer_rsrc_t r_lam, r_lab, r_th, r_tp, r_w, r_pf, r_sa, r_fa, r_out;
  {
    const size_t off = (size_t)xb * np;
    const size_t rest = (size_t)(nx - xb) * np;
    r_lam = make_rsrc(a.lam_in + off, rest * 4);
    r_lab = make_rsrc(a.lab + off, rest);
    r_th = make_rsrc(a.theta + off, rest * 4);
    r_tp = make_rsrc(a.theta_prev + off, rest * 4);
    r_w = make_rsrc(a.w + off, rest * 4);
    r_pf = PERF ? make_rsrc(a.perf + off, rest * 4) : r_w;
    r_sa = make_rsrc(a.sacc + off, rest * 4);
    r_fa = make_rsrc(a.facc + off, rest * 4);
    r_out = make_rsrc(a.lam_out + off, rest * 4);
  }

  // the forward kernel's lanes (rfa_pair_kernel.h)
  const int first = pair_first(fp + V * tid, V, np);
  const int cell = lead + first - fp;
  const unsigned col = first < np ? (unsigned)first : 0u;
  bool owns = false;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int f = first + v, q = f - fp;
    owns = owns || (f < np && (q >= lead || sg == 0) && (q < lead + seg || sg == segs - 1));
  }
  const unsigned col4 = col * 4u, own4 = owns ? col4 : kOob;
  const bool wave_valid = first < np, wave_owns = owns;
  const bool do_mid = __ballot(wave_valid) != 0ull;  // uniform
  const bool do_out = __ballot(wave_owns) != 0ull;   // uniform
  const bool has_halo = tid < 2 * nz;
  int hcell = 0;
  unsigned hoff = kOob;
  if (has_halo) {
    const int f = tid < nz ? fp - nz + tid : fp - nz + P + tid;
    hcell = lead - nz + (tid < nz ? tid : P + tid);
    if (f >= 0 && f < np) hoff = (unsigned)f;
  }
  const unsigned hoff4 = hoff == kOob ? kOob : hoff * 4u;
  const bool sacc_all = a.sacc_all;
  // class bytes of voxels whose Lambda is summed: free, and flagged unless all are
  const unsigned sum_bits = sacc_all ? kHeld : kHeld | kSource;
  const unsigned sum_want = sacc_all ? 0u : kSource;

  auto plane_of = [&](int x) { return min(max(x, 0), nx - 1) - xb; };  // uniform
  auto load = [&](int x, AdjPairPlane<V>& q) {
    const int so1 = plane_of(x) * np, so4 = so1 * 4;
    ld_u8v<V>(q.b, r_lab, col, so1);
    ld_f32v<V>(q.lam, r_lam, col4, so4);
    q.hl = ld_f32(r_lam, hoff4, so4);
    q.hb = ld_u8(r_lab, hoff, so1);
  };
  // Whether a lane's Lambda moves: all, or where one of its voxels is flagged.
  auto sums_at = [&](const unsigned (&b)[V]) {
    unsigned any = 0u;
#pragma unroll
    for (int v = 0; v < V; ++v) any |= b[v];
    return sacc_all || (any & kSource) != 0u;
  };
  // what only the own steps of plane x need
  auto load_own = [&](int x, AdjPairPlane<V>& q) {
    const int so4 = plane_of(x) * np * 4;
    ld_f32v<V>(q.th, r_th, col4, so4);
    ld_f32v<V>(q.w, r_w, col4, so4);
    if constexpr (PERF) {
      ld_f32v<V>(q.pf, r_pf, col4, so4);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) q.pf[v] = 1.0f;
    }
    ld_f32v<V>(q.fa, r_fa, own4, so4);
    ld_f32v<V>(q.sa, r_sa, sums_at(q.b) ? own4 : kOob, so4);
  };

  AdjPairPlane<V> ring[kRing];
  const int xs = x0 - 1;
  float lp[V];  // lambda^{n+1} of plane x - 1
  {
    const int so = plane_of(xs - 1) * np;
    unsigned b0[V];
    ld_f32v<V>(lp, r_lam, col4, so * 4);
    ld_u8v<V>(b0, r_lab, col, so);
    load(xs, ring[0]);
    load(xs + 1, ring[1]);
    stage_pairs(sm.pc, sm.cls, a.tab, NT);
    load_own(xs, ring[0]);
#pragma unroll
    for (int v = 0; v < V; ++v) sm.lab[3][cell + v] = (uint8_t)b0[v];
  }
#pragma unroll
  for (int v = 0; v < V; ++v) ring[3].w[v] = 0.0f, ring[3].pf[v] = 1.0f;
  // halo cells of the first-step planes enter only lanes whose results are dropped
  for (int c = tid; c < 2 * nz; c += NT) {
    const int e = lead - nz + (c < nz ? c : P + c);
    sm.mid[0][e] = sm.mid[1][e] = 0.0f;
  }
  // nor is the cell after a voxel that two lanes share ever written
  if (first != fp + V * tid) {
    sm.in[0][cell + V] = sm.in[1][cell + V] = sm.mid[0][cell + V] = sm.mid[1][cell + V] = 0.0f;
#pragma unroll
    for (int k = 0; k < kRing; ++k) sm.lab[k][cell + V] = 0;
  }
  // first-step results of planes x - 1 and x - 2, accumulators of x - 1
  float m1[V], m2[V], mfa[V], msa[V], tp[V];
  unsigned mb[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    m1[v] = m2[v] = mfa[v] = msa[v] = tp[v] = 0.0f;
    mb[v] = kHeld;
  }

  // One step of this lane's voxels: lambda l of the plane (t: in LDS, with
  // class bytes tl, those of x - 1 in tpv), its x neighbours lm / ln, class
  // bytes lb (and bn of x + 1), theta th, weight w.
  auto step = [&](const float* t, const uint8_t* tl, const uint8_t* tpv, unsigned code,
                  const float (&l)[V], const float (&lm)[V], const float (&ln)[V],
                  const unsigned (&lb)[V], const unsigned (&bn)[V], const float (&th)[V],
                  const float (&w)[V], const float (&pf)[V], float (&nl)[V], float (&sa)[V],
                  float (&fa)[V]) {
    uintptr_t tab = (uintptr_t)a.tab;
    asm volatile("" : "+s"(tab));  // constants are read here, not kept in registers
    ConstF* q = (ConstF*)tab + offsetof(Tables, K) / 4;
    PairConst K;
    K.dtka = q[0];
    K.c2 = q[1];
    K.tak = q[2];
    K.clamp2 = q[3];
    K.cold = q[7];
    float2 rm, rp;  // rows y - 1 and y + 1
    if constexpr (EVEN) {
      rm = *reinterpret_cast<const float2*>(t + (cell - nz));
      rp = *reinterpret_cast<const float2*>(t + (cell + nz));
    }
    auto row = [&](int v, int o, const float2& r) {
      if constexpr (EVEN) return v == 0 ? r.x : r.y;
      return t[cell + v + o];
    };
    if (code != kPairIrregular) {
      ConstF* c = (ConstF*)tab + offsetof(Tables, adj) / 4 + 4 * (code & (kMaxClasses - 1));
      const float kx = c[0], ky = c[1], kz = c[2], B1 = c[3];
      bool warm = false;
      float off[V], diag[V], dr[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        diag[v] = 1.0f - (PERF ? B1 * pf[v] : B1);
        diag[v] -= kx;
        diag[v] -= kx;
        diag[v] -= ky;
        diag[v] -= ky;
        diag[v] -= kz;
        diag[v] -= kz;
        float o = kx * lm[v];
        o = __builtin_fmaf(kx, ln[v], o);
        o = __builtin_fmaf(ky, row(v, -nz, rm), o);
        o = __builtin_fmaf(ky, row(v, nz, rp), o);
        o = __builtin_fmaf(kz, v > 0 ? l[v - 1] : t[cell - 1], o);
        off[v] = __builtin_fmaf(kz, v < V - 1 ? l[v + 1] : t[cell + V], o);
        warm = warm || !(fabsf(th[v]) < K.cold);
      }
      const float kr = K.c2 * 0.69314718f;
      const float r0 = __builtin_amdgcn_rcpf(K.tak);
      const float cold = K.dtka * kr * K.tak * (r0 * r0);
#pragma unroll
      for (int v = 0; v < V; ++v) dr[v] = cold;
      if (__ballot(warm) != 0ull) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float r = __builtin_amdgcn_rcpf(K.tak + th[v]);
          const float x = K.c2 * th[v] * r;
          const float rate = K.dtka * __builtin_amdgcn_exp2f(fminf(x, K.clamp2));
          const float dr0 = rate * kr * K.tak * (r * r);
          dr[v] = x < K.clamp2 ? dr0 : 0.0f;
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const bool held = (lb[v] & kHeld) != 0u;
        const float d = (lb[v] & kTissue) ? dr[v] : 0.0f;
        const float lo = __builtin_fmaf(diag[v], l[v], off[v]) + w[v] * d;
        nl[v] = held ? 0.0f : lo;
        sa[v] = (lb[v] & sum_bits) == sum_want ? sa[v] + l[v] : sa[v];
        fa[v] = held ? fa[v] : __builtin_fmaf(-B1, th[v] * l[v], fa[v]);
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int e = cell + v;
        const float nlam[6] = {lm[v], ln[v], row(v, -nz, rm), row(v, nz, rp), t[e - 1], t[e + 1]};
        const unsigned nlab[6] = {tpv[e], bn[v], tl[e - nz], tl[e + nz], tl[e - 1], tl[e + 1]};
        const float2* pc = sm.pc;
        const float sa0 = sa[v];
        adjoint_voxel(
            l[v], th[v], lb[v], pf[v], w[v], nlam, nlab,
            [pc](int ax, unsigned cq, unsigned cp) { return pair_from_pairs(pc, ax, cq, cp); },
            sm.cls, K, nl[v], sa[v], fa[v]);
        sa[v] = (lb[v] & sum_bits) == sum_want ? sa[v] : sa0;
      }
    }
  };

  auto put = [&](float* p, const float (&l)[V]) {
    if constexpr (EVEN) {
      *reinterpret_cast<float2*>(p) = make_float2(l[0], l[1]);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) p[v] = l[v];
    }
  };

  auto publish = [&](auto SL_, const AdjPairPlane<V>& q) {
    constexpr int SL = decltype(SL_)::value;
    put(sm.in[SL & 1] + cell, q.lam);
#pragma unroll
    for (int v = 0; v < V; ++v) sm.lab[SL][cell + v] = (uint8_t)q.b[v];
    if (has_halo) {
      sm.in[SL & 1][hcell] = q.hl;
      sm.lab[SL][hcell] = (uint8_t)q.hb;
    }
  };

  // wave codes of planes x - 1 and x, and the dword with that of x + 1
  unsigned code = 0u, code_next, code_shift;
  auto fetch_code = [&](int x) {
    code_next = code_word(a.codes, ((size_t)(plane_of(x) + xb) * segs + sg) * NW + wave,
                          code_shift);
  };
  fetch_code(xs);

  // The buffers' reuse is that of the forward kernel: what iteration x writes
  // was last read before its barrier.
  auto iterate = [&](auto SL_, int x) {
    constexpr int SL = decltype(SL_)::value;  // plane x
    constexpr int SP = (SL + 3) % kRing;      // plane x - 1
    constexpr int SN = (SL + 1) % kRing;      // plane x + 1
    constexpr int SA = (SL + 2) % kRing;      // receives plane x + 2; in LDS still x - 2
    constexpr int BUF = SL & 1;
    AdjPairPlane<V>& C = ring[SL];
    AdjPairPlane<V>& N = ring[SN];
    const AdjPairPlane<V>& B = ring[SP];
    __syncthreads();
    load(x + 2, ring[SA]);
    const unsigned pcode = code;
    code = (code_next >> code_shift) & 0xffu;
    fetch_code(x + 1);
    float n1[V], fa[V], sa[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      n1[v] = 0.0f;
      fa[v] = C.fa[v];
      sa[v] = C.sa[v];
    }
    if (do_mid)
      step(sm.in[BUF], sm.lab[SL], sm.lab[SP], code, C.lam, lp, N.lam, C.b, N.b, C.th, C.w, C.pf,
           n1, sa, fa);
    put(sm.mid[BUF] + cell, n1);
#pragma unroll
    for (int v = 0; v < V; ++v) lp[v] = C.lam[v];
    publish(std::integral_constant<int, SN>{}, N);
    load_own(x + 1, N);
    float tn[V];  // theta^{n-1} of plane x, for the next iteration
    ld_f32v<V>(tn, r_tp, own4, plane_of(x) * np * 4);
    {
      float o[V];
      const bool out = x > x0;  // uniform: plane x - 1 is in the chunk
#pragma unroll
      for (int v = 0; v < V; ++v) o[v] = 0.0f;
      if (do_out && out)
        step(sm.mid[BUF ^ 1], sm.lab[SP], sm.lab[SA], pcode, m1, m2, n1, mb, C.b, tp, B.w, B.pf, o,
             msa, mfa);
      const int so4 = plane_of(x - 1) * np * 4;
      const unsigned v4 = out ? own4 : kOob;
      st_f32v<kStoreThrough, V>(o, r_out, v4, so4);
      st_f32v<kStoreThrough, V>(mfa, r_fa, v4, so4);
      st_f32v<kStoreThrough, V>(msa, r_sa, sums_at(mb) ? v4 : kOob, so4);
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      m2[v] = m1[v];
      m1[v] = n1[v];
      mfa[v] = fa[v];
      msa[v] = sa[v];
      tp[v] = tn[v];
      mb[v] = C.b[v];
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  static_assert(kRing == 4, "unrolled for a ring of four planes");
  publish(I0{}, ring[0]);
  for (int x = xs;; x += kRing) {
    iterate(I0{}, x);
    if (x + 1 > x1) break;
    iterate(I1{}, x + 1);
    if (x + 2 > x1) break;
    iterate(I2{}, x + 2);
    if (x + 3 > x1) break;
    iterate(I3{}, x + 3);
    if (x + 4 > x1) break;
  }
}

namespace {

template <int NT, int V, int MAXNZ>
hipError_t launch_kind(const PairShape& s, Grid3 g, const AdjointBuffers& a, hipStream_t st) {
  const dim3 grid(s.nwg), block(NT);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, a, g.nx, g.ny, g.nz, s.xc, s.seg, s.segs,
                       s.nwg);
    return hipGetLastError();
  };
  if constexpr (V == 2)
    if (g.nz % 2 == 0)
      return a.perf ? go(k_adjoint_pair<NT, V, MAXNZ, true, true>)
                    : go(k_adjoint_pair<NT, V, MAXNZ, false, true>);
  return a.perf ? go(k_adjoint_pair<NT, V, MAXNZ, true, false>)
                : go(k_adjoint_pair<NT, V, MAXNZ, false, false>);
}

}  // namespace

int adjoint_pair_chunk(Grid3 g, int waves, int v) {
  int best = 1;
  double least = 1e300;
  for (int xc = 1; xc <= std::min(g.nx, 64); ++xc) {
    if (!pair_fits(g, waves, v, xc)) break;
    const double us = pair_estimate(waves, v, pair_shape(g, waves, v, xc).nwg, xc);
    if (us < least) {
      least = us;
      best = xc;
    }
  }
  return best;
}

hipError_t launch_adjoint_pair(const PairShape& s, Grid3 g, const AdjointBuffers& a,
                               hipStream_t st) {
  if (!pair_fits(g, s.waves, s.v, s.xc) || !a.codes || !a.theta_prev) return hipErrorInvalidValue;
  if (s.waves == 16 && s.v == 2) return launch_kind<1024, 2, 256>(s, g, a, st);
  if (s.waves == 8 && s.v == 2) return launch_kind<512, 2, 128>(s, g, a, st);
  if (s.waves == 8 && s.v == 1) return launch_kind<512, 1, 128>(s, g, a, st);
  if (s.waves == 4 && s.v == 1) return launch_kind<256, 1, 96>(s, g, a, st);
  return hipErrorInvalidValue;
}

}  // namespace rfa
