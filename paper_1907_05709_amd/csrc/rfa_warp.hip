// rfa_warp.hip -- breathing-motion view of the temperature image.
//
// The simulated temperature is shown in the breathing phase given by a
// surrogate signal beta(t) by pulling it back through the inverse motion
// field (Eq. (eq:breathing)): T_view(x) = T(x + beta v(x)).  z is the fastest
// index and the motion is smooth, so a wave's corner gathers fall on a few
// contiguous cache lines of four source rows.  Bytes that must move per
// voxel: the three displacement components, one output and the state's hi
// word once (20 bytes; lo words only where they matter, see kLoAll); the
// 2 x 2 corner re-reads are served by the caches.
//
// What bounds it: memory on large grids (256^3 69 us, 4.9 TB/s at 20 bytes a
// voxel; 256x256x234 58 us, 5.3 TB/s).  The kernel issues about 75 vector
// instructions a voxel; with float-float positions and one dword of
// displacement a load it issued 175 and was bound by them (76 and 71 us;
// 151x140x133 with two fields 22.3 -> 17.6 us).
//
// Accuracy (the view is within 1e-4 K of the FP64 interpolant of the state):
//  * sample positions are formed in double, i + c v with the FP64 factor
//    c = surrogate / spacing: the displacement is up to tens of voxels, where
//    one FP32 product would misplace the sample by ~1e-6 voxel, i.e. ~1e-4 K
//    on the steepest slopes next to the needle.  A double multiply-add costs
//    what a float one costs here; only the fraction within the cell, in
//    [0, 1], is rounded to float;
//  * the eight corners are interpolated as excess over the hi word of the
//    corner nearest to the sample, so the lerps act on local differences (a
//    few K) instead of the full 900 K.  Their lo words are read where they
//    matter at this tolerance: in cells with a corner at or above 1024 degC
//    and for samples on a voxel centre (see kLoAll); elsewhere they move the
//    view by less than half an ulp of the hi word;
//  * 37 + that hi word + the interpolated excess is summed in double and
//    rounded once.  A sample on a voxel centre (fractions 0 or 1: integer
//    shifts, positions clamped to a wall) is that voxel's float-float state
//    rounded once.
//
// Launch shape: a thread takes four voxels adjacent in z, so that the
// displacement comes and the output goes as 16 bytes a lane (a multi-dword
// access needs only 4-byte alignment) and four independent gather chains are
// in flight; two voxels a thread are equal on one field and 5 % slower on
// two.  The two z corners of a row are one 8-byte load.  The eighths of a
// plane go to the eight XCDs, so the planes x and x + 1 that a cell needs
// meet in one L2 while all XCDs read one plane's neighbourhood at a time:
// slabs of x planes per XCD put their streams a power of two apart (256^3
// with two fields 116 us against 98).  Asking for more waves than the
// registers allow spills (256^3 84 us).  The displacement is read with the
// ordinary cache policy, so the part of it that stays in the last-level
// cache between frames is reused, and the output is stored non-temporally.
#include "rfa_warp.h"

#include <type_traits>

#include "rfa_tile_common.h"

namespace rfa {
namespace {

constexpr int kWarpThreads = 256;
constexpr int kXcds = 8;
// Excess temperature (K) from which a cell reads its corners' lo words.
// Below it (T < 1024 degC) the lo words, each at most ulp(hi) / 2 <= 3.1e-5
// K, move the interpolant by at most that much, and the output's rounding
// adds at most as much again: 6.1e-5 K together.  Above it the output's
// rounding alone reaches 6.1e-5 K, so hotter cells keep every lo word.
constexpr float kLoAll = 987.0f;

// One displacement field: x, y, z component planes (metres) and the factors
// that turn them into voxels (surrogate / spacing per axis).
struct WarpField {
  const float* x;
  const float* y;
  const float* z;
  double c[3];
};

// Quotient by a divisor d known to the host: q / d for q < 2^31 is the high
// word of q m, shifted (m = floor(2^(31 + l) / d) + 1, l = ceil(log2 d) >= 1;
// d = 1 is its own case).
struct Divisor {
  unsigned d, m, shift;
};
inline Divisor divisor(unsigned d) {
  unsigned l = 1;
  while (l < 31 && (1u << l) < d) ++l;
  return Divisor{d, d > 1 ? (unsigned)((1ull << (31 + l)) / d + 1) : 0u, l - 1};
}
__device__ __forceinline__ unsigned quotient(unsigned q, Divisor v) {
  return v.d > 1 ? __umulhi(q, v.m) >> v.shift : q;
}

// Two or four consecutive floats, 4-byte aligned.
typedef float pair_f32 __attribute__((ext_vector_type(2), aligned(4)));
typedef float quad_f32 __attribute__((ext_vector_type(4), aligned(4)));

// Split a position s (voxels) into a base index k in [0, n - 2] and a
// fraction f in [0, 1], positions beyond the walls taken at the wall (a NaN
// at the lower one).  Where the fraction rounds to 1 the sample is the far
// corner with weight 1, the same value as the next cell's near corner.
__device__ __forceinline__ void locate(double s, int n, double top, int& k, float& f) {
  s = fmin(fmax(s, 0.0), top);
  k = min((int)s, n - 2);
  f = (float)(s - (double)k);
  asm("" : "+v"(f));  // the float is what is kept, not the difference it came from
}

// max(m, |u|, |w|) in one instruction (fmaxf would quiet each operand first)
__device__ __forceinline__ float max_abs(float m, float u, float w) {
  asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(u), "v"(w));
  return m;
}

// (1 - t) a + t b as two FMAs: exactly a at t = 0 and exactly b at t = 1, so
// positions on a voxel centre (integer shifts, positions clamped to a wall)
// return that voxel's value unrounded.
__device__ __forceinline__ float lerp(float a, float b, float t) {
  return __builtin_fmaf(t, b, __builtin_fmaf(-t, a, a));
}

// Excess of the float-float corner (h, l) over the base b, rounded once
// (h - b is exact for neighbouring values within a factor of two; 0 for
// the base corner itself, whose excess is then exactly l).
__device__ __forceinline__ float rel(float h, float l, float b) { return (h - b) + l; }

// Positions i_a + c_a v_a (+ c2_a v2_a with a second field), in voxels.
// A thread takes VZ voxels consecutive in z (the last of a row start at
// nz - VZ, so that where VZ does not divide nz a few voxels are computed
// twice, to the same bits); XCD k takes the k-th eighth of every plane's
// threads (part.d of them), plane by plane.
// ACCESS: kBuffer if every offset fits a 32-bit buffer descriptor (n < 2^29),
// so that the eight corner gathers share one vector offset and take the row and
// plane strides as scalar offsets, with indices and strides below 2^24 (24-bit
// multiplies); kBufferWide the same where a plane has 2^24 voxels or more
// (8x4200x4200: 694 us, 741 with plain loads; 896 and 1080 where neighbouring
// displacements differ by voxels); kPlain otherwise.
enum Access { kPlain, kBuffer, kBufferWide };
template <bool kTwo, Access ACCESS, int VZ>
__global__ __launch_bounds__(kWarpThreads) void k_warp(const float* __restrict__ hi,
                                                       const float* __restrict__ lo,
                                                       WarpField a, WarpField b,
                                                       float* __restrict__ out, int nx, int ny,
                                                       int nz, Divisor groups, Divisor part) {
  constexpr bool kBuf = ACCESS != kPlain;
  const unsigned t = blockIdx.x / kXcds * kWarpThreads + threadIdx.x;
  const unsigned x = quotient(t, part);
  const unsigned q = (blockIdx.x % kXcds) * part.d + (t - x * part.d);
  const unsigned y = quotient(q, groups);
  if (x >= (unsigned)nx || y >= (unsigned)ny) return;  // no barrier follows
  const int z0 = min((int)(q - y * groups.d) * VZ, nz - VZ);
  const unsigned sy = (unsigned)nz, sx = (unsigned)ny * (unsigned)nz;
  auto mul = [](unsigned u, unsigned w) { return kBuf ? __umul24(u, w) : u * w; };
  auto mul_x = [](unsigned u, unsigned w) {
    return ACCESS == kBuffer ? __umul24(u, w) : u * w;
  };
  const unsigned o = mul_x(x, sx) + (mul(y, sy) + (unsigned)z0);
  const unsigned n = sx * (unsigned)nx;
  __amdgpu_buffer_rsrc_t rh, rl, ro;
  if constexpr (kBuf) {
    const size_t bytes = (size_t)n * 4;
    rh = tile::make_rsrc(hi, bytes);
    rl = tile::make_rsrc(lo, bytes);
    ro = tile::make_rsrc(out, bytes);
  }
  // component w of a displacement at the thread's voxels
  auto disp = [&](const float* w, float (&v)[VZ]) {
    if constexpr (VZ == 4) {
      quad_f32 t;
      if constexpr (kBuf)
        t = __builtin_bit_cast(quad_f32,
                               __builtin_amdgcn_raw_buffer_load_b128(
                                   tile::make_rsrc(w, (size_t)n * 4), (int)(o * 4u), 0, 0));
      else
        t = *(const quad_f32*)(w + o);
      v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
    } else {
      for (int j = 0; j < VZ; ++j) v[j] = w[o + j];
    }
  };
  const int so1 = (int)(sy * 4u), so2 = (int)(sx * 4u), so3 = (int)((sx + sy) * 4u);
  auto corners = [&](const float* base, __amdgpu_buffer_rsrc_t r, unsigned c, pair_f32& c00,
                     pair_f32& c01, pair_f32& c10, pair_f32& c11) {
    if constexpr (kBuf) {
      const int vo = (int)(c * 4u);
      c00 = __builtin_bit_cast(pair_f32, __builtin_amdgcn_raw_buffer_load_b64(r, vo, 0, 0));
      c01 = __builtin_bit_cast(pair_f32, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so1, 0));
      c10 = __builtin_bit_cast(pair_f32, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so2, 0));
      c11 = __builtin_bit_cast(pair_f32, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so3, 0));
    } else {
      const float* p = base + c;
      c00 = *(const pair_f32*)p;
      c01 = *(const pair_f32*)(p + sy);
      c10 = *(const pair_f32*)(p + sx);
      c11 = *(const pair_f32*)(p + sx + sy);
    }
  };

  // Phase 1: cell, fractions and the four hi pairs of every voxel, all
  // gathers issued before any use.
  unsigned cc[VZ];
  float fx[VZ], fy[VZ], fz[VZ];
  pair_f32 h[VZ][4];
  {
    float ax[VZ], ay[VZ], az[VZ], bx[VZ], by[VZ], bz[VZ];
    disp(a.x, ax);
    disp(a.y, ay);
    disp(a.z, az);
    if constexpr (kTwo) {
      disp(b.x, bx);
      disp(b.y, by);
      disp(b.z, bz);
    }
    const double dx = x, dy = y, dz = z0;
    const double tx = nx - 1, ty = ny - 1, tz = nz - 1;
#pragma unroll
    for (int j = 0; j < VZ; ++j) {
      double px = __builtin_fma(a.c[0], (double)ax[j], dx);
      double py = __builtin_fma(a.c[1], (double)ay[j], dy);
      double pz = __builtin_fma(a.c[2], (double)az[j], dz + (double)j);
      if constexpr (kTwo) {
        px = __builtin_fma(b.c[0], (double)bx[j], px);
        py = __builtin_fma(b.c[1], (double)by[j], py);
        pz = __builtin_fma(b.c[2], (double)bz[j], pz);
      }
      int kx, ky, kz;
      locate(px, nx, tx, kx, fx[j]);
      locate(py, ny, ty, ky, fy[j]);
      locate(pz, nz, tz, kz, fz[j]);
      cc[j] = mul_x((unsigned)kx, sx) + (mul((unsigned)ky, sy) + (unsigned)kz);
      corners(hi, rh, cc[j], h[j][0], h[j][1], h[j][2], h[j][3]);
    }
  }
  // A sample on a voxel centre (every fraction 0 or 1) also reads that
  // voxel's lo word (the nearest corner's): the interpolant there is
  // exactly its excess, so the view is the state rounded once.  Known from
  // the fractions alone, so these loads fly with the hi gathers; a branch,
  // taken only by waves that hold such a sample.
  bool any_ctr = false;
  bool ctr[VZ];
  float lb[VZ];
#pragma unroll
  for (int j = 0; j < VZ; ++j) {
    auto off = [](float f) { return __builtin_fmaf(-f, f, f); };  // 0 for 0 and 1 alone
    ctr[j] = fmaxf(off(fx[j]), fmaxf(off(fy[j]), off(fz[j]))) == 0.0f;
    any_ctr |= ctr[j];
    lb[j] = 0.0f;
  }
  if (any_ctr) {
#pragma unroll
    for (int j = 0; j < VZ; ++j) {
      const unsigned cb = cc[j] + (fz[j] >= 0.5f ? 1u : 0u) + (fy[j] >= 0.5f ? sy : 0u) +
                          (fx[j] >= 0.5f ? sx : 0u);
      if constexpr (kBuf)
        lb[j] = tile::ld_f32(rl, ctr[j] ? cb * 4u : tile::kOob, 0);
      else
        lb[j] = ctr[j] ? lo[cb] : 0.0f;
    }
  }
  // hi word of the corner nearest to the sample (ties to the lower one)
  auto nearest = [&](int j) {
    auto sel = [](bool c, float u, float w) { return c ? u : w; };
    const bool cz = fz[j] >= 0.5f, cy = fy[j] >= 0.5f;
    const float b0 = sel(cy, sel(cz, h[j][1].y, h[j][1].x), sel(cz, h[j][0].y, h[j][0].x));
    const float b1 = sel(cy, sel(cz, h[j][3].y, h[j][3].x), sel(cz, h[j][2].y, h[j][2].x));
    return sel(fx[j] >= 0.5f, b1, b0);
  };
  // 37 + b + d rounded once (the double sum is exact to ~2^-43)
  auto finish = [](float b, float d) { return (float)((37.0 + (double)b) + (double)d); };
  // Phase 2: every voxel from the hi words.
  float r[VZ];
  bool hot[VZ];
  bool any_hot = false;
#pragma unroll
  for (int j = 0; j < VZ; ++j) {
    const float b0 = nearest(j);
    auto along_z = [&](pair_f32 p) {
      return __builtin_fmaf(fz[j], p.y - p.x, p.x - b0);
    };
    const float e00 = along_z(h[j][0]), e01 = along_z(h[j][1]);
    const float e10 = along_z(h[j][2]), e11 = along_z(h[j][3]);
    const float e0 = __builtin_fmaf(fy[j], e01 - e00, e00);
    const float e1 = __builtin_fmaf(fy[j], e11 - e10, e10);
    r[j] = finish(b0, __builtin_fmaf(fx[j], e1 - e0, e0));
    float m = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) m = max_abs(m, h[j][c].x, h[j][c].y);
    hot[j] = m >= kLoAll;
    any_hot |= hot[j];
  }
  if (any_ctr) {
#pragma unroll
    for (int j = 0; j < VZ; ++j) r[j] = ctr[j] ? finish(nearest(j), lb[j]) : r[j];
  }
  // Phase 3: cells with a corner at or above kLoAll read their eight lo
  // words and are redone over the nearest corner (a branch, taken only by
  // waves that hold such a cell: gathers masked out by offset cost as much
  // as real ones).
  if (any_hot) {
#pragma unroll
    for (int j = 0; j < VZ; ++j) {
      pair_f32 l[4];
      if constexpr (kBuf) {
        corners(lo, rl, hot[j] ? cc[j] : tile::kOob / 4u, l[0], l[1], l[2], l[3]);
      } else {
        l[0] = l[1] = l[2] = l[3] = pair_f32{0.0f, 0.0f};
        if (hot[j]) corners(lo, rl, cc[j], l[0], l[1], l[2], l[3]);
      }
      const float b0 = nearest(j);
      auto along_z = [&](int c) {
        return lerp(rel(h[j][c].x, l[c].x, b0), rel(h[j][c].y, l[c].y, b0), fz[j]);
      };
      const float d = lerp(lerp(along_z(0), along_z(1), fy[j]),
                           lerp(along_z(2), along_z(3), fy[j]), fx[j]);
      r[j] = hot[j] ? finish(b0, d) : r[j];
    }
  }
  if constexpr (VZ == 4) {
    const quad_f32 t = {r[0], r[1], r[2], r[3]};
    if constexpr (kBuf)
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, t), ro,
          (int)(o * 4u), 0, tile::kStoreStream);
    else
      __builtin_nontemporal_store(t, (quad_f32*)(out + o));
  } else {
    for (int j = 0; j < VZ; ++j) __builtin_nontemporal_store(r[j], out + (o + j));
  }
}

template <bool kTwo, Access ACCESS, int VZ>
hipError_t launch(Grid3 g, const float* hi, const float* lo, const WarpField& a,
                  const WarpField& b, float* out, hipStream_t st) {
  const size_t groups = (size_t)(g.nz + VZ - 1) / VZ;
  const size_t part = (groups * g.ny + kXcds - 1) / kXcds;  // of a plane, per XCD
  const size_t nwg = (part * g.nx + kWarpThreads - 1) / kWarpThreads * kXcds;
  if (nwg > 0x7fffffffu) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_warp<kTwo, ACCESS, VZ>), dim3((unsigned)nwg), dim3(kWarpThreads), 0, st,
                     hi, lo, a, b, out, g.nx, g.ny, g.nz, divisor((unsigned)groups),
                     divisor((unsigned)part));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_warp(Grid3 g, const float* hi, const float* lo, const float* v,
                       const double (&scale)[3], const float* v2, const double (&scale2)[3],
                       float* out, hipStream_t st) {
  const size_t n = g.n();
  if (n == 0) return hipSuccess;
  if (n >= (size_t(1) << 31) || g.nx < 2 || g.ny < 2 || g.nz < 2) return hipErrorInvalidValue;
  auto field = [&](const float* w, const double(&c)[3]) {
    return WarpField{w, w + n, w + 2 * n, {c[0], c[1], c[2]}};
  };
  const unsigned k24 = 1u << 24;
  const bool buf = n * 4 <= 0x7fffffffu && (unsigned)g.ny < k24 && (unsigned)g.nz < k24;
  const bool wide = (unsigned)g.nx >= k24 || (size_t)g.ny * g.nz >= k24;
  const WarpField a = field(v, scale);
  const WarpField b = v2 ? field(v2, scale2) : a;
  auto go = [&](auto access, auto vz) {
    constexpr Access A = decltype(access)::value;
    return v2 ? launch<true, A, decltype(vz)::value>(g, hi, lo, a, b, out, st)
              : launch<false, A, decltype(vz)::value>(g, hi, lo, a, b, out, st);
  };
  using Plain = std::integral_constant<Access, kPlain>;
  using Buffer = std::integral_constant<Access, kBuffer>;
  using BufferWide = std::integral_constant<Access, kBufferWide>;
  using One = std::integral_constant<int, 1>;
  using Four = std::integral_constant<int, 4>;
  // rows of two or three voxels hold no group of four
  if (g.nz < 4) return go(Plain{}, One{});
  if (!buf) return go(Plain{}, Four{});
  return wide ? go(BufferWide{}, Four{}) : go(Buffer{}, Four{});
}

}  // namespace rfa
