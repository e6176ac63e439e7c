// Ray set-up of the bricked ray caster: the samples that a pixel's ray takes in
// a brick, from the view's FP64 quantities.  A lane does this once per brick
// its ray may cross; everything after it is integer and FP32 arithmetic.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

// 1 / x and 1 / sqrt(x): the hardware values (about 2^-26) refined twice by
// Newton steps, each of which squares the relative error
__device__ __forceinline__ double ray_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double ray_rsqrt(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = __builtin_fma(0.5 * r, __builtin_fma(-(x * r), r, 1.0), r);
  return __builtin_fma(0.5 * r, __builtin_fma(-(x * r), r, 1.0), r);
}

// smallest j >= 0 with t_in + (j + 1/2) dt >= t, that is ceil((t - t_in) / dt -
// 1/2) (below 2^22: the boundary refuses steps with more samples along the
// cube's diagonal)
__device__ __forceinline__ int first_index(double t_in, double idt, double t) {
  return (int)__builtin_fmax(__builtin_ceil(__builtin_fma(t - t_in, idt, -0.5)), 0.0);
}

// 32.32 fixed point of |p| < 2^18: of its FP32 value and of the rest, each
// truncated (error < 2^-31).  Rounding to the nearest instead moves every sample
// by up to 2^-32, and a network in BF16 makes 5e-4 of a pixel of that.  Whole
// numbers below 2^51 are the low bits of their sum with 3 * 2^51.
__device__ __forceinline__ int64_t q32(double p) {
  constexpr double one = 4294967296.0, bias = 6755399441055744.0;
  const double hi = (double)(float)p;
  const double whole = __builtin_trunc(hi * one) + __builtin_trunc((p - hi) * one);
  return __builtin_bit_cast(int64_t, whole + bias) - __builtin_bit_cast(int64_t, bias);
}

struct RaySeg {
  int n;                 // samples of the ray inside the brick
  int64_t u[3];          // first sample, ghosted brick-local coordinate minus 1/2, 32.32
  int64_t s[3];          // step vector, 32.32 (zero for a single sample)
};

// Ray of pixel (px, py) against brick br: the samples t_j = t_in + (j+1/2) dt
// of the ray's cube interval that fall in the brick's half-open box.  The step
// is the view's, or with the per-voxel policy 1 / max_a |d_a| (consecutive
// samples one voxel apart along the ray's dominant axis, the discrete ray
// casting of Section 2.3.2).
//
// Of the cube only the entry is needed: the brick lies inside it, so a ray
// that misses the cube misses the brick, one behind the eye ends the brick
// before its first sample, and the brick's exit is never past the cube's (where
// their faces coincide both come from the same arithmetic).
//
// FP64, not pairs of FP32: before the fixed point's truncation the samples are
// off by 2e-13 voxels (RMS) for an eye 3,000 voxels away and 5e-11 for one 10^6
// away.  Pairs had 6e-12 and 1.6e-9 with divisions of three digits, 1.1e-11 and
// 1.9e-9 with divisions of one correction, and were not faster: 1024^3 FP32
// frame 1332 us (now 1326), four FP16 views of 864 bricks 4989 (4895), 256x256
// frame of 128^3 48.5 (47.1).
template <typename View, typename Brick>
__device__ bool ray_segment(View& vp, Brick& br, int px, int py, bool per_voxel, RaySeg& seg) {
  const double x = vp.iw * (double)(2 * px + 1 - vp.width), y = vp.ih * (double)(vp.height - 2 * py - 1);
  double o[3], d[3];
  if (vp.kind == 0) {
    double u[3];
    for (int a = 0; a < 3; ++a) {
      o[a] = vp.e[a];
      u[a] = __builtin_fma(vp.a[a], x, __builtin_fma(vp.b[a], y, vp.c[a]));
    }
    const double ilen = ray_rsqrt(__builtin_fma(u[0], u[0], __builtin_fma(u[1], u[1], u[2] * u[2])));
    for (int a = 0; a < 3; ++a) d[a] = u[a] * ilen;
  } else {
    for (int a = 0; a < 3; ++a) {
      o[a] = __builtin_fma(vp.a[a], x, __builtin_fma(vp.b[a], y, vp.e[a]));
      d[a] = vp.c[a];
    }
  }
  // slab tests: entry into the cube, entry into and exit from the brick
  double g0 = -INFINITY, b0 = g0, b1 = INFINITY;
  bool miss = false;
  for (int a = 0; a < 3; ++a) {
    const double blo = (double)br.lo[a], bhi = (double)br.hi[a];
    // (an axis along which the ray does not move: inside its slab or not at all)
    const bool still = d[a] == 0.0, up = d[a] > 0.0;
    miss = miss || (still && !(o[a] >= blo && o[a] < bhi));
    const double id = ray_rcp(still ? 1.0 : d[a]);
    g0 = still ? g0 : __builtin_fmax(g0, ((up ? 0.0 : vp.dims[a]) - o[a]) * id);
    b0 = still ? b0 : __builtin_fmax(b0, ((up ? blo : bhi) - o[a]) * id);
    b1 = still ? b1 : __builtin_fmin(b1, ((up ? bhi : blo) - o[a]) * id);
  }
  if (miss || !(b0 < b1)) return false;
  const double t_in = __builtin_fmax(g0, 0.0);
  double dt = vp.dt, idt = vp.idt;
  if (per_voxel) {
    idt = __builtin_fmax(__builtin_fmax(__builtin_fabs(d[0]), __builtin_fabs(d[1])), __builtin_fabs(d[2]));
    dt = ray_rcp(idt);
  }
  // (a ray has a direction: at least one axis took part)
  const int j0 = first_index(t_in, idt, b0), j1 = first_index(t_in, idt, b1);
  if (j1 <= j0) return false;
  seg.n = j1 - j0;
  const double t0 = __builtin_fma(dt, (double)j0 + 0.5, t_in);
  // (one sample needs no step, and its view's may be longer than the form holds)
  const double ds = seg.n > 1 ? dt : 0.0;
  for (int a = 0; a < 3; ++a) {
    seg.u[a] = q32(__builtin_fma(t0, d[a], o[a]) + (0.5 - (double)br.lo[a]));
    seg.s[a] = q32(ds * d[a]);
  }
  return true;
}
