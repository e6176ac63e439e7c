// Ray set-up of the bricked ray caster: the samples that a pixel's ray takes in
// a brick, in pairs of FP32.  A lane does this once per brick its ray may
// cross; everything after it is integer and FP32 arithmetic.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include "bc_df.h"

// How far the rays' origins are moved towards the cube, in lengths of c (the
// ray through the image's centre): to the plane at the cube's centre, if that
// lies more than two of the cube's diagonals away along c and the whole cube in
// front of the viewer (who looks along dir), else not at all.  A pair holds 2^-48
// of the larger of a ray's origin and its way to the sample; from the plane both
// are of the cube's size, from an eye 10^6 voxels away they are 10^6, and the
// samples were off by 1.9e-9 voxels (RMS).  Nearer, where the fixed point's
// truncation (1.3e-10) is 20 times the pairs' error and more, rays keep the eye.
__device__ __forceinline__ double ray_shift(const double* e, const double* c, const double* dir, const int32_t* dims) {
  double ec = 0.0, ed = 0.0, cc = 0.0, dd = 0.0;
  for (int a = 0; a < 3; ++a) {
    const double to = 0.5 * (double)dims[a] - e[a];
    ec += to * c[a];
    ed += to * dir[a];
    cc += c[a] * c[a];
    dd += (double)dims[a] * (double)dims[a];
  }
  return ec > 0.0 && ec * ec > 4.0 * dd * cc && ed > 0.0 && 4.0 * ed * ed > dd ? ec / cc : 0.0;
}

// a pair for e + s c; the product is not rounded before the sum, so that along
// an axis on which a view hardly moves its rays keep to the right side of a face
__device__ __forceinline__ void ray_moved(double e, double s, double c, float& hi, float& lo) {
  hi = (float)__builtin_fma(s, c, e);
  lo = (float)__builtin_fma(s, c, e - (double)hi);
}

__device__ __forceinline__ df dfv(float hi, float lo) { return df_make(hi, lo); }

// smallest j >= 0 with t_in + (j + 1/2) dt >= t, that is ceil(q - 1/2) for
// q = (t - t_in) / dt, taken exactly from the double-float q: q.hi - 1/2 is
// exact (q stays below 2^22: the boundary refuses steps with more samples
// along the cube's diagonal), and unless it is an integer the trailing part
// (below half its ulp) cannot carry it past one
__device__ __forceinline__ int first_index(df t_in, df idt, df t) {
  const df q = df_mul(df_sub(t, t_in), idt);
  const float c = q.hi - 0.5f;
  const float j = ceilf(c);
  return (int)fmaxf((j == c && q.lo > 0.0f) ? j + 1.0f : j, 0.0f);
}

// 32.32 fixed point of a double-float (each part truncated; error < 2^-31).
// The leading part goes in two steps of 16 bits, each exact, so that no 64-bit
// conversion (a dozen instructions) is needed; it stays below 2^15 for
// positions in a brick and for every step that takes two samples in one.
__device__ __forceinline__ int64_t q32(df a) {
#pragma clang fp contract(off)
  const float x = a.hi * 65536.0f, t = __builtin_truncf(x);
  const int lo = (int)((x - t) * 65536.0f) + (int)(a.lo * 4294967296.0f);
  return (int64_t)(int)t * 65536 + lo;
}

struct RaySeg {
  int n;                 // samples of the ray inside the brick
  int64_t u[3];          // first sample, ghosted brick-local coordinate minus 1/2, 32.32
  int64_t s[3];          // step vector, 32.32
};

__device__ __forceinline__ df df_abs(df a) { return df_lt(a, df_from(0.0f)) ? df_neg(a) : a; }

// Ray of pixel (px, py) against brick br: the samples t_j = t_in + (j+1/2) dt
// of the ray's cube interval that fall in the brick's half-open box.  The step
// is the view's, or with the per-voxel policy 1 / max_a |d_a| (consecutive
// samples one voxel apart along the ray's dominant axis, the discrete ray
// casting of Section 2.3.2).
//
// Of the cube only the entry is needed: the brick lies inside it, so a ray
// that misses the cube misses the brick, one behind the eye ends the brick
// before its first sample, and the brick's exit is never past the cube's (where
// their faces coincide both come from the same arithmetic).  Every lane does
// this once per brick its ray may cross, so it is kept short: about 700 vector
// instructions where general double-float operations took 1900.
template <typename View, typename Brick>
__device__ bool ray_segment(View& vp, const int32_t* gdims, Brick& br, int px, int py, bool per_voxel, RaySeg& seg) {
  const int W = vp.width, H = vp.height;
  const df x = df_mul_f(dfv(vp.iw_hi, vp.iw_lo), (float)(2 * px + 1 - W));
  const df y = df_mul_f(dfv(vp.ih_hi, vp.ih_lo), (float)(H - 2 * py - 1));
  df o[3], d[3];
  auto direction = [&] {
    df u[3];
    for (int a = 0; a < 3; ++a)
      u[a] = df_fma2(dfv(vp.a_hi[a], vp.a_lo[a]), x, dfv(vp.b_hi[a], vp.b_lo[a]), y, dfv(vp.c_hi[a], vp.c_lo[a]));
    const df ilen = df_rsqrt(df_norm2(u));
    for (int a = 0; a < 3; ++a) d[a] = df_mul(u[a], ilen);
  };
  // (moved origins beside the orthographic ones: a branch of their own behind
  // the near views' directions cost those up to 1.7%)
  if (vp.kind == 0) {
    for (int a = 0; a < 3; ++a) o[a] = dfv(vp.e_hi[a], vp.e_lo[a]);
    direction();
  } else {
    for (int a = 0; a < 3; ++a) {
      o[a] = df_fma2(dfv(vp.oa_hi[a], vp.oa_lo[a]), x, dfv(vp.ob_hi[a], vp.ob_lo[a]), y, dfv(vp.e_hi[a], vp.e_lo[a]));
      d[a] = dfv(vp.c_hi[a], vp.c_lo[a]);
    }
    if (vp.kind == 2) direction();
  }
  // slab tests: entry into the cube, entry into and exit from the brick
  df g0 = df_from(-INFINITY), b0 = g0, b1 = df_from(INFINITY);
  bool miss = false;
  for (int a = 0; a < 3; ++a) {
    const float blo = (float)br.lo[a], bhi = (float)br.hi[a];
    // (an axis along which the ray does not move: inside its slab or not at all)
    const bool still = d[a].hi == 0.0f && d[a].lo == 0.0f;
    miss = miss || (still && !(df_ge(o[a], df_from(blo)) && df_lt(o[a], df_from(bhi))));
    const df id = df_rcp(df_make(still ? 1.0f : d[a].hi, d[a].lo));
    const bool up = d[a].hi > 0.0f;
    g0 = df_pick(still, g0, df_max(g0, df_plane(up ? 0.0f : (float)gdims[a], o[a], id)));
    b0 = df_pick(still, b0, df_max(b0, df_plane(up ? blo : bhi, o[a], id)));
    b1 = df_pick(still, b1, df_min(b1, df_plane(up ? bhi : blo, o[a], id)));
  }
  if (miss || !df_lt(b0, b1)) return false;
  const df t_in = df_max(df_from(vp.t_min), g0);
  df dt = dfv(vp.dt_hi, vp.dt_lo), idt = dfv(vp.idt_hi, vp.idt_lo);
  if (per_voxel) {
    idt = df_max(df_max(df_abs(d[0]), df_abs(d[1])), df_abs(d[2]));
    dt = df_rcp(idt);
  }
  // (a ray has a direction: at least one axis took part)
  const int j0 = first_index(t_in, idt, b0), j1 = first_index(t_in, idt, b1);
  if (j1 <= j0) return false;
  seg.n = j1 - j0;
  const df t0 = df_add(t_in, df_mul_f(dt, (float)j0 + 0.5f));
  for (int a = 0; a < 3; ++a) {
    const df p = df_add(o[a], df_mul(t0, d[a]));
    seg.u[a] = q32(df_add_f(p, 0.5f - (float)br.lo[a]));
    seg.s[a] = q32(df_mul(dt, d[a]));
  }
  return true;
}
