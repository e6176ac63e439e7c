// Double-float ("df") arithmetic on FP32 pairs (hi + lo, |lo| <= ulp(hi)/2).
// Used once per ray and per brick / sample chunk so that sample positions keep
// about 44 bits of precision while every per-sample operation stays FP32.
// Error-free transformations: Knuth's two-sum, Dekker's fast two-sum and the
// FMA-based exact product.  Contraction is switched off so that the compiler
// cannot fuse the additions these transformations rely on.
#pragma once
#include <hip/hip_runtime.h>

struct df { float hi, lo; };

__device__ __forceinline__ df df_make(float hi, float lo) { df r; r.hi = hi; r.lo = lo; return r; }
__device__ __forceinline__ df df_from(float a) { return df_make(a, 0.0f); }

__device__ __forceinline__ df two_sum(float a, float b) {
#pragma clang fp contract(off)
  float s = a + b;
  float bb = s - a;
  float e = (a - (s - bb)) + (b - bb);
  return df_make(s, e);
}

__device__ __forceinline__ df fast_two_sum(float a, float b) {
#pragma clang fp contract(off)
  float s = a + b;
  float e = b - (s - a);
  return df_make(s, e);
}

__device__ __forceinline__ df two_prod(float a, float b) {
#pragma clang fp contract(off)
  float p = a * b;
  float e = __builtin_fmaf(a, b, -p);
  return df_make(p, e);
}

// a + b with an error of a few 2^-48 of |a| + |b| (the trailing parts are not
// summed exactly): where a result much smaller than its terms needs no more
// than the terms' own accuracy, which every use here can say of itself
__device__ __forceinline__ df df_add(df a, df b) {
#pragma clang fp contract(off)
  df s = two_sum(a.hi, b.hi);
  s.lo = s.lo + (a.lo + b.lo);
  return fast_two_sum(s.hi, s.lo);
}

__device__ __forceinline__ df df_neg(df a) { return df_make(-a.hi, -a.lo); }
__device__ __forceinline__ df df_sub(df a, df b) { return df_add(a, df_neg(b)); }

__device__ __forceinline__ df df_mul(df a, df b) {
#pragma clang fp contract(off)
  df p = two_prod(a.hi, b.hi);
  float c = __builtin_fmaf(a.hi, b.lo, a.lo * b.hi);
  p.lo = p.lo + c;
  return fast_two_sum(p.hi, p.lo);
}

__device__ __forceinline__ df df_mul_f(df a, float b) {
#pragma clang fp contract(off)
  df p = two_prod(a.hi, b);
  p.lo = __builtin_fmaf(a.lo, b, p.lo);
  return fast_two_sum(p.hi, p.lo);
}

// a + b for a float b: the leading parts summed exactly, the trailing part
// added to the error once
__device__ __forceinline__ df df_add_f(df a, float b) {
#pragma clang fp contract(off)
  df s = two_sum(a.hi, b);
  s.lo = s.lo + a.lo;
  return fast_two_sum(s.hi, s.lo);
}

// 1 / a: the hardware reciprocal (about 1 ulp) refined once in FP32, so that
// an FMA leaves its remainder exact, then corrected by that remainder
// e = 1 - a r (with the trailing part's product): r (1 + e + e^2), e below
// 2^-22; a.hi is a normal number at the call sites (ray directions of order
// one, down to those of nearly axis-parallel rays)
__device__ __forceinline__ df df_rcp(df a) {
#pragma clang fp contract(off)
  const float r0 = __builtin_amdgcn_rcpf(a.hi);
  const float r = __builtin_fmaf(r0, __builtin_fmaf(-a.hi, r0, 1.0f), r0);
  const float e = __builtin_fmaf(-a.lo, r, __builtin_fmaf(-a.hi, r, 1.0f));
  return fast_two_sum(r, r * __builtin_fmaf(e, e, e));
}

// 1 / sqrt(a): the hardware value r (about 1 ulp) corrected by e = 1 - a r^2:
// r (1 + e/2 + 3/8 e^2)
__device__ __forceinline__ df df_rsqrt(df a) {
#pragma clang fp contract(off)
  const float r = __builtin_amdgcn_rsqf(a.hi);
  const df r2 = two_prod(r, r);
  const df p = two_prod(a.hi, r2.hi);
  float e = (1.0f - p.hi) - p.lo;
  e = __builtin_fmaf(-a.hi, r2.lo, e);
  e = __builtin_fmaf(-a.lo, r2.hi, e);
  return fast_two_sum(r, r * (e * __builtin_fmaf(0.375f, e, 0.5f)));
}

// a x + b y + c: exact products and sums of the leading parts, the trailing
// parts added to their errors
__device__ __forceinline__ df df_fma2(df a, df x, df b, df y, df c) {
#pragma clang fp contract(off)
  const df p = two_prod(a.hi, x.hi), q = two_prod(b.hi, y.hi);
  const df s = two_sum(p.hi, q.hi), r = two_sum(s.hi, c.hi);
  const float el = __builtin_fmaf(a.hi, x.lo, a.lo * x.hi), fl = __builtin_fmaf(b.hi, y.lo, b.lo * y.hi);
  return fast_two_sum(r.hi, ((p.lo + q.lo) + (el + fl)) + ((s.lo + r.lo) + c.lo));
}

// u.u of a vector
__device__ __forceinline__ df df_norm2(const df* u) {
#pragma clang fp contract(off)
  const df p = two_prod(u[0].hi, u[0].hi), q = two_prod(u[1].hi, u[1].hi), r = two_prod(u[2].hi, u[2].hi);
  const df s = two_sum(p.hi, q.hi), t = two_sum(s.hi, r.hi);
  const float l = __builtin_fmaf(u[0].hi, u[0].lo, __builtin_fmaf(u[1].hi, u[1].lo, u[2].hi * u[2].lo));
  return fast_two_sum(t.hi, __builtin_fmaf(2.0f, l, ((p.lo + q.lo) + r.lo) + (s.lo + t.lo)));
}

// (f - o) id for a float f (the difference normalised first: near a face its
// parts are of one size)
__device__ __forceinline__ df df_plane(float f, df o, df id) { return df_mul(df_add_f(df_neg(o), f), id); }

// exact comparisons of normalised pairs
__device__ __forceinline__ bool df_lt(df a, df b) { return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo); }
__device__ __forceinline__ bool df_ge(df a, df b) { return !df_lt(a, b); }
__device__ __forceinline__ df df_min(df a, df b) { return df_lt(a, b) ? a : b; }
__device__ __forceinline__ df df_max(df a, df b) { return df_lt(a, b) ? b : a; }

__device__ __forceinline__ df df_pick(bool c, df a, df b) { return df_make(c ? a.hi : b.hi, c ? a.lo : b.lo); }
