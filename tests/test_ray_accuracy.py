"""The ray caster's ray set-up (bc_ray.h) on the CPU, against the same ray in
128-bit arithmetic: the sample range of every brick and the sample
positions, for eyes from inside the cube to a million voxels away."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1205_0282_amd", "csrc")

# The hardware's reciprocals are off by an ulp: here correctly rounded ones, put
# off by up to half of one.
RUNTIME = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __forceinline__ inline
inline float off(float r, float x) {
  uint32_t u;
  std::memcpy(&u, &x, 4);
  u = (u ^ (u >> 13)) * 2654435761u;
  return r * (1.0f + ((float)(u >> 8) / 8388608.0f - 1.0f) * 6e-8f);
}
inline float __builtin_amdgcn_rcpf(float x) { return off(1.0f / x, x); }
inline float __builtin_amdgcn_rsqf(float x) { return off(1.0f / std::sqrt(x), x); }
"""

MAIN = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <quadmath.h>
#include <random>
#include "bc_types.h"
#include "bc_ray.h"
typedef __float128 Q;

static void split(double v, float& hi, float& lo) {
  hi = (float)v;
  lo = (float)(v - (double)hi);
}

int main(int argc, char** argv) {
  const double D = atof(argv[1]), step = atof(argv[5]);
  const int kind = atoi(argv[2]), pv = atoi(argv[3]), n = atoi(argv[4]), brick = atoi(argv[6]), axis = atoi(argv[7]);
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> U(0, 1);
  Q sum = 0, last_over = 0;
  long hits = 0, wrong = 0, near_tie = 0, moved = 0;
  for (int view = 0; view < 8000 && hits < 6000; ++view) {
    const double az = axis ? 0.0 : 6.283185307179586 * U(g), el = axis ? 0.0 : 1.4 * (2 * U(g) - 1);
    // (a nearly axis-parallel view keeps the tiny components that cos(pi/2) leaves)
    const double tiny = axis == 2 ? 6.1e-17 : 0.0;
    const double c[3] = {axis ? tiny : -cos(el) * sin(az), -sin(el), -cos(el) * cos(az)};
    double r[3] = {-c[2], 0.0, c[0]};
    const double rl = sqrt(r[0] * r[0] + r[2] * r[2]);
    for (double& x : r) x /= rl;
    const double up[3] = {r[1] * c[2] - r[2] * c[1], r[2] * c[0] - r[0] * c[2], r[0] * c[1] - r[1] * c[0]};
    const int W = 1919, H = 1081;
    const double R = 0.9 * n, spread = kind ? R : (D > R ? R / D : 0.5);
    const int dims[3] = {n, n, n};
    double E[3], A[3], B[3];
    for (int a = 0; a < 3; ++a) {
      E[a] = 0.5 * n - D * c[a];
      A[a] = r[a] * spread * W / H;
      B[a] = up[a] * spread;
    }
    // the view's record, as the set-up kernel writes it
    BcViewParams vp{};
    vp.width = W;
    vp.height = H;
    split(step, vp.dt_hi, vp.dt_lo);
    split(1.0 / step, vp.idt_hi, vp.idt_lo);
    split(1.0 / W, vp.iw_hi, vp.iw_lo);
    split(1.0 / H, vp.ih_hi, vp.ih_lo);
    const double s = ray_shift(E, c, c, dims);
    moved += s != 0.0;
    vp.kind = kind ? 1 : (s != 0.0 ? 2 : 0);
    vp.t_min = s != 0.0 ? -INFINITY : 0.0f;
    for (int a = 0; a < 3; ++a) {
      ray_moved(E[a], s, c[a], vp.e_hi[a], vp.e_lo[a]);
      split(kind ? A[a] : s * A[a], vp.oa_hi[a], vp.oa_lo[a]);
      split(kind ? B[a] : s * B[a], vp.ob_hi[a], vp.ob_lo[a]);
      split(A[a], vp.a_hi[a], vp.a_lo[a]);
      split(B[a], vp.b_hi[a], vp.b_lo[a]);
      split(c[a], vp.c_hi[a], vp.c_lo[a]);
    }
    const int nb = (n + brick - 1) / brick;
    for (int k = 0; k < 400; ++k) {
      const int px = k < 3 ? W / 2 : (int)(U(g) * W), py = k < 6 ? H / 2 : (int)(U(g) * H);
      BcBrick br{};
      for (int a = 0; a < 3; ++a) {
        br.lo[a] = brick * (int)(U(g) * nb);
        br.hi[a] = std::min(n, br.lo[a] + brick);
      }
      // the ray in 128 bits
      const Q x = (Q)(2 * px + 1 - W) / W, y = (Q)(H - 2 * py - 1) / H;
      Q o[3], d[3], len = 0;
      for (int a = 0; a < 3; ++a) {
        const Q t = (Q)A[a] * x + (Q)B[a] * y;
        o[a] = kind ? t + E[a] : (Q)E[a];
        d[a] = kind ? (Q)c[a] : t + c[a];
        len += d[a] * d[a];
      }
      if (!kind) for (Q& v : d) v /= sqrtq(len);
      Q t_in = 0, b0 = -1e30Q, b1 = 1e30Q, most = 0;
      bool miss = false;
      for (int a = 0; a < 3; ++a) {
        most = fmaxq(most, fabsq(d[a]));
        if (d[a] == 0) {
          miss = miss || o[a] < br.lo[a] || o[a] >= br.hi[a];
          continue;
        }
        const Q f0 = (0 - o[a]) / d[a], f1 = (n - o[a]) / d[a];
        t_in = fmaxq(t_in, fminq(f0, f1));
        const Q e0 = (br.lo[a] - o[a]) / d[a], e1 = (br.hi[a] - o[a]) / d[a];
        b0 = fmaxq(b0, fminq(e0, e1));
        b1 = fminq(b1, fmaxq(e0, e1));
      }
      const Q dt = pv ? 1 / most : (Q)step;
      const Q q0 = (b0 - t_in) / dt - 0.5Q, q1 = (b1 - t_in) / dt - 0.5Q;
      const Q j0 = fmaxq(ceilq(q0), 0), j1 = fmaxq(ceilq(q1), 0);
      const long count = miss || !(b0 < b1) || j1 <= j0 ? 0 : (long)(j1 - j0);
      RaySeg s;
      const bool hit = ray_segment(vp, dims, br, px, py, pv != 0, s);
      // a sample within 1e-6 of a face may fall to either side
      if (fabsq(q0 - rintq(q0)) < 1e-6Q || fabsq(q1 - rintq(q1)) < 1e-6Q || fabsq(b0 - b1) < 1e-6Q) {
        ++near_tie;
        continue;
      }
      if ((hit ? s.n : 0) != count) {
        ++wrong;
        continue;
      }
      if (!hit) continue;
      ++hits;
      for (int a = 0; a < 3; ++a) {
        const Q want = o[a] + (t_in + (j0 + 0.5Q) * dt) * d[a] - br.lo[a] + 0.5Q;
        const Q e = (Q)s.u[a] / 4294967296.0Q - want;
        sum += e * e;
        const Q l = ((Q)s.u[a] + (Q)(s.n - 1) * (Q)s.s[a]) / 4294967296.0Q - (want + (s.n - 1) * dt * d[a]);
        last_over = fmaxq(last_over, (fabsq(l) - fabsq(e)) / s.n);
      }
    }
  }
  printf("%ld %ld %ld %.6e %.6e %ld\n", hits, wrong, near_tie, (double)sqrtq(sum / (3 * std::max(hits, 1l))), (double)last_over, moved);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "g++ is needed"
    d = tmp_path_factory.mktemp("ray")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "ray")
    subprocess.run([gxx, "-std=gnu++17", "-O2", "-ffp-contract=off", "-mfma", "-I", str(d), "-I", CSRC, str(d / "main.cpp"),
                    "-lquadmath", "-o", exe], check=True, timeout=120)
    return exe


@pytest.mark.parametrize("eye,kind,voxel,n,step,brick,axis,moved", [
    (300, 0, 0, 1024, 0.5, 256, 0, False), (3000, 0, 0, 1024, 0.5, 256, 0, False), (3000, 0, 1, 1024, 0.5, 256, 0, False),
    (3500, 0, 0, 1024, 0.5, 256, 0, False), (3600, 0, 0, 1024, 0.5, 256, 0, True), (3600, 1, 0, 1024, 0.5, 256, 0, True),
    (3e4, 0, 0, 1024, 0.5, 256, 0, True), (1e6, 0, 0, 1024, 0.5, 256, 0, True), (1e6, 0, 1, 1721, 0.5, 256, 0, True),
    (1e6, 1, 0, 1024, 0.37, 256, 0, True), (60, 0, 0, 23, 0.37, 16, 0, False), (900, 0, 0, 700, 0.05, 700, 0, False),
    (2500, 0, 0, 1024, 700.0, 512, 0, False), (900, 1, 0, 512, 0.3, 128, 1, False), (900, 0, 0, 512, 0.3, 128, 1, False),
    (1800, 0, 0, 512, 0.3, 128, 1, True), (900, 1, 1, 512, 0.5, 128, 2, False), (1800, 1, 1, 512, 0.5, 128, 2, True)])
def test_samples_of_a_brick(program, eye, kind, voxel, n, step, brick, axis, moved):
    """The sample range is exact.  The first sample is off by the fixed point's
    truncation (2^-32, its RMS over sqrt(3)), a few roundings of the view's FP64
    quantities at the eye's distance, and a few roundings of pairs of FP32 (2^-48)
    at the distance of the rays' origin: at most two of the cube's diagonals from
    its centre, and half of one to its corners (1% for the scatter of an RMS over
    5,000 rays and more).  Rays from an eye a million voxels away had 1.9e-9.  A
    step adds the truncation of its fixed point, twice where a component is below
    2^-8, and of a pair."""
    out = subprocess.run([program] + [str(v) for v in (eye, kind, voxel, n, step, brick, axis)], check=True,
                         capture_output=True, text=True, timeout=120).stdout.split()
    hits, wrong, near_tie = (int(v) for v in out[:3])
    first, last = float(out[3]), float(out[4])
    print(out)
    assert hits > 5000 and wrong == 0
    assert (int(out[5]) > 0) == moved
    way = 2.5 * 3 ** 0.5 * n
    assert first <= 1.01 * ((2.0 ** -32 / 3 ** 0.5) ** 2 + (4 * 2.0 ** -53 * (eye + n)) ** 2 + (4 * 2.0 ** -48 * way) ** 2) ** 0.5
    assert last <= 2.0 ** -31 + 4 * 2.0 ** -48 * n
