// Per-frame kernels of the bricked ray caster.
//
//  setup     (FP64, one workgroup per view): inverse view transform, eye,
//            per-brick visibility keys and their sort, per-brick rendering
//            rectangles (Section 2.3.2, Figure 4), and the work-item prefix sums.
//  composite per pixel, folds the brick sub-images in visibility order with
//            "over" (Section 2.3.3; associativity of alpha blending).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <float.h>
#include "bc_types.h"
#include "bc_kernels.h"
#include "bc_ray.h"

namespace {

// ------------------------------------------------------------------ FP64 setup
// One workgroup per view derives the view, orders its bricks and finds their
// rectangles; one workgroup then numbers the work items (the same one, in the
// same launch, for a single view).  Every step of it stands between the frame
// and its ray casting with nothing else on the GPU, so it is arranged for its
// latency: the pass inputs are read once, from where the host wrote them, the
// inverse runs a column to a lane, a rectangle's corners go to eight lanes, and
// the order of up to 1024 bricks is sorted in registers.  8 bricks 11.6 us, 64
// bricks 10.9, 245 bricks 17.7, 864 bricks and four views 28 + 12.7; with the
// inverse in one lane, a brick per lane and the order through LDS 16.0, 18.9,
// 25.7 and 115.
constexpr int kRankSortMax = 256;   // up to here the order is a rank count: no barriers between its steps

// a view's derived values, as the later steps of its workgroup read them
struct SetupView {
  double in[32];       // modelview, projection (OpenGL order)
  double pm[16];       // P*M, row-major
  double eye[3], dir[3];
  double e[3], a[3], b[3], c[3];   // ray generator: origin and its derivatives, direction of the centre
  double step, tau;
  int32_t persp, width, height, skip;
};

__device__ __forceinline__ void split(double v, float& hi, float& lo) {
  hi = (float)v;
  lo = (float)(v - (double)hi);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One wave: P*M and its Gauss-Jordan inverse with partial pivoting (a column
// of the augmented matrix per lane, lanes 0-3 and 4-7; never singular: the host
// refuses such projections, and the modelview is rigid), the eye, and the ray
// generator's vectors (an axis per lane).
__device__ void view_params(SetupView& sv, BcViewParams& vp, int tile_shift) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, col = lane & 7;
  const double* mv = sv.in;
  const double* pr = sv.in + 16;
  const int32_t width = sv.width, height = sv.height;
  const double step = sv.step;
  // P*M: row r, column c = sum over k of P[r][k] M[k][c], in order
  double a[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) s = s + pr[k * 4 + r] * mv[(col & 3) * 4 + k];
    if (lane < 4) sv.pm[r * 4 + lane] = s;
    a[r] = col < 4 ? s : (r == col - 4 ? 1.0 : 0.0);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = lane_value(a[r], c);
    int p = c;
    double best = fabs(v[c]);
#pragma unroll
    for (int r = c + 1; r < 4; ++r)
      if (fabs(v[r]) > best) { p = r; best = fabs(v[r]); }
    // (swapped in by selects, so that the columns stay in registers)
#pragma unroll
    for (int r = c + 1; r < 4; ++r) {
      const bool sw = r == p;
      const double x = a[c], y = a[r], vx = v[c], vy = v[r];
      a[c] = sw ? y : x;
      a[r] = sw ? x : y;
      v[c] = sw ? vy : vx;
      v[r] = sw ? vx : vy;
    }
    a[c] = a[c] / v[c];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r == c) continue;
      a[r] = v[r] == 0.0 ? a[r] : a[r] - v[r] * a[c];
    }
  }
  double Q[16];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) Q[r * 4 + c] = lane_value(a[r], 4 + c);
  const bool persp = pr[3] == 0.0 && pr[7] == 0.0 && pr[11] == -1.0 && pr[15] == 0.0;
  if (lane == 0) {
    sv.persp = persp;
    vp.width = width;
    vp.height = height;
    vp.tile_shift = tile_shift;
    vp.tiles_x = (width + (1 << tile_shift) - 1) >> tile_shift;
    vp.tiles_y = (height + (64 >> tile_shift) - 1) >> (6 - tile_shift);
    vp.tau = (float)sv.tau;
    split(step, vp.dt_hi, vp.dt_lo);
  }
  if (lane == 3) split(1.0 / step, vp.idt_hi, vp.idt_lo);
  if (lane == 4) split(1.0 / (double)width, vp.iw_hi, vp.iw_lo);
  if (lane == 5) split(1.0 / (double)height, vp.ih_hi, vp.ih_lo);
  if (lane < 3) {
    const int x = lane;
    // eye e_a = -((R0a t0 + R1a t1) + R2a t2), without fused multiply-add
    const double e = -((mv[x * 4 + 0] * mv[12] + mv[x * 4 + 1] * mv[13]) + mv[x * 4 + 2] * mv[14]);
    const double dir = -mv[x * 4 + 2];
    sv.eye[x] = e;
    sv.dir[x] = dir;
    const double q0 = x == 0 ? Q[0] : (x == 1 ? Q[4] : Q[8]), q1 = x == 0 ? Q[1] : (x == 1 ? Q[5] : Q[9]);
    const double q2 = x == 0 ? Q[2] : (x == 1 ? Q[6] : Q[10]), q3 = x == 0 ? Q[3] : (x == 1 ? Q[7] : Q[11]);
    double E, A, B, C;
    if (persp) {
      // far point w(x, y) = Q (x, y, 1, 1); direction of dehom(w) - e is w.xyz - e w.w
      double sgn = 1.0;
      const double w00 = -Q[12] - Q[13] + Q[14] + Q[15];
      if (w00 < 0.0) sgn = -1.0;
      E = e;
      A = sgn * (q0 - e * Q[12]);
      B = sgn * (q1 - e * Q[13]);
      C = sgn * ((q2 + q3) - e * (Q[14] + Q[15]));
    } else {
      // origin on the near plane o(x, y) = Q (x, y, -1, 1); direction Q (0, 0, 2, 0)
      double n = 0.0;
      for (int k = 0; k < 3; ++k) n = n + Q[k * 4 + 2] * Q[k * 4 + 2];
      n = sqrt(n);
      E = q3 - q2;
      A = q0;
      B = q1;
      C = q2 / n;
    }
    split(A, vp.a_hi[x], vp.a_lo[x]);
    split(B, vp.b_hi[x], vp.b_lo[x]);
    split(C, vp.c_hi[x], vp.c_lo[x]);
    sv.e[x] = E;
    sv.a[x] = A;
    sv.b[x] = B;
    sv.c[x] = C;
  }
}

// where the rays start, an axis per lane
__device__ void ray_origins(const SetupView& sv, BcViewParams& vp, const int32_t* gdims) {
  const int x = threadIdx.x & 63;
  if (x >= 3) return;
  const double s = ray_shift(sv.e, sv.c, sv.persp ? sv.dir : sv.c, gdims);
  const double by = sv.persp ? s : 1.0;
  ray_moved(sv.e[x], s, sv.c[x], vp.e_hi[x], vp.e_lo[x]);
  split(by * sv.a[x], vp.oa_hi[x], vp.oa_lo[x]);
  split(by * sv.b[x], vp.ob_hi[x], vp.ob_lo[x]);
  if (x == 0) {
    vp.kind = !sv.persp ? 1 : (s != 0.0 ? 2 : 0);
    vp.t_min = s != 0.0 ? -INFINITY : 0.0f;
  }
}

// visibility key: power distance from the eye (perspective) or the centre's
// projection on the view direction (orthographic), FP64 left to right, no FMA
__device__ double brick_key(const SetupView& sv, const BcBrick& b) {
#pragma clang fp contract(off)
  double k = 0.0;
  if (sv.persp) {
    for (int a = 0; a < 3; ++a) {
      const double p = (sv.eye[a] - (double)b.lo[a]) * (sv.eye[a] - (double)b.hi[a]);
      k = k + p;
    }
  } else {
    for (int a = 0; a < 3; ++a) {
      const double c = ((double)b.lo[a] + (double)b.hi[a]) / 2.0;
      k = k + c * sv.dir[a];
    }
  }
  return k;
}

// conservative rendering rectangle in whole tiles: bounding box of the eight
// projected corners widened by one pixel; the whole frame when a corner lies
// behind the eye or the eye is inside the brick.  Eight neighbouring lanes, one
// corner each; the first of them writes.
__device__ void brick_rect(const SetupView& sv, const BcBrick& b, int tile_shift, int32_t* r) {
#pragma clang fp contract(off)
  const int W = sv.width, H = sv.height;
  const int lane = threadIdx.x & 63, c = lane & 7;
  bool full = false;
  if (sv.persp) {
    bool inside = true;
    for (int a = 0; a < 3; ++a) inside = inside && sv.eye[a] >= b.lo[a] && sv.eye[a] <= b.hi[a];
    full = inside;
  }
  const double X = (c & 1) ? b.hi[0] : b.lo[0];
  const double Y = (c & 2) ? b.hi[1] : b.lo[1];
  const double Z = (c & 4) ? b.hi[2] : b.lo[2];
  double clip[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    clip[i] = ((sv.pm[i * 4 + 0] * X + sv.pm[i * 4 + 1] * Y) + sv.pm[i * 4 + 2] * Z) + sv.pm[i * 4 + 3];
  full = full || ((__ballot(!(clip[3] > 0.0)) >> (lane & 56)) & 0xffull) != 0;
  double xmin = (clip[0] / clip[3] + 1.0) * (0.5 * W) - 0.5, xmax = xmin;
  double ymin = (1.0 - clip[1] / clip[3]) * (0.5 * H) - 0.5, ymax = ymin;
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    xmin = fmin(xmin, __shfl_xor(xmin, o));
    xmax = fmax(xmax, __shfl_xor(xmax, o));
    ymin = fmin(ymin, __shfl_xor(ymin, o));
    ymax = fmax(ymax, __shfl_xor(ymax, o));
  }
  if (c != 0) return;
  int x0, x1, y0, y1;   // inclusive pixel bounds
  if (full) {
    x0 = 0; y0 = 0; x1 = W - 1; y1 = H - 1;
  } else {
    if (xmax < -1.0 || ymax < -1.0 || xmin > W || ymin > H) {
      r[0] = r[1] = r[2] = r[3] = 0;
      return;
    }
    x0 = (int)fmax(floor(xmin) - 1.0, 0.0);
    y0 = (int)fmax(floor(ymin) - 1.0, 0.0);
    x1 = (int)fmin(ceil(xmax) + 1.0, (double)(W - 1));
    y1 = (int)fmin(ceil(ymax) + 1.0, (double)(H - 1));
    if (x1 < x0 || y1 < y0) {
      r[0] = r[1] = r[2] = r[3] = 0;
      return;
    }
  }
  const int sx = tile_shift, sy = 6 - tile_shift;
  r[0] = x0 >> sx;
  r[1] = y0 >> sy;
  r[2] = (x1 >> sx) + 1;
  r[3] = (y1 >> sy) + 1;
}

// the decision from the shares, by one wave: true if the frame falls back
__device__ bool psnr_decide(const BcFramePtrs& f, float threshold, bool write) {
  const int lane = threadIdx.x & 63;
  float acc = f.ctr->psnr_sum[lane];
  int cnt = f.ctr->psnr_count[lane];
  for (int s = 32; s > 0; s >>= 1) {
    acc += __shfl_xor(acc, s);
    cnt += __shfl_xor(cnt, s);
  }
  const float mse = cnt > 0 ? acc / (float)cnt : 0.0f;
  const float p = mse > 0.0f ? 10.0f * log10f(1.0f / mse) : INFINITY;
  const bool back = p < threshold;
  if (lane == 0 && write) {
    f.ctr->psnr_db = p;
    f.ctr->fallback = back ? 1u : 0u;
  }
  return back;
}

// One view: its parameters, visibility order and rectangles.  A conditional
// pass decides first (by the validation shares) and has no work unless the
// frame falls back: sv.skip is set.
__device__ void setup_view(const BcFramePtrs& f, int v, bool copy, SetupView& sv, double* skey, int32_t* sidx) {
  const int tid = threadIdx.x;
  const int nb = f.n_bricks;
  // The pass inputs, read straight from the host's pinned buffer (two words
  // per thread for a 256-entry table) instead of a separate copy ahead of the
  // kernel: the view by the first wave, everything by the others for the
  // kernels that follow.
  const BcFrameIn* src = f.fin_src ? f.fin_src : f.fin;
  if (tid < 32) sv.in[tid] = (tid < 16 ? src->views[v].mv : src->views[v].pr)[tid & 15];
  if (tid >= 64 && tid < 128) {
    bool skip = false;
    if (src->conditional) skip = !psnr_decide(f, src->psnr_threshold, copy);
    if (tid == 64) sv.skip = skip;
  }
  if (tid == 33) sv.step = src->views[v].step;
  if (tid == 34) sv.tau = src->views[v].tau;
  if (tid == 35) sv.width = src->views[v].width;
  if (tid == 36) sv.height = src->views[v].height;
  if (copy && f.fin_src && tid >= 64) {
    const uint32_t* from = reinterpret_cast<const uint32_t*>(f.fin_src);
    uint32_t* to = reinterpret_cast<uint32_t*>(const_cast<BcFrameIn*>(f.fin));
    for (int i = tid - 64; i < f.fin_bytes / 4; i += blockDim.x - 64) to[i] = from[i];
  }
  __syncthreads();
  if (sv.skip) return;
  if (tid < 64) view_params(sv, f.views[v], f.tile_shift);
  __syncthreads();
  if (tid >= (int)blockDim.x - 64) ray_origins(sv, f.views[v], f.gdims);   // (beside the bricks, in the wave that they reach last)
  // (eight lanes to a brick: whole groups are in or out)
  for (int i = tid; i < 8 * nb; i += blockDim.x)
    brick_rect(sv, f.bricks[i >> 3], f.tile_shift, f.rects + ((int64_t)v * nb + (i >> 3)) * 4);
  int32_t* order = f.order + v * nb;
  if (nb <= kRankSortMax) {
    // each brick's place is the number of (key, index) pairs below its own,
    // counted by `parts` neighbouring lanes
    int np2 = 1;
    while (np2 < nb) np2 <<= 1;
    const int parts = min(16, (int)blockDim.x / np2);
    for (int i = tid; i < nb; i += blockDim.x) skey[i] = brick_key(sv, f.bricks[i]);
    __syncthreads();
    const int b = tid / parts, part = tid % parts;
    int rank = 0;
    if (b < nb) {
      const double k = skey[b];
      for (int j = part; j < nb; j += parts) {
        const double kj = skey[j];
        rank += (kj < k || (kj == k && j < b)) ? 1 : 0;
      }
    }
    for (int o = 1; o < parts; o <<= 1) rank += __shfl_xor(rank, o);
    if (b < nb && part == 0) order[rank] = b;
  } else if (nb <= 1024) {
    // bitonic network, a (key, index) pair per thread: partners within a wave
    // trade through registers, the others through LDS
    double k = tid < nb ? brick_key(sv, f.bricks[tid]) : DBL_MAX;
    int32_t id = tid < nb ? tid : 0x7fffffff;
    for (int size = 2; size <= 1024; size <<= 1)
      for (int j = size >> 1; j > 0; j >>= 1) {
        double ok;
        int32_t oid;
        if (j < 64) {
          ok = __shfl_xor(k, j);
          oid = __shfl_xor(id, j);
        } else {
          __syncthreads();
          skey[tid] = k;
          sidx[tid] = id;
          __syncthreads();
          ok = skey[tid ^ j];
          oid = sidx[tid ^ j];
        }
        const bool gt = k > ok || (k == ok && id > oid);
        const bool take = ((tid & size) == 0) == ((tid & j) == 0) ? gt : !gt;
        k = take ? ok : k;
        id = take ? oid : id;
      }
    if (tid < nb) order[tid] = id;
  } else {
    int np2 = 1;
    while (np2 < nb) np2 <<= 1;
    for (int i = tid; i < np2; i += blockDim.x) {
      skey[i] = i < nb ? brick_key(sv, f.bricks[i]) : DBL_MAX;
      sidx[i] = i < nb ? i : 0x7fffffff;
    }
    __syncthreads();
    for (int k = 2; k <= np2; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < np2; i += blockDim.x) {
          const int ixj = i ^ j;
          if (ixj > i) {
            const bool up = (i & k) == 0;
            const double ka = skey[i], kb = skey[ixj];
            const int ia = sidx[i], ib = sidx[ixj];
            const bool gt = (ka > kb) || (ka == kb && ia > ib);
            if (gt == up) {
              skey[i] = kb; skey[ixj] = ka;
              sidx[i] = ib; sidx[ixj] = ia;
            }
          }
        }
        __syncthreads();
      }
    }
    for (int i = tid; i < nb; i += blockDim.x) order[i] = sidx[i];
  }
}

// Work items: entry (b, v) owns the selected tiles of its rectangle.  Entries
// are numbered in queue order -- bricks grouped by b % Q -- so that queue q
// (served first by the waves of XCD q) holds whole bricks and the XCDs' L2
// caches hold different bricks.
__device__ void setup_items(const BcFramePtrs& f, bool skip, int32_t* spart) {
  const int tid = threadIdx.x;
  const int nv = f.n_views, nb = f.n_bricks;
  if (skip) {
    // no items: every later kernel of the pass returns at once
    if (tid <= 8) f.ctr->qbound[tid] = 0u;
    if (tid == 0) {
      f.ctr->n_items = 0u;
      f.ctr->n_queues = (uint32_t)f.n_queues;
    }
    return;
  }
  const int ts = f.fin->tile_stride, tox = f.fin->tile_ox, toy = f.fin->tile_oy;
  const int Q = f.n_queues;
  const int K = nb * nv;
  const int seg = (K + blockDim.x - 1) / blockDim.x;
  const int k0 = tid * seg, k1 = min(k0 + seg, K);
  struct Entry { int b, v, cx, cy, fx, fy; };
  auto entry = [&](int pos) -> Entry {
    Entry e;
    queue_entry(pos, nb, nv, Q, e.b, e.v);
    const int4 r = reinterpret_cast<const int4*>(f.rects)[(int64_t)e.v * nb + e.b];
    e.fx = sel_first(r.x, ts, tox);
    e.fy = sel_first(r.y, ts, toy);
    e.cx = sel_count(r.x, r.z, ts, tox);
    e.cy = sel_count(r.y, r.w, ts, toy);
    return e;
  };
  int32_t sum = 0;
  for (int k = k0; k < k1; ++k) {
    const Entry e = entry(k);
    sum += e.cx * e.cy;
  }
  // exclusive scan of the threads' sums: within each wave by shuffles, then
  // over the waves' totals
  const int lane = tid & 63, wave = tid >> 6;
  int32_t x = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) spart[wave] = x;
  __syncthreads();
  int32_t run = x - sum, total = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    const int32_t t = spart[w];
    run += w < wave ? t : 0;
    total += t;
  }
  for (int k = k0; k < k1; ++k) {
    const Entry e = entry(k);
    f.item_perm[k] = run;
    f.item_base[e.b * nv + e.v] = run;
    f.item_entry[k] = make_int4(e.b | (e.v << 16), e.cx, e.fx, e.fy);
    run += e.cx * e.cy;
  }
  if (tid == 0) {
    f.item_perm[K] = total;
    f.item_base[K] = total;
    const uint32_t n_items = (uint32_t)min((int64_t)total, f.max_items);
    f.ctr->n_items = n_items;
    if (f.fin->reset_counters) {
      f.ctr->nominal = 0ull;
      f.ctr->evaluated = 0ull;
      f.ctr->total_items = n_items;
    } else {
      f.ctr->total_items += n_items;
    }
  }
  __syncthreads();
  if (f.fin->reset_counters && tid >= 64 && tid < 64 + 2 * BC_COUNT_PARTS)
    f.ctr->part[(tid - 64) >> 1].count[tid & 1] = 0ull;
  if (tid < 8) {
    f.ctr->q[tid].next = 0u;
    int g0 = 0;
    for (int g = 0; g < min(tid, Q); ++g) g0 += group_size(nb, Q, g);
    f.ctr->qbound[tid] = tid < Q ? (uint32_t)f.item_perm[g0 * nv] : (uint32_t)total;
  }
  if (tid == 8) {
    f.ctr->qbound[8] = (uint32_t)total;
    f.ctr->n_queues = (uint32_t)Q;
  }
}

// a single view: everything in one workgroup
__global__ __launch_bounds__(1024) void setup_kernel(BcFramePtrs f) {
  __shared__ SetupView sv;
  __shared__ double skey[BC_MAX_BRICKS];
  __shared__ int32_t sidx[BC_MAX_BRICKS];
  __shared__ int32_t spart[16];
  setup_view(f, 0, true, sv, skey, sidx);
  __syncthreads();
  setup_items(f, sv.skip, spart);
}

// several: a workgroup each, then the items in a launch of their own
__global__ __launch_bounds__(1024) void setup_views_kernel(BcFramePtrs f) {
  __shared__ SetupView sv;
  __shared__ double skey[BC_MAX_BRICKS];
  __shared__ int32_t sidx[BC_MAX_BRICKS];
  setup_view(f, (int)blockIdx.x, blockIdx.x == 0, sv, skey, sidx);
}
__global__ __launch_bounds__(1024) void setup_items_kernel(BcFramePtrs f) {
  __shared__ int32_t spart[16];
  setup_items(f, f.fin->conditional && !f.ctr->fallback, spart);
}

// One workgroup per 4x4 block of screen tiles (16 waves, one tile each).  The
// workgroup first culls the view's visibility order down to the bricks whose
// rectangle meets the block (order kept, in LDS), so each wave folds only the
// sub-images that can cover its tile.
constexpr int kCompBlock = 4;
__global__ __launch_bounds__(1024) void composite_kernel(BcFramePtrs f, float4* __restrict__ out) {
  __shared__ int32_t list[BC_MAX_BRICKS];
  __shared__ int32_t wave_count[16];
  __shared__ int32_t n_list;
  if (f.fin->conditional && !f.ctr->fallback) return;
  const int v = blockIdx.z;
  const int nb = f.n_bricks, nv = f.n_views;
  const int W = f.width, H = f.height;
  const int ts = f.fin->tile_stride, tox = f.fin->tile_ox, toy = f.fin->tile_oy;
  const int bx0 = blockIdx.x * kCompBlock, by0 = blockIdx.y * kCompBlock;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // ordered compaction of the bricks whose rectangle meets this block of tiles
  if (tid == 0) n_list = 0;
  __syncthreads();
  for (int base = 0; base < nb; base += 1024) {
    const int k = base + tid;
    bool keep = false;
    int b = 0;
    if (k < nb) {
      b = f.order[v * nb + k];
      const int32_t* r = f.rects + ((int64_t)v * nb + b) * 4;
      keep = r[0] < bx0 + kCompBlock && r[2] > bx0 && r[1] < by0 + kCompBlock && r[3] > by0;
    }
    const uint64_t bal = __ballot(keep);
    if (lane == 0) wave_count[wave] = __popcll(bal);
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wave_count[w];
    if (keep) list[n_list + before + __popcll(bal & ((1ull << lane) - 1ull))] = b;
    __syncthreads();
    if (tid == 0) {
      int t = 0;
      for (int w = 0; w < 16; ++w) t += wave_count[w];
      n_list += t;
    }
    __syncthreads();
  }
  const int tx = bx0 + (wave % kCompBlock), ty = by0 + (wave / kCompBlock);
  const int tsh = f.tile_shift, tw = 1 << tsh, th = 64 >> tsh;
  const int tiles_x = (W + tw - 1) >> tsh, tiles_y = (H + th - 1) >> (6 - tsh);
  if (tx >= tiles_x || ty >= tiles_y) return;
  if (tx % ts != tox || ty % ts != toy) return;
  const int px = tx * tw + (lane & (tw - 1));
  const int py = ty * th + (lane >> tsh);
  float4 F = make_float4(0.f, 0.f, 0.f, 0.f);
  float M = -INFINITY;
  const int n = n_list;
  // the list in groups of 64 entries: lane j finds the sub-image tile of
  // entry j for this wave's screen tile (-1: its rectangle misses the tile),
  // all lanes' loads in flight together; then the wave folds the tiles in
  // list order, four sub-image loads in flight
  for (int base = 0; base < n; base += 64) {
    const int m = min(64, n - base);
    int my_item = -1;
    if (lane < m) {
      const int b = list[base + lane];
      const int32_t* r = f.rects + ((int64_t)v * nb + b) * 4;
      const int r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
      if (tx >= r0 && tx < r2 && ty >= r1 && ty < r3) {
        const int fx = sel_first(r0, ts, tox), fy = sel_first(r1, ts, toy);
        const int cx = sel_count(r0, r2, ts, tox);
        const int64_t item = (int64_t)f.item_base[b * nv + v] + (int64_t)((ty - fy) / ts) * cx + (tx - fx) / ts;
        if (item < (int64_t)f.max_items) my_item = (int)item;
      }
    }
    for (int k0 = 0; k0 < m; k0 += 4) {
      int it[4];
      float4 S[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) it[u] = k0 + u < m ? __shfl(my_item, k0 + u) : -1;
      if (f.op == 1) {
        const float* subf = reinterpret_cast<const float*>(f.sub);
        float m4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) m4[u] = it[u] >= 0 ? subf[(int64_t)it[u] * 64 + lane] : -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u) M = fmaxf(M, m4[u]);
        continue;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        S[u] = it[u] >= 0 ? f.sub[(int64_t)it[u] * 64 + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float om = 1.0f - F.w;
        F.x = __builtin_fmaf(om, S[u].x, F.x);
        F.y = __builtin_fmaf(om, S[u].y, F.y);
        F.z = __builtin_fmaf(om, S[u].z, F.z);
        F.w = __builtin_fmaf(om, S[u].w, F.w);
      }
    }
  }
  if (f.op == 1 && M != -INFINITY) {
    // maximum intensity projection: the largest brick maximum (any order),
    // then the colour map; no sample anywhere leaves the pixel clear
    const int K = f.fin->K;
    const float4* tab = reinterpret_cast<const float4*>(f.fin->table);
    float x = __builtin_fmaf(M, f.fin->tf_scale, f.fin->tf_bias);
    x = fminf(fmaxf(x, 0.0f), (float)(K - 1));
    const int i = min((int)x, K - 2);
    const float t = x - (float)i;
    const float4 a = tab[i], b = tab[i + 1];
    F = make_float4(__builtin_fmaf(t, b.x - a.x, a.x), __builtin_fmaf(t, b.y - a.y, a.y),
                    __builtin_fmaf(t, b.z - a.z, a.z), __builtin_fmaf(t, b.w - a.w, a.w));
  }
  if (px < W && py < H) out[((int64_t)v * H + py) * W + px] = F;
}

// Few bricks (up to kTileCompMax): one wave per screen tile, four per
// workgroup (a 2x2 block of tiles), no culling pass and no barrier.  Lane j
// takes entries j, j + 64, ... of the view's visibility order and finds the
// brick's sub-image tile for this screen tile (its rectangle, and the brick's
// first work item, loaded together); the wave then folds the covering tiles
// in visibility order, four sub-image loads in flight.  Entries that do not
// cover the tile fold as zero in composite_kernel, which changes no bit, so
// the two kernels' images are identical.
constexpr int kTileCompMax = 128;
__global__ __launch_bounds__(256) void composite_tile_kernel(BcFramePtrs f, float4* __restrict__ out) {
  if (f.fin->conditional && !f.ctr->fallback) return;
  const int v = blockIdx.z;
  const int nb = f.n_bricks, nv = f.n_views;
  const int W = f.width, H = f.height;
  const int ts = f.fin->tile_stride, tox = f.fin->tile_ox, toy = f.fin->tile_oy;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tx = (int)blockIdx.x * 2 + (wave & 1), ty = (int)blockIdx.y * 2 + (wave >> 1);
  const int tsh = f.tile_shift, tw = 1 << tsh, th = 64 >> tsh;
  const int tiles_x = (W + tw - 1) >> tsh, tiles_y = (H + th - 1) >> (6 - tsh);
  if (tx >= tiles_x || ty >= tiles_y) return;
  if (tx % ts != tox || ty % ts != toy) return;
  const int px = tx * tw + (lane & (tw - 1));
  const int py = ty * th + (lane >> tsh);
  float4 F = make_float4(0.f, 0.f, 0.f, 0.f);
  float M = -INFINITY;
  for (int base = 0; base < nb; base += 64) {
    const int k = base + lane;
    int my_item = -1;
    if (k < nb) {
      const int b = f.order[v * nb + k];
      const int32_t* r = f.rects + ((int64_t)v * nb + b) * 4;
      const int r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
      const int64_t first = f.item_base[b * nv + v];
      if (tx >= r0 && tx < r2 && ty >= r1 && ty < r3) {
        const int fx = sel_first(r0, ts, tox), fy = sel_first(r1, ts, toy);
        const int cx = sel_count(r0, r2, ts, tox);
        const int64_t item = first + (int64_t)((ty - fy) / ts) * cx + (tx - fx) / ts;
        if (item < (int64_t)f.max_items) my_item = (int)item;
      }
    }
    uint64_t cover = __ballot(my_item >= 0);
    while (cover) {
      int it[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        it[u] = -1;
        if (cover) {
          const int j = __builtin_ctzll(cover);
          cover &= cover - 1ull;
          it[u] = __shfl(my_item, j);
        }
      }
      if (f.op == 1) {
        const float* subf = reinterpret_cast<const float*>(f.sub);
        float m4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) m4[u] = it[u] >= 0 ? subf[(int64_t)it[u] * 64 + lane] : -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u) M = fmaxf(M, m4[u]);
        continue;
      }
      float4 S[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        S[u] = it[u] >= 0 ? f.sub[(int64_t)it[u] * 64 + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float om = 1.0f - F.w;
        F.x = __builtin_fmaf(om, S[u].x, F.x);
        F.y = __builtin_fmaf(om, S[u].y, F.y);
        F.z = __builtin_fmaf(om, S[u].z, F.z);
        F.w = __builtin_fmaf(om, S[u].w, F.w);
      }
    }
  }
  if (f.op == 1 && M != -INFINITY) {
    const int K = f.fin->K;
    const float4* tab = reinterpret_cast<const float4*>(f.fin->table);
    float x = __builtin_fmaf(M, f.fin->tf_scale, f.fin->tf_bias);
    x = fminf(fmaxf(x, 0.0f), (float)(K - 1));
    const int i = min((int)x, K - 2);
    const float t = x - (float)i;
    const float4 a = tab[i], b = tab[i + 1];
    F = make_float4(__builtin_fmaf(t, b.x - a.x, a.x), __builtin_fmaf(t, b.y - a.y, a.y),
                    __builtin_fmaf(t, b.z - a.z, a.z), __builtin_fmaf(t, b.w - a.w, a.w));
  }
  if (px < W && py < H) out[((int64_t)v * H + py) * W + px] = F;
}

// Learned frame: squared differences of the upsampled image and the plain
// render over the validation tiles, a share per workgroup; the conditional
// pass's set-up adds them up and decides (setup_view).  One workgroup for all
// of it was bound by what a compute unit can have in flight: 510 tiles of a
// 1920x1080 frame, 1 MB, took 24 us, now 5.
__global__ __launch_bounds__(256) void psnr_kernel(BcFramePtrs f, const float4* __restrict__ ref,
                                                   const float4* __restrict__ img) {
  // FP32 throughout: each thread keeps a compensated (Kahan) sum of its
  // pixels' squared differences, and the partial sums are added pairwise
  // (relative error about 14 roundings).  A wave takes tiles in turn, a lane
  // one pixel of each.
  __shared__ float red[4];
  __shared__ int nred[4];
  const int ts = f.fin->tile_stride, tox = f.fin->tile_ox, toy = f.fin->tile_oy;
  const int W = f.width, H = f.height, nv = f.n_views;
  const int tsh = f.tile_shift, tw = 1 << tsh, th = 64 >> tsh;
  const int tiles_x = (W + tw - 1) >> tsh, tiles_y = (H + th - 1) >> (6 - tsh);
  const int sx = sel_count(0, tiles_x, ts, tox), sy = sel_count(0, tiles_y, ts, toy);
  const int fx = sel_first(0, ts, tox), fy = sel_first(0, ts, toy);
  const int total = nv * sx * sy;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int lx = lane & (tw - 1), ly = lane >> tsh;
  float acc = 0.0f, comp = 0.0f;
  int cnt = 0;
  for (int t = 4 * (int)blockIdx.x + wave; t < total; t += 4 * BC_PSNR_PARTS) {
    const int v = t / (sx * sy), rem = t - v * (sx * sy), row = rem / sx;
    const int px = (fx + (rem - row * sx) * ts) * tw + lx, py = (fy + row * ts) * th + ly;
    if (px >= W || py >= H) continue;
    const int64_t i = ((int64_t)v * H + py) * W + px;
    const float4 a = ref[i], b = img[i];
    const float dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z, dw = a.w - b.w;
    const float term = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, __builtin_fmaf(dz, dz, dw * dw)));
    const float y = term - comp;
    const float t2 = acc + y;
    comp = (t2 - acc) - y;
    acc = t2;
    cnt += 4;
  }
  for (int s = 32; s > 0; s >>= 1) {
    acc += __shfl_xor(acc, s);
    cnt += __shfl_xor(cnt, s);
  }
  if (lane == 0) {
    red[wave] = acc;
    nred[wave] = cnt;
  }
  __syncthreads();
  if (tid == 0) {
    f.ctr->psnr_sum[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    f.ctr->psnr_count[blockIdx.x] = nred[0] + nred[1] + nred[2] + nred[3];
  }
}

}  // namespace

hipError_t bc_launch_setup(const BcFramePtrs& f, hipStream_t st) {
  if (f.n_views == 1) {
    setup_kernel<<<1, 1024, 0, st>>>(f);
  } else {
    setup_views_kernel<<<f.n_views, 1024, 0, st>>>(f);
    setup_items_kernel<<<1, 1024, 0, st>>>(f);
  }
  return hipGetLastError();
}

hipError_t bc_launch_psnr(const BcFramePtrs& f, const float4* ref, const float4* img, hipStream_t st) {
  psnr_kernel<<<BC_PSNR_PARTS, 256, 0, st>>>(f, ref, img);
  return hipGetLastError();
}

hipError_t bc_launch_composite(const BcFramePtrs& f, float4* out, hipStream_t st) {
  const int tsh = f.tile_shift;
  const int tiles_x = (f.width + (1 << tsh) - 1) >> tsh, tiles_y = (f.height + (64 >> tsh) - 1) >> (6 - tsh);
  if (f.n_bricks <= kTileCompMax) {
    dim3 grid((tiles_x + 1) / 2, (tiles_y + 1) / 2, f.n_views);
    composite_tile_kernel<<<grid, 256, 0, st>>>(f, out);
  } else {
    dim3 grid((tiles_x + kCompBlock - 1) / kCompBlock, (tiles_y + kCompBlock - 1) / kCompBlock, f.n_views);
    composite_kernel<<<grid, 1024, 0, st>>>(f, out);
  }
  return hipGetLastError();
}
