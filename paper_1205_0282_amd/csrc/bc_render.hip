// Ray casting of bricks into sub-images (the per-GPU ray-casting step of
// Sections 1.2 and 2.3.2) and the empty-space classification it uses.
//
//  classify  once per transfer-function table: one bit per interpolation cell
//            of every brick (the cube between 2x2x2 neighbouring stored
//            voxels) telling whether any value the cell can interpolate to
//            maps to a non-zero table entry.  A sample in a clear cell adds
//            exactly zero to its ray, so it is counted but not evaluated.
//            For maximum intensity projection a cell is clear when every
//            value it can take lies in the leading run of colour-map entries
//            equal to the first one: such a maximum, and every smaller one,
//            maps to that first entry, so it never changes the pixel.
//  render    persistent kernel: every wave pulls (brick, view, 8x8 tile) work
//            items from a device counter and casts the tile's 64 rays
//            through the brick: ray from the viewer's matrices, clipping to
//            the cube and the brick, samples at a fixed step anchored at the
//            cube entry, trilinear interpolation, transfer-function lookup,
//            front-to-back compositing with early ray termination.
//
// Sample positions.  Per ray and brick the first sample's brick-local
// position and the step vector are formed in double-float arithmetic (bc_ray.h) and
// turned into 32.32 fixed point; every later sample position is an exact
// integer sum, so the cell index and the interpolation weights of sample j
// carry about 2^-32 voxels of error however far the ray has travelled.
//
// Lane schedule.  Each lane walks its own ray in chunks of 32 samples.  For a
// chunk it first gathers the 32 occupancy bits (cheap, all lanes in step),
// then evaluates only the samples whose cell is occupied, lowest first, so a
// lane's evaluations do not wait for the empty stretches of other lanes.
// FP32 compositing takes them two at a time: both samples' cells are
// gathered together (those gathers mostly miss the L1, so two in flight hide
// part of the wait), then the two are folded in order.
//
// Fewer gathers, fewer instructions.  The kernel is bound by the latency of
// its gathers (the L1 misses above all) together with instruction issue, not
// by HBM bandwidth.  So each lane avoids loads it can do without: consecutive
// samples in the same occupancy word reuse the word (the repeated load gets an
// out-of-range offset, answered by the range check without a cache access),
// and consecutive evaluated samples in the same interpolation cell reuse the
// cell's 8 voxels held in registers.  And the per-sample arithmetic is kept to
// single instructions where it can be: 24-bit multiply-adds with the strides
// in scalar registers, a floor-convert, a fract, a median-of-three clamp.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <float.h>
#include <type_traits>
#include "bc_types.h"
#include "bc_kernels.h"
#include "bc_ray.h"
#include "bc_e4m3.h"

// Launch data that no wave writes while the ray caster runs (frame inputs,
// view and brick records, the queue tables), addressed in the constant address
// space so that wave-uniform reads of it become scalar loads: they then wait on
// the scalar counter, not behind the vector loads and atomics in flight.
#define KC(T) const __attribute__((address_space(4))) T
template <typename T> __device__ __forceinline__ KC(T)* kc(const T* p) { return (KC(T)*)p; }

namespace {

// ------------------------------------------------------------------ storage
template <int FMT>
__device__ __forceinline__ float decode(uint32_t raw, float s, float o) {
  if (FMT == 0) return __uint_as_float(raw);
  if (FMT == 1) return __half2float(__ushort_as_half((unsigned short)raw));
  return __builtin_fmaf(bc_e4m3_decode(raw), s, o);
}

// Buffer resources: the hardware range check turns an offset outside the
// brick (or its occupancy bits) into a zero instead of a fault.  Base and size
// are made wave-uniform explicitly so that the resource lives in scalar
// registers (a resource the compiler cannot prove uniform is rebuilt lane by
// lane around every load).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  void* ub = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// a voxel and its +x neighbour (the next element) at a byte offset inside
// the brick, with one load
template <int FMT>
__device__ __forceinline__ void load_pair(__amdgpu_buffer_rsrc_t r, uint32_t ofs, float s, float o, float& a, float& b) {
  if (FMT == 0) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 p = __builtin_amdgcn_raw_buffer_load_b64(r, ofs, 0, 0);
    a = decode<0>(p.x, s, o);
    b = decode<0>(p.y, s, o);
  } else if (FMT == 1) {
    const uint32_t p = __builtin_amdgcn_raw_buffer_load_b32(r, ofs, 0, 0);
    a = decode<1>(p & 0xffffu, s, o);
    b = decode<1>(p >> 16, s, o);
  } else {
    // the hardware conversion of two E4M3 bytes is exact, as is the decode
    // above (the pool never holds the NaN codes: the encoder saturates)
    typedef float f2 __attribute__((ext_vector_type(2)));
    const uint32_t p = __builtin_amdgcn_raw_buffer_load_b16(r, ofs, 0, 0);
    const f2 v = __builtin_amdgcn_cvt_pk_f32_fp8((int)p, false);
    if (FMT == 3) {   // the codes' values only: the caller applies scale and offset
      a = v.x;
      b = v.y;
    } else {
      a = __builtin_fmaf(v.x, s, o);
      b = __builtin_fmaf(v.y, s, o);
    }
  }
}

// a * b + c on the low 24 bits of a and b (one multiply-add instruction)
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) { return __umul24(a, b) + c; }

// (a & mask) | (b & ~mask) in one instruction (the compiler splits the
// expression into ands and ors)
__device__ __forceinline__ uint32_t bfi_u32(uint32_t mask, uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(a), "v"(b));
  return r;
}

// a * b + c on signed 24-bit a and b (one multiply-add instruction)
__device__ __forceinline__ int mad_i24(int a, int b, int c) { return __mul24(a, b) + c; }

// floor(x) as an integer in one instruction
__device__ __forceinline__ int floor_i32(float x) {
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

// ------------------------------------------------------------------ classify
struct ClassifyArgs {
  const BcBrick* bricks;
  const BcFrameIn* fin;
  uint32_t* occ;
  const void* pool;
  int32_t n_bricks;
  int32_t x_tiles;        // 4-word tiles along x of the widest brick
  int32_t y_tiles;        // 16-word tiles along y of the deepest brick
  int32_t z_words;        // words along z of one walk (even)
  int32_t z_chunks;       // walks along z of the tallest brick
  uint32_t run;           // tiles dealt to an XCD at a time
  int32_t max_words;      // words of the largest brick (a thread per word)
  int32_t mip;            // classify for maximum intensity projection
};

// one stored row: the 4 voxels of a micro-block row and the first one of the
// next micro-block along x, as decoded values
template <int FMT>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, uint32_t ofs, float* v) {
  if (FMT == 0) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    const u4 p = __builtin_amdgcn_raw_buffer_load_b128(r, ofs, 0, 0);
    const uint32_t e = __builtin_amdgcn_raw_buffer_load_b32(r, ofs + 16u, 0, 0);
    v[0] = __uint_as_float(p.x);
    v[1] = __uint_as_float(p.y);
    v[2] = __uint_as_float(p.z);
    v[3] = __uint_as_float(p.w);
    v[4] = __uint_as_float(e);
  } else if (FMT == 1) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 p = __builtin_amdgcn_raw_buffer_load_b64(r, ofs, 0, 0);
    const uint32_t e = __builtin_amdgcn_raw_buffer_load_b16(r, ofs + 8u, 0, 0);
    v[0] = decode<1>(p.x & 0xffffu, 1.f, 0.f);
    v[1] = decode<1>(p.x >> 16, 1.f, 0.f);
    v[2] = decode<1>(p.y & 0xffffu, 1.f, 0.f);
    v[3] = decode<1>(p.y >> 16, 1.f, 0.f);
    v[4] = decode<1>(e, 1.f, 0.f);
  }
}

// before[k] = the entry ahead of the first one at or after k that matters, by a
// whole workgroup.  Those are the entries of non-zero opacity when compositing
// (premultiplied colour is zero wherever opacity is), those different from the
// first entry for maximum intensity projection.  Each thread takes a run of
// entries; the first one that matters behind its run comes from a suffix scan.
__device__ __forceinline__ void table_before(const ClassifyArgs& a, float* before, int32_t* wave_first) {
  constexpr int kNone = 0x7fff;
  const int K = a.fin->K, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float4* tab = reinterpret_cast<const float4*>(a.fin->table);
  const float4 e0 = tab[0];
  auto matters = [&](int k) -> bool {
    const float4 e = tab[k];
    if (!a.mip) return e.w != 0.0f;
    return e.x != e0.x || e.y != e0.y || e.z != e0.z || e.w != e0.w;
  };
  const int per = (K + 255) / 256, k0 = min(K, tid * per), k1 = min(K, k0 + per);
  int first = kNone;
  for (int k = k1 - 1; k >= k0; --k)
    if (matters(k)) first = k;
  int run = first;   // smallest over this lane and those above it
  for (int o = 1; o < 64; o <<= 1) {
    const int other = __shfl_down(run, o);
    if (lane + o < 64) run = min(run, other);
  }
  int behind = __shfl_down(run, 1);
  if (lane == 63) behind = kNone;
  if (lane == 0) wave_first[wave] = run;
  __syncthreads();
  for (int w = wave + 1; w < 4; ++w) behind = min(behind, wave_first[w]);
  for (int k = k1 - 1; k >= k0; --k) {
    if (matters(k)) behind = k;
    before[k] = (float)(behind - 1);
  }
  __syncthreads();
}

// A brick's mapping of stored values to the table, and the cells that can reach
// an entry that matters.
//
// FP8 compositing: the ray caster interpolates the codes' values and maps the
// result to the table with the brick's scale and offset folded in, fma(q, scale
// * s, fma(o, scale, bias)); the cells are bounded through the same mapping of
// the same values, so that every index the ray caster can form lies inside the
// checked range.  Projection compares decoded values: the decode is monotone, so
// it is taken of the two bounds.
template <int FMT>
struct CellMap {
  float csc, cbi, ds, dof, klast;
  int il_mask;   // projection: every entry from the first one on
  bool fold;
  __device__ __forceinline__ CellMap(const ClassifyArgs& a, const BcBrick& br) {
    const float sc = a.fin->tf_scale, bi = a.fin->tf_bias;
    fold = FMT == 2 && !a.mip;
    csc = fold ? sc * br.scale : sc;
    cbi = fold ? __builtin_fmaf(br.offs, sc, bi) : bi;
    ds = br.scale;
    dof = br.offs;
    klast = (float)(a.fin->K - 2);
    il_mask = a.mip ? 0 : -1;
  }
  // bits of the four cells between two slices' rows, of which l and h are the
  // smallest and largest of a row and its +y row at the 5 voxels along x
  __device__ __forceinline__ uint32_t cells(const float* l0, const float* h0, const float* l1, const float* h1,
                                            const float* before) const {
    uint32_t bits = 0;
    float l[5], h[5];
#pragma unroll
    for (int x = 0; x < 5; ++x) {
      l[x] = fminf(l0[x], l1[x]);
      h[x] = fmaxf(h0[x], h1[x]);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      float lo = fminf(fminf(l[x], l[x + 1]), FLT_MAX), hi = fmaxf(fmaxf(h[x], h[x + 1]), -FLT_MAX);
      if (FMT == 2 && !fold) {
        lo = __builtin_fmaf(lo, ds, dof);
        hi = __builtin_fmaf(hi, ds, dof);
      }
      // trilinear values lie within the corner range up to a few roundings
      const float m = fmaxf(fabsf(lo), fabsf(hi)) * 9.5367431640625e-07f + 1e-30f;   // 2^-20
      float xl = __builtin_fmaf(lo - m, csc, cbi), xh = __builtin_fmaf(hi + m, csc, cbi);
      // entries [il, ih] with il = min(floor(xl), K - 2) and ih =
      // min(floor(xh), K - 2) + 1: one of them matters if the first that
      // does from il on, less one, is at most floor(xh)
      xl = __builtin_amdgcn_fmed3f(xl, 0.0f, klast);
      xh = __builtin_amdgcn_fmed3f(xh, 0.0f, klast);
      bits |= before[(int)xl & il_mask] <= xh ? 1u << x : 0u;
    }
    return bits;
  }
};

// Bound by the one read of the pool.  A stored row holds what the 4 cells of a
// word's row need along x.  So a lane takes one row of cells and walks up z;
// 16 neighbouring lanes take 16 rows along y (4 words), each with its +y row
// from the lane above it; a wave has 4 such columns along x, a workgroup four
// waves along y, the last row of a wave taking its +y row from the next wave
// through LDS and that of the last wave from memory.  A word's 32 bits meet by
// two cross-lane ORs.  1024^3 FP32 cube (5.5 GB): 1.52 ms, 6.6 GB read, 4.3
// TB/s; a thread per word with 75 loads of its own took 5.74 ms, and with
// every lane loading its +y rows this form read 8.4 GB in 1.78 ms.
template <int FMT>
__global__ __launch_bounds__(256) void classify_kernel(ClassifyArgs a) {
  __shared__ float before[BC_MAX_K];   // before[k] = the entry ahead of the first one at or after k that matters
  __shared__ int32_t wave_first[4];
  __shared__ __attribute__((aligned(16))) float edge[2][4][4][20];   // first rows: [turn parity][wave][column][slice][x]
  table_before(a, before, wave_first);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  static_assert(FMT < 2, "FP8: a thread per word");
  constexpr uint32_t esz = FMT == 0 ? 4 : 2;
  const int cy = tid & 3;                                  // the lane's cell row in its word
  const bool top = (lane & 15) == 15, bottom = (lane & 15) == 0;   // the last and the first of its 16 rows
  int parity = 0;
  // neighbouring tiles share rows: the tiles are dealt out in runs, to the
  // workgroups of each XCD in turn (as these are dispatched), so that
  // neighbours meet in one L2
  const int per_plane = a.x_tiles * a.y_tiles;
  const uint32_t per_brick = (uint32_t)per_plane * a.z_chunks, total = per_brick * a.n_bricks;   // (65 * 17 * 129 * 4096 at most)
  for (uint32_t at = blockIdx.x >> 3;; at += gridDim.x >> 3) {
    const uint32_t round = at / a.run * 8 * a.run, item = round + (blockIdx.x & 7) * a.run + at % a.run;
    if (round >= total) break;
    if (item >= total) continue;
    const int b = (int)(item / per_brick), rem = (int)(item - (uint32_t)b * per_brick);
    const int zc = rem / per_plane, tile = rem - zc * per_plane, ty = tile / a.x_tiles, tx = tile - ty * a.x_tiles;
    const BcBrick& br = a.bricks[b];
    const int WX = br.occ_w[0], WY = br.occ_w[1], WZ = br.occ_w[2];
    const int w0 = zc * a.z_words, w1 = min(w0 + a.z_words, WZ);
    const int wx = tx * 4 + (lane >> 4), wy = ty * 16 + wave * 4 + ((lane & 15) >> 2);
    if (w0 >= w1 || tx * 4 >= WX || ty * 16 >= WY) continue;   // (the whole workgroup)
    // cells 0..nc-1 per axis; cell i spans ghosted voxels i and i+1
    const int ncx = br.hi[0] - br.lo[0] + 1, ncy = br.hi[1] - br.lo[1] + 1, ncz = br.hi[2] - br.lo[2] + 1;
    const bool word = wx < WX && wy < WY, stored = wx < WX && wy < br.mb[1];   // (a last row of cells may need one more row)
    const bool live = ty * 16 + wave * 4 < WY;   // (other waves only bring the row above)
    const uint32_t row_mask = word && wy * 4 + cy < ncy ? (1u << clampi(ncx - wx * 4, 0, 4)) - 1u : 0u;
    const uint32_t mbx = (uint32_t)br.mb[0], mby = (uint32_t)br.mb[1];
    const uint32_t slab = mbx * mby * (BC_MB_ELEMS * esz);
    const __amdgpu_buffer_rsrc_t pool =
        make_rsrc(static_cast<const char*>(a.pool) + br.offset * esz, slab * (uint32_t)br.mb[2]);
    // the lane's row in slice z (rows past the brick read as zero; their cells are masked)
    const uint32_t row0 = (((uint32_t)wy * mbx + (uint32_t)wx) * BC_MB_ELEMS + (uint32_t)cy * BC_ROW) * esz;
    const uint32_t dy = (mbx * BC_MB_ELEMS - 3u * BC_ROW) * esz;   // from a word's last row to the next word's first
    const CellMap<FMT> map(a, br);
    // N slices from z on: smallest and largest of the lane's row and its +y
    // row, at the 5 voxels along x
    auto slices = [&](int z, auto count, float (*lo)[5], float (*hi)[5]) {
      constexpr int N = decltype(count)::value;
      float u[N][5], v[N][5];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const uint32_t ofs = row0 + (uint32_t)((z + k) >> 2) * slab + (uint32_t)((z + k) & 3) * (4u * BC_ROW * esz);
        load_row<FMT>(pool, stored ? ofs : 0xffffff00u, u[k]);   // (past the range: no access)
        if (wave == 3) load_row<FMT>(pool, word && top ? ofs + dy : 0xffffff00u, v[k]);
      }
      if (bottom) {
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
          for (int x = 0; x < 5; ++x) edge[parity][wave][lane >> 4][5 * k + x] = u[k][x];
      }
      __syncthreads();
      if (wave != 3) {
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
          for (int x = 0; x < 5; ++x) v[k][x] = edge[parity][wave + 1][lane >> 4][5 * k + x];
      }
      parity ^= 1;   // (the next turn's rows go beside these: one barrier a turn)
#pragma unroll
      for (int k = 0; k < N; ++k)
#pragma unroll
        for (int x = 0; x < 5; ++x) {
          // the row of the lane above (row_shl:1), the next wave's first one in the last lane
          const float y1 = __int_as_float(
              __builtin_amdgcn_update_dpp(__float_as_int(v[k][x]), __float_as_int(u[k][x]), 0x101, 0xf, 0xf, false));
          lo[k][x] = fminf(u[k][x], y1);
          hi[k][x] = fmaxf(u[k][x], y1);
        }
    };
    auto cells = [&](const float* l0, const float* h0, const float* l1, const float* h1) -> uint32_t {
      return map.cells(l0, h0, l1, h1, before) & row_mask;
    };
    auto put = [&](int w, uint32_t bits) {
      bits <<= 4 * cy;
      bits |= (uint32_t)__builtin_amdgcn_mov_dpp((int)bits, 0xb1, 0xf, 0xf, true);   // lane ^ 1
      bits |= (uint32_t)__builtin_amdgcn_mov_dpp((int)bits, 0x4e, 0xf, 0xf, true);   // lane ^ 2
      if (cy == 0 && word) a.occ[br.occ_offset + ((int64_t)w * WY + wy) * WX + wx] = bits;
    };
    // A micro-block (four slices, two words) per turn, all of its rows in
    // flight together: its 320 bytes are two or three lines that would be
    // fetched again if a turn took some of them.  The second word's last cells
    // wait for the next turn's first slice.
    float l[4][5], h[4][5], pl[5], ph[5];
    uint32_t half = 0;
    for (int w = w0; w < w1; w += 2) {
      slices(2 * w, std::integral_constant<int, 4>{}, l, h);
      if (live) {
        if (w > w0) put(w - 1, half | cells(pl, ph, l[0], h[0]) << 16);
        uint32_t bits = cells(l[0], h[0], l[1], h[1]);
        const uint32_t odd = cells(l[1], h[1], l[2], h[2]);
        if (2 * w + 1 < ncz) bits |= odd << 16;
        put(w, bits);
        half = cells(l[2], h[2], l[3], h[3]);
      }
#pragma unroll
      for (int x = 0; x < 5; ++x) {
        pl[x] = l[3][x];
        ph[x] = h[3][x];
      }
    }
    if (!((w1 - w0) & 1)) {   // the last word is a second one
      slices(2 * w1, std::integral_constant<int, 1>{}, l, h);
      if (live) {
        const uint32_t odd = cells(pl, ph, l[0], h[0]);
        if (2 * w1 - 1 < ncz) half |= odd << 16;
        put(w1 - 1, half);
      }
    }
  }
}

// FP8, and bricks so thin that few of those lanes would have a row: a thread per
// word, with the word's 15 rows read through registers, three slices at a time
// up y.  Bound by its loads, 15 rows of 64 lanes each; an FP8 row is one line's
// part for several lanes, an FP32 one is not (1024^3 in 256^3 bricks: FP8 1.43
// ms against 1.51 by rows; FP32 2.6 times as long as by rows).
template <int FMT>
__global__ __launch_bounds__(256) void classify_words_kernel(ClassifyArgs a) {
  __shared__ float before[BC_MAX_K];
  __shared__ int32_t wave_first[4];
  table_before(a, before, wave_first);
  constexpr uint32_t esz = FMT == 0 ? 4 : (FMT == 1 ? 2 : 1);
  const int64_t total = (int64_t)a.n_bricks * a.max_words;
  for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < total; g += (int64_t)gridDim.x * 256) {
    const int b = (int)(g / a.max_words), w = (int)(g - (int64_t)b * a.max_words);
    const BcBrick& br = a.bricks[b];
    const int WX = br.occ_w[0], WY = br.occ_w[1];
    if (w >= WX * WY * br.occ_w[2]) continue;
    const int wx = w % WX, wy = w / WX % WY, wz = w / (WX * WY);
    const int ncx = br.hi[0] - br.lo[0] + 1, ncy = br.hi[1] - br.lo[1] + 1, ncz = br.hi[2] - br.lo[2] + 1;
    const uint32_t mask = (1u << clampi(ncx - wx * 4, 0, 4)) - 1u;
    const uint32_t mbx = (uint32_t)br.mb[0], slab = mbx * (uint32_t)br.mb[1] * (BC_MB_ELEMS * esz);
    // (the lanes' bricks differ: an address each, clamped to the last row and
    // slice, whose copies belong to cells that are masked)
    const char* pool = static_cast<const char*>(a.pool) + br.offset * esz;
    const CellMap<FMT> map(a, br);
    auto row = [&](int y, int z, float* v) {
      y = min(y, ncy);
      z = min(z, ncz);
      const uint32_t ofs = (((uint32_t)(y >> 2) * mbx + (uint32_t)wx) * BC_MB_ELEMS + (uint32_t)(4 * (z & 3) + (y & 3)) * BC_ROW) * esz +
                           (uint32_t)(z >> 2) * slab;
#pragma unroll
      for (int x = 0; x < 5; ++x) {
        if (FMT == 0) v[x] = *reinterpret_cast<const float*>(pool + ofs + 4 * x);
        else if (FMT == 1) v[x] = __half2float(*reinterpret_cast<const __half*>(pool + ofs + 2 * x));
        else v[x] = bc_e4m3_decode(*reinterpret_cast<const uint8_t*>(pool + ofs + x));
      }
    };
    uint32_t bits = 0;
    float p[3][5];
#pragma unroll
    for (int z = 0; z < 3; ++z) row(4 * wy, 2 * wz + z, p[z]);
#pragma unroll
    for (int cy = 0; cy < 4; ++cy) {
      float q[3][5], l[3][5], h[3][5];
#pragma unroll
      for (int z = 0; z < 3; ++z) {
        row(4 * wy + cy + 1, 2 * wz + z, q[z]);
#pragma unroll
        for (int x = 0; x < 5; ++x) {
          l[z][x] = fminf(p[z][x], q[z][x]);
          h[z][x] = fmaxf(p[z][x], q[z][x]);
          p[z][x] = q[z][x];
        }
      }
      if (4 * wy + cy >= ncy) break;
      bits |= (map.cells(l[0], h[0], l[1], h[1], before) & mask) << (4 * cy);
      if (2 * wz + 1 < ncz) bits |= (map.cells(l[1], h[1], l[2], h[2], before) & mask) << (16 + 4 * cy);
    }
    a.occ[br.occ_offset + w] = bits;
  }
}

__device__ __forceinline__ int hi32(int64_t v) { return (int)(v >> 32); }
__device__ __forceinline__ float frac32(int64_t v) { return (float)(uint32_t)v * 2.3283064365386963e-10f; }

// ------------------------------------------------------------------ render
// OP 0: front-to-back compositing into premultiplied RGBA with early
// termination at opacity tau.  OP 1: maximum intensity projection, the largest
// sample value per ray (-inf for a ray with no sample in the brick, -FLT_MAX
// when all its samples fell in clear cells), stopping once it reaches the
// largest value the brick stores.
// URGENT: the waves issue at the raised priority levels (2, and 3 while they
// evaluate occupied samples) instead of the base levels (0 and 1): the plain
// passes' setting, while a pass that runs beside a more urgent one (a learned
// frame's coarse pass beside its validation pass) keeps the base levels; a
// template parameter so that each instantiation holds one setting.
template <int FMT, bool TF_LDS, int CHUNK, int OP, bool URGENT>
__global__ __launch_bounds__(256, 4) void render_kernel(BcFramePtrs f) {
  // table entry k at 2k, its difference to entry k+1 at 2k+1
  __shared__ float4 s_tab[(TF_LDS && OP == 0) ? 2 * BC_TF_LDS : 2];
  const int lane = threadIdx.x & 63;
  KC(BcFrameIn)* fin = kc(f.fin);
  KC(BcCounters)* cr = kc(f.ctr);   // the lines the waves read, not the queue counters
  if (cr->n_items == 0) return;   // e.g. a conditional pass that is not needed
  if (URGENT) __builtin_amdgcn_s_setprio(2);
  const int K = fin->K;
  const float tf_scale = fin->tf_scale;
  // held in a vector register: an FMA can read only one scalar operand
  float tf_bias = fin->tf_bias;
  if (OP == 0) asm volatile("" : "+v"(tf_bias));
  const float kmax_f = (float)(K - 1);
  const float4* gtab = reinterpret_cast<const float4*>(f.fin->table);   // gathered per lane
  if (TF_LDS && OP == 0) {
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
      const float4 a = gtab[k], b = gtab[min(k + 1, K - 1)];
      s_tab[2 * k] = a;
      s_tab[2 * k + 1] = make_float4(b.x - a.x, b.y - a.y, b.z - a.z, b.w - a.w);
    }
    __syncthreads();
  }

  const int nv = f.n_views, nb = f.n_bricks;
  const int KB = nb * nv;
  const uint32_t n_items = cr->n_items;
  const bool ess = f.ess != 0;
  const bool per_voxel = f.step_policy != 0;
  const int ts = fin->tile_stride;
  constexpr uint32_t esz = FMT == 0 ? 4 : (FMT == 1 ? 2 : 1);
  // per-lane sample counts (a lane takes at most a few thousand samples per
  // item and a few dozen items per launch, far below 2^32)
  uint32_t nominal = 0, evaluated = 0;
  // the queue of the XCD this workgroup runs on first, then the others once
  // it is drained; the XCD comes from its hardware id register (XCC_ID, bits
  // 0-3), not from the block index, so that the choice holds however the
  // dispatcher deals workgroups to the XCDs (0.2% faster on the bench orbit).
  // Q is 8 or 1, so Q - 1 masks the id to a queue (written without a branch,
  // which left the projection kernels out of scalar registers)
  const int Q = (int)cr->n_queues;
  int q = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & (uint32_t)(Q - 1)), drained = 0;
  uint32_t q_lo = cr->qbound[q], q_hi = cr->qbound[q + 1];
  // a slot is claimed when the wave needs it: claiming one item ahead, the
  // atomic in flight during the item before, made the launch 8% slower
  for (;;) {
    uint32_t item = 0;
    bool have = false;
    while (drained < Q) {
      const uint32_t claim = lane == 0 ? atomicAdd(&f.ctr->q[q].next, 1u) : 0u;
      const uint32_t it = q_lo + (uint32_t)__builtin_amdgcn_readlane((int)claim, 0);
      if (it < q_hi && it < n_items) {
        item = it;
        have = true;
        break;
      }
      ++drained;
      q = (q + 1 == Q) ? 0 : q + 1;
      q_lo = cr->qbound[q];
      q_hi = cr->qbound[q + 1];
    }
    if (!have) break;
    KC(int32_t)* perm = kc(f.item_perm);
    int lo = 0, hi = KB;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((uint32_t)perm[mid] <= item) lo = mid; else hi = mid;
    }
    KC(int4)& ent = kc(f.item_entry)[lo];
    const int b = ent.x & 0xffff, v = ent.x >> 16, cx = ent.y;
    const int local = (int)(item - (uint32_t)perm[lo]);
    const int tx = ent.z + (local % cx) * ts, ty = ent.w + (local / cx) * ts;
    KC(BcViewParams)& vp = kc(f.views)[v];
    const int tsh = f.tile_shift;
    const int px = (tx << tsh) + (lane & ((1 << tsh) - 1));
    const int py = ty * (64 >> tsh) + (lane >> tsh);
    KC(BcBrick)& br = kc(f.bricks)[b];
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float mx = -INFINITY;
    RaySeg seg;
    if (px < vp.width && py < vp.height && ray_segment(vp, f.gdims, br, px, py, per_voxel, seg)) {
      const float tau = vp.tau;
      const float bound = br.dmax;
      mx = -FLT_MAX;
      const int cmx = br.hi[0] - br.lo[0], cmy = br.hi[1] - br.lo[1], cmz = br.hi[2] - br.lo[2];
      const int mbx = br.mb[0], mby = br.mb[1];
      const uint32_t WX = (uint32_t)br.occ_w[0], WY = (uint32_t)br.occ_w[1], WX4 = 4u * WX;
      const uint32_t n_occ = WX * WY * (uint32_t)br.occ_w[2];
      const __amdgpu_buffer_rsrc_t occ = make_rsrc(f.occ + br.occ_offset, n_occ * 4u);
      const uint32_t n_vox = (uint32_t)br.mb[0] * (uint32_t)br.mb[1] * (uint32_t)br.mb[2] * BC_MB_ELEMS;
      const __amdgpu_buffer_rsrc_t pool = make_rsrc(static_cast<const char*>(f.pool) + br.offset * esz, n_vox * esz);
      const float s_q = br.scale, o_q = br.offs;
      // FP8 compositing: interpolation is linear, so the brick's scale and
      // offset move from the 8 decoded voxels into the table index (one
      // multiply-add per sample); MIP compares decoded values with the
      // brick maximum and decodes each voxel
      constexpr bool FOLD = FMT == 2 && OP == 0;
      // FP32 evaluates its occupied samples two at a time (its gathers miss
      // the L1 most; 1.305 -> 1.229 ms on the bench orbit, and 0.915 -> 0.879
      // ms with maximum intensity projection at the per-voxel step); the
      // narrower forms, whose cells more often share cached lines, one at a
      // time, and so does projection with 64-sample chunks, which would spill
      constexpr bool PAIRS = FMT == 0 && (OP == 0 || CHUNK == 32);
      const float tsc = FOLD ? tf_scale * s_q : tf_scale, tbi = FOLD ? __builtin_fmaf(o_q, tf_scale, tf_bias) : tf_bias;
      // byte steps to the +y/+z neighbour: inside a micro-block, or across
      // into the next one (from its last row or slice)
      constexpr uint32_t sh = FMT == 0 ? 2 : (FMT == 1 ? 1 : 0);
      uint32_t dyb = ((uint32_t)mbx * BC_MB_ELEMS - 3u * BC_ROW) << sh,
               dzb = ((uint32_t)mbx * (uint32_t)mby * BC_MB_ELEMS - 12u * BC_ROW) << sh;
      asm volatile("" : "+v"(dyb), "+v"(dzb));   // (selected per lane below)
      // the element index of ghosted local voxel (x, y, z) in the brick: 4x4x4
      // micro-blocks stored row-major, each as 16 rows (y, then z) of 5
      // elements, x fastest.  As a sum of per-axis terms: along x
      // 80 (x>>2) + (x&3) = 20 x - 19 (x&3), along y and z likewise with the
      // micro-block row and slice strides; in bytes
      const uint32_t cxb = 20u << sh;
      uint32_t cyb = (20u * (uint32_t)mbx) << sh, czb = (20u * (uint32_t)mbx * (uint32_t)mby) << sh;
      const int rxb = -(int)(19u << sh);
      int ryb = (int)(BC_ROW << sh) - (int)cyb, rzb = (int)((4u * BC_ROW) << sh) - (int)czb;
      // (projection has vector registers to spare and no scalar ones)
      if (OP == 1) asm volatile("" : "+v"(cyb), "+v"(czb), "+v"(ryb), "+v"(rzb));
      int64_t uc0 = seg.u[0], uc1 = seg.u[1], uc2 = seg.u[2];
      // the step, with y and z scaled by 4 and 16 (kept only so, to save
      // registers) so that in the occupancy pass bits 2-3 of the integer part
      // of y' hold y%4 and bit 4 of z' holds z%2
      const int64_t s0 = seg.s[0], s1q = seg.s[1] * 4, s2q = seg.s[2] * 16;
      const float sfx = (float)s0 * 2.3283064365386963e-10f, sfy = (float)seg.s[1] * 2.3283064365386963e-10f,
                  sfz = (float)seg.s[2] * 2.3283064365386963e-10f;
      int used = seg.n;
      // the voxels of the cell the lane interpolated last, and its offset
      // (none yet)
      uint32_t cell_ofs = 0xffffffffu;
      float cv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int k = 0; k < seg.n; k += CHUNK) {
        const int cnt = min(CHUNK, seg.n - k);
        uint64_t mask = cnt >= 64 ? ~0ull : ((1ull << cnt) - 1ull);
        if (ess) {
          int64_t un0 = uc0, un1 = uc1 * 4, un2 = uc2 * 16;
          // occupancy bits of the chunk's samples (cells outside the brick
          // read as clear through the buffer range check)
          // all addresses first, then all loads in flight together
          uint64_t m = 0;
          uint32_t occ_ofs = 0xffffffffu, occ_word = 0u;   // the occupancy word loaded last
#pragma unroll
          for (int h = 0; h < CHUNK / 8; ++h) {
            uint32_t wofs[8], bit[8], word[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              // x, 4 y + (2 bits), 16 z + (4 bits)
              const uint32_t ix = (uint32_t)hi32(un0), iy4 = (uint32_t)hi32(un1), iz16 = (uint32_t)hi32(un2);
              // word (x/4, y/4, z/2) as a byte offset; bit (x%4) + 4 (y%4) + 16 (z%2), of
              // which the bit-field extract below reads only the low five bits
              wofs[i] = mad_u24(mad_u24(iz16 >> 5, WY, iy4 >> 4), WX4, ix & ~3u);
              // two bit-field inserts: x%4 into 4 (y%4), then into 16 (z%2)
              bit[i] = bfi_u32(15u, bfi_u32(3u, ix, iy4), iz16);
              un0 += s0; un1 += s1q; un2 += s2q;
            }
            // a sample in the same word as the one before it reuses that
            // word: its load gets an offset past the end of the bits, which
            // the range check answers without a cache access
            bool fresh[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) fresh[i] = wofs[i] != (i ? wofs[i - 1] : occ_ofs);
            occ_ofs = wofs[7];
#pragma unroll
            for (int i = 0; i < 8; ++i)
              word[i] = __builtin_amdgcn_raw_buffer_load_b32(occ, fresh[i] ? wofs[i] : 0xfffffff0u, 0, 0);
            uint32_t mh = 0;
            // (a reused sample's load returned zero: keep the word before)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              occ_word = word[i] | (fresh[i] ? 0u : occ_word);
              mh |= __builtin_amdgcn_ubfe(occ_word, bit[i], 1u) << i;
            }
            m |= (uint64_t)mh << (8 * h);
          }
          mask &= m;
        }
        bool stop = false;
        if (mask) {
          // a wave evaluating samples waits on dependent gathers; letting it
          // issue ahead of the waves gathering occupancy bits (whose loads are
          // all in flight together) shortens the frame
          __builtin_amdgcn_s_setprio(URGENT ? 3 : 1);
          // sample positions inside the chunk in FP32, relative to the
          // chunk's first sample: integer cell of that sample plus a
          // fraction that stays below 1 + CHUNK/2 voxels
          const int bx = hi32(uc0), by = hi32(uc1), bz = hi32(uc2);
          const float fx0 = frac32(uc0), fy0 = frac32(uc1), fz0 = frac32(uc2);
          // the sample that ended the ray (the loop runs out instead of
          // breaking, which keeps the loop's registers in place)
          int last = CHUNK - 1;
          for (int half = 0; half < CHUNK / 32; ++half) {
            uint32_t m32 = stop ? 0u : (uint32_t)(mask >> (32 * half));
            if constexpr (PAIRS) {
              // occupied samples two at a time: both cells' gathers in flight
              // together (the second sample's only if its cell differs from the
              // first's), then the samples folded in order; the arithmetic of
              // each sample is that of one taken alone
              while (m32) {
                const int i0 = 32 * half + (int)__builtin_ctz(m32);
                m32 &= m32 - 1u;
                const bool two = m32 != 0u;
                const int i1 = two ? 32 * half + (int)__builtin_ctz(m32) : i0;
                if (two) m32 &= m32 - 1u;
                float w0[3], w1[3];
                uint32_t a0, a1;
                int ry0, rz0, ry1, rz1;
                auto cell = [&](int i, float* w, uint32_t& a, int& ry, int& rz) {
                  const float fi = (float)i;
                  const float ux = __builtin_fmaf(fi, sfx, fx0), uy = __builtin_fmaf(fi, sfy, fy0),
                              uz = __builtin_fmaf(fi, sfz, fz0);
                  w[0] = __builtin_amdgcn_fractf(ux);
                  w[1] = __builtin_amdgcn_fractf(uy);
                  w[2] = __builtin_amdgcn_fractf(uz);
                  const uint32_t ix = (uint32_t)(bx + floor_i32(ux)), iy = (uint32_t)(by + floor_i32(uy)),
                                 iz = (uint32_t)(bz + floor_i32(uz));
                  ry = (int)(iy & 3u);
                  rz = (int)(iz & 3u);
                  a = (uint32_t)mad_i24(rz, rzb, mad_i24(ry, ryb, mad_i24((int)(ix & 3u), rxb,
                                        (int)mad_u24(ix, cxb, mad_u24(iy, cyb, __umul24(iz, czb))))));
                };
                auto gather = [&](uint32_t a, int ry, int rz, float* v) {
                  const uint32_t dy = ry == 3 ? dyb : (BC_ROW << sh);
                  const uint32_t dz = rz == 3 ? dzb : ((4u * BC_ROW) << sh);
                  const uint32_t a010 = a + dy, a001 = a + dz, a011 = a001 + dy;
                  load_pair<FOLD ? 3 : FMT>(pool, a, s_q, o_q, v[0], v[1]);
                  load_pair<FOLD ? 3 : FMT>(pool, a010, s_q, o_q, v[2], v[3]);
                  load_pair<FOLD ? 3 : FMT>(pool, a001, s_q, o_q, v[4], v[5]);
                  load_pair<FOLD ? 3 : FMT>(pool, a011, s_q, o_q, v[6], v[7]);
                };
                cell(i0, w0, a0, ry0, rz0);
                cell(i1, w1, a1, ry1, rz1);
                if (a0 != cell_ofs) {
                  gather(a0, ry0, rz0, cv);
                  cell_ofs = a0;
                }
                float cw[8];
                const bool own1 = two && a1 != a0;
                if (own1) gather(a1, ry1, rz1, cw);
                auto sample = [&](const float* v, const float* w, int i) {
                  const float c00 = __builtin_fmaf(w[0], v[1] - v[0], v[0]);
                  const float c10 = __builtin_fmaf(w[0], v[3] - v[2], v[2]);
                  const float c01 = __builtin_fmaf(w[0], v[5] - v[4], v[4]);
                  const float c11 = __builtin_fmaf(w[0], v[7] - v[6], v[6]);
                  const float c0 = __builtin_fmaf(w[1], c10 - c00, c00);
                  const float c1 = __builtin_fmaf(w[1], c11 - c01, c01);
                  const float val = __builtin_fmaf(w[2], c1 - c0, c0);
                  if (OP == 1) {
                    mx = fmaxf(mx, val);
                    if (mx >= bound) {
                      last = i;
                      stop = true;
                      m32 = 0u;
                    }
                    return;
                  }
                  const float xt = __builtin_amdgcn_fmed3f(__builtin_fmaf(val, tsc, tbi), 0.0f, kmax_f);
                  const int it = TF_LDS ? (int)xt : min((int)xt, K - 2);
                  const float ft = TF_LDS ? __builtin_amdgcn_fractf(xt) : xt - (float)it;
                  float4 q0, dq;
                  if (TF_LDS) {
                    q0 = s_tab[2 * it];
                    dq = s_tab[2 * it + 1];
                  } else {
                    q0 = gtab[it];
                    const float4 q1 = gtab[it + 1];
                    dq = make_float4(q1.x - q0.x, q1.y - q0.y, q1.z - q0.z, q1.w - q0.w);
                  }
                  const float om = 1.0f - acc.w;
                  acc.x = __builtin_fmaf(om, __builtin_fmaf(ft, dq.x, q0.x), acc.x);
                  acc.y = __builtin_fmaf(om, __builtin_fmaf(ft, dq.y, q0.y), acc.y);
                  acc.z = __builtin_fmaf(om, __builtin_fmaf(ft, dq.z, q0.z), acc.z);
                  acc.w = __builtin_fmaf(om, __builtin_fmaf(ft, dq.w, q0.w), acc.w);
                  if (acc.w >= tau) {
                    last = i;
                    stop = true;
                    m32 = 0u;
                  }
                };
                sample(cv, w0, i0);
                if (two && !stop) {
                  if (own1) {
  #pragma unroll
                    for (int q = 0; q < 8; ++q) cv[q] = cw[q];
                    cell_ofs = a1;
                  }
                  sample(cv, w1, i1);
                }
              }
            } else {
              while (m32) {
                const int i = 32 * half + (int)__builtin_ctz(m32);
                m32 &= m32 - 1u;
                const float fi = (float)i;
                const float ux = __builtin_fmaf(fi, sfx, fx0), uy = __builtin_fmaf(fi, sfy, fy0),
                            uz = __builtin_fmaf(fi, sfz, fz0);
                const float wx = __builtin_amdgcn_fractf(ux), wy = __builtin_amdgcn_fractf(uy),
                            wz = __builtin_amdgcn_fractf(uz);
                // the sample's cell (inside the brick: 0 <= ix, iy, iz < 2^24)
                const uint32_t ix = (uint32_t)(bx + floor_i32(ux)), iy = (uint32_t)(by + floor_i32(uy)),
                               iz = (uint32_t)(bz + floor_i32(uz));
                const int ry = (int)(iy & 3u), rz = (int)(iz & 3u);
                const uint32_t a000 = (uint32_t)mad_i24(
                    rz, rzb, mad_i24(ry, ryb, mad_i24((int)(ix & 3u), rxb,
                                                      (int)mad_u24(ix, cxb, mad_u24(iy, cyb, __umul24(iz, czb))))));
                // the 8 voxels of the sample's cell, loaded only when the cell
                // differs from the one the lane interpolated last
                if (a000 != cell_ofs) {
                  const uint32_t dy = ry == 3 ? dyb : (BC_ROW << sh);
                  const uint32_t dz = rz == 3 ? dzb : ((4u * BC_ROW) << sh);
                  const uint32_t a010 = a000 + dy, a001 = a000 + dz, a011 = a001 + dy;
                  load_pair<FOLD ? 3 : FMT>(pool, a000, s_q, o_q, cv[0], cv[1]);
                  load_pair<FOLD ? 3 : FMT>(pool, a010, s_q, o_q, cv[2], cv[3]);
                  load_pair<FOLD ? 3 : FMT>(pool, a001, s_q, o_q, cv[4], cv[5]);
                  load_pair<FOLD ? 3 : FMT>(pool, a011, s_q, o_q, cv[6], cv[7]);
                  cell_ofs = a000;
                }
                const float c00 = __builtin_fmaf(wx, cv[1] - cv[0], cv[0]);
                const float c10 = __builtin_fmaf(wx, cv[3] - cv[2], cv[2]);
                const float c01 = __builtin_fmaf(wx, cv[5] - cv[4], cv[4]);
                const float c11 = __builtin_fmaf(wx, cv[7] - cv[6], cv[6]);
                const float c0 = __builtin_fmaf(wy, c10 - c00, c00);
                const float c1 = __builtin_fmaf(wy, c11 - c01, c01);
                const float val = __builtin_fmaf(wz, c1 - c0, c0);
                if (OP == 1) {
                  mx = fmaxf(mx, val);
                  if (mx >= bound) {
                    last = i;
                    stop = true;
                    m32 = 0u;
                  }
                  continue;
                }
                // clamp to [0, K-1] (the median of three, exact)
                const float xt = __builtin_amdgcn_fmed3f(__builtin_fmaf(val, tsc, tbi), 0.0f, kmax_f);
                // (the table in LDS has an entry K-1 with a zero difference)
                const int it = TF_LDS ? (int)xt : min((int)xt, K - 2);
                const float ft = TF_LDS ? __builtin_amdgcn_fractf(xt) : xt - (float)it;
                // table entry and its difference to the next entry
                float4 q0, dq;
                if (TF_LDS) {
                  q0 = s_tab[2 * it];
                  dq = s_tab[2 * it + 1];
                } else {
                  q0 = gtab[it];
                  const float4 q1 = gtab[it + 1];
                  dq = make_float4(q1.x - q0.x, q1.y - q0.y, q1.z - q0.z, q1.w - q0.w);
                }
                const float om = 1.0f - acc.w;
                acc.x = __builtin_fmaf(om, __builtin_fmaf(ft, dq.x, q0.x), acc.x);
                acc.y = __builtin_fmaf(om, __builtin_fmaf(ft, dq.y, q0.y), acc.y);
                acc.z = __builtin_fmaf(om, __builtin_fmaf(ft, dq.z, q0.z), acc.z);
                acc.w = __builtin_fmaf(om, __builtin_fmaf(ft, dq.w, q0.w), acc.w);
                if (acc.w >= tau) {
                  last = i;
                  stop = true;
                  m32 = 0u;
                }
              }
            }
          }
          __builtin_amdgcn_s_setprio(URGENT ? 2 : 0);
          // the occupied samples up to the last one evaluated
          evaluated += (uint32_t)__builtin_popcountll(mask & (~0ull >> (63 - last)));
          if (stop) used = k + last + 1;
        }
        if (stop) break;
        uc0 += CHUNK * s0; uc1 += (CHUNK * s1q) >> 2; uc2 += (CHUNK * s2q) >> 4;
      }
      nominal += (uint32_t)used;
    }
    if (OP == 0) f.sub[(int64_t)item * 64 + lane] = acc;
    else reinterpret_cast<float*>(f.sub)[(int64_t)item * 64 + lane] = mx;
  }
  uint64_t wave_nominal = nominal, wave_evaluated = evaluated;
  for (int off = 32; off > 0; off >>= 1) {
    wave_nominal += __shfl_xor(wave_nominal, off);
    wave_evaluated += __shfl_xor(wave_evaluated, off);
  }
  if (lane == 0 && wave_nominal) {
    atomicAdd(&f.ctr->nominal, (unsigned long long)wave_nominal);
    atomicAdd(&f.ctr->evaluated, (unsigned long long)wave_evaluated);
  }
}

// ------------------------------------------------------------------ render, few work items
// A frame of few work items leaves most of the chip idle while each wave walks
// a whole tile: its time is one wave's chain of dependent gathers.  Here a
// workgroup takes one item, a wave 16 of its rays, and four neighbouring lanes
// one ray: they gather a quarter of a chunk's occupancy bits each, evaluate four
// occupied samples at a time, and each folds all four colours in order, so that
// images, counts and early termination are those of render_kernel bit for bit.
// No queue: the launch has about a workgroup per item.  61x47 frame of a
// 37x29x23 cube 19.4 -> 13.3 us, 256x256 of 128^3 63 -> 31; with enough items
// to fill the chip the persistent kernel's waves, each with 64 rays, do the
// same in fewer instructions (1024^3 frame 1308 against 1994 us).
template <int J>
__device__ __forceinline__ float quad_lane(float v) {   // lane J of the lane's four
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x55 * J, 0xf, 0xf, true));
}

template <int FMT, bool TF_LDS, int OP>
__global__ __launch_bounds__(256) void render_quad_kernel(BcFramePtrs f) {
  extern __shared__ float4 q_tab[];   // table entry k at 2k, its difference to entry k+1 at 2k+1
  __shared__ uint32_t wave_count[2][4];
  KC(BcFrameIn)* fin = kc(f.fin);
  KC(BcCounters)* cr = kc(f.ctr);
  const uint32_t n_items = cr->n_items;
  if (blockIdx.x >= n_items) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6), sub = lane & 3;
  const int K = fin->K;
  const float4* gtab = reinterpret_cast<const float4*>(f.fin->table);
  // (on its way during the ray set-up)
  float4 ta = make_float4(0.f, 0.f, 0.f, 0.f), tb = ta;
  if (TF_LDS && OP == 0 && tid < K) {
    ta = gtab[tid];
    tb = gtab[min(tid + 1, K - 1)];
  }
  const float tf_scale = fin->tf_scale, tf_bias = fin->tf_bias, kmax_f = (float)(K - 1);
  uint32_t nominal = 0, evaluated = 0;
  bool staged = false;
  for (uint32_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    KC(int32_t)* perm = kc(f.item_perm);
    int lo = 0, hi = f.n_bricks * f.n_views;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((uint32_t)perm[mid] <= item) lo = mid; else hi = mid;
    }
    KC(int4)& ent = kc(f.item_entry)[lo];
    const int b = ent.x & 0xffff, v = ent.x >> 16, cx = ent.y, ts = fin->tile_stride;
    const int local = (int)(item - (uint32_t)perm[lo]);
    const int tx = ent.z + (local % cx) * ts, ty = ent.w + (local / cx) * ts;
    KC(BcViewParams)& vp = kc(f.views)[v];
    KC(BcBrick)& br = kc(f.bricks)[b];
    const int tsh = f.tile_shift, pix = 16 * wave + (lane >> 2);
    const int px = (tx << tsh) + (pix & ((1 << tsh) - 1)), py = ty * (64 >> tsh) + (pix >> tsh);
    RaySeg seg;
    const bool hit = px < vp.width && py < vp.height && ray_segment(vp, f.gdims, br, px, py, f.step_policy != 0, seg);
    if (TF_LDS && OP == 0 && !staged) {
      staged = true;
      for (int k = tid; k < K; k += 256) {
        if (k != tid) {
          ta = gtab[k];
          tb = gtab[min(k + 1, K - 1)];
        }
        q_tab[2 * k] = ta;
        q_tab[2 * k + 1] = make_float4(tb.x - ta.x, tb.y - ta.y, tb.z - ta.z, tb.w - ta.w);
      }
      __syncthreads();
    }
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float mx = -INFINITY;
    if (hit) {
      constexpr uint32_t esz = FMT == 0 ? 4 : (FMT == 1 ? 2 : 1);
      constexpr uint32_t sh = FMT == 0 ? 2 : (FMT == 1 ? 1 : 0);
      constexpr bool FOLD = FMT == 2 && OP == 0;
      const float tau = vp.tau, bound = br.dmax;
      mx = -FLT_MAX;
      // strides and resources as in render_kernel
      const uint32_t mbx = (uint32_t)br.mb[0], mby = (uint32_t)br.mb[1];
      const uint32_t WX = (uint32_t)br.occ_w[0], WY = (uint32_t)br.occ_w[1], WX4 = 4u * WX;
      const __amdgpu_buffer_rsrc_t occ = make_rsrc(f.occ + br.occ_offset, WX * WY * (uint32_t)br.occ_w[2] * 4u);
      const __amdgpu_buffer_rsrc_t pool = make_rsrc(static_cast<const char*>(f.pool) + br.offset * esz,
                                                    mbx * mby * (uint32_t)br.mb[2] * BC_MB_ELEMS * esz);
      const float s_q = br.scale, o_q = br.offs;
      const float tsc = FOLD ? tf_scale * s_q : tf_scale, tbi = FOLD ? __builtin_fmaf(o_q, tf_scale, tf_bias) : tf_bias;
      const uint32_t dyb = (mbx * BC_MB_ELEMS - 3u * BC_ROW) << sh, dzb = (mbx * mby * BC_MB_ELEMS - 12u * BC_ROW) << sh;
      const uint32_t cxb = 20u << sh, cyb = (20u * mbx) << sh, czb = (20u * mbx * mby) << sh;
      const int rxb = -(int)(19u << sh), ryb = (int)(BC_ROW << sh) - (int)cyb, rzb = (int)((4u * BC_ROW) << sh) - (int)czb;
      int64_t uc0 = seg.u[0], uc1 = seg.u[1], uc2 = seg.u[2];
      const int64_t s0 = seg.s[0], s1 = seg.s[1], s2 = seg.s[2];
      const float sfx = (float)s0 * 2.3283064365386963e-10f, sfy = (float)s1 * 2.3283064365386963e-10f,
                  sfz = (float)s2 * 2.3283064365386963e-10f;
      int used = seg.n;
      for (int k = 0; k < seg.n; k += 32) {
        const int cnt = min(32, seg.n - k);
        uint32_t mask = cnt >= 32 ? ~0u : (1u << cnt) - 1u;
        if (f.ess) {
          // the lane's eight samples; the words all in flight together
          int64_t un0 = uc0 + 8 * sub * s0, un1 = (uc1 + 8 * sub * s1) * 4, un2 = (uc2 + 8 * sub * s2) * 16;
          uint32_t bit[8], ofs[8], word[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t ix = (uint32_t)hi32(un0), iy4 = (uint32_t)hi32(un1), iz16 = (uint32_t)hi32(un2);
            ofs[i] = mad_u24(mad_u24(iz16 >> 5, WY, iy4 >> 4), WX4, ix & ~3u);
            bit[i] = bfi_u32(15u, bfi_u32(3u, ix, iy4), iz16);
            un0 += s0; un1 += 4 * s1; un2 += 16 * s2;
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
            word[i] = __builtin_amdgcn_raw_buffer_load_b32(occ, i && ofs[i] == ofs[i - 1] ? 0xfffffff0u : ofs[i], 0, 0);
          uint32_t m = 0, w = 0;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            w = word[i] | (i && ofs[i] == ofs[i - 1] ? w : 0u);
            m |= __builtin_amdgcn_ubfe(w, bit[i], 1u) << i;
          }
          m <<= 8 * sub;
          m |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xb1, 0xf, 0xf, true);   // lane ^ 1
          m |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4e, 0xf, 0xf, true);   // lane ^ 2
          mask &= m;
        }
        const int bx = hi32(uc0), by = hi32(uc1), bz = hi32(uc2);
        const float fx0 = frac32(uc0), fy0 = frac32(uc1), fz0 = frac32(uc2);
        int last = 31;
        bool stop = false;
        uint32_t left = mask;
        while (left) {
          // the four lowest samples left, one to a lane (the last one again where there are fewer)
          int idx[4];
          bool on[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            on[j] = left != 0u;
            idx[j] = on[j] ? (int)__builtin_ctz(left) : idx[j > 0 ? j - 1 : 0];
            left &= left - 1u;
          }
          const int i = sub == 0 ? idx[0] : (sub == 1 ? idx[1] : (sub == 2 ? idx[2] : idx[3]));
          const float fi = (float)i;
          const float ux = __builtin_fmaf(fi, sfx, fx0), uy = __builtin_fmaf(fi, sfy, fy0), uz = __builtin_fmaf(fi, sfz, fz0);
          const float wx = __builtin_amdgcn_fractf(ux), wy = __builtin_amdgcn_fractf(uy), wz = __builtin_amdgcn_fractf(uz);
          const uint32_t ix = (uint32_t)(bx + floor_i32(ux)), iy = (uint32_t)(by + floor_i32(uy)),
                         iz = (uint32_t)(bz + floor_i32(uz));
          const int ry = (int)(iy & 3u), rz = (int)(iz & 3u);
          const uint32_t a000 = (uint32_t)mad_i24(
              rz, rzb, mad_i24(ry, ryb, mad_i24((int)(ix & 3u), rxb, (int)mad_u24(ix, cxb, mad_u24(iy, cyb, __umul24(iz, czb))))));
          const uint32_t dy = ry == 3 ? dyb : (BC_ROW << sh), dz = rz == 3 ? dzb : ((4u * BC_ROW) << sh);
          float c[8];
          load_pair<FOLD ? 3 : FMT>(pool, a000, s_q, o_q, c[0], c[1]);
          load_pair<FOLD ? 3 : FMT>(pool, a000 + dy, s_q, o_q, c[2], c[3]);
          load_pair<FOLD ? 3 : FMT>(pool, a000 + dz, s_q, o_q, c[4], c[5]);
          load_pair<FOLD ? 3 : FMT>(pool, a000 + dz + dy, s_q, o_q, c[6], c[7]);
          const float c00 = __builtin_fmaf(wx, c[1] - c[0], c[0]), c10 = __builtin_fmaf(wx, c[3] - c[2], c[2]);
          const float c01 = __builtin_fmaf(wx, c[5] - c[4], c[4]), c11 = __builtin_fmaf(wx, c[7] - c[6], c[6]);
          const float c0 = __builtin_fmaf(wy, c10 - c00, c00), c1 = __builtin_fmaf(wy, c11 - c01, c01);
          const float val = __builtin_fmaf(wz, c1 - c0, c0);
          if (OP == 1) {
            const float val4[4] = {quad_lane<0>(val), quad_lane<1>(val), quad_lane<2>(val), quad_lane<3>(val)};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (!on[j] || stop) continue;
              mx = fmaxf(mx, val4[j]);
              if (mx >= bound) {
                last = idx[j];
                stop = true;
              }
            }
          } else {
            const float xt = __builtin_amdgcn_fmed3f(__builtin_fmaf(val, tsc, tbi), 0.0f, kmax_f);
            const int it = TF_LDS ? (int)xt : min((int)xt, K - 2);
            const float ft = TF_LDS ? __builtin_amdgcn_fractf(xt) : xt - (float)it;
            float4 q0, dq;
            if (TF_LDS) {
              q0 = q_tab[2 * it];
              dq = q_tab[2 * it + 1];
            } else {
              q0 = gtab[it];
              const float4 q1 = gtab[it + 1];
              dq = make_float4(q1.x - q0.x, q1.y - q0.y, q1.z - q0.z, q1.w - q0.w);
            }
            const float4 col = make_float4(__builtin_fmaf(ft, dq.x, q0.x), __builtin_fmaf(ft, dq.y, q0.y),
                                           __builtin_fmaf(ft, dq.z, q0.z), __builtin_fmaf(ft, dq.w, q0.w));
            const float4 col4[4] = {
                make_float4(quad_lane<0>(col.x), quad_lane<0>(col.y), quad_lane<0>(col.z), quad_lane<0>(col.w)),
                make_float4(quad_lane<1>(col.x), quad_lane<1>(col.y), quad_lane<1>(col.z), quad_lane<1>(col.w)),
                make_float4(quad_lane<2>(col.x), quad_lane<2>(col.y), quad_lane<2>(col.z), quad_lane<2>(col.w)),
                make_float4(quad_lane<3>(col.x), quad_lane<3>(col.y), quad_lane<3>(col.z), quad_lane<3>(col.w))};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (!on[j] || stop) continue;
              const float om = 1.0f - acc.w;
              acc.x = __builtin_fmaf(om, col4[j].x, acc.x);
              acc.y = __builtin_fmaf(om, col4[j].y, acc.y);
              acc.z = __builtin_fmaf(om, col4[j].z, acc.z);
              acc.w = __builtin_fmaf(om, col4[j].w, acc.w);
              if (acc.w >= tau) {
                last = idx[j];
                stop = true;
              }
            }
          }
          if (stop) left = 0u;
        }
        if (sub == 0) evaluated += (uint32_t)__builtin_popcount(mask & (~0u >> (31 - last)));
        if (stop) {
          used = k + last + 1;
          break;
        }
        uc0 += 32 * s0; uc1 += 32 * s1; uc2 += 32 * s2;
      }
      if (sub == 0) nominal += (uint32_t)used;
    }
    if (sub == 0) {
      if (OP == 0) f.sub[(int64_t)item * 64 + pix] = acc;
      else reinterpret_cast<float*>(f.sub)[(int64_t)item * 64 + pix] = mx;
    }
  }
  // one addition per workgroup, spread over a few cache lines
  for (int off = 32; off > 0; off >>= 1) {
    nominal += __shfl_xor(nominal, off);
    evaluated += __shfl_xor(evaluated, off);
  }
  if (lane == 0) {
    wave_count[0][wave] = nominal;
    wave_count[1][wave] = evaluated;
  }
  __syncthreads();
  if (tid < 2) {
    unsigned long long n = 0;
    for (int w = 0; w < 4; ++w) n += wave_count[tid][w];
    if (n) atomicAdd(&f.ctr->part[blockIdx.x % BC_COUNT_PARTS].count[tid], n);
  }
}

template <int FMT>
hipError_t launch_render_fmt(const BcFramePtrs& f, int n_workgroups, hipStream_t st) {
  const bool lds = f.K <= BC_TF_LDS;
  if (f.item_bound > 0) {
    const int n = (int)f.item_bound;   // (a further item, if the bound were short, is a workgroup's second)
    if (f.op == 1) render_quad_kernel<FMT, false, 1><<<n, 256, 0, st>>>(f);
    else if (lds) render_quad_kernel<FMT, true, 0><<<n, 256, sizeof(float4) * 2 * f.K, st>>>(f);
    else render_quad_kernel<FMT, false, 0><<<n, 256, 0, st>>>(f);
    return hipGetLastError();
  }
  if (f.op == 1) {
    // the colour map is applied after the merge: no table in the ray caster
    if (f.chunk == 32) render_kernel<FMT, false, 32, 1, false><<<n_workgroups, 256, 0, st>>>(f);
    else render_kernel<FMT, false, 64, 1, false><<<n_workgroups, 256, 0, st>>>(f);
  } else if (f.chunk == 32) {
    if (lds && f.urgent) render_kernel<FMT, true, 32, 0, true><<<n_workgroups, 256, 0, st>>>(f);
    else if (lds) render_kernel<FMT, true, 32, 0, false><<<n_workgroups, 256, 0, st>>>(f);
    else render_kernel<FMT, false, 32, 0, false><<<n_workgroups, 256, 0, st>>>(f);
  } else {
    if (lds && f.urgent) render_kernel<FMT, true, 64, 0, true><<<n_workgroups, 256, 0, st>>>(f);
    else if (lds) render_kernel<FMT, true, 64, 0, false><<<n_workgroups, 256, 0, st>>>(f);
    else render_kernel<FMT, false, 64, 0, false><<<n_workgroups, 256, 0, st>>>(f);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t bc_launch_classify(const BcFramePtrs& f, const int max_w[3], int64_t words, hipStream_t st) {
  ClassifyArgs a;
  a.bricks = f.bricks;
  a.fin = f.fin;
  a.occ = f.occ;
  a.pool = f.pool;
  a.n_bricks = f.n_bricks;
  a.x_tiles = (max_w[0] + 3) / 4;
  a.y_tiles = (max_w[1] + 15) / 16;
  // a walk re-reads the slice that the next one starts with: long walks where
  // there are enough of them to fill the chip a few times over (1024^3 FP32
  // cube: 8 words 1620, 32 words 1518, 128 words 1586 us)
  const int64_t columns = (int64_t)f.n_bricks * a.x_tiles * a.y_tiles;
  a.z_words = 32;
  while (a.z_words > 4 && columns * ((max_w[2] + a.z_words - 1) / a.z_words) < 4096) a.z_words /= 2;
  a.z_chunks = (max_w[2] + a.z_words - 1) / a.z_words;
  a.max_words = max_w[0] * max_w[1] * max_w[2];
  a.mip = f.op == 1;
  // Each workgroup looks the table over for itself, 16 entries a thread at 4096:
  // fewer of them on a long one (1024^3 FP32, 4096 entries: 2.10 ms with a
  // workgroup per tile, 1.80 with 4096 of them; FP8 by words 3 % less with 1024
  // than with 8192, 512^3 in bricks of 64^3 36 %; at 256 entries these grids cost
  // 3 to 8 %).
  const bool long_table = f.K > 1024;
  const double rows = (double)max_w[0] * max_w[1] / (64.0 * a.x_tiles * a.y_tiles);   // of a walk's lanes, those with one
  // By words: FP8 always (512^3, 256 entries, us that a change of the transfer
  // function adds to a frame, by rows / by words: bricks of
  // 64^3 346 / 175, of 512 x 8 x 512 626 / 229, of 8 x 512 x 512 290 / 240, of
  // 600^3 in 12 x 300 x 300 326 / 354, the one shape where rows were ahead).
  // The others where few lanes have a row: 1000 x 1 x 64 (a 16th) FP32 2192 / 899,
  // FP16 2011 / 496; 512 x 8 x 512 (0.18) FP32 603 / 808, FP16 534 / 448; 300 x
  // 12 x 300 (0.25) FP32 668 / 1174, FP16 608 / 661.
  if (f.storage == 2 || rows < (f.storage == 0 ? 0.15 : 0.2)) {
    const int64_t need = ((int64_t)f.n_bricks * a.max_words + 255) / 256;
    const int grid = (int)std::min<int64_t>(need, long_table ? 1024 : 8192);
    if (f.storage == 0) classify_words_kernel<0><<<grid, 256, 0, st>>>(a);
    else if (f.storage == 1) classify_words_kernel<1><<<grid, 256, 0, st>>>(a);
    else classify_words_kernel<2><<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
  }
  const int64_t total = columns * a.z_chunks;
  a.run = (uint32_t)((total + 7) / 8);
  // An eighth of the tiles to each XCD, unless the bricks' sizes differ: then most
  // tiles of the small ones are empty, and they lie together (300 x 1000 x 1000 in
  // 5 x 900 x 900, FP32, the same measure: 2.50 ms in eighths, 0.93 in runs of
  // 64; 1024^3 in 256^3 4 % the other way).
  if ((double)words < 0.9 * f.n_bricks * a.max_words) a.run = (uint32_t)std::min<int64_t>(std::max<int64_t>(total / 64, 1), 64);
  const int grid = (int)std::min<int64_t>((total + 8 * (int64_t)a.run - 1) / (8 * (int64_t)a.run) * (8 * (int64_t)a.run), long_table ? 4096 : 1 << 20);
  if (f.storage == 0) classify_kernel<0><<<grid, 256, 0, st>>>(a);
  else classify_kernel<1><<<grid, 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t bc_launch_render(const BcFramePtrs& f, int n_workgroups, hipStream_t st) {
  if (f.storage == 0) return launch_render_fmt<0>(f, n_workgroups, st);
  if (f.storage == 1) return launch_render_fmt<1>(f, n_workgroups, st);
  return launch_render_fmt<2>(f, n_workgroups, st);
}
