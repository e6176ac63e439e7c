// Kernel launchers called by the host runtime.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "bc_types.h"

struct BcLoadSrc {
  const void* ptr;        // device pointer
  int64_t strides[3];     // elements (x, y, z)
  int32_t origin[3];      // global voxel coordinates of element [0][0][0]
  int32_t dims[3];        // global cube dims
  int32_t dtype;          // 0 float32, 1 float16
};

hipError_t bc_launch_init_minmax(BcCounters* ctr, int n, hipStream_t st);
// bricks [first, first + count): max_rows bounds each brick's ghosted rows
// (y * z extent); the encode's max_rows bounds its rows of micro-blocks along x
// (y * z extent in micro-blocks), max_mb0 its micro-blocks along x.  FP8
// storage: minmax, finalize, encode; otherwise the encode takes the min/max:
// encode, finalize.
hipError_t bc_launch_minmax(const BcLoadSrc& src, const BcBrick* bricks, int first, int count, int max_rows,
                            BcCounters* ctr, hipStream_t st);
hipError_t bc_launch_finalize(BcBrick* bricks, const BcCounters* ctr, int first, int count, int storage,
                              hipStream_t st);
hipError_t bc_launch_encode(const BcLoadSrc& src, const BcBrick* bricks, int first, int count, int64_t max_rows,
                            int max_mb0, int storage, void* pool, BcCounters* ctr, hipStream_t st);

struct BcFramePtrs {
  const BcFrameIn* fin;
  BcViewParams* views;
  const BcBrick* bricks;
  int32_t* order;         // [BC_MAX_VIEWS][n_bricks]
  int32_t* rects;         // [BC_MAX_VIEWS][n_bricks][4] tiles (x0, y0, x1, y1)
  int32_t* item_base;     // [n_bricks * n_views + 1] first item of entry b * n_views + v
  int32_t* item_perm;     // [n_bricks * n_views + 1] first item of the entry at each queue-order position
  int4* item_entry;       // [n_bricks * n_views] the entry at each queue-order position: brick | view << 16,
                          // its selected tile columns, its first selected tile x and y
  BcCounters* ctr;
  float4* sub;            // sub-image tiles: [max_items][64] (one float per ray, read as
                          // float[max_items][64], for maximum intensity projection)
  const void* pool;
  uint32_t* occ;          // cell-occupancy bits of every brick
  int32_t ess;            // skip samples in clear cells
  int32_t chunk;          // samples per occupancy-mask chunk of the ray caster (32 or 64)
  int32_t n_queues;       // 8: bricks split over one work queue per XCD; 1: one queue
  int32_t K;              // transfer-function entries
  int32_t op;             // 0 front-to-back compositing, 1 maximum intensity projection
  int32_t step_policy;    // 0 the view's fixed step, 1 one sample per voxel slice
  int32_t n_bricks, n_views;
  int32_t gdims[3];
  int64_t max_items;
  int64_t item_bound;     // ray caster with a workgroup per item: the bound on the items (0: persistent)
  int32_t storage;
  int32_t width, height;  // frame size (all views share it)
  int32_t urgent;         // persistent ray casting: 1: its waves issue at raised priority (2, and 3
                          // while evaluating); 0: at the base levels (0 and 1), for a pass that runs
                          // beside a more urgent one
  int32_t tile_shift;     // screen tiles are (1 << tile_shift) x (64 >> tile_shift) pixels
  // the pass inputs in host-coherent pinned memory, which the set-up kernel
  // copies to `fin` before it reads them (nullptr: `fin` already holds them)
  const BcFrameIn* fin_src;
  int32_t fin_bytes;      // bytes of the pass inputs to copy (a multiple of 4)
};

hipError_t bc_launch_setup(const BcFramePtrs& f, hipStream_t st);
// max_w bounds the bricks' occupancy words per axis; `words` of them are used
hipError_t bc_launch_classify(const BcFramePtrs& f, const int max_w[3], int64_t words, hipStream_t st);
hipError_t bc_launch_render(const BcFramePtrs& f, int n_workgroups, hipStream_t st);
hipError_t bc_launch_composite(const BcFramePtrs& f, float4* out, hipStream_t st);
hipError_t bc_launch_psnr(const BcFramePtrs& f, const float4* ref, const float4* img, hipStream_t st);

// Queue order of the (brick, view) entries: bricks grouped by b % Q, then b,
// then view: the bricks of a group, and the entry at a position.
__device__ __forceinline__ int group_size(int nb, int Q, int x) { return x < nb ? (nb - x + Q - 1) / Q : 0; }
__device__ __forceinline__ void queue_entry(int pos, int nb, int nv, int Q, int& b, int& v) {
  const uint32_t e = (uint32_t)pos / (uint32_t)nv;
  v = pos - (int)e * nv;
  // the first `more` groups hold one brick more than the others
  const uint32_t size = (uint32_t)nb / (uint32_t)Q, more = (uint32_t)nb - size * (uint32_t)Q, big = more * (size + 1);
  const uint32_t r = e < big ? e : e - big, s = e < big ? size + 1 : size;   // (s > 0: e is an entry)
  const uint32_t g = r / s;
  b = (int)((e < big ? g : more + g) + (r - g * s) * (uint32_t)Q);
}

// tile selection {t : t % s == o}: first selected tile >= lo, count in [lo, hi)
__device__ __forceinline__ int sel_first(int lo, int s, int o) { return s == 1 ? lo : lo + ((o - lo) % s + s) % s; }
__device__ __forceinline__ int sel_count(int lo, int hi, int s, int o) {
  if (s == 1) return max(hi - lo, 0);
  const int f = sel_first(lo, s, o);
  return f < hi ? (hi - 1 - f) / s + 1 : 0;
}
