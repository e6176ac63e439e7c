// Load-time kernels: per-brick minimum/maximum of the stored values (the
// paper's min/max task after the data reaches GPU memory, Section 2.3.1; of
// its own ahead of an FP8 encode, which needs it, and within the others), the
// FP8 scale/offset, the largest decoded value, and the encode + layout of
// ghosted bricks into 4x4x4 micro-blocks (micro-blocks row-major inside the
// brick; a micro-block is 16 rows of 5 elements, x fastest, the fifth
// repeating the first voxel of the next micro-block along x).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "bc_types.h"
#include "bc_kernels.h"
#include "bc_e4m3.h"

namespace {

__device__ __forceinline__ uint32_t ordered_bits(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<__half>(__half v) { return __half2float(v); }

struct SrcView {
  const void* ptr;
  int64_t sx, sy, sz;   // strides (elements)
  int32_t ox, oy, oz;   // global voxel coordinates of element [0][0][0]
  int32_t nx, ny, nz;   // global cube dims (for clamping)
};

// Four source rows along x, read by one wave together: lane offsets along x are
// shared, row starts are uniform, and the four loads are in flight at once.
template <typename T>
struct Rows {
  const T* row[4];
  __device__ __forceinline__ void start(const SrcView& s, int k, int gy, int gz) {
    gy = min(max(gy, 0), s.ny - 1);
    gz = min(max(gz, 0), s.nz - 1);
    row[k] = static_cast<const T*>(s.ptr) + ((int64_t)(gy - s.oy) * s.sy + (int64_t)(gz - s.oz) * s.sz);
  }
  __device__ __forceinline__ void load(const SrcView& s, int gx, float* v) const {
    const int64_t o = (int64_t)(min(max(gx, 0), s.nx - 1) - s.ox) * s.sx;
    T e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = row[k][o];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = to_f32<T>(e[k]);
  }
};

// folds a workgroup's smallest and largest value into the brick's pair; most
// workgroups find a pair that already covers theirs (it only ever widens, so a
// value read late costs at most an atomic that changes nothing)
__device__ __forceinline__ void fold_minmax(float mn, float mx, uint32_t* pair) {
  __shared__ float red[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    mn = fminf(mn, __shfl_xor(mn, off));
    mx = fmaxf(mx, __shfl_xor(mx, off));
  }
  if (lane == 0) {
    red[0][wave] = mn;
    red[1][wave] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      mn = fminf(mn, red[0][w]);
      mx = fmaxf(mx, red[1][w]);
    }
    if (mn <= mx) {
      const uint32_t lo = ordered_bits(mn), hi = ordered_bits(mx);
      if (lo < __hip_atomic_load(&pair[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&pair[0], lo);
      if (hi > __hip_atomic_load(&pair[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&pair[1], hi);
    }
  }
}

// min/max over each brick's ghosted region [lo-1, hi+1) (clamped to the
// cube): brick first + blockIdx.x; every wave takes four rows along x at a time
template <typename T>
__global__ __launch_bounds__(256) void minmax_kernel(SrcView s, const BcBrick* __restrict__ bricks, int first,
                                                     BcCounters* ctr) {
  const int b = first + (int)blockIdx.x;
  const BcBrick& br = bricks[b];
  const int ex = br.hi[0] - br.lo[0] + 2, ey = br.hi[1] - br.lo[1] + 2, ez = br.hi[2] - br.lo[2] + 2;
  const int rows = ey * ez;
  const int lane = threadIdx.x & 63, wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float mn = INFINITY, mx = -INFINITY;
  for (int r0 = 16 * (int)blockIdx.y + 4 * wave; r0 < rows; r0 += 16 * (int)gridDim.y) {
    Rows<T> in;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = min(r0 + k, rows - 1);
      in.start(s, k, br.lo[1] - 1 + r % ey, br.lo[2] - 1 + r / ey);
    }
#pragma unroll 2
    for (int x = lane; x < ex; x += 64) {
      float v[4];
      in.load(s, br.lo[0] - 1 + x, v);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        mn = fminf(mn, v[k]);
        mx = fmaxf(mx, v[k]);
      }
    }
  }
  fold_minmax(mn, mx, ctr->minmax[b]);
}

__global__ void init_minmax_kernel(BcCounters* ctr, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    ctr->minmax[i][0] = 0xffffffffu;
    ctr->minmax[i][1] = 0u;
  }
}

// scale/offset of each brick from its stored range (FP32 formulas:
// o = (min+max)/2, s = (max-min)/896, s = 1 when max == min)
__global__ void finalize_kernel(BcBrick* bricks, const BcCounters* ctr, int first, int count, int storage) {
  const int b = first + blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= first + count) return;
  const float mn = from_ordered(ctr->minmax[b][0]);
  const float mx = from_ordered(ctr->minmax[b][1]);
  bricks[b].vmin = mn;
  bricks[b].vmax = mx;
  float s = 1.0f, o = 0.0f;
  if (storage == 2) {
    if (mx == mn) {
      s = 1.0f;
      o = mn;
    } else {
      o = (mn + mx) / 2.0f;
      s = (mx - mn) / 896.0f;
    }
  }
  bricks[b].scale = s;
  bricks[b].offs = o;
  // the encodes below are monotone (round to nearest, saturating), so the
  // largest stored element is the encode of the largest source value; its
  // decode bounds every value the brick can produce (maximum intensity
  // projection stops a ray there)
  float dmax = mx;
  if (storage == 1) dmax = __half2float(__float2half_rn(mx));
  if (storage == 2) dmax = __builtin_fmaf(bc_e4m3_decode(bc_e4m3_encode((mx - o) * (1.0f / s))), s, o);
  bricks[b].dmax = dmax;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// LDS floats of a staged source row (n stored voxels along x): rows start 4
// banks apart, so that the elements of neighbouring rows, which neighbouring
// threads pick up, fall on different banks
constexpr int kEncodeThreads = 240;   // of 256 write: a multiple of every form's 16-byte chunks per micro-block
__host__ __device__ __forceinline__ int staged_row(int mb0) { return (4 * mb0 + 64) / 64 * 64 + 4; }

// encode + layout: brick first + blockIdx.x; a workgroup fills the row of
// micro-blocks (all x) at micro-block coordinates (y, z) = blockIdx.y.  Its 16
// source rows are read once, whole rows by whole waves, into LDS, and leave in
// stored order as 16 bytes per thread (4 of FP8, whose conversion is the longer
// part: 512^3 in bricks 62 wide 580 us with the min/max, 709 with 16); FP32 and FP16 storage, which need no
// scale, take the brick's min/max on the way (one read of the source instead
// of two).  Bound by that read and write: 1024^3 FP32
// (4.3 GB in, 5.5 GB out) takes 1.95 ms, 5.0 TB/s; 1.60 ms of min/max and 3.20
// of an encode with a thread per element before
template <typename T, int FMT>
__global__ __launch_bounds__(256) void encode_kernel(SrcView s, const BcBrick* __restrict__ bricks, int first,
                                                     void* pool, BcCounters* ctr) {
  extern __shared__ float stage[];
  constexpr int EPC = FMT == 1 ? 8 : 4;    // elements of a chunk: 16 bytes, or 4 of FP8
  constexpr int CPM = BC_MB_ELEMS / EPC;   // chunks of a micro-block
  constexpr int esz = FMT == 0 ? 4 : (FMT == 1 ? 2 : 1);
  static_assert(kEncodeThreads % CPM == 0, "a thread's place in a micro-block is fixed");
  const int b = first + (int)blockIdx.x;
  const BcBrick& br = bricks[b];
  const int mb0 = br.mb[0], mb1 = br.mb[1];
  const int slabs = mb1 * br.mb[2];
  const int cx = br.hi[0] - br.lo[0], cy = br.hi[1] - br.lo[1], cz = br.hi[2] - br.lo[2];
  const float inv = 1.0f / br.scale, offs = br.offs;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = staged_row(mb0), nx = 4 * mb0 + 1;
  // the thread's chunk of every kEncodeThreads / CPM-th micro-block: its elements' rows and places
  const int chunk = tid % CPM;
  int at[EPC];
#pragma unroll
  for (int i = 0; i < EPC; ++i) {
    const int in = chunk * EPC + i, row = in / BC_ROW;
    at[i] = row * S + (in - row * BC_ROW);   // the fifth of a row is the next micro-block's first voxel
  }
  float mn = INFINITY, mx = -INFINITY;
  for (int sl = (int)blockIdx.y; sl < slabs; sl += (int)gridDim.y) {
    const int mby = sl % mb1, mbz = sl / mb1;
    // local ghosted index (0 <-> voxel lo-1); padding replicates the last ghost
    Rows<T> in;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      in.start(s, k, br.lo[1] - 1 + min(mby * 4 + k, cy + 1), br.lo[2] - 1 + min(mbz * 4 + wave, cz + 1));
    float* rows = stage + (4 * wave) * S;
#pragma unroll 2
    for (int x = lane; x < nx; x += 64) {
      float v[4];
      in.load(s, br.lo[0] - 1 + min(x, cx + 1), v);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        rows[k * S + x] = v[k];
        if (FMT != 2) {
          mn = fminf(mn, v[k]);
          mx = fmaxf(mx, v[k]);
        }
      }
    }
    __syncthreads();
    if (tid < kEncodeThreads) {
      char* out = static_cast<char*>(pool) + (br.offset + (int64_t)sl * mb0 * BC_MB_ELEMS) * esz;
      for (int m = tid / CPM; m < mb0; m += kEncodeThreads / CPM) {
        const float* from = stage + 4 * m;
        constexpr int W = EPC * esz / 4;
        uint32_t w[W];
        if (FMT == 0) {
#pragma unroll
          for (int i = 0; i < W; ++i) w[i] = __float_as_uint(from[at[i]]);
        } else if (FMT == 1) {
#pragma unroll
          for (int i = 0; i < W; ++i)
            w[i] = __half_as_ushort(__float2half_rn(from[at[(2 * i) % EPC]])) |
                   (uint32_t)__half_as_ushort(__float2half_rn(from[at[(2 * i + 1) % EPC]])) << 16;
        } else {
#pragma unroll
          for (int i = 0; i < W; ++i) {
            w[i] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float xq = (from[at[(4 * i + j) % EPC]] - offs) * inv;
              w[i] |= (uint32_t)bc_e4m3_encode(xq) << (8 * j);
            }
          }
        }
        // (nothing reads them before the pool is whole: not kept in the caches)
        char* to = out + (m * CPM + chunk) * (EPC * esz);
        if constexpr (W == 4)
          __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4*>(to));
        else
          __builtin_nontemporal_store(w[0], reinterpret_cast<uint32_t*>(to));
      }
    }
    __syncthreads();
  }
  if (FMT != 2) fold_minmax(mn, mx, ctr->minmax[b]);
}

// FP8 bricks narrow along x: the rows are too short for whole waves to read
// them, so a thread takes four stored elements, anywhere in the brick, with a
// load each.  Bound by the loads of partial lines and, in the load as a whole,
// by the min/max that goes before.
template <typename T>
__global__ __launch_bounds__(256) void encode_narrow_kernel(SrcView s, const BcBrick* __restrict__ bricks, int first,
                                                            void* pool) {
  constexpr uint32_t UPM = BC_MB_ELEMS / 4;   // units of four elements of a micro-block
  const BcBrick& br = bricks[first + (int)blockIdx.x];
  const uint32_t mb0 = (uint32_t)br.mb[0], mb1 = (uint32_t)br.mb[1], units = mb0 * mb1 * (uint32_t)br.mb[2] * UPM;
  const int cx = br.hi[0] - br.lo[0], cy = br.hi[1] - br.lo[1], cz = br.hi[2] - br.lo[2];
  const float inv = 1.0f / br.scale, offs = br.offs;
  for (uint32_t u = blockIdx.y * 256u + threadIdx.x; u < units; u += gridDim.y * 256u) {
    const uint32_t mb = u / UPM, in = u - mb * UPM, sl = mb / mb0, mbx = mb - sl * mb0, mbz = sl / mb1, mby = sl - mbz * mb1;
    T v[4];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t e = 4 * in + j, row = e / BC_ROW, wx = e - row * BC_ROW;   // the fifth is the next micro-block's first voxel
      // local ghosted index (0 <-> voxel lo-1); padding replicates the last ghost
      const int lx = min((int)(mbx * 4 + wx), cx + 1), ly = min((int)(mby * 4 + (row & 3)), cy + 1),
                lz = min((int)(mbz * 4 + (row >> 2)), cz + 1);
      const int gx = min(max(br.lo[0] - 1 + lx, 0), s.nx - 1), gy = min(max(br.lo[1] - 1 + ly, 0), s.ny - 1),
                gz = min(max(br.lo[2] - 1 + lz, 0), s.nz - 1);
      v[j] = static_cast<const T*>(s.ptr)[(int64_t)(gx - s.ox) * s.sx + (int64_t)(gy - s.oy) * s.sy + (int64_t)(gz - s.oz) * s.sz];
    }
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) w |= (uint32_t)bc_e4m3_encode((to_f32<T>(v[j]) - offs) * inv) << (8 * j);
    __builtin_nontemporal_store(w, reinterpret_cast<uint32_t*>(static_cast<char*>(pool) + br.offset) + u);
  }
}

inline SrcView make_src(const BcLoadSrc& s) {
  SrcView v;
  v.ptr = s.ptr;
  v.sx = s.strides[0]; v.sy = s.strides[1]; v.sz = s.strides[2];
  v.ox = s.origin[0]; v.oy = s.origin[1]; v.oz = s.origin[2];
  v.nx = s.dims[0]; v.ny = s.dims[1]; v.nz = s.dims[2];
  return v;
}

}  // namespace

hipError_t bc_launch_init_minmax(BcCounters* ctr, int n, hipStream_t st) {
  init_minmax_kernel<<<(n + 255) / 256, 256, 0, st>>>(ctr, n);
  return hipGetLastError();
}

hipError_t bc_launch_minmax(const BcLoadSrc& src, const BcBrick* bricks, int first, int count, int max_rows,
                            BcCounters* ctr, hipStream_t st) {
  SrcView s = make_src(src);
  // 16 rows to a workgroup at a time: enough workgroups for a few thousand in
  // all, and otherwise at least four turns each (fewer folds into the pair)
  const int turns = (max_rows + 15) / 16;
  const dim3 grid((unsigned)count,
                  (unsigned)std::max(1, std::min(std::min(turns, 65535), std::max((turns + 3) / 4, 4096 / count))));
  if (src.dtype == 0)
    minmax_kernel<float><<<grid, 256, 0, st>>>(s, bricks, first, ctr);
  else
    minmax_kernel<__half><<<grid, 256, 0, st>>>(s, bricks, first, ctr);
  return hipGetLastError();
}

hipError_t bc_launch_finalize(BcBrick* bricks, const BcCounters* ctr, int first, int count, int storage,
                              hipStream_t st) {
  finalize_kernel<<<(count + 255) / 256, 256, 0, st>>>(bricks, ctr, first, count, storage);
  return hipGetLastError();
}

hipError_t bc_launch_encode(const BcLoadSrc& src, const BcBrick* bricks, int first, int count, int64_t max_rows,
                            int max_mb0, int storage, void* pool, BcCounters* ctr, hipStream_t st) {
  SrcView s = make_src(src);
  // One workgroup per row of micro-blocks (up to the largest brick's y * z
  // count in micro-blocks), the same row of every brick before the next row:
  // bricks side by side then read their shared source lines together, and the
  // reads and writes spread over all of the memory (1024^3 FP32: 1.95 ms,
  // against 2.67 brick by brick).
  const dim3 grid((unsigned)count, (unsigned)std::max<int64_t>(1, std::min<int64_t>(max_rows, 65535)));
  const size_t lds = sizeof(float) * 16 * staged_row(max_mb0);
  auto launch = [&](auto* kernel) -> hipError_t {
    // (over 64 KiB for bricks wider than 950 voxels)
    if (lds > 65536) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    kernel<<<grid, 256, lds, st>>>(s, bricks, first, pool, ctr);
    return hipGetLastError();
  };
  // FP8 bricks up to 38 voxels wide by elements (512^3 in bricks of b x 512 x 512,
  // min/max and encode, us staged / by elements: b = 1 22900 / 13200, 6 3910 /
  // 2490, 14 1780 / 1260, 30 928 / 822, 38 761 / 726, 46 665 / 697, 62 582 / 607)
  if (storage == 2 && max_mb0 <= 10) {
    const int64_t units = max_rows * max_mb0 * (BC_MB_ELEMS / 4);
    const dim3 flat((unsigned)count, (unsigned)std::max<int64_t>(1, std::min<int64_t>((units + 511) / 512, 65535)));
    if (src.dtype == 0) encode_narrow_kernel<float><<<flat, 256, 0, st>>>(s, bricks, first, pool);
    else encode_narrow_kernel<__half><<<flat, 256, 0, st>>>(s, bricks, first, pool);
    return hipGetLastError();
  }
  if (src.dtype == 0) {
    if (storage == 0) return launch(encode_kernel<float, 0>);
    if (storage == 1) return launch(encode_kernel<float, 1>);
    return launch(encode_kernel<float, 2>);
  }
  if (storage == 0) return launch(encode_kernel<__half, 0>);
  if (storage == 1) return launch(encode_kernel<__half, 1>);
  return launch(encode_kernel<__half, 2>);
}
