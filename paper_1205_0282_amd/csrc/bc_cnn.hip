// Learned upsampler: a three-layer 3x3 convolutional network that turns a
// half-resolution, coarse-step render into a full-resolution image
// (no passage in the paper; the network is a stated reading):
//
//   a1 = relu(conv(x;  W1 32x4))   a2 = relu(conv(a1; W2 32x32))
//   y  = conv(a2; W3 16x32)        out = pixel_shuffle2(y) + bilinear2(x)
//
// Every convolution is an implicit GEMM on the matrix cores: rows are output
// pixels, columns output channels, and the reduction runs over (tap, input
// channel) in steps of 32 with v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32
// accumulation).  The weights are pre-packed per (k-step, n-tile) in the lane
// order of the instruction, so one 16-byte load per lane fetches a fragment.
// The pixels are read from an LDS tile of the layer input (NHWC, BF16).
//
// Kernels: fused inference (all three layers of a 16x16 output tile with
// LDS-resident activations), per-layer training forward with the loss in the
// last layer's epilogue, backward-data (a forward convolution with flipped,
// channel-transposed weights and the ReLU mask in the epilogue),
// backward-weights (GEMM over the pixels, partial sums per workgroup), their
// deterministic reduction with the Adam step, and the weight packer.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "bc_cnn.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// round to nearest, ties to even (one hardware conversion on gfx950)
__device__ __forceinline__ uint16_t bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// ------------------------------------------------------------------ pixel operand
// Lane (g = lane/16, r = lane%16) of an M-tile supplies pixel r (output pixel p)
// and reduction indices k0 .. k0+7 with k0 = 32 ks + 8 g; k = tap*CIN + c.
// `in` is an LDS tile, WIN pixels wide, SIN BF16 elements per pixel; the
// output pixel with input offset `pix` (its element index in the tile) reads
// input pixel pix + dy*WIN + dx for tap dy*3 + dx.  Tile shapes are template
// parameters, so that with the k-steps unrolled every tap offset is a
// constant of the LDS instruction.
template <int CIN, int WIN, int SIN>
__device__ __forceinline__ int tap_offset(int tap) {
  return tap < 9 ? ((tap / 3) * WIN + tap % 3) * SIN : -1;
}

// element offsets (from the output pixel's input position) of the lane's
// reduction indices at k-step ks: for CIN = 16 one run of 8 channels of one
// tap, for CIN = 4 two taps of 4 channels; -1 for the zero padding past tap 8
template <int CIN, int WIN, int SIN>
__device__ __forceinline__ int2 lane_offsets(int g, int ks) {
  static_assert(CIN == 4 || CIN == 16, "tiles of 32 channels go through conv_hold");
  if (CIN == 16) {
    const int o = tap_offset<CIN, WIN, SIN>(2 * ks + g / 2);
    return make_int2(o < 0 ? -1 : o + 8 * (g % 2), -1);
  }
  const int t0 = (ks * 32 + 8 * g) / 4;
  return make_int2(tap_offset<CIN, WIN, SIN>(t0), tap_offset<CIN, WIN, SIN>(t0 + 1));
}

// Tiles of 32 channels at 64 bytes per pixel: the 16 pixels that a 16-byte read
// touches would start in four places of the banks' 256 bytes.  So channels
// 8 c .. 8 c + 7 of a pixel at column x lie at its place c ^ (x / 4 % 4), which
// spreads 16 neighbouring columns over all of it.
__device__ __forceinline__ int swizzle(int c, int x) { return 8 * (c ^ ((x >> 2) & 3)); }

template <int CIN>
__device__ __forceinline__ bf16x8 load_a(const uint16_t* in, int pix, int2 off) {
  if (CIN == 16) {
    if (off.x < 0) return as_bf16x8(make_uint4(0, 0, 0, 0));
    return as_bf16x8(*reinterpret_cast<const uint4*>(in + pix + off.x));
  }
  const uint2 h0 = off.x >= 0 ? *reinterpret_cast<const uint2*>(in + pix + off.x) : make_uint2(0, 0);
  const uint2 h1 = off.y >= 0 ? *reinterpret_cast<const uint2*>(in + pix + off.y) : make_uint2(0, 0);
  return as_bf16x8(make_uint4(h0.x, h0.y, h1.x, h1.y));
}

// wave-uniform buffer resource over `bytes` bytes at `base` (scalar registers)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  void* ub = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, (int)bytes, 0x00020000);
}

// a layer's packed weights in registers: one 16-byte load per lane and fragment
// (through a buffer resource: one lane offset, the fragments' are constants)
template <int N>
__device__ __forceinline__ void load_weights(const uint4* __restrict__ wf, bf16x8 (&w)[N]) {
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  const __amdgpu_buffer_rsrc_t wr = wave_rsrc(wf, (uint32_t)(N * 64 * 16));
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < N; ++i)
    w[i] = __builtin_bit_cast(bf16x8, (u4)__builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, i * 1024, 0));
}

// One convolution layer over an LDS tile: M output pixels in raster order of
// an output tile WOUT wide; KS k-steps, NT n-tiles of weights `w`.  The weights
// stay in registers: read again for each pair of M-tiles they took more of the
// L1's 64 bytes a cycle than the matrix cores left it.  A wave takes R of its
// M-tiles at a time (R x NT accumulations in flight).  The weights are the
// first operand, so that a lane ends up with four consecutive channels of one
// pixel: epi(p, v) receives them for pixel p < M (bias not added), v[nt][i] of
// channel 16 nt + 4 (lane / 16) + i.
template <int CIN, int KS, int NT, int R, int WIN, int SIN, int M, int WOUT, typename Epi>
__device__ __forceinline__ void conv_tile(const uint16_t* in, const bf16x8 (&w)[KS * NT], Epi epi) {
  // (every kernel here runs 256-thread workgroups: 4 waves; the wave index is
  // made explicitly uniform so that the per-tile guards below are scalar branches)
  constexpr int nwaves = 4;
  const int lane = threadIdx.x & 63, wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  constexpr int n_mt = (M + 15) / 16;
  // the lane's tap offsets do not depend on the pixel: computed once
  int2 off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) off[ks] = lane_offsets<CIN, WIN, SIN>(g, ks);
  for (int base = wave; base < n_mt; base += nwaves * R) {
    f32x4 acc[R][NT];
    int pix[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int p = min((base + nwaves * j) * 16 + r, M - 1);
      pix[j] = ((p / WOUT) * WIN + p % WOUT) * SIN;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // (every slot is computed: a slot past the last M-tile reads clamped
    // pixels and is not stored; a guard here would cost more than it saves)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 a[R];
#pragma unroll
      for (int j = 0; j < R; ++j) a[j] = load_a<CIN>(in, pix[j], off[ks]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < R; ++j) acc[j][nt] = mfma(w[ks * NT + nt], a[j], acc[j][nt]);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int mt = base + nwaves * j;
      if (mt >= n_mt) break;
      const int p = mt * 16 + r;
      if (p < M) epi(p, acc[j]);
    }
  }
}

// The same for a tile of 32 channels (swizzled at 64 bytes per pixel), all M-tiles of a wave at once:
// M-tile wave + 4 j in acc[j], left in registers so that the caller can write
// the results over the input.  Each fragment of the weights is used once, so
// it is read AHEAD k-steps before its use and not kept (1, 2 and 3 steps: 35.7,
// 35.0 and 36.1 us for the kernel below; left to the compiler's order, 36.6).
template <int NT, int R, int WIN, int SIN, int M, int WOUT>
__device__ __forceinline__ void conv_hold(const uint16_t* in, const uint4* __restrict__ wf, f32x4 (&acc)[R][NT]) {
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  constexpr int KS = 9, AHEAD = 2;
  const __amdgpu_buffer_rsrc_t wr = wave_rsrc(wf, (uint32_t)(KS * NT * 64 * 16));
  const int lane = threadIdx.x & 63, wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15;
  bf16x8 w[KS][NT];
  auto fetch = [&](int ks) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      w[ks][nt] = __builtin_bit_cast(bf16x8, (u4)__builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16, (ks * NT + nt) * 1024, 0));
  };
#pragma unroll
  for (int ks = 0; ks < AHEAD; ++ks) fetch(ks);
  int at[R], cx[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int p = min((wave + 4 * j) * 16 + r, M - 1);
    at[j] = ((p / WOUT) * WIN + p % WOUT) * SIN;
    cx[j] = p % WOUT;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + AHEAD < KS) fetch(ks + AHEAD);
    bf16x8 a[R];
#pragma unroll
    for (int j = 0; j < R; ++j)
      a[j] = as_bf16x8(*reinterpret_cast<const uint4*>(in + at[j] + (SIN == 32 ? swizzle(g, cx[j] + ks % 3) : 8 * g) +
                                                   ((ks / 3) * WIN + ks % 3) * SIN));
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int j = 0; j < R; ++j) acc[j][nt] = mfma(w[ks][nt], a[j], acc[j][nt]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// four values as BF16
__device__ __forceinline__ uint2 bf16_pack(float a, float b, float c, float d) {
  return make_uint2(bf16_bits(a) | (uint32_t)bf16_bits(b) << 16, bf16_bits(c) | (uint32_t)bf16_bits(d) << 16);
}

constexpr int PSTRIDE = 40;   // BF16 elements per pixel of a 32-channel LDS tile: 80 bytes, so that the 16 pixels
                               // that a 16-byte read touches start 4 banks apart and cover all banks once

// ------------------------------------------------------------------ inference
// One 16x16 tile of coarse pixels per workgroup: input tile with a 3-pixel
// halo, the hidden activations in LDS, output 32x32 fine pixels.  Bound by the
// latency of its phases (matrix cores busy 18% of the cycles), so it is built
// to have four workgroups on a compute unit: a hidden layer's results wait in
// registers until all of its input is read and then take the input's place
// (31 KB of LDS), and no layer's weights stay in registers (126 of them).  The last
// layer's results go to an LDS output tile (in the activation's space again) and
// leave as whole fine pixels, with the bilinear skip read from an FP32 copy of
// the input (in the BF16 input tile's space, free after the first layer).
// 960x540, whose 2040 tiles then fill the chip twice instead of 2.7 times: 39.6
// -> 34.7 us; with two activations in LDS and three workgroups, swizzled 38.9,
// not swizzled 39.6.
constexpr int XF = 18;        // FP32 input pixels per side for the bilinear skip of a tile
constexpr int ISTRIDE = 32;   // BF16 elements per pixel of the hidden activations (swizzled)
__global__ __launch_bounds__(256, 4) void infer_kernel(CnnInferArgs a) {
  __shared__ __attribute__((aligned(16))) float xbuf[XF * XF * 4];   // BF16 22x22x4 input, then FP32 18x18x4
  __shared__ __attribute__((aligned(16))) uint16_t a1[20 * 20 * ISTRIDE];
  static_assert(sizeof(uint16_t) * 22 * 22 * 4 <= sizeof(float) * XF * XF * 4, "input tile fits");
  static_assert(sizeof(a1) >= sizeof(float) * 32 * 32 * 4, "output tile fits");
  uint16_t* xs = reinterpret_cast<uint16_t*>(xbuf);
  const int H = a.h, W = a.w;
  const int n = blockIdx.z;
  const int oy = blockIdx.y * 16, ox = blockIdx.x * 16;
  const float4* __restrict__ x = reinterpret_cast<const float4*>(a.x) + (int64_t)n * H * W;
  float* __restrict__ out = a.out + (int64_t)n * 4 * H * W * 4;
  const int tid = threadIdx.x, g = (tid & 63) >> 4;
  float4 in[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + 256 * k, gy = oy - 3 + i / 22, gx = ox - 3 + i % 22;
    in[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < 22 * 22 && gy >= 0 && gy < H && gx >= 0 && gx < W) in[k] = x[(int64_t)gy * W + gx];
  }
  bf16x8 w1[4];
  load_weights(a.wf1, w1);
  const float* __restrict__ bias = a.params;
  float bv[2][4];
  auto biases = [&](int at, int nt_count) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (nt < nt_count) bv[nt][i] = bias[at + 16 * nt + 4 * g + i];
  };
  biases(CNN_OFF_B1, 2);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + 256 * k;
    if (i < 22 * 22) *reinterpret_cast<uint2*>(xs + 4 * i) = bf16_pack(in[k].x, in[k].y, in[k].z, in[k].w);
  }
  __syncthreads();
  // a hidden layer's outputs are zero outside the image (the next one's padding)
  const bool inner = oy >= 2 && ox >= 2 && oy + 18 <= H && ox + 18 <= W;
  auto hidden = [&](uint16_t* d, int col, int y, int z, const f32x4* v) {
    const bool keep = inner || (y >= 0 && y < H && z >= 0 && z < W);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      float q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = fmaxf(v[nt][i] + bv[nt][i], 0.0f);
      const uint2 u = bf16_pack(q[0], q[1], q[2], q[3]);
      *reinterpret_cast<uint2*>(d + swizzle(2 * nt + (g >> 1), col) + 4 * (g & 1)) =
          make_uint2(keep ? u.x : 0u, keep ? u.y : 0u);
    }
  };
  conv_tile<4, 2, 2, 7, 22, 4, 400, 20>(xs, w1, [&](int p, const f32x4* v) {
    hidden(a1 + p * ISTRIDE, p % 20, oy - 2 + p / 20, ox - 2 + p % 20, v);
  });
  __syncthreads();
  // FP32 input rows oy-1 .. oy+16 and columns ox-1 .. ox+16, clamped to the
  // image as the bilinear skip clamps them
  for (int i = tid; i < XF * XF; i += 256) {
    const int gy = min(max(oy - 1 + i / XF, 0), H - 1), gx = min(max(ox - 1 + i % XF, 0), W - 1);
    reinterpret_cast<float4*>(xbuf)[i] = x[(int64_t)gy * W + gx];
  }
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6), r = tid & 15;
  {
    f32x4 acc[6][2];
    conv_hold<2, 6, 20, ISTRIDE, 324, 18>(a1, a.wf2, acc);
    biases(CNN_OFF_B2, 2);
    __syncthreads();   // (all of a1 read: the second activation takes its place)
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const int p = (wave + 4 * j) * 16 + r;
      if (p < 324) hidden(a1 + p * ISTRIDE, p % 18, oy - 1 + p / 18, ox - 1 + p % 18, acc[j]);
    }
  }
  __syncthreads();
  float* ot = reinterpret_cast<float*>(a1);   // [32][32] fine pixels x 4 channels
  {
    f32x4 acc[4][1];
    conv_hold<1, 4, 18, ISTRIDE, 256, 16>(a1, a.wf3, acc);
    biases(CNN_OFF_B3, 1);
    __syncthreads();
    // channel 4c + 2dy + dx goes to fine pixel (2i + dy, 2j + dx), channel c: the lane's four are c = g
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float* d = ot + ((2 * (wave + 4 * j)) * 32 + 2 * r) * 4 + g;
      d[0] = acc[j][0][0] + bv[0][0];
      d[4] = acc[j][0][1] + bv[0][1];
      d[128] = acc[j][0][2] + bv[0][2];
      d[132] = acc[j][0][3] + bv[0][3];
    }
  }
  __syncthreads();
  // out = shuffled network output + bilinear x2 of x (half-pixel centres,
  // clamp to edge), whole fine pixels per thread; fine coordinates lie a
  // quarter to either side of the coarse one (xbuf holds the clamped
  // neighbours)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = tid + 256 * k, fy = i / 32, fx = i % 32;
    const int Y = 2 * oy + fy, X = 2 * ox + fx;
    const float ty = (fy & 1) ? 0.25f : 0.75f, tx = (fx & 1) ? 0.25f : 0.75f;
    const int at = ((fy + 1) >> 1) * XF + ((fx + 1) >> 1);
    const float4* xv = reinterpret_cast<const float4*>(xbuf) + at;
    const float4 v00 = xv[0], v01 = xv[1], v10 = xv[XF], v11 = xv[XF + 1];
    const float4 z = reinterpret_cast<const float4*>(ot)[i];
    auto bl = [&](float a00, float a01, float a10, float a11) {
      const float top = a00 * (1.0f - tx) + a01 * tx;
      const float bot = a10 * (1.0f - tx) + a11 * tx;
      return top * (1.0f - ty) + bot * ty;
    };
    float4 o;
    o.x = z.x + bl(v00.x, v01.x, v10.x, v11.x);
    o.y = z.y + bl(v00.y, v01.y, v10.y, v11.y);
    o.z = z.z + bl(v00.z, v01.z, v10.z, v11.z);
    o.w = z.w + bl(v00.w, v01.w, v10.w, v11.w);
    if (Y < 2 * H && X < 2 * W) reinterpret_cast<float4*>(out)[(int64_t)Y * 2 * W + X] = o;
  }
}

// ------------------------------------------------------------------ training forward / backward-data
// Stage an 18x18 input tile (output tile 16x16 plus a 1-pixel halo) of CIN
// channels into LDS: from the FP32 image (CIN = 4) or a BF16 NHWC tensor.
template <int CIN>
__device__ void stage_tile(uint16_t* t, int sin, const float* __restrict__ img, const uint16_t* __restrict__ act,
                           int H, int W, int oy, int ox) {
  for (int i = threadIdx.x; i < 18 * 18; i += blockDim.x) {
    const int gy = oy - 1 + i / 18, gx = ox - 1 + i % 18;
    const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
    if (CIN == 4) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (in) v = reinterpret_cast<const float4*>(img)[(int64_t)gy * W + gx];
      t[i * sin + 0] = bf16_bits(v.x);
      t[i * sin + 1] = bf16_bits(v.y);
      t[i * sin + 2] = bf16_bits(v.z);
      t[i * sin + 3] = bf16_bits(v.w);
    } else {
      const uint4* src = reinterpret_cast<const uint4*>(act + ((int64_t)gy * W + gx) * CIN);
      for (int q = 0; q < CIN / 8; ++q)
        *reinterpret_cast<uint4*>(t + i * sin + 8 * q) = in ? src[q] : make_uint4(0, 0, 0, 0);
    }
  }
}

// Bound by HBM and the latency of a tile's phases.  At 960x540: forward 14.7,
// 21.7 and (with the loss) 25.9 us, backward 17.6 and 25.2 us.  The layers of 32
// input channels stream their weights and the loss layer keeps its outputs and
// gradients in its input's place, so that four workgroups share a compute
// unit: with the weights in registers and LDS of their own 22.3, 32.8 and 26.0.
// With a lane's results in one channel of four pixels (2-byte stores, 4-byte
// loads of the target) 14.6, 24, 37.6, 28.6 and 33.
// mode 0: a = bf16(relu(z + b)) stored NHWC (COUT channels)
// mode 1: g = bf16(z * [mask > 0]) stored NHWC (backward-data with ReLU mask)
// mode 2: last layer + loss: y = z + b, out = shuffle(y) + bilinear(x),
//         g_y = bf16(2 (out - target) / count), squared error summed per tile
template <int CIN, int COUT, int MODE>
__global__ __launch_bounds__(256, CIN == 32 ? 4 : 1) void layer_kernel(CnnLayerArgs a) {
  constexpr int KS = (9 * CIN + 31) / 32;   // k-steps of 32 (tap, channel) pairs
  constexpr int SIN = CIN == 4 ? 4 : PSTRIDE;
  constexpr int NT = COUT / 16;
  __shared__ __attribute__((aligned(16))) uint16_t t[18 * 18 * SIN];
  // last layer: the image around the tile, and in the input's place its
  // outputs as fine pixels and their gradients
  __shared__ float4 xi[MODE == 2 ? 18 * 18 : 1];
  __shared__ float red[MODE == 2 ? 256 : 1];
  float4* ot = reinterpret_cast<float4*>(t);
  uint16_t* gt = t + 32 * 32 * 8;
  static_assert(MODE != 2 || 18 * 18 * SIN >= 32 * 32 * 8 + 256 * 16, "outputs and gradients fit");
  const int H = a.h, W = a.w;
  const int n = blockIdx.z;
  const int oy = blockIdx.y * 16, ox = blockIdx.x * 16;
  const int64_t plane = (int64_t)H * W;
  bf16x8 w[CIN == 32 ? 1 : KS * NT];
  if constexpr (CIN != 32) load_weights(a.wf, w);
  stage_tile<CIN>(t, SIN, a.img ? a.img + n * plane * 4 : nullptr, a.in ? a.in + n * plane * CIN : nullptr, H, W, oy, ox);
  if (MODE == 2)
    for (int i = threadIdx.x; i < 18 * 18; i += 256) {
      const int gy = min(max(oy - 1 + i / 18, 0), H - 1), gx = min(max(ox - 1 + i % 18, 0), W - 1);
      xi[i] = reinterpret_cast<const float4*>(a.img)[n * plane + (int64_t)gy * W + gx];
    }
  const int g = (threadIdx.x & 63) >> 4;
  float bv[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int i = 0; i < 4; ++i) bv[nt][i] = MODE == 1 ? 0.0f : a.bias[16 * nt + 4 * g + i];
  __syncthreads();
  auto result = [&](int p, const f32x4* v) {
    if (MODE == 2) {
      // channel 4c + 2dy + dx is channel c of fine pixel (2 gy + dy, 2 gx + dx): the lane's four are c = g
      float* d = reinterpret_cast<float*>(ot) + ((2 * (p >> 4)) * 32 + 2 * (p & 15)) * 4 + g;
      d[0] = v[0][0] + bv[0][0];
      d[4] = v[0][1] + bv[0][1];
      d[128] = v[0][2] + bv[0][2];
      d[132] = v[0][3] + bv[0][3];
      return;
    }
    const int gy = oy + p / 16, gx = ox + p % 16;
    if (gy >= H || gx >= W) return;
    const int64_t pix = n * plane + (int64_t)gy * W + gx;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // four consecutive channels of one pixel: 8-byte loads and stores
      const int64_t at = pix * COUT + 16 * nt + 4 * g;
      uint2* out = reinterpret_cast<uint2*>(a.out + at);
      if (MODE == 0) {
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = fmaxf(v[nt][i] + bv[nt][i], 0.0f);
        *out = bf16_pack(z[0], z[1], z[2], z[3]);
      } else if (MODE == 1) {
        const uint2 m = *reinterpret_cast<const uint2*>(a.mask + at);
        *out = bf16_pack((m.x & 0x7fffu) ? v[nt][0] : 0.0f, (m.x & 0x7fff0000u) ? v[nt][1] : 0.0f,
                         (m.y & 0x7fffu) ? v[nt][2] : 0.0f, (m.y & 0x7fff0000u) ? v[nt][3] : 0.0f);
      }
    }
  };
  if constexpr (CIN == 32) {
    f32x4 acc[4][NT];
    conv_hold<NT, 4, 18, SIN, 256, 16>(t, a.wf, acc);
    if (MODE == 2) __syncthreads();   // (all of the input read)
#pragma unroll
    for (int j = 0; j < 4; ++j) result(((int)(threadIdx.x >> 6) + 4 * j) * 16 + (int)(threadIdx.x & 15), acc[j]);
  } else {
    conv_tile<CIN, KS, NT, 4, 18, SIN, 256, 16>(t, w, result);
  }
  if (MODE == 2) {
    // whole fine pixels per thread, so that the target is read and the
    // gradient written in whole lines
    float sq = 0.0f;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = threadIdx.x + 256 * k, fy = i / 32, fx = i % 32, Y = 2 * oy + fy, X = 2 * ox + fx;
      // bilinear x2 (half-pixel centres, clamp to edge): fine coordinates lie
      // a quarter to either side of the coarse one
      const float ty = (fy & 1) ? 0.25f : 0.75f, tx = (fx & 1) ? 0.25f : 0.75f;
      const float4* xv = xi + ((fy + 1) >> 1) * 18 + ((fx + 1) >> 1);
      const float4 v00 = xv[0], v01 = xv[1], v10 = xv[18], v11 = xv[19], z = ot[i];
      const bool in = Y < 2 * H && X < 2 * W;
      float4 tg = make_float4(0.f, 0.f, 0.f, 0.f);
      if (in) tg = reinterpret_cast<const float4*>(a.target)[n * 4 * plane + (int64_t)Y * 2 * W + X];
      auto diff = [&](float zc, float a00, float a01, float a10, float a11, float t) {
        const float top = a00 * (1.0f - tx) + a01 * tx;
        const float bot = a10 * (1.0f - tx) + a11 * tx;
        return (zc + (top * (1.0f - ty) + bot * ty)) - t;
      };
      const float d[4] = {diff(z.x, v00.x, v01.x, v10.x, v11.x, tg.x), diff(z.y, v00.y, v01.y, v10.y, v11.y, tg.y),
                          diff(z.z, v00.z, v01.z, v10.z, v11.z, tg.z), diff(z.w, v00.w, v01.w, v10.w, v11.w, tg.w)};
      // channel 4c + 2dy + dx of the coarse pixel is channel c of fine pixel (dy, dx)
      uint16_t* gp = gt + ((fy >> 1) * 16 + (fx >> 1)) * 16 + 2 * (fy & 1) + (fx & 1);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (in) sq += d[c] * d[c];
        gp[4 * c] = bf16_bits(d[c] * a.grad_scale);
      }
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int i = threadIdx.x; i < 512; i += 256) {
      const int gy = oy + i / 32, gx = ox + (i >> 1) % 16;
      if (gy < H && gx < W)
        reinterpret_cast<uint4*>(a.out + (n * plane + (int64_t)gy * W + gx) * 16)[i & 1] = reinterpret_cast<const uint4*>(gt)[i];
    }
    for (int s = 128; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0)
      a.loss_part[((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = red[0];
  }
}

// ------------------------------------------------------------------ backward-weights
// dW[o][c][tap] = sum_p g[p][o] x[p + tap][c] and db[o] = sum_p g[p][o], as a
// GEMM with rows o, columns (tap, c) and the reduction over pixels, 32 to a
// matrix instruction (two rows of a 16x16 tile).  Both operands need eight
// consecutive pixels of one channel per lane, so a tile is staged in LDS
// channel by channel (pixels contiguous): operand A is then one 16-byte read,
// and one 20-byte read of a row of x gives operand B of the row's three taps
// (the tap one to the right is the same bytes shifted by one pixel).  A
// workgroup keeps its sums in the accumulators over all its tiles
// (blockIdx.x, + gridDim.x, ...) and writes one partial vector at its end, in
// the layout of the parameters; the next tile's inputs come to registers during
// a tile.  At 960x540 the three launches take 18, 25 and 11 us and the reduction
// of all layers with the update 11 us; without the loads ahead 34, 45 and 25;
// with one partial vector per tile, gathered element by element from LDS, 46,
// 85 and 37, and 473 us for each layer's reduction (one thread per parameter).
constexpr int XROW = 24;               // elements per staged row of x: 18 pixels, rows 16-byte aligned
constexpr int XCH = 18 * XROW + 8;     // elements per staged channel of x and of g: the 16 channels that
constexpr int GCH = 256 + 8;           // a read touches start 4 banks apart, so their 16 bytes cover all banks once

// the 16-bit elements j of eight channels of two neighbouring pixels, as one
// pair (a in the low half) per channel at d[j * stride] (in pairs)
__device__ __forceinline__ void store_pairs(uint32_t* d, int stride, uint4 a, uint4 b) {
  const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    d[(2 * j) * stride] = __builtin_amdgcn_perm(bv[j], av[j], 0x05040100u);
    d[(2 * j + 1) * stride] = __builtin_amdgcn_perm(bv[j], av[j], 0x07060302u);
  }
}

template <int CIN, int COUT>
__global__ __launch_bounds__(256) void wgrad_kernel(CnnWgradArgs a) {
  constexpr int NCOL = 9 * CIN;
  constexpr bool IMG = CIN == 4;
  // the four waves share the work as (o tile) x (c tile) x (half of the rows)
  constexpr int OT = COUT / 16, CT = IMG ? 1 : CIN / 16, KH = 4 / (OT * CT);
  constexpr int NB = IMG ? 3 : 9;      // accumulators: taps, or rows of taps (columns 4 dx + c) of the image
  __shared__ __attribute__((aligned(16))) uint16_t xt[CIN * XCH];
  __shared__ __attribute__((aligned(16))) uint16_t gt[COUT * GCH];
  const int H = a.h, W = a.w;
  const int64_t plane = (int64_t)H * W;
  const int tx = (W + 15) >> 4, ty = (H + 15) >> 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15;
  const int ot = wave % OT, ct = (wave / OT) % CT, kh = wave / (OT * CT);
  f32x4 acc[NB], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16x8 ones = as_bf16x8(make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  // the thread's share of a tile, on its way while the tile before is summed:
  // 18 rows of nine pixel pairs of x (zero outside the image), 128 pairs of g
  constexpr int XQ = IMG ? 1 : CIN / 8, XN = (162 * XQ + 255) / 256, GQ = COUT / 8, GN = 128 * GQ / 256;
  uint4 xr[XN][2], gr[GN][2];
  float4 fr[2];
  auto fetch = [&](int tile) {
    const int n = tile / (tx * ty), rem = tile - n * (tx * ty), oy = (rem / tx) * 16, ox = (rem % tx) * 16;
    const uint4 z = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < XN; ++t) {
      const int i = tid + 256 * t, q = i % XQ, pr = i / XQ, row = pr / 9, k = pr % 9;
      const int gy = oy - 1 + row, gx = ox - 1 + 2 * k;
      const bool in = i < 162 * XQ && gy >= 0 && gy < H, in0 = in && gx >= 0 && gx < W, in1 = in && gx + 1 < W;
      const int64_t pix = n * plane + (int64_t)gy * W + gx;
      if constexpr (IMG) {
        fr[0] = fr[1] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in0) fr[0] = reinterpret_cast<const float4*>(a.img)[pix];
        if (in1) fr[1] = reinterpret_cast<const float4*>(a.img)[pix + 1];
      } else {
        xr[t][0] = xr[t][1] = z;
        if (in0) xr[t][0] = reinterpret_cast<const uint4*>(a.x + pix * CIN)[q];
        if (in1) xr[t][1] = reinterpret_cast<const uint4*>(a.x + (pix + 1) * CIN)[q];
      }
    }
#pragma unroll
    for (int t = 0; t < GN; ++t) {
      const int i = tid + 256 * t, q = i % GQ, pr = i / GQ, gy = oy + (pr >> 3), gx = ox + 2 * (pr & 7);
      const int64_t pix = n * plane + (int64_t)gy * W + gx;
      gr[t][0] = gr[t][1] = z;
      if (gy < H && gx < W) gr[t][0] = reinterpret_cast<const uint4*>(a.g + pix * COUT)[q];
      if (gy < H && gx + 1 < W) gr[t][1] = reinterpret_cast<const uint4*>(a.g + (pix + 1) * COUT)[q];
    }
  };
  fetch(blockIdx.x);
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    __syncthreads();   // the tile before has been read
    uint32_t* xp = reinterpret_cast<uint32_t*>(xt);
    uint32_t* gp = reinterpret_cast<uint32_t*>(gt);
#pragma unroll
    for (int t = 0; t < XN; ++t) {
      const int i = tid + 256 * t, q = i % XQ, pr = i / XQ;
      if (i >= 162 * XQ) break;
      uint32_t* d = xp + (8 * q) * (XCH / 2) + (pr / 9) * (XROW / 2) + pr % 9;
      if constexpr (IMG) {
        d[0] = bf16_bits(fr[0].x) | (uint32_t)bf16_bits(fr[1].x) << 16;
        d[XCH / 2] = bf16_bits(fr[0].y) | (uint32_t)bf16_bits(fr[1].y) << 16;
        d[XCH] = bf16_bits(fr[0].z) | (uint32_t)bf16_bits(fr[1].z) << 16;
        d[3 * (XCH / 2)] = bf16_bits(fr[0].w) | (uint32_t)bf16_bits(fr[1].w) << 16;
      } else {
        store_pairs(d, XCH / 2, xr[t][0], xr[t][1]);
      }
    }
#pragma unroll
    for (int t = 0; t < GN; ++t) {
      const int i = tid + 256 * t, q = i % GQ, pr = i / GQ;
      store_pairs(gp + (8 * q) * (GCH / 2) + pr, GCH / 2, gr[t][0], gr[t][1]);
    }
    __syncthreads();
    if (tile + (int)gridDim.x < a.n_tiles) fetch(tile + gridDim.x);
#pragma unroll
    for (int s = 0; s < 8 / KH; ++s) {
      const int row = 2 * (s + (8 / KH) * kh) + (g >> 1), xo = 8 * (g & 1);
      const bf16x8 av = as_bf16x8(*reinterpret_cast<const uint4*>(gt + (ot * 16 + r) * GCH + row * 16 + xo));
      if (ct == 0) accb = mfma(av, ones, accb);
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        // pixels xo .. xo + 9 of the row dy of the lane's channel
        const uint16_t* src = xt + (IMG ? (r & 3) : ct * 16 + r) * XCH + (row + dy) * XROW + xo;
        const uint4 lo = *reinterpret_cast<const uint4*>(src);
        const uint32_t hi = *reinterpret_cast<const uint32_t*>(src + 8);
        if constexpr (IMG) {
          // columns 4 dx + c: the lane's dx = r / 4 (columns 12-15 are not used)
          const int sh = 16 * min(r >> 2, 2);
          auto pick = [&](uint32_t p, uint32_t q) { return (uint32_t)((((uint64_t)q << 32) | p) >> sh); };
          acc[dy] = mfma(av, as_bf16x8(make_uint4(pick(lo.x, lo.y), pick(lo.y, lo.z), pick(lo.z, lo.w), pick(lo.w, hi))),
                         acc[dy]);
        } else {
          auto mid = [&](uint32_t p, uint32_t q) { return __builtin_amdgcn_alignbit(q, p, 16); };
          acc[3 * dy] = mfma(av, as_bf16x8(lo), acc[3 * dy]);
          acc[3 * dy + 1] = mfma(
              av, as_bf16x8(make_uint4(mid(lo.x, lo.y), mid(lo.y, lo.z), mid(lo.z, lo.w), mid(lo.w, hi))), acc[3 * dy + 1]);
          acc[3 * dy + 2] = mfma(av, as_bf16x8(make_uint4(lo.y, lo.z, lo.w, hi)), acc[3 * dy + 2]);
        }
      }
    }
  }
  if constexpr (KH == 2) {
    // the two halves of the rows meet in LDS
    float* mine = reinterpret_cast<float*>(IMG ? gt : xt) + ((wave & 1) * 64 + lane) * 4;
    static_assert((IMG ? sizeof(gt) : sizeof(xt)) >= 512 * (NB + 1) * sizeof(float), "accumulators fit");
    __syncthreads();
    if (kh == 1) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) mine[j * 512 + i] = acc[j][i];
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[NB * 512 + i] = accb[i];
    }
    __syncthreads();
    if (kh == 1) return;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[j][i] += mine[j * 512 + i];
#pragma unroll
    for (int i = 0; i < 4; ++i) accb[i] += mine[NB * 512 + i];
  }
  // rows o = 16 ot + 4 g + i, layout W[o][c][dy][dx], then b[o]
  float* part = a.part + (int64_t)blockIdx.x * CNN_N_PARAMS + a.off;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = ot * 16 + 4 * g + i;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (IMG) {
        if (r < 12) part[o * NCOL + (r & 3) * 9 + 3 * j + (r >> 2)] = acc[j][i];
      } else {
        part[o * NCOL + (ct * 16 + r) * 9 + j] = acc[j][i];
      }
    }
    if (ct == 0 && r == 0) part[COUT * NCOL + o] = accb[i];
  }
}

// ------------------------------------------------------------------ reduction, Adam and packing
// element of the packed fragments (see pack_kernel) that holds B[k][n]
__device__ __forceinline__ int frag_index(int k, int n, int nt) {
  return (((k >> 5) * nt + (n >> 4)) * 64 + 16 * ((k >> 3) & 3) + (n & 15)) * 8 + (k & 7);
}

// Sums the workgroups' partial vectors into the gradient, 64 parameters per
// workgroup: wave k adds the vectors k, k + 16, ... and the sixteen sums are
// added in order (fixed orders: deterministic).  With an update (u.w), the
// thread that holds a parameter's gradient also takes its Adam step and
// writes the weight's BF16 value into the fragments that the layers read, in
// place of two more launches.
__global__ __launch_bounds__(1024) void reduce_kernel(const float* __restrict__ part, int n_part,
                                                      float* __restrict__ grad, CnnUpdate u, CnnPackTable tab) {
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + lane;
  float s = 0.0f;
  if (j < CNN_N_PARAMS) {
#pragma unroll 8
    for (int t = wave; t < n_part; t += 16) s += part[(int64_t)t * CNN_N_PARAMS + j];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0 || j >= CNN_N_PARAMS) return;
  float gi = red[0][lane];
#pragma unroll
  for (int k = 1; k < 16; ++k) gi += red[k][lane];
  grad[j] = gi;
  if (!u.w) return;
  const float mi = u.b1 * u.m[j] + (1.0f - u.b1) * gi;
  const float vi = u.b2 * u.v[j] + (1.0f - u.b2) * gi * gi;
  u.m[j] = mi;
  u.v[j] = vi;
  const float w = u.w[j] - u.lr * (mi / u.c1) / (sqrtf(vi / u.c2) + u.eps);
  u.w[j] = w;
  const uint16_t h = bf16_bits(w);
  for (int e = 0; e < tab.n; ++e) {
    const CnnPackEntry& p = tab.e[e];
    const int x = j - p.w_off;
    if (x < 0 || x >= p.cout * p.cin * 9) continue;   // another layer's weight, or a bias
    const int o = x / (9 * p.cin), c = (x / 9) % p.cin, tap = x % 9;
    p.dst[p.transposed ? frag_index((8 - tap) * p.cout + o, c, p.nt) : frag_index(tap * p.cin + c, o, p.nt)] = h;
  }
}

// B fragments: element i of lane l of (ks, nt) is B[k][n] with
// k = 32 ks + 8 (l / 16) + i, n = 16 nt + l % 16.  Forward layers:
// B[tap*CIN + c][o] = W[o][c][tap]; backward-data (a convolution of the output
// gradient): B[tap*COUT + o][c] = W[o][c][8 - tap].
__global__ void pack_kernel(const float* __restrict__ w, CnnPackTable tab) {
  const int gidx = blockIdx.x * blockDim.x + threadIdx.x;
  int rem = gidx;
  for (int e = 0; e < tab.n; ++e) {
    const CnnPackEntry& p = tab.e[e];
    const int count = p.ks * p.nt * 64 * 8;
    if (rem < count) {
      const int i = rem & 7, lane = (rem >> 3) & 63, frag = rem >> 9;
      const int ks = frag / p.nt, nt = frag % p.nt;
      const int k = 32 * ks + 8 * (lane >> 4) + i, ncol = 16 * nt + (lane & 15);
      float val = 0.0f;
      if (!p.transposed) {
        // forward: k = tap*cin + c, ncol = o
        if (k < 9 * p.cin) {
          const int tap = k / p.cin, c = k % p.cin;
          val = w[p.w_off + (ncol * p.cin + c) * 9 + tap];
        }
      } else {
        // backward-data: k = tap*cout + o, ncol = c
        if (k < 9 * p.cout) {
          const int tap = k / p.cout, o = k % p.cout;
          val = w[p.w_off + (o * p.cin + ncol) * 9 + (8 - tap)];
        }
      }
      p.dst[rem] = bf16_bits(val);
      return;
    }
    rem -= count;
  }
}

}  // namespace

hipError_t cnn_launch_infer(const CnnInferArgs& a, int n, hipStream_t st) {
  dim3 grid((a.w + 15) / 16, (a.h + 15) / 16, n);
  infer_kernel<<<grid, 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t cnn_launch_layer(int layer, int mode, const CnnLayerArgs& a, int n, hipStream_t st) {
  dim3 grid((a.w + 15) / 16, (a.h + 15) / 16, n);
  if (layer == 1 && mode == 0) layer_kernel<4, 32, 0><<<grid, 256, 0, st>>>(a);
  else if (layer == 2 && mode == 0) layer_kernel<32, 32, 0><<<grid, 256, 0, st>>>(a);
  else if (layer == 3 && mode == 2) layer_kernel<32, 16, 2><<<grid, 256, 0, st>>>(a);
  // backward-data of layer 3: input g_y (16 ch) -> g_a2 (32 ch) masked by a2
  else if (layer == 3 && mode == 1) layer_kernel<16, 32, 1><<<grid, 256, 0, st>>>(a);
  // backward-data of layer 2: input g_z2 (32 ch) -> g_a1 (32 ch) masked by a1
  else if (layer == 2 && mode == 1) layer_kernel<32, 32, 1><<<grid, 256, 0, st>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t cnn_launch_wgrad(int layer, const CnnWgradArgs& a, int n_workgroups, hipStream_t st) {
  if (layer == 1) wgrad_kernel<4, 32><<<n_workgroups, 256, 0, st>>>(a);
  else if (layer == 2) wgrad_kernel<32, 32><<<n_workgroups, 256, 0, st>>>(a);
  else if (layer == 3) wgrad_kernel<32, 16><<<n_workgroups, 256, 0, st>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t cnn_launch_reduce(const float* part, int n_part, float* grad, const CnnUpdate& u, const CnnPackTable& tab,
                             hipStream_t st) {
  reduce_kernel<<<(CNN_N_PARAMS + 63) / 64, 1024, 0, st>>>(part, n_part, grad, u, tab);
  return hipGetLastError();
}

CnnUpdate cnn_adam(float* w, float* m, float* v, float lr, int64_t step) {
  const double b1 = 0.9, b2 = 0.999;
  CnnUpdate u;
  u.w = w;
  u.m = m;
  u.v = v;
  u.lr = lr;
  u.b1 = (float)b1;
  u.b2 = (float)b2;
  u.eps = 1e-8f;
  u.c1 = (float)(1.0 - pow(b1, (double)step));
  u.c2 = (float)(1.0 - pow(b2, (double)step));
  return u;
}

hipError_t cnn_launch_pack(const float* w, const CnnPackTable& tab, hipStream_t st) {
  int total = 0;
  for (int e = 0; e < tab.n; ++e) total += tab.e[e].ks * tab.e[e].nt * 64 * 8;
  pack_kernel<<<(total + 255) / 256, 256, 0, st>>>(w, tab);
  return hipGetLastError();
}
