// cnn.hip -- the camera decoder of the rendered features (SplatAD, arXiv 2411.16816, Sec. 3.2: a
// small CNN maps the feature image, the ray directions and a camera embedding to a per-pixel
// affine map of the rendered colour; the training-details appendix: two residual blocks of
// width 32, kernel size 3, then a final linear layer).
//
//   x  = [F, d, e]                       (D_f + 3 + E <= 32 channels, zero-padded to 32)
//   h0 = ReLU(conv_in(x)),  r_k = ReLU(conv_k1(h_{k-1})),  h_k = ReLU(h_{k-1} + conv_k2(r_k))
//   (M, b) = W_out h_2 + b_out,  I = M * F_rgb + b
//
// Activations are NHWC float32 with 32 channels.  The 3x3 convolutions are dense contractions
// (K = 9 taps x 32 channels per output) and run on the matrix cores, FP32 in and FP32 accumulate:
//   * forward (k_conv3x3): v_mfma_f32_16x16x4_f32, whose results the ReLU decisions of the adjoint
//     depend on (a change of rounding here flips some of them).  1920 x 1080, per convolution:
//     0.354 ms, 108 TFLOP/s of the 137 that the instruction reaches from registers; as three
//     independent workgroups per compute unit it took 0.46 ms.  The epilogue also leaves the signs
//     of the activations (a bit per channel) for the adjoint, which would otherwise read the whole
//     activation image for them;
//   * input gradient (k_conv3x3_bwd) and weight gradient (k_conv3x3_wgrad): the bf16 matrix
//     instructions on operands split into three bf16 parts (see below).  1920 x 1080: 0.22 ms
//     (0.46 with the FP32 instructions) and 0.23 ms (0.445) per convolution.  Their matrix work alone
//     is 0.095 ms and their HBM traffic about 0.12 ms; what they cannot overlap is the splitting and
//     the barriers of one workgroup per compute unit;
//   * the stem input, the 1x1 head and their adjoints are per-pixel kernels.
#include "kernels.hpp"
#include "reduce.hpp"
#include "wave_ops.hpp"

namespace splat {

constexpr int kCC = 32;            // padded channel count of every activation
constexpr int kTS = 16;            // forward tile side
constexpr int kHalo = kTS + 2;     // 18
constexpr int kLS = 36;            // floats per pixel in LDS (32 + 4: 16-byte aligned rows)
constexpr int kWTH = 8;            // weight-gradient tile: 8 rows x 16 columns
constexpr int kWOut = 9 * kCC * kCC + kCC;   // partial sums per workgroup: dW [tap][ci][co], db
constexpr int kHeadOut = 6 * kCC + 6;        // dW_out [6][32], db_out [6]
constexpr int kCnnBlock = 128;               // per-pixel kernels with LDS contractions

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---- FP32 contractions on the bf16 matrix cores ------------------------------------------------
// A float is the exact sum of three bf16 values (8 significand bits each, rounded to nearest: the
// remainders are exact): x = h + m + l.  A product of two floats is then the six products
// hh + hm + mh + mm + hl + lh up to 2^-24 of it, each exact in FP32; v_mfma_f32_32x32x16_bf16 adds
// sixteen of them per output in FP32.  Its rate is 17.5x that of the FP32 matrix instructions
// (2400 against 137 TFLOP/s measured from registers), so six products are 2.9x as fast.
//
// The instruction rounds its sums of mixed magnitudes downwards: with all six products in one
// accumulator a dot product of 288 normal values errs by 2.5e-7 rms of its own rms (FP32
// instructions: 3.0e-7), of which -1.7e-8 is a bias that sums over many pixels would collect.  With
// the hh products, which align, in an accumulator of their own the error is 9.5e-8 and the bias below
// 1e-9.  Where the registers do not allow that, half of the terms are contracted negated and
// subtracted, so that the bias cancels.
//
// Operands are split scaled by 2^24, and the sums scaled back: the last bit of any FP32 value is then
// 2^-125 at least, so that no part falls among bf16's subnormals, which would cost it bits (unscaled,
// operands of 1e-36 gave sums off by 3e-5).  Infinities and NaN do not split, and products or sums above
// 2^79 do not fit the scaled range: the kernels find the outputs that are not finite and contract them
// with the FP32 instructions.
constexpr float kSplitScale = 16777216.f;                            // 2^24
constexpr float kSplitBack = 1.f / (kSplitScale * kSplitScale);
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}

// parts[0..2] = the (high, middle, low) bf16 parts of the pair (a, b) times `scale`, a in the low half
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&parts)[3], float scale = kSplitScale) {
  a *= scale;
  b *= scale;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    parts[p] = pack_bf16(a, b);
    a -= __uint_as_float(parts[p] << 16);
    b -= __uint_as_float(parts[p] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ floatx16 mfma16(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// the six products of a split contraction: part of A, part of B, and the accumulator of a kernel that
// keeps one per magnitude (0: hl lh mm, 1: hm mh, 2: hh); two products on one are far apart
constexpr int kProd = 6;
__device__ constexpr int prod_a(int i) { return i == 0 ? 0 : i == 1 ? 0 : i == 2 ? 0 : i == 3 ? 2 : i == 4 ? 1 : 1; }
__device__ constexpr int prod_b(int i) { return i == 0 ? 2 : i == 1 ? 1 : i == 2 ? 0 : i == 3 ? 0 : i == 4 ? 0 : 1; }
__device__ constexpr int prod_acc(int i) { return i == 0 ? 0 : i == 1 ? 1 : i == 2 ? 2 : i == 3 ? 0 : i == 4 ? 1 : 0; }

// 16-byte image loads through a buffer descriptor: an offset past its size reads zeros, so pixels
// outside the image cost a select instead of a branch around each load.  The window starts at pixel
// row y0 of a 32-channel image (rows before the image are only ever given the outside offset), and its
// bytes stay below 2^31 up to kMaxWidth.  WIDE: for wider images, plain 64-bit addresses, the first
// pixel's where there is none (1000000 x 16, forward and adjoint: 38 ms; with an output per lane on the
// vector units instead of these kernels 3.7 s).
constexpr int kMaxWidth = 900000;

template <bool WIDE>
struct Window {
  const float4* img;
  int W, y0;
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ Window(const float* img, int W, int y0, int rows)
      : img(reinterpret_cast<const float4*>(img)), W(W), y0(y0) {
    if (!WIDE)
      rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(img + (int64_t)y0 * W * 32), 0, rows * W * 128, 0x00027000);
  }
  // piece q (16 bytes) of pixel (x, y0 + row), at `offset` from the window's start
  __device__ __forceinline__ float4 load(bool inside, int offset, int row, int x, int q) const {
    if (WIDE) {
      const float4 v = img[inside ? ((int64_t)(y0 + row) * W + x) * 8 + q : 0];
      return inside ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, inside ? offset : -1, 0, 0));
  }
};

struct ConvArgs {
  const float* in;      // [H*W][32]
  float* out;           // [H*W][32]
  const float* w;       // [co_n][ci_n][3][3] (OIHW)
  int ci_n, co_n;       // channels of w
  int transpose;        // 0: out[co] = sum w[co][ci][t] in[p + t][ci]; 1: input gradient
  const float* bias;    // [co_n] or null
  const float* addend;  // [H*W][32] or null, added before the activation
  uint32_t* bits_out;       // [H*W] or null: bit c of a pixel = out[c] > 0
  const uint32_t* mask;     // [H*W] or null: out = v where the channel's bit is set, else 0
  int H, W;
};

// B operand element: the weight taking input channel `cin` of the convolution's input to its
// output channel `cout` at tap (ky, kx); zero outside the weight's channels (a select, not a branch
// around each load).
__device__ __forceinline__ float conv_w(const ConvArgs& a, int cin, int cout, int ky, int kx) {
  // input gradient: the input holds gradients of the layer's outputs (co), the output its inputs (ci)
  const int co = a.transpose ? cin : cout, ci = a.transpose ? cout : cin;
  const int tap = a.transpose ? 8 - (3 * ky + kx) : 3 * ky + kx;
  const bool ok = co < a.co_n && ci < a.ci_n;
  const float w = a.w[ok ? (co * a.ci_n + ci) * 9 + tap : 0];
  return ok ? w : 0.f;
}

constexpr int kFrag = 9 * 16 * 64;           // A fragments of one convolution: [tap][quad][lane][4]
constexpr int kSplitFrag = 9 * 2 * 3 * 64;   // A fragments (16 bytes) of one split convolution:
                                             // [tap][channel half][part][lane]
constexpr int kConvs = 5;                    // convolutions of the network

struct ConvWeights {
  const float* w[kConvs];
  int ci_n[kConvs];
};

// The A operands of every MFMA of k_conv3x3 in lane order (quad: output half x four of the eight
// contraction steps); all five convolutions in one launch (blockIdx.y).
__global__ void k_conv_frag(ConvWeights cw, float* __restrict__ frag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kFrag) return;
  const ConvArgs a{nullptr, nullptr, cw.w[blockIdx.y], cw.ci_n[blockIdx.y], kCC, 0};
  const int lane = (i >> 2) & 63, q = (i >> 8) & 3, tap = i >> 10;
  const int h = q >> 1, s = 4 * (q & 1) + (i & 3);
  frag[blockIdx.y * kFrag + i] = conv_w(a, 8 * (lane >> 4) + s, 16 * h + (lane & 15), tap / 3, tap % 3);
}

// The split A operands (flipped, transposed weights) of every MFMA of k_conv3x3_bwd in lane
// order, all five input-gradient convolutions in one launch (blockIdx.y).
__global__ void k_conv_split_frag(ConvWeights cw, uint4* __restrict__ frag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 9 * 2 * 64) return;
  const ConvArgs a{nullptr, nullptr, cw.w[blockIdx.y], cw.ci_n[blockIdx.y], kCC, 1};
  const int lane = i & 63, ks = (i >> 6) & 1, tap = i >> 7;
  const int cin = 16 * ks + 8 * (lane >> 5), cout = lane & 31;
  uint32_t part[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t q[3];
    split_pair(conv_w(a, cin + 2 * e, cout, tap / 3, tap % 3), conv_w(a, cin + 2 * e + 1, cout, tap / 3, tap % 3), q);
#pragma unroll
    for (int p = 0; p < 3; ++p) part[p][e] = q[p];
  }
#pragma unroll
  for (int p = 0; p < 3; ++p)
    frag[blockIdx.y * kSplitFrag + ((tap * 2 + ks) * 3 + p) * 64 + lane] =
        make_uint4(part[p][0], part[p][1], part[p][2], part[p][3]);
}

// Forward convolution (FP32 matrix instructions).  Persistent workgroups of eight wavefronts, one
// workgroup per compute unit, compute 16 x 16-pixel tiles from their 18 x 18 input halo in LDS; a
// wavefront owns 2 pixel rows.  In an MFMA the A operand is 16 output channels x 4 input channels (the
// weights, which stay in LDS), the B operand 4 input channels x 16 pixels; the contraction order
// inside a tap is permuted so that a lane's eight B values of a tap are eight consecutive channels of
// one pixel (two 16-byte LDS reads), with A laid out to match, and a lane ends up with runs of four
// output channels of one pixel.  The halo is double-buffered, so that one workgroup's matrix work
// overlaps its own loads: three independent workgroups per compute unit, each staging, contracting
// and storing in step with the others, left the matrix cores idle 43 % of the time.
constexpr int kConvBlock = 512;
constexpr int kHaloVec = kHalo * kHalo * 8;                                  // 16-byte pieces of a halo
constexpr int kHaloPer = (kHaloVec + kConvBlock - 1) / kConvBlock;           // per thread

// A thread's pieces of a halo: their place in the window and in memory, the same for every tile.
template <bool WIDE>
struct HaloLoad {
  int off[kHaloPer], row[kHaloPer], col[kHaloPer];
  __device__ __forceinline__ explicit HaloLoad(int W) {
#pragma unroll
    for (int j = 0; j < kHaloPer; ++j) {
      const int i = threadIdx.x + kConvBlock * j, pix = i >> 3;
      row[j] = i < kHaloVec ? pix / kHalo : (1 << 30);   // past every image
      col[j] = pix % kHalo;
      off[j] = WIDE ? 0 : (pix / kHalo * W + col[j]) * 128 + 16 * (i & 7);
    }
  }
  __device__ __forceinline__ void load(float4 (&v)[kHaloPer], const ConvArgs& a, int tile, int tiles_x) const {
    const int ty0 = tile / tiles_x * kTS - 1, tx0 = tile % tiles_x * kTS - 1;
    const Window<WIDE> win(a.in, a.W, ty0, kHalo);
#pragma unroll
    for (int j = 0; j < kHaloPer; ++j)
      v[j] = win.load((unsigned)(ty0 + row[j]) < (unsigned)a.H && (unsigned)(tx0 + col[j]) < (unsigned)a.W,
                      WIDE ? 0 : off[j] + tx0 * 128, row[j], tx0 + col[j], threadIdx.x & 7);
  }
};

template <bool WIDE>
__global__ __launch_bounds__(kConvBlock) void k_conv3x3(ConvArgs a, const float4* __restrict__ frag) {
  __shared__ float4 s_in[2][kHalo * kHalo * kLS / 4];
  __shared__ float4 s_w[kFrag / 4];
  const int tiles_x = (a.W + kTS - 1) / kTS, n_tiles = tiles_x * ((a.H + kTS - 1) / kTS);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int li = lane & 15, lk = lane >> 4;
  const HaloLoad<WIDE> halo(a.W);
  float4 v[kHaloPer];
  auto load = [&](int tile) { halo.load(v, a, tile < n_tiles ? tile : n_tiles - 1, tiles_x); };
  auto stage = [&](float4* dst) {
#pragma unroll
    for (int j = 0; j < kHaloPer; ++j) {
      const int i = tid + kConvBlock * j;
      if (i < kHaloVec) dst[(i >> 3) * (kLS / 4) + (i & 7)] = v[j];
    }
  };
  load(blockIdx.x);   // the grid has at most n_tiles workgroups
  for (int i = tid; i < kFrag / 4; i += kConvBlock) s_w[i] = frag[i];
  float bias[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) bias[h][e] = a.bias[16 * h + 4 * lk + e];
  stage(s_in[0]);
  load(blockIdx.x + gridDim.x);
  int buf = 0;
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x, buf ^= 1) {
    const int x = tile % tiles_x * kTS + li, y0 = tile / tiles_x * kTS + wave * 2;
    __syncthreads();   // this tile is staged, and the other buffer's readers are done
    float4 add[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t at = y0 + r < a.H && x < a.W ? (int64_t)(y0 + r) * a.W + x : 0;
        add[r][h] = a.addend ? reinterpret_cast<const float4*>(a.addend)[at * 8 + 4 * h + lk]
                             : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    floatx4 acc[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[r][h] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      float wf[2][8], xf[2][8];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 w4 = s_w[(tap * 4 + 2 * r + q) * 64 + lane];
          const float4 x4 = s_in[buf][((wave * 2 + r + tap / 3) * kHalo + li + tap % 3) * (kLS / 4) + 2 * lk + q];
          wf[r][4 * q] = w4.x; wf[r][4 * q + 1] = w4.y; wf[r][4 * q + 2] = w4.z; wf[r][4 * q + 3] = w4.w;
          xf[r][4 * q] = x4.x; xf[r][4 * q + 1] = x4.y; xf[r][4 * q + 2] = x4.z; xf[r][4 * q + 3] = x4.w;
        }
      // four independent accumulators between two MFMAs on the same one
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int h = 0; h < 2; ++h) acc[r][h] = mfma4(wf[h][s], xf[r][s], acc[r][h]);
    }
    // D[i][j]: output channel 16 h + 4 lk + e, pixel column li of the row
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const bool ok = y0 + r < a.H && x < a.W;
      const int64_t at = (int64_t)(y0 + r) * a.W + x;
      uint32_t on = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float ad[4] = {add[r][h].x, add[r][h].y, add[r][h].z, add[r][h].w};
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = acc[r][h][e] + bias[h][e];
          if (a.addend) o[e] += ad[e];
          o[e] = fmaxf(o[e], 0.f);
          on |= o[e] > 0.f ? 1u << (16 * h + e) : 0u;
        }
        if (ok) reinterpret_cast<float4*>(a.out)[at * 8 + 4 * h + lk] = make_float4(o[0], o[1], o[2], o[3]);
      }
      if (a.bits_out) {   // the ReLU's signs for the adjoint: the four lanes of a pixel together
        on <<= 4 * lk;
        on |= (uint32_t)__shfl_xor((int)on, 16, 64);
        on |= (uint32_t)__shfl_xor((int)on, 32, 64);
        if (ok && lk == 0) a.bits_out[at] = on;
      }
    }
    if (tile + (int)gridDim.x < n_tiles) {   // uniform
      stage(s_in[buf ^ 1]);
      load(tile + 2 * gridDim.x);
    }
  }
}

// Input-gradient convolution on the bf16 matrix cores (split operands, see above).  Persistent
// workgroups of eight wavefronts, one workgroup per compute unit, compute 16 x 16-pixel tiles; a
// wavefront owns 2 pixel rows, and an MFMA contracts 16 channels for 32 output channels (operand A,
// the weights) x 32 pixels (operand B).  The split weights (55 KB) stay in LDS: fetched per tap and
// wavefront they cost as many bytes through the L1 as the matrix cores could use, and held in
// registers (216) they leave one wavefront per SIMD and nothing to hide the LDS latency.  The 18 x 18
// halo is split while it is staged (each value once, not once per tap), three 64-byte parts per pixel
// in LDS rows of 13 x 16 bytes (an odd count, so that 16 pixels read by one instruction spread over
// all banks).  The next two tiles' loads are in flight while this one is contracted (one tile's 41 KB
// per compute unit do not keep HBM busy).
constexpr int kSplitRow = 13;     // uint4 per pixel in LDS: 3 parts x 4, and one of padding

// The outputs of the wavefront's tiles that are not finite, once more with the FP32 instructions, from
// global memory (operands as in k_conv3x3).  Masked outputs are zero and stay.  With an output at a time
// on the vector units an upstream gradient without a finite value made 640 x 360 pixels take 39.6 ms
// forward and adjoint, this way and with wgrad_fp32 2.4; with one such value 16.1, now 1.5; with none 0.73.
__device__ __forceinline__ void conv_bwd_fp32(const ConvArgs& a, int n_tiles, int tiles_x) {
  const int wave = threadIdx.x >> 6, li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
  __threadfence_block();   // the stores of the wavefront's other lanes
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int x = tile % tiles_x * kTS + li, y0 = tile / tiles_x * kTS + wave * 2;
    float o[2][2][4];   // as stored: [pixel row][channel half]; zero outside the image
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool ok = y0 + r < a.H && x < a.W;
        const int64_t at = ok ? (int64_t)(y0 + r) * a.W + x : 0;
        const float4 v = reinterpret_cast<const float4*>(a.out)[at * 8 + 4 * h + lk];
        o[r][h][0] = ok ? v.x : 0.f;
        o[r][h][1] = ok ? v.y : 0.f;
        o[r][h][2] = ok ? v.z : 0.f;
        o[r][h][3] = ok ? v.w : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) bad = bad || !finite_f(o[r][h][e]);
      }
    if (!__any(bad)) continue;
    floatx4 acc[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[r][h] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int tap = 0; tap < 9; ++tap) {
      float xf[2][8];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int yy = y0 + r + tap / 3 - 1, xx = x + tap % 3 - 1;
        const bool ok = (unsigned)yy < (unsigned)a.H && (unsigned)xx < (unsigned)a.W;
        const float4* in = reinterpret_cast<const float4*>(a.in) + (ok ? (int64_t)yy * a.W + xx : 0) * 8 + 2 * lk;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float4 v = in[q];
          xf[r][4 * q] = ok ? v.x : 0.f;
          xf[r][4 * q + 1] = ok ? v.y : 0.f;
          xf[r][4 * q + 2] = ok ? v.z : 0.f;
          xf[r][4 * q + 3] = ok ? v.w : 0.f;
        }
      }
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float wf = conv_w(a, 8 * lk + s, 16 * h + li, tap / 3, tap % 3);
#pragma unroll
          for (int r = 0; r < 2; ++r) acc[r][h] = mfma4(wf, xf[r][s], acc[r][h]);
        }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (finite_f(o[r][h][e])) continue;
          const int64_t i = ((int64_t)(y0 + r) * a.W + x) * kCC + 16 * h + 4 * lk + e;
          a.out[i] = a.addend ? acc[r][h][e] + a.addend[i] : acc[r][h][e];
        }
  }
}

template <bool WIDE>
__global__ __launch_bounds__(kConvBlock) void k_conv3x3_bwd(ConvArgs a, const uint4* __restrict__ frag) {
  __shared__ uint4 s_in[kHalo * kHalo * kSplitRow];
  __shared__ uint4 s_w[kSplitFrag];
  const int tiles_x = (a.W + kTS - 1) / kTS, n_tiles = tiles_x * ((a.H + kTS - 1) / kTS);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int px = lane & 15, pr = (lane >> 4) & 1, kh = lane >> 5;
  // after the swap below a lane holds, of the pixels (px, row 0 and 1 of the wavefront), the 16-byte
  // pieces c4 and c4 + 4: 64 contiguous bytes per 4 lanes (16-byte pieces of other lines would cost
  // twice the bytes written to HBM)
  const int c4 = 2 * pr + kh;
  const HaloLoad<WIDE> halo(a.W);
  float4 va[kHaloPer], vb[kHaloPer];   // the next two tiles' halos
  // unconditional: no branch around the loads
  auto load = [&](float4 (&v)[kHaloPer], int tile) { halo.load(v, a, tile < n_tiles ? tile : n_tiles - 1, tiles_x); };
  float bad = 0.f;   // not a number once an output is not finite
  load(va, blockIdx.x);
  load(vb, blockIdx.x + gridDim.x);
  for (int i = tid; i < kSplitFrag; i += kConvBlock) s_w[i] = frag[i];
  auto tile_step = [&](float4 (&v)[kHaloPer], int tile) {
    const int ty0 = tile / tiles_x * kTS, tx0 = tile % tiles_x * kTS;
    __syncthreads();   // the previous tile's readers are done
#pragma unroll
    for (int j = 0; j < kHaloPer; ++j) {
      const int i = tid + kConvBlock * j, pix = i >> 3, q = i & 7;
      if (i >= kHaloVec) break;
      uint32_t lo[3], hi[3];
      split_pair(v[j].x, v[j].y, lo);
      split_pair(v[j].z, v[j].w, hi);
#pragma unroll
      for (int p = 0; p < 3; ++p)
        reinterpret_cast<uint2*>(&s_in[pix * kSplitRow + 4 * p])[q] = make_uint2(lo[p], hi[p]);
    }
    __syncthreads();
    // the epilogue's inputs first (they are needed first), then the halo two tiles ahead
    const int x = tx0 + px, y0 = ty0 + wave * 2;
    float4 add[2][2];
    uint32_t msk[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const bool ok = y0 + r < a.H && x < a.W;
      const int64_t at = ok ? (int64_t)(y0 + r) * a.W + x : 0;
      msk[r] = a.mask ? a.mask[at] : ~0u;
#pragma unroll
      for (int u = 0; u < 2; ++u)
        add[r][u] = a.addend ? reinterpret_cast<const float4*>(a.addend)[at * 8 + c4 + 4 * u]
                             : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    load(v, tile + 2 * gridDim.x);
    floatx16 acc[3];   // by magnitude
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = acc[2][e] = 0.f;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const uint4* src = &s_in[((wave * 2 + pr + tap / 3) * kHalo + px + tap % 3) * kSplitRow + kh];
      uint4 xf[2][3], wf[2][3];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          wf[ks][p] = s_w[((tap * 2 + ks) * 3 + p) * 64 + lane];
          xf[ks][p] = src[4 * p + 2 * ks];
        }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < kProd; ++i)
          acc[prod_acc(i)] = mfma16(wf[ks][prod_a(i)], xf[ks][prod_b(i)], acc[prod_acc(i)]);
    }
    // D: column lane & 31 = pixel, row 8 g + 4 kh + e = channel
    float o[2][2][4];   // [pixel row][piece][channel]
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g0 = (acc[0][8 * u + e] + acc[1][8 * u + e]) + acc[2][8 * u + e];
        const float g1 = (acc[0][8 * u + 4 + e] + acc[1][8 * u + 4 + e]) + acc[2][8 * u + 4 + e];
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(g0), __float_as_uint(g1), false, false);
        o[0][u][e] = __uint_as_float(r[0]);
        o[1][u][e] = __uint_as_float(r[1]);
      }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (y0 + r >= a.H || x >= a.W) continue;
      const int64_t at = (int64_t)(y0 + r) * a.W + x;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float ad[4] = {add[r][u].x, add[r][u].y, add[r][u].z, add[r][u].w};
        const uint32_t m = msk[r] >> (4 * c4 + 16 * u);
        float w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t keep = (uint32_t)((int32_t)(m << (31 - e)) >> 31);   // all ones where the bit is set
          w[e] = __uint_as_float(__float_as_uint(SPLAT_FMA(o[r][u][e], kSplitBack, ad[e])) & keep);
          bad = SPLAT_FMA(w[e], 0.f, bad);
        }
        reinterpret_cast<float4*>(a.out)[at * 8 + c4 + 4 * u] = make_float4(w[0], w[1], w[2], w[3]);
      }
    }
  };
  for (int tile = blockIdx.x; tile < n_tiles; tile += 2 * gridDim.x) {
    tile_step(va, tile);
    if (tile + (int)gridDim.x < n_tiles) tile_step(vb, tile + gridDim.x);   // uniform
  }
  if (__any(bad != 0.f)) conv_bwd_fp32(a, n_tiles, tiles_x);
}

// Weight gradient dW[tap][ci][co] = sum_p x[p + tap][ci] dy[p][co] on the bf16 matrix cores (split
// operands, see above): persistent workgroups stage 8-row x 16-column tiles.  An MFMA contracts 16
// pixels (2 columns x 8 rows) for 32 input x 32 output channels, so a lane needs 8 rows of one
// channel: the staging transposes, a thread reading a column of 8 rows x 4 channels and writing each
// channel's rows as 16 bytes.  A tap's column offset is then another 16-byte slot, and its row
// offset a funnel shift of the ten staged rows (registers), so each x fragment serves three taps.
// Twelve wavefronts, three per SIMD: three column offsets x four quarters of the columns, three
// 32 x 32 blocks each.  The tile is double-buffered: the next one's loads are in flight while this one
// is contracted, and are split into the other buffer before the one barrier per tile.  The quarters
// are added at the end, and a second kernel adds the workgroups' partial sums in a fixed order.
constexpr int kWgradBlock = 768;
constexpr int kXCol = 19;   // uint4 slots of a channel's 18 halo columns (odd: spreads over banks)
constexpr int kDyCol = 17;  // the same for its 16 columns

struct WgradSmem {
  uint4 x[3][kCC][kXCol];        // rows 0-7 of the ten halo rows, two per word
  uint32_t x_tail[3][kCC][kXCol];  // rows 8, 9
  uint4 dy[3][kCC][kDyCol];
};

// splits NR rows of four channels; put(part, channel, words) stores a channel's rows, two per word
template <int NR, typename Put>
__device__ __forceinline__ void split_rows(const float4 (&v)[NR], float scale, Put put) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t w[3][NR / 2];
#pragma unroll
    for (int h = 0; h < NR / 2; ++h) {
      const float4 u0 = v[2 * h], u1 = v[2 * h + 1];
      uint32_t q[3];
      split_pair(c == 0 ? u0.x : c == 1 ? u0.y : c == 2 ? u0.z : u0.w,
                 c == 0 ? u1.x : c == 1 ? u1.y : c == 2 ? u1.z : u1.w, q, scale);
#pragma unroll
      for (int p = 0; p < 3; ++p) w[p][h] = q[p];
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) put(p, c, w[p]);
  }
}

// The workgroup's partial sums that are not finite, once more with the FP32 instructions, from global
// memory: a block of 16 input x 16 output channels of a tap is contracted over four pixels at a time, three
// blocks to a wavefront.  A tap's pixels outside the image add nothing, whatever the other operand.
__device__ __forceinline__ void wgrad_fp32(const float* __restrict__ x, const float* __restrict__ dy, int H, int W,
                                           float* __restrict__ dst) {
  const int tiles_x = (W + kTS - 1) / kTS, tiles_y = (H + kWTH - 1) / kWTH;
  const int li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
  constexpr int kBlocks = 36 / (kWgradBlock / 64);
  for (int b = 0; b < kBlocks; ++b) {
    const int blk = (int)(threadIdx.x >> 6) * kBlocks + b, tap = blk >> 2;
    const int ci0 = 16 * ((blk >> 1) & 1), co0 = 16 * (blk & 1);
    floatx4 acc{0.f, 0.f, 0.f, 0.f};
    for (int tile = blockIdx.x; tile < tiles_x * tiles_y; tile += gridDim.x)
      for (int y = 0; y < kWTH; ++y) {
        const int yy = tile / tiles_x * kWTH + y, ys = yy + tap / 3 - 1;
        if (yy >= H || ys < 0 || ys >= H) continue;   // uniform
#pragma unroll
        for (int c = 0; c < kTS; c += 4) {
          const int xx = tile % tiles_x * kTS + c + lk, xs = xx + tap % 3 - 1;
          const bool ok = xx < W && xs >= 0 && xs < W;
          const float xv = x[((int64_t)ys * W + (ok ? xs : 0)) * kCC + ci0 + li];
          const float dv = dy[((int64_t)yy * W + (ok ? xx : 0)) * kCC + co0 + li];
          acc = mfma4(ok ? xv : 0.f, ok ? dv : 0.f, acc);
        }
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = (tap * kCC + ci0 + 4 * lk + e) * kCC + co0 + li;
      if (!finite_f(dst[i])) dst[i] = acc[e];
    }
  }
}

template <bool WIDE>
__global__ __launch_bounds__(kWgradBlock)
void k_conv3x3_wgrad(const float* __restrict__ x, const float* __restrict__ dy, int H, int W, float* __restrict__ partial) {
  __shared__ union {
    WgradSmem t[2];
    float red[9 * kCC * kCC];
    float b[16 * 8][2][4];
  } sm;
  __shared__ int s_bad;   // a sum is not finite
  const int tiles_x = (W + kTS - 1) / kTS, tiles_y = (H + kWTH - 1) / kWTH;
  const int n_tiles = tiles_x * tiles_y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int ch = lane & 31, kh = lane >> 5;
  const int kx = wave % 3, quarter = wave / 3;
  float* dst = partial + (int64_t)blockIdx.x * kWOut;
  floatx16 acc[3];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[m][e] = 0.f;
  float accb[4] = {0.f, 0.f, 0.f, 0.f};
  // the odd workgroups contract -dy and negate their sums: the instruction's rounding bias cancels (an
  // image of one tile has none of them and needs none: 16 x 8 pixels err by 2.0e-7 to 3.5e-7 over the
  // blocks' weights, where the FP32 instructions err by 3.9e-7 to 4.8e-7)
  const float sign = (blockIdx.x & 1) ? -1.f : 1.f;
  // staging tasks of (column, four channels, four rows): threads 0-255 the 16 dy columns, threads
  // 256-543 the 18 x columns (rows 0-7); threads 544-687 rows 8, 9 of the x columns
  const int q = tid & 7;
  const bool is_dy = tid < 256, is_tail = tid >= 544;
  const bool is_dy_wave = __builtin_amdgcn_readfirstlane(tid) < 256;   // the same, as a scalar
  const int part = tid < 544 ? (tid >> 3) & 1 : 2;   // rows 4 part ...
  const int col = is_dy ? tid >> 4 : is_tail ? (tid - 544) >> 3 : (tid - 256) >> 4;
  const int r0 = 4 * part + (is_dy ? 1 : 0);   // from the row above the tile
  const int off = WIDE ? 0 : (r0 * W + (is_dy ? col : col - 1)) * 128 + 16 * q;
  const int rows = tid < 544 ? 4 : tid < 688 ? 2 : 0;
  float4 v[4];
  auto load = [&](int tile) {   // in flight while the previous tile is contracted
    tile = tile < n_tiles ? tile : n_tiles - 1;   // unconditional: no branch around the loads
    const int ty0 = tile / tiles_x * kWTH - 1, tx0 = tile % tiles_x * kTS;
    const int px = tx0 + (is_dy ? col : col - 1);
    const bool in_x = (unsigned)px < (unsigned)W;
    const Window<WIDE> win(is_dy_wave ? dy : x, W, ty0, kWTH + 2);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      v[r] = win.load(in_x && r < rows && (unsigned)(ty0 + r0 + r) < (unsigned)H, WIDE ? 0 : off + (r * W + tx0) * 128,
                      r0 + r, px, q);
  };
  auto stage = [&](WgradSmem& t) {   // splits the loaded values into a buffer
    if (is_dy) {   // uniform over the wavefront
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        accb[0] += v[r].x;
        accb[1] += v[r].y;
        accb[2] += v[r].z;
        accb[3] += v[r].w;
      }
    }
    if (is_tail) {
      if (rows)
        split_rows<2>({v[0], v[1]}, kSplitScale, [&](int p, int c, const uint32_t (&w)[1]) { t.x_tail[p][4 * q + c][col] = w[0]; });
    } else {
      split_rows<4>(v, is_dy ? sign * kSplitScale : kSplitScale, [&](int p, int c, const uint32_t (&w)[2]) {
        uint4* dst = is_dy ? &t.dy[p][4 * q + c][col] : &t.x[p][4 * q + c][col];
        reinterpret_cast<uint2*>(dst)[part] = make_uint2(w[0], w[1]);
      });
    }
  };
  if (tid == 0) s_bad = 0;
  load(blockIdx.x);   // the grid has at most n_tiles workgroups
  stage(sm.t[0]);
  load(blockIdx.x + gridDim.x);
  int buf = 0;
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x, buf ^= 1) {
    __syncthreads();
    const WgradSmem& t = sm.t[buf];
#pragma unroll
    for (int k = 0; k < 2; ++k) {   // the wavefront's two pairs of columns
      const int cx = 4 * quarter + 2 * k + kh;
      uint4 g[3], f[3][3];   // f: [row offset][part]
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        g[p] = t.dy[p][ch][cx];
        const uint4 u = t.x[p][ch][cx + kx];
        const uint32_t w = t.x_tail[p][ch][cx + kx];
        f[0][p] = u;
        f[1][p] = make_uint4(__builtin_amdgcn_alignbit(u.y, u.x, 16), __builtin_amdgcn_alignbit(u.z, u.y, 16),
                             __builtin_amdgcn_alignbit(u.w, u.z, 16), __builtin_amdgcn_alignbit(w, u.w, 16));
        f[2][p] = make_uint4(u.y, u.z, u.w, w);
      }
#pragma unroll
      for (int i = 0; i < kProd; ++i)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) acc[ky] = mfma16(f[ky][prod_a(i)], g[prod_b(i)], acc[ky]);
    }
    // the other buffer was last read before this iteration's barrier
    if (tile + (int)gridDim.x < n_tiles) {   // uniform
      stage(sm.t[buf ^ 1]);
      load(tile + 2 * gridDim.x);
    }
  }
  for (int w = 0; w < 4; ++w) {   // the column quarters, in order
    __syncthreads();
    if (quarter == w) {
#pragma unroll
      for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int i = ((3 * m + kx) * kCC + 8 * (e >> 2) + 4 * kh + (e & 3)) * kCC + ch;
          sm.red[i] = w == 0 ? acc[m][e] : sm.red[i] + acc[m][e];
        }
    }
  }
  __syncthreads();
  float bad = 0.f;   // not a number once a sum is not finite
  for (int i = tid; i < 9 * kCC * kCC; i += kWgradBlock) {
    const float s = sm.red[i] * (sign * kSplitBack);
    bad = SPLAT_FMA(s, 0.f, bad);
    dst[i] = s;
  }
  if (bad != 0.f) s_bad = 1;
  __syncthreads();   // all of dst is stored
  if (is_dy) {
#pragma unroll
    for (int c = 0; c < 4; ++c) sm.b[col * 8 + q][part][c] = accb[c];
  }
  __syncthreads();
  if (tid < kCC) {   // channel 4 q + c: the 16 dy columns in order
    float s = 0.f;
    for (int c = 0; c < 16; ++c) s += sm.b[c * 8 + (tid >> 2)][0][tid & 3] + sm.b[c * 8 + (tid >> 2)][1][tid & 3];
    dst[9 * kCC * kCC + tid] = s;
  }
  if (s_bad) wgrad_fp32(x, dy, H, W, dst);
}

// dW (OIHW, +=) and db (+=) of one convolution from the column sums of the partials
struct ConvGradStore {
  float* dw;
  float* db;
  int ci_n, co_n;
  __device__ void operator()(int o, float s) const {
    if (o < 9 * kCC * kCC) {
      const int tap = o / (kCC * kCC), ci = (o / kCC) % kCC, co = o % kCC;
      if (dw && ci < ci_n && co < co_n) dw[(co * ci_n + ci) * 9 + tap] += s;
    } else {
      const int co = o - 9 * kCC * kCC;
      if (db && co < co_n) db[co] += s;
    }
  }
};

struct CnnGeo {
  float R[9];         // world -> camera rotation
  float fx, fy, cx, cy;
  int W, H;
};

// x = [F, d, e, 0...] per pixel; eight lanes per pixel, lane q writing channels 4q .. 4q + 3, so
// that a wavefront reads and writes contiguous rows (vec: 16-byte feature rows, C and Df multiples
// of 4)
__global__ __launch_bounds__(256) void k_cnn_input(const float* __restrict__ feat, int C, int Df, int E,
                                                   const float* __restrict__ embed, CnnGeo g, int vec,
                                                   float* __restrict__ x0) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t p = t >> 3;
  const int k0 = 4 * (int)(t & 7);
  if (p >= (int64_t)g.W * g.H) return;
  const float* row = feat + p * C;
  float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
  if (vec && k0 + 4 <= Df) {
    out = *reinterpret_cast<const float4*>(row + k0);
  } else if (k0 < Df + 3 + E) {
    const int u = (int)(p % g.W), v = (int)(p / g.W);
    float dc0 = ((float)u + 0.5f - g.cx) / g.fx, dc1 = ((float)v + 0.5f - g.cy) / g.fy, dc2 = 1.f;
    const float inv = rsqrtf(dc0 * dc0 + dc1 * dc1 + 1.f);
    dc0 *= inv;
    dc1 *= inv;
    dc2 *= inv;
    // world direction R^T d_c
    const float dw0 = g.R[0] * dc0 + g.R[3] * dc1 + g.R[6] * dc2, dw1 = g.R[1] * dc0 + g.R[4] * dc1 + g.R[7] * dc2,
                dw2 = g.R[2] * dc0 + g.R[5] * dc1 + g.R[8] * dc2;
    float o4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + j;
      o4[j] = k < Df            ? row[k]
              : k == Df         ? dw0
              : k == Df + 1     ? dw1
              : k == Df + 2     ? dw2
              : k < Df + 3 + E  ? embed[k - Df - 3]
                                : 0.f;
    }
    out = make_float4(o4[0], o4[1], o4[2], o4[3]);
  }
  reinterpret_cast<float4*>(x0 + p * kCC)[t & 7] = out;
}

// the stem's input gradient: d_feat += dx[0:Df]; per-workgroup sums of dx[Df+3 : Df+3+E] (embedding)
// vec: the host found d_feat 16-byte aligned and C, Df multiples of 4 (16-byte rows)
__global__ __launch_bounds__(256) void k_cnn_input_bwd(const float* __restrict__ dx0, int64_t n, int C, int Df, int E,
                                                        int vec, float* __restrict__ d_feat,
                                                        float* __restrict__ partial_e) {
  __shared__ float s_e[256][9];
  __shared__ float s_p[8][9];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float e[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) e[k] = 0.f;
  if (p < n) {
    const float* src = dx0 + p * kCC;
    float v[kCC];
#pragma unroll
    for (int q = 0; q < 8; ++q) {   // every load issued before any store
      const float4 x = reinterpret_cast<const float4*>(src)[q];
      v[4 * q] = x.x;
      v[4 * q + 1] = x.y;
      v[4 * q + 2] = x.z;
      v[4 * q + 3] = x.w;
    }
    if (d_feat) {
      float* row = d_feat + p * C;
      if (vec) {   // uniform: 16-byte rows
        float4 old[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (4 * q < Df) old[q] = reinterpret_cast<const float4*>(row)[q];
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (4 * q < Df)
            reinterpret_cast<float4*>(row)[q] =
                make_float4(old[q].x + v[4 * q], old[q].y + v[4 * q + 1], old[q].z + v[4 * q + 2], old[q].w + v[4 * q + 3]);
      } else {
        float old[kCC];
#pragma unroll
        for (int k = 0; k < kCC; ++k) old[k] = k < Df ? row[k] : 0.f;
#pragma unroll
        for (int k = 0; k < kCC; ++k)
          if (k < Df) row[k] = old[k] + v[k];
      }
    }
    // the embedding's channels Df + 3 .. Df + 3 + E - 1, picked from the registers already loaded
#pragma unroll
    for (int k = 0; k < kCC; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j < E && k == Df + 3 + j) e[j] = v[k];
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) s_e[threadIdx.x][k] = e[k];
  __syncthreads();
  if (threadIdx.x < 64) {   // 8 slices of 32 rows per embedding entry, then the 8 slices in order
    const int k = threadIdx.x & 7, part = threadIdx.x >> 3;
    float s = 0.f;
    for (int t = 32 * part; t < 32 * part + 32; ++t) s += s_e[t][k];
    s_p[part][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    float s = 0.f;
    for (int part = 0; part < 8; ++part) s += s_p[part][threadIdx.x];
    partial_e[(int64_t)blockIdx.x * 8 + threadIdx.x] = s;
  }
}

struct HeadW {
  float w[6][kCC];
  float b[6];
};

__device__ __forceinline__ void stage_head(HeadW& Hw, const float* w_out, const float* b_out) {
  for (int i = threadIdx.x; i < 6 * kCC; i += blockDim.x) Hw.w[i / kCC][i % kCC] = w_out[i];
  if (threadIdx.x < 6) Hw.b[threadIdx.x] = b_out[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_cnn_head(const float* __restrict__ h2, const float* __restrict__ feat, int C,
                                                   const float* __restrict__ w_out, const float* __restrict__ b_out,
                                                   int64_t n, float* __restrict__ image) {
  __shared__ HeadW Hw;
  stage_head(Hw, w_out, b_out);
  __syncthreads();
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  float z[6];
#pragma unroll
  for (int o = 0; o < 6; ++o) z[o] = Hw.b[o];
  const float4* hp = reinterpret_cast<const float4*>(h2 + p * kCC);
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float4 h = hp[q];
#pragma unroll
    for (int o = 0; o < 6; ++o) {
      z[o] = fmaf(Hw.w[o][4 * q], h.x, z[o]);
      z[o] = fmaf(Hw.w[o][4 * q + 1], h.y, z[o]);
      z[o] = fmaf(Hw.w[o][4 * q + 2], h.z, z[o]);
      z[o] = fmaf(Hw.w[o][4 * q + 3], h.w, z[o]);
    }
  }
  const float* f = feat + p * C;
#pragma unroll
  for (int c = 0; c < 3; ++c) image[p * 3 + c] = fmaf(z[c], f[c], z[3 + c]);
}

// head adjoint: dI -> dz -> d_feat (colour part), dpre2 = (W_out^T dz) * [h2 > 0]; dW_out, db_out
// as per-workgroup contractions over the workgroup's pixels (partials, summed later)
__global__ __launch_bounds__(kCnnBlock) void k_cnn_head_bwd(const float* __restrict__ h2, const float* __restrict__ feat,
                                                            int C, const float* __restrict__ w_out,
                                                            const float* __restrict__ b_out, int64_t n,
                                                            const float* __restrict__ d_image, float* __restrict__ d_feat,
                                                            float* __restrict__ dpre2, float* __restrict__ partial) {
  __shared__ HeadW Hw;
  __shared__ float s_h[kCnnBlock][kCC + 1];
  __shared__ float s_dz[kCnnBlock][6];
  stage_head(Hw, w_out, b_out);
  constexpr int NPT = (kHeadOut + kCnnBlock - 1) / kCnnBlock;
  float acc[NPT];
#pragma unroll
  for (int i = 0; i < NPT; ++i) acc[i] = 0.f;
  const int t = threadIdx.x;
  for (int64_t base = (int64_t)blockIdx.x * kCnnBlock; base < n; base += (int64_t)gridDim.x * kCnnBlock) {
    __syncthreads();
    const int64_t p = base + t;
    if (p < n) {
      float h[kCC];
      const float4* hp = reinterpret_cast<const float4*>(h2 + p * kCC);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float4 v = hp[q];
        h[4 * q] = v.x;
        h[4 * q + 1] = v.y;
        h[4 * q + 2] = v.z;
        h[4 * q + 3] = v.w;
      }
      float z[3];
#pragma unroll
      for (int o = 0; o < 3; ++o) {
        float s = Hw.b[o];
#pragma unroll
        for (int c = 0; c < kCC; ++c) s = fmaf(Hw.w[o][c], h[c], s);
        z[o] = s;   // M
      }
      const float* f = feat + p * C;
      float dz[6];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float di = d_image[p * 3 + c];
        dz[c] = di * f[c];      // dL/dM
        dz[3 + c] = di;         // dL/db
        if (d_feat) d_feat[p * C + c] += di * z[c];
      }
      float4* gp = reinterpret_cast<float4*>(dpre2 + p * kCC);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float g4[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int c = 4 * q + m;
          float s = 0.f;
#pragma unroll
          for (int o = 0; o < 6; ++o) s = fmaf(Hw.w[o][c], dz[o], s);
          g4[m] = h[c] > 0.f ? s : 0.f;
        }
        gp[q] = make_float4(g4[0], g4[1], g4[2], g4[3]);
      }
#pragma unroll
      for (int c = 0; c < kCC; ++c) s_h[t][c] = h[c];
#pragma unroll
      for (int o = 0; o < 6; ++o) s_dz[t][o] = dz[o];
    } else {
#pragma unroll
      for (int c = 0; c < kCC; ++c) s_h[t][c] = 0.f;
#pragma unroll
      for (int o = 0; o < 6; ++o) s_dz[t][o] = 0.f;
    }
    __syncthreads();
    const int rows = (n - base) < kCnnBlock ? (int)(n - base) : kCnnBlock;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int o = t + i * kCnnBlock;
      if (o >= kHeadOut) break;
      float s = 0.f;
      if (o < 6 * kCC) {
        const int oo = o / kCC, c = o % kCC;
        for (int q = 0; q < rows; ++q) s = fmaf(s_dz[q][oo], s_h[q][c], s);
      } else {
        const int oo = o - 6 * kCC;
        for (int q = 0; q < rows; ++q) s += s_dz[q][oo];
      }
      acc[i] += s;
    }
  }
#pragma unroll
  for (int i = 0; i < NPT; ++i) {
    const int o = t + i * kCnnBlock;
    if (o < kHeadOut) partial[(int64_t)blockIdx.x * kHeadOut + o] = acc[i];
  }
}

// ---- workspace --------------------------------------------------------------------------------
struct CnnWs {
  float* act[6];   // x0, h0, r1, h1, r2, h2
  float* g[3];     // gradient buffers
  uint32_t* bits[4];   // the signs of act[1 .. 4], a bit per channel
  float* frag;     // A fragments of the five forward convolutions
  uint4* sfrag;    // split A fragments of the five input-gradient convolutions
  float* partial;  // partial sums
  size_t bytes;
};

inline int wgrad_blocks(int W, int H) {
  const int tiles = ((W + kTS - 1) / kTS) * ((H + kWTH - 1) / kWTH);
  return tiles < 256 ? tiles : 256;   // one workgroup per compute unit
}
inline int head_blocks(int64_t n) {
  const int64_t b = (n + kCnnBlock - 1) / kCnnBlock;
  return (int)(b < 1024 ? b : 1024);
}
inline int64_t input_bwd_blocks(int64_t n) { return (n + 255) / 256; }

// base == nullptr: sizes only (every pointer stays null; no arithmetic on the null base)
inline CnnWs carve_cnn(void* base, int W, int H) {
  CnnWs w;
  const int64_t n = (int64_t)W * H;
  const size_t act = ((size_t)n * kCC * sizeof(float) + 255) / 256 * 256;
  size_t off = 0;
  char* b = (char*)base;
  auto at = [&](size_t o) { return b ? (float*)(b + o) : nullptr; };
  for (int i = 0; i < 6; ++i, off += act) w.act[i] = at(off);
  for (int i = 0; i < 3; ++i, off += act) w.g[i] = at(off);
  for (int i = 0; i < 4; ++i, off += ((size_t)n * 4 + 255) / 256 * 256) w.bits[i] = (uint32_t*)at(off);
  w.frag = at(off);
  off += (size_t)kConvs * kFrag * sizeof(float);
  w.sfrag = (uint4*)at(off);
  off += (size_t)kConvs * kSplitFrag * sizeof(uint4);
  size_t part = (size_t)wgrad_blocks(W, H) * kWOut;
  const size_t hp = (size_t)head_blocks(n) * kHeadOut;
  const size_t ep = (size_t)input_bwd_blocks(n) * 8;
  part = part > hp ? part : hp;
  part = part > ep ? part : ep;
  w.partial = at(off);
  off += (part * sizeof(float) + 255) / 256 * 256;
  w.bytes = off;
  return w;
}

static bool cnn_ok(const SplatCamera* cam, const SplatCameraCNN* m) {
  if (!cam || !m || cam->width <= 0 || cam->height <= 0) return false;
  if (m->n_feat < 3 || m->n_embed < 0 || m->n_embed > 8 || m->n_feat + 3 + m->n_embed > kCC) return false;
  if (!m->w_in || !m->b_in || !m->w_out || !m->b_out || (m->n_embed > 0 && !m->embed)) return false;
  for (int k = 0; k < 4; ++k)
    if (!m->w_block[k] || !m->b_block[k]) return false;
  return true;
}

static CnnGeo cnn_geo(const SplatCamera* cam) {
  CnnGeo g;
  for (int k = 0; k < 9; ++k) g.R[k] = cam->R[k];
  g.fx = cam->fx;
  g.fy = cam->fy;
  g.cx = cam->cx;
  g.cy = cam->cy;
  g.W = cam->width;
  g.H = cam->height;
  return g;
}

// one persistent workgroup per compute unit
static unsigned conv_grid(int W, int H) {
  const int64_t tiles = (int64_t)((W + kTS - 1) / kTS) * ((H + kTS - 1) / kTS);
  return (unsigned)(tiles < 256 ? tiles : 256);
}

static ConvWeights conv_weights(const SplatCameraCNN* cnn, int cin) {
  ConvWeights cw;
  for (int k = 0; k < kConvs; ++k) {
    cw.w[k] = k == 0 ? cnn->w_in : cnn->w_block[k - 1];
    cw.ci_n[k] = k == 0 ? cin : kCC;
  }
  return cw;
}

// forward convolution k (0: the stem, 1-4: the blocks'), ReLU after the optional addend
static hipError_t conv(int k, const float* in, float* out, const ConvWeights& cw, const float* bias, const float* addend,
                       int W, int H, const CnnWs& w, hipStream_t s) {
  ConvArgs a{in, out, cw.w[k], cw.ci_n[k], kCC, 0, bias, addend, k < 4 ? w.bits[k] : nullptr, nullptr, H, W};
  hipLaunchKernelGGL(W > kMaxWidth ? k_conv3x3<true> : k_conv3x3<false>, dim3(conv_grid(W, H)), dim3(kConvBlock), 0, s,
                     a, (const float4*)(w.frag + (size_t)k * kFrag));
  return hipGetLastError();
}

// its input gradient: (addend + conv^T(in)) where mask > 0
static hipError_t conv_bwd(int k, const float* in, float* out, const ConvWeights& cw, const float* addend,
                           const uint32_t* mask, int W, int H, const CnnWs& w, hipStream_t s) {
  ConvArgs a{in, out, cw.w[k], cw.ci_n[k], kCC, 1, nullptr, addend, nullptr, mask, H, W};
  hipLaunchKernelGGL(W > kMaxWidth ? k_conv3x3_bwd<true> : k_conv3x3_bwd<false>, dim3(conv_grid(W, H)),
                     dim3(kConvBlock), 0, s, a, (const uint4*)(w.sfrag + (size_t)k * kSplitFrag));
  return hipGetLastError();
}

static hipError_t wgrad(const float* x, const float* dy, int ci_n, int co_n, float* dw, float* db, float* partial, int W,
                        int H, hipStream_t s) {
  const int nb = wgrad_blocks(W, H);
  hipLaunchKernelGGL(W > kMaxWidth ? k_conv3x3_wgrad<true> : k_conv3x3_wgrad<false>, dim3((unsigned)nb),
                     dim3(kWgradBlock), 0, s, x, dy, H, W, partial);
  launch_column_sums((const float*)partial, kWOut, nb, kWOut, ConvGradStore{dw, db, ci_n, co_n}, s);
  return hipGetLastError();
}

}  // namespace splat

using namespace splat;

extern "C" {

size_t splat_camera_decode_workspace_bytes(int32_t width, int32_t height) {
  if (width <= 0 || height <= 0) return 0;
  return carve_cnn(nullptr, width, height).bytes;
}

int splat_camera_decode(const SplatCamera* cam, const float* feat, const SplatCameraCNN* cnn, float* image, void* ws,
                        size_t ws_bytes, void* stream) {
  if (!cnn_ok(cam, cnn) || !feat || !image) return SPLAT_ERR_INVALID_ARG;
  const int W = cam->width, H = cam->height;
  const int64_t n = (int64_t)W * H;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < splat_camera_decode_workspace_bytes(W, H)) return SPLAT_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  CnnWs w = carve_cnn(ws, W, H);
  const int C = cam->n_channels > 0 ? cam->n_channels : cnn->n_feat;
  if (cnn->n_feat > C) return SPLAT_ERR_INVALID_ARG;
  const int cin = cnn->n_feat + 3 + cnn->n_embed;
  const int vec = (((uintptr_t)feat & 15) == 0 && ((C | cnn->n_feat) & 3) == 0) ? 1 : 0;
  hipLaunchKernelGGL(k_cnn_input, dim3((unsigned)div_up(8 * n, 256)), dim3(256), 0, s, feat, C, cnn->n_feat,
                     cnn->n_embed, cnn->embed, cnn_geo(cam), vec, w.act[0]);
  const ConvWeights cw = conv_weights(cnn, cin);
  hipLaunchKernelGGL(k_conv_frag, dim3(kFrag / 256, kConvs), dim3(256), 0, s, cw, w.frag);
  hipError_t e = conv(0, w.act[0], w.act[1], cw, cnn->b_in, nullptr, W, H, w, s);
  for (int k = 0; k < 2 && e == hipSuccess; ++k) {
    float* hin = w.act[1 + 2 * k];
    e = conv(1 + 2 * k, hin, w.act[2 + 2 * k], cw, cnn->b_block[2 * k], nullptr, W, H, w, s);
    if (e == hipSuccess)
      e = conv(2 + 2 * k, w.act[2 + 2 * k], w.act[3 + 2 * k], cw, cnn->b_block[2 * k + 1], hin, W, H, w, s);
  }
  if (e != hipSuccess) return SPLAT_ERR_DEVICE;
  hipLaunchKernelGGL(k_cnn_head, dim3((unsigned)div_up(n, 256)), dim3(256), 0, s, (const float*)w.act[5], feat, C,
                     cnn->w_out, cnn->b_out, n, image);
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

int splat_camera_decode_bwd(const SplatCamera* cam, const float* feat, const SplatCameraCNN* cnn, const float* d_image,
                            float* d_feat, const SplatCameraCNNGrads* d_cnn, void* ws, size_t ws_bytes, void* stream) {
  if (!cnn_ok(cam, cnn) || !feat || !d_image || !d_cnn) return SPLAT_ERR_INVALID_ARG;
  const int W = cam->width, H = cam->height;
  const int64_t n = (int64_t)W * H;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < splat_camera_decode_workspace_bytes(W, H)) return SPLAT_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  CnnWs w = carve_cnn(ws, W, H);
  const int C = cam->n_channels > 0 ? cam->n_channels : cnn->n_feat;
  if (cnn->n_feat > C) return SPLAT_ERR_INVALID_ARG;
  const int cin = cnn->n_feat + 3 + cnn->n_embed;
  float *x0 = w.act[0], *h0 = w.act[1], *r1 = w.act[2], *h1 = w.act[3], *r2 = w.act[4], *h2 = w.act[5];
  float *ga = w.g[0], *gb = w.g[1], *gc = w.g[2];
  const ConvWeights cw = conv_weights(cnn, cin);
  hipLaunchKernelGGL(k_conv_split_frag, dim3((9 * 2 * 64 + 255) / 256, kConvs), dim3(256), 0, s, cw, w.sfrag);
  // head: dpre2 -> ga
  const int hb = head_blocks(n);
  hipLaunchKernelGGL(k_cnn_head_bwd, dim3((unsigned)hb), dim3(kCnnBlock), 0, s, (const float*)h2, feat, C, cnn->w_out,
                     cnn->b_out, n, d_image, d_feat, ga, w.partial);
  launch_column_sums((const float*)w.partial, kHeadOut, hb, 6 * kCC, AddTo{d_cnn->w_out}, s);
  launch_column_sums((const float*)(w.partial + 6 * kCC), kHeadOut, hb, 6, AddTo{d_cnn->b_out}, s);
  hipError_t e = hipGetLastError();
  // blocks, last first: dpre_k in `dp`, h_{k-1}, r_k the saved activations
  float* dp = ga;
  float* spare[2] = {gb, gc};
  for (int k = 1; k >= 0 && e == hipSuccess; --k) {
    float* hin = w.act[1 + 2 * k];
    float* r = w.act[2 + 2 * k];
    float* du = spare[0];
    float* dnext = spare[1];
    // conv_k2: its input r_k, output gradient dpre_k
    e = wgrad(r, dp, kCC, kCC, d_cnn->w_block[2 * k + 1], d_cnn->b_block[2 * k + 1], w.partial, W, H, s);
    if (e == hipSuccess)   // du_k = conv_k2^T(dpre_k) * [r_k > 0]
      e = conv_bwd(2 + 2 * k, dp, du, cw, nullptr, w.bits[1 + 2 * k], W, H, w, s);
    if (e == hipSuccess)   // conv_k1: input h_{k-1}, output gradient du_k
      e = wgrad(hin, du, kCC, kCC, d_cnn->w_block[2 * k], d_cnn->b_block[2 * k], w.partial, W, H, s);
    if (e == hipSuccess)   // dpre_{k-1} = (dpre_k + conv_k1^T(du_k)) * [h_{k-1} > 0]
      e = conv_bwd(1 + 2 * k, du, dnext, cw, dp, w.bits[2 * k], W, H, w, s);
    spare[0] = dp;
    spare[1] = du;
    dp = dnext;
  }
  (void)h1;
  (void)r1;
  (void)r2;
  (void)h0;
  // stem: dW_in, db_in; dx0 = conv_in^T(dpre0)
  if (e == hipSuccess) e = wgrad(x0, dp, cin, kCC, d_cnn->w_in, d_cnn->b_in, w.partial, W, H, s);
  float* dx0 = spare[0];
  if (e == hipSuccess) e = conv_bwd(0, dp, dx0, cw, nullptr, nullptr, W, H, w, s);
  if (e != hipSuccess) return SPLAT_ERR_DEVICE;
  const int64_t eb = input_bwd_blocks(n);
  const int vec = (((uintptr_t)d_feat & 15) == 0 && ((C | cnn->n_feat) & 3) == 0) ? 1 : 0;
  hipLaunchKernelGGL(k_cnn_input_bwd, dim3((unsigned)eb), dim3(256), 0, s, (const float*)dx0, n, C, cnn->n_feat,
                     cnn->n_embed, vec, d_feat, w.partial);
  if (cnn->n_embed > 0) launch_column_sums((const float*)w.partial, 8, (int)eb, cnn->n_embed, AddTo{d_cnn->embed}, s);
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

}  // extern "C"
