// decoders.hip -- the lidar decoder of the rendered features (SplatAD, arXiv 2411.16816, Sec. 3.3;
// the training-details appendix gives its size: two layers, hidden width 32).
//
// Per lidar ray, the rendered feature row F (C channels) and the ray's unit direction
// d = (cos el cos az, cos el sin az, sin el) in the sensor frame are decoded:
//   h = ReLU(W1 [F, d] + b1),  z = W2 h + b2,  intensity = sigmoid(z0),  drop = sigmoid(z1).
//
// Both directions run the first layer on the matrix cores (v_mfma_f32_32x32x2_f32: 32 hidden units x
// 32 rays, two of the inputs [F, d] per instruction; FP32 in, FP32 accumulate).  A lane holds one ray's
// inputs, and one v_permlane32_swap of two of them makes the operands of both of the wavefront's 32-ray
// blocks.  A result register then holds one hidden unit of the lane's ray, sixteen per lane, so that the
// ReLU and the output layer stay in registers, their two halves added by another swap.  Rows are loaded
// one step ahead.  On the vector units the first layer took 416 of about 600 instructions per ray at
// C = 8 and bounded the forward: 16.8M rays 288 -> 239 us (40 bytes in and 8 out per ray: 164 us at
// 4.9 TB/s); with 3 channels, which the vector form ran as 8 with selects on the weights, 1M rays
// 58 -> 19 us, and with 16, 4M rays 136 -> 80 us.
//
// Adjoint: one wavefront per workgroup, persistent over chunks of 64 rays.  The wavefront recomputes
// the forward, sums the output layer's gradients (W2, b2) per lane in registers, and stages x and the
// pre-activation gradient dpre in LDS, from which the matrix cores contract over the hidden units
// (dL/dF, 16x16x4) and over the rays ([dW1 | db1] = sum of dpre^T [x, 1], 16x16x4, accumulating
// across chunks).  At the end every workgroup stores its partial sums (the W2 / b2 sums reduced over
// its lanes), and a second kernel adds them in workgroup order: deterministic, no atomics.  It is
// bound by the vector and matrix instructions, which share their multipliers in FP32: with 3 channels
// 1M rays 152 -> 71 us, with 16 4M rays 396 -> 276 us against the vector form; aligned rows of 8
// channels keep the vector form (k_lidar_decode_bwd_valu).
#include "kernels.hpp"
#include "reduce.hpp"
#include "wave_ops.hpp"

namespace splat {

constexpr int kDecHidden = 32;
constexpr int kDecBlock = 128;
constexpr int kDecMaxC = 32;

inline int dec_outputs(int C) { return kDecHidden * (C + 3) + kDecHidden + 2 * kDecHidden + 2; }

__device__ __forceinline__ float sigmoid_f(float z) { return 1.f / (1.f + expf(-z)); }

// One ray's inputs as loaded: a chunk's loads are issued while the chunk before it is computed.
// VEC: C == CM and the rows are 16-byte aligned (whole-row vector loads)
template <int CM, bool VEC>
struct DecRay {
  float F[CM], az, el;
  __device__ __forceinline__ void load(const float* feat, const float* az_, const float* el_, int64_t r, int C) {
    if (VEC) {
      const float4* row = reinterpret_cast<const float4*>(feat + r * CM);
#pragma unroll
      for (int q = 0; q < CM / 4; ++q) {
        const float4 v = row[q];
        F[4 * q] = v.x;
        F[4 * q + 1] = v.y;
        F[4 * q + 2] = v.z;
        F[4 * q + 3] = v.w;
      }
    } else {
      const float* row = feat + r * C;
#pragma unroll
      for (int k = 0; k < CM; ++k) F[k] = k < C ? row[k] : 0.f;
    }
    az = az_[r];
    el = el_[r];
  }
  // [F, d, 1]
  __device__ __forceinline__ void inputs(float (&x)[CM + 4]) const {
    float sa, ca, se, ce;
    sincosf(az, &sa, &ca);
    sincosf(el, &se, &ce);
#pragma unroll
    for (int k = 0; k < CM; ++k) x[k] = F[k];
    x[CM] = ce * ca;
    x[CM + 1] = ce * sa;
    x[CM + 2] = se;
    x[CM + 3] = 1.f;
  }
};

typedef float decx4 __attribute__((ext_vector_type(4)));
typedef float decx16 __attribute__((ext_vector_type(16)));

// W1's column of input k of [F (CM, zero beyond the C features), d]; zero where there is none
template <int CM>
__device__ __forceinline__ float dec_w1(const SplatLidarMLP& m, int C, int j, int k) {
  if (k < CM) return k < C ? m.w1[j * (C + 3) + k] : 0.f;
  return k < CM + 3 ? m.w1[j * (C + 3) + C + (k - CM)] : 0.f;
}

// hidden unit of result register r of a 32x32 block
__device__ __forceinline__ int dec_hidden(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// {lanes 0-31 of a, lanes 0-31 of b} and {lanes 32-63 of a, lanes 32-63 of b}
__device__ __forceinline__ void half_swap(uint32_t a, uint32_t b, uint32_t& lo, uint32_t& hi) {
  auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  lo = r[0];
  hi = r[1];
}
__device__ __forceinline__ void half_swap(float a, float b, float& lo, float& hi) {
  uint32_t l, h;
  half_swap(__float_as_uint(a), __float_as_uint(b), l, h);
  lo = __uint_as_float(l);
  hi = __uint_as_float(h);
}

// max(x, 0) in one instruction (NaN gives 0, as fmaxf)
__device__ __forceinline__ float relu(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, INFINITY); }

// The output layer's weights of a lane's hidden units.
struct DecOutput {
  float w2[2][16];
  float b2[2];
  __device__ __forceinline__ DecOutput(const SplatLidarMLP& m, int half) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      w2[0][r] = m.w2[dec_hidden(r, half)];
      w2[1][r] = m.w2[kDecHidden + dec_hidden(r, half)];
    }
    b2[0] = m.b2[0];
    b2[1] = m.b2[1];
  }
  // z: the outputs of the lane's own ray, from its 16 pre-activations of each block
  __device__ __forceinline__ void outputs(const decx16 (&pre)[2], float (&z)[2]) const {
    float p[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float h = relu(pre[b][r]);
        p[b][0] = fmaf(w2[0][r], h, p[b][0]);
        p[b][1] = fmaf(w2[1][r], h, p[b][1]);
      }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      float lo, hi;
      half_swap(p[0][c], p[1][c], lo, hi);   // the halves of block 0 on lanes 0-31, of block 1 on 32-63
      z[c] = (lo + hi) + b2[c];
    }
  }
};

// The first layer: pre[b] = the lane's 16 pre-activations of block b (ray 32 b + (lane & 31)).  The FP32
// matrix instructions add their products in order, like a chain of fmaf (b1 first, then the features
// and the direction), so that the ReLU decisions of both directions are those of such a chain.
template <int CM>
struct DecFirst {
  float a1[CM / 2 + 2], b1[16];
  __device__ __forceinline__ DecFirst(const SplatLidarMLP& m, int C, int lane) {
    const int half = lane >> 5;
#pragma unroll
    for (int s = 0; s < CM / 2 + 2; ++s) a1[s] = dec_w1<CM>(m, C, lane & 31, 2 * s + half);
#pragma unroll
    for (int r = 0; r < 16; ++r) b1[r] = m.b1[dec_hidden(r, half)];
  }
  __device__ __forceinline__ void operator()(const float (&x)[CM + 4], decx16 (&pre)[2]) const {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) pre[b][r] = b1[r];
#pragma unroll
    for (int s = 0; s < CM / 2 + 2; ++s) {
      float x0, x1;
      half_swap(x[2 * s], 2 * s + 1 < CM + 3 ? x[2 * s + 1] : 0.f, x0, x1);
      pre[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s], x0, pre[0], 0, 0, 0);
      pre[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s], x1, pre[1], 0, 0, 0);
    }
  }
};

// One wavefront takes 64 rays at a time; lanes past the end work on the last ray and store nothing.
template <int CM, bool VEC>
__global__ __launch_bounds__(kDecBlock) void k_lidar_decode(int64_t n, const float* __restrict__ feat,
                                                            const float* __restrict__ az, const float* __restrict__ el,
                                                            SplatLidarMLP m, float* __restrict__ intensity,
                                                            float* __restrict__ drop) {
  const int C = VEC ? CM : m.n_feat, lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t r0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63);
  DecRay<CM, VEC> ray;
  ray.load(feat, az, el, r0 + lane < n ? r0 + lane : n - 1, C);
  const DecFirst<CM> first(m, C, lane);
  const DecOutput w(m, lane >> 5);
  for (; r0 < n; r0 += stride) {   // uniform over the wavefront
    float x[CM + 4], z[2];
    ray.inputs(x);
    const int64_t next = r0 + stride + lane;
    ray.load(feat, az, el, next < n ? next : n - 1, C);
    decx16 pre[2];
    first(x, pre);
    w.outputs(pre, z);
    if (r0 + lane < n) {
      if (intensity) intensity[r0 + lane] = sigmoid_f(z[0]);
      if (drop) drop[r0 + lane] = sigmoid_f(z[1]);
    }
  }
}

// N-tiles of 16 columns of the x rows: [F (CM), d (3), 1] padded with zeros
template <int CM>
constexpr int dec_xtiles() { return (CM + 4 + 15) / 16; }

constexpr int kDecChunk = 64;   // rays per chunk of the adjoint: one per lane of its wavefront

// One chunk's operands of the contractions.  Row strides: x odd (a lane writes its own row); dpre 4
// modulo 64 banks, so that the reads of both contractions (16 hidden units x 4 rays, 16 rays x 4 hidden
// units four apart) meet every bank once.
template <int CM>
struct DecRows {
  float x[kDecChunk][16 * dec_xtiles<CM>() + 1];   // [F (zero beyond C), d, 1, 0...]
  float dpre[kDecHidden][kDecChunk + 4];
};

// A workgroup's sums to its row of partial sums: W1 and b1 (the blocks of the contraction over its rays)
template <int CM>
__device__ __forceinline__ void dec_store_first(float* __restrict__ dst, int C, int lane,
                                                const decx4 (&acc)[2 * dec_xtiles<CM>()]) {
  constexpr int NXT = dec_xtiles<CM>(), NT = 2 * NXT;
  const int XC = C + 3, nw1 = kDecHidden * XC, li = lane & 15, lk = lane >> 4;
  // D[i][j] of a block: lane j + 16 (i / 4), element i % 4
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    const int jh = b / NXT, nt = b % NXT;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = 16 * jh + 4 * lk + e, col = 16 * nt + li;
      const float v = acc[b][e];
      if (col < C) dst[j * XC + col] = v;                                     // feature columns of W1
      else if (col >= CM && col < CM + 3) dst[j * XC + C + (col - CM)] = v;   // direction columns
      else if (col == CM + 3) dst[nw1 + j] = v;                               // b1
    }
  }
}

// ... and b2 (a sum per lane)
__device__ __forceinline__ void dec_store_b2(float* __restrict__ dst, int C, int lane, float gb0, float gb1) {
  const int nw2 = kDecHidden * (C + 3) + 3 * kDecHidden;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    gb0 += __shfl_xor(gb0, o, 64);
    gb1 += __shfl_xor(gb1, o, 64);
  }
  if (lane == 0) {
    dst[nw2] = gb0;
    dst[nw2 + 1] = gb1;
  }
}

template <int CM, bool VEC>
__global__ __launch_bounds__(kDecChunk) __attribute__((amdgpu_waves_per_eu(2)))
void k_lidar_decode_bwd(int64_t n, const float* __restrict__ feat, const float* __restrict__ az,
                        const float* __restrict__ el, SplatLidarMLP m, const float* __restrict__ d_int,
                        const float* __restrict__ d_drop, float* __restrict__ d_feat, float* __restrict__ partial,
                        int n_out) {
  constexpr int NXT = dec_xtiles<CM>();
  constexpr int NT = 2 * NXT;            // [dW1 | db1] blocks: hidden rows 16 (b / NXT) .., x columns 16 (b % NXT) ..
  constexpr int NF = (CM + 15) / 16;     // tiles of 16 features of dL/dF
  __shared__ DecRows<CM> S;
  const int C = VEC ? CM : m.n_feat, XC = C + 3;
  const int nb1 = kDecHidden * XC + kDecHidden;
  const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4, half = lane >> 5;
  const DecFirst<CM> first(m, C, lane);
  const DecOutput w(m, half);
  float aF[NF][8];   // W1^T operands of dL/dF: feature 16 t + li, hidden unit 16 (s >> 2) + 4 lk + (s & 3)
#pragma unroll
  for (int t = 0; t < NF; ++t)
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 16 * t + li;
      aF[t][s] = k < C ? m.w1[(16 * (s >> 2) + 4 * lk + (s & 3)) * XC + k] : 0.f;
    }
  decx4 acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = decx4{0.f, 0.f, 0.f, 0.f};
  float gw2[32];   // this lane's sums of dz_c h over its rays: output c, register r at 16 c + r
#pragma unroll
  for (int i = 0; i < 32; ++i) gw2[i] = 0.f;
  float gb0 = 0.f, gb1 = 0.f;
  const int64_t step = (int64_t)gridDim.x * kDecChunk;
  DecRay<CM, VEC> ray;
  float ui, ud;
  // Lanes past the end work on the last ray with zero upstream gradients: they add nothing, and
  // every load of a chunk is unconditional (issued together, not one branch at a time).
  auto load = [&](int64_t base) {
    const int64_t r = base + lane, rr = r < n ? r : n - 1;
    ray.load(feat, az, el, rr, C);
    ui = d_int ? d_int[rr] : 0.f;
    ud = d_drop ? d_drop[rr] : 0.f;
    ui = r < n ? ui : 0.f;
    ud = r < n ? ud : 0.f;
  };
  load((int64_t)blockIdx.x * kDecChunk);
  for (int64_t base = (int64_t)blockIdx.x * kDecChunk; base < n; base += step) {
    float x[CM + 4];
    ray.inputs(x);
    const float di = ui, dd = ud;
    load(base + step);
    __syncthreads();   // the previous chunk's rows are consumed
#pragma unroll
    for (int k = 0; k < 16 * NXT; ++k) S.x[lane][k] = k < CM + 4 ? x[k < CM + 4 ? k : 0] : 0.f;
    decx16 pre[2];
    float z[2];
    first(x, pre);
    w.outputs(pre, z);
    const float s0 = sigmoid_f(z[0]), s1 = sigmoid_f(z[1]);
    const float g0 = di * s0 * (1.f - s0);
    const float g1 = dd * s1 * (1.f - s1);
    gb0 += g0;
    gb1 += g1;
    float gb[2][2];   // [output][block]: the upstream gradients of the lane's ray in each block
    half_swap(g0, g0, gb[0][0], gb[0][1]);
    half_swap(g1, g1, gb[1][0], gb[1][1]);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float p = pre[b][q], h = relu(p);
        gw2[q] = fmaf(gb[0][b], h, gw2[q]);
        gw2[16 + q] = fmaf(gb[1][b], h, gw2[16 + q]);
        const float u = fmaf(w.w2[0][q], gb[0][b], w.w2[1][q] * gb[1][b]);
        S.dpre[dec_hidden(q, half)][32 * b + (lane & 31)] = u * (p > 0.f ? 1.f : 0.f);   // ReLU'
      }
    __syncthreads();
    // dL/dF = W1^T dpre: 16 rays at a time; a lane ends up with features 4 lk .. 4 lk + 3 of ray li
    if (d_feat) {
#pragma unroll 1
      for (int rb = 0; rb < kDecChunk / 16; ++rb) {
        const int64_t ray = base + 16 * rb + li;
        decx4 o[NF];
#pragma unroll
        for (int t = 0; t < NF; ++t) o[t] = decx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const float bv = S.dpre[16 * (s >> 2) + 4 * lk + (s & 3)][16 * rb + li];
#pragma unroll
          for (int t = 0; t < NF; ++t) o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(aF[t][s], bv, o[t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < NF; ++t) {
          const int k0 = 16 * t + 4 * lk;
          if (ray >= n || k0 >= C) continue;
          float* row = d_feat + ray * C + k0;
          if (VEC) {
            float4 v = *reinterpret_cast<const float4*>(row);
            v.x += o[t][0];
            v.y += o[t][1];
            v.z += o[t][2];
            v.w += o[t][3];
            *reinterpret_cast<float4*>(row) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (k0 + e < C) row[e] += o[t][e];
          }
        }
      }
    }
    // [dW1 | db1] += dpre^T [x, 1] over the chunk's 64 rays: K in 16 steps of 4 rows (4 s + lk)
    // (the blocks' accumulation chains are independent: interleaved, their latencies overlap)
#pragma unroll 4
    for (int s4 = 0; s4 < kDecChunk / 4; ++s4) {
      const int q = 4 * s4 + lk;
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        const int jh = b / NXT, nt = b % NXT;
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.dpre[16 * jh + li][q], S.x[q][16 * nt + li], acc[b], 0, 0, 0);
      }
    }
  }
  float* dst = partial + (int64_t)blockIdx.x * n_out;
  dec_store_first<CM>(dst, C, lane, acc);
  // W2: the sums over the 32 lanes of each half (the two halves hold different hidden units)
#pragma unroll
  for (int i = 0; i < 32; ++i) {
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) gw2[i] += __shfl_xor(gw2[i], o, 64);
    if ((lane & 31) == 0) dst[nb1 + kDecHidden * (i >> 4) + dec_hidden(i & 15, half)] = gw2[i];
  }
  dec_store_b2(dst, C, lane, gb0, gb1);
}

// ---- the adjoint at 8 channels on the vector units --------------------------------------------
// With 8 channels in 16-byte rows the first layer is short enough that one lane per ray, with the
// weights in scalar registers (every lane uses the same weight: scalar loads through the constant
// address space, a row's loads merged), needs no more instructions than the matrix form spends around
// its products, at 3 wavefronts per SIMD instead of 2: 16.8M rays 0.82 to 0.83 ms against 0.84 to 0.85 (262144
// rays, two latency chains: 33.4 us against 32.9).
typedef const __attribute__((address_space(4))) float* ConstF;

__device__ __forceinline__ float hidden_pre_s(ConstF w1, ConstF b1, int j, const float (&F)[8], const float (&d)[3]) {
  constexpr int CM = 8;
  const int row = j * (CM + 3);
  float p = b1[j];
#pragma unroll
  for (int k = 0; k < CM; ++k) p = fmaf(w1[row + k], F[k], p);
  p = fmaf(w1[row + CM], d[0], p);
  p = fmaf(w1[row + CM + 1], d[1], p);
  return fmaf(w1[row + CM + 2], d[2], p);
}

// One chunk's rows for the first-layer contraction (+1 column: conflict-free row writes)
struct DecLaneRows {
  float x[kDecChunk][16 * dec_xtiles<8>() + 1];     // [F, d, 1, 0...]
  float dpre[kDecChunk][kDecHidden + 1];            // pre-activation, then its gradient
};

// at least 3 wavefronts per SIMD: the output-layer sums take 66 registers per lane
__global__ __launch_bounds__(kDecChunk) __attribute__((amdgpu_waves_per_eu(3)))
void k_lidar_decode_bwd_valu(int64_t n, const float* __restrict__ feat, const float* __restrict__ az,
                             const float* __restrict__ el, SplatLidarMLP m, const float* __restrict__ d_int,
                             const float* __restrict__ d_drop, float* __restrict__ d_feat,
                             float* __restrict__ partial, int n_out) {
  constexpr int CM = 8;
  constexpr int NXT = dec_xtiles<CM>();
  constexpr int NT = 2 * NXT;   // [dW1 | db1] blocks: hidden rows 16 (b / NXT) .., x columns 16 (b % NXT) ..
  constexpr int UNR = 4;        // hidden units per unrolled step
  __shared__ DecLaneRows S;
  const ConstF w1 = (ConstF)m.w1, b1 = (ConstF)m.b1, w2 = (ConstF)m.w2, b2 = (ConstF)m.b2;
  constexpr int C = CM, XC = C + 3, nb1 = kDecHidden * XC + kDecHidden;
  decx4 acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = decx4{0.f, 0.f, 0.f, 0.f};
  float gw2[2 * kDecHidden];   // this lane's sums of dz_c h_j over its rays: W2[c][j] at c * 32 + j
#pragma unroll
  for (int i = 0; i < 2 * kDecHidden; ++i) gw2[i] = 0.f;
  float gb0 = 0.f, gb1 = 0.f;
  const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4;
  const int64_t step = (int64_t)gridDim.x * kDecChunk;
  for (int64_t base = (int64_t)blockIdx.x * kDecChunk; base < n; base += step) {
    __syncthreads();   // the previous chunk's rows are consumed
    // Lanes past the end work on the last ray with zero upstream gradients: they add nothing,
    // and every load of the chunk is unconditional (issued together, not one branch at a time).
    const int64_t r = base + lane;
    const bool valid = r < n;
    const int64_t rr = valid ? r : n - 1;
    float F[CM], d[3];
    const float4* frow = reinterpret_cast<const float4*>(feat + rr * CM);
#pragma unroll
    for (int q = 0; q < CM / 4; ++q) {
      const float4 v = frow[q];
      F[4 * q] = v.x;
      F[4 * q + 1] = v.y;
      F[4 * q + 2] = v.z;
      F[4 * q + 3] = v.w;
    }
    const float a_r = az[rr], e_r = el[rr];
    float di = d_int ? d_int[rr] : 0.f, dd = d_drop ? d_drop[rr] : 0.f;
    di = valid ? di : 0.f;
    dd = valid ? dd : 0.f;
    {
      float sa, ca, se, ce;
      sincosf(a_r, &sa, &ca);
      sincosf(e_r, &se, &ce);
      d[0] = ce * ca;
      d[1] = ce * sa;
      d[2] = se;
    }
#pragma unroll
    for (int k = 0; k < CM; ++k) S.x[lane][k] = F[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) S.x[lane][CM + k] = d[k];   // x = [F, d]: direction after the features
#pragma unroll
    for (int k = CM + 3; k < 16 * NXT; ++k) S.x[lane][k] = k == CM + 3 ? 1.f : 0.f;   // ones: the bias
    // forward again; the pre-activations wait in this lane's own LDS row
    float z0 = b2[0], z1 = b2[1];
#pragma unroll UNR
    for (int j = 0; j < kDecHidden; ++j) {
      const float p = hidden_pre_s(w1, b1, j, F, d);
      S.dpre[lane][j] = p;
      const float h = fmaxf(p, 0.f);
      z0 = fmaf(w2[j], h, z0);
      z1 = fmaf(w2[kDecHidden + j], h, z1);
    }
    const float s0 = sigmoid_f(z0), s1 = sigmoid_f(z1);
    const float g0 = di * s0 * (1.f - s0);
    const float g1 = dd * s1 * (1.f - s1);
    gb0 += g0;
    gb1 += g1;
    // output layer: sums of dz_c h_j (a pass of its own, fully unrolled: the sums stay in
    // registers, while the first layer's loop below is only partly unrolled)
#pragma unroll
    for (int j = 0; j < kDecHidden; ++j) {
      const float h = fmaxf(S.dpre[lane][j], 0.f);
      gw2[j] = fmaf(g0, h, gw2[j]);
      gw2[kDecHidden + j] = fmaf(g1, h, gw2[kDecHidden + j]);
    }
    float dF[CM];
#pragma unroll
    for (int k = 0; k < CM; ++k) dF[k] = 0.f;
#pragma unroll UNR
    for (int j = 0; j < kDecHidden; ++j) {
      const float p = S.dpre[lane][j];
      const float t = fmaf(w2[j], g0, w2[kDecHidden + j] * g1);
      const float dp = t * (p > 0.f ? 1.f : 0.f);   // ReLU'
      S.dpre[lane][j] = dp;
      const int row = j * XC;
#pragma unroll
      for (int k = 0; k < CM; ++k) dF[k] = fmaf(w1[row + k], dp, dF[k]);
    }
    if (d_feat && valid) {
      float4* row = reinterpret_cast<float4*>(d_feat + r * CM);
#pragma unroll
      for (int q = 0; q < CM / 4; ++q) {
        float4 v = row[q];
        v.x += dF[4 * q];
        v.y += dF[4 * q + 1];
        v.z += dF[4 * q + 2];
        v.w += dF[4 * q + 3];
        row[q] = v;
      }
    }
    __syncthreads();
    // [dW1 | db1] += dpre^T [x, 1] over the chunk's 64 rays: K in 16 steps of 4 rows (4 s + lk)
    // (the blocks' accumulation chains are independent: interleaved, their latencies overlap)
#pragma unroll 4
    for (int s4 = 0; s4 < kDecChunk / 4; ++s4) {
      const int q = 4 * s4 + lk;
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        const int jh = b / NXT, nt = b % NXT;
        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.dpre[q][16 * jh + li], S.x[q][16 * nt + li], acc[b], 0, 0, 0);
      }
    }
  }
  float* dst = partial + (int64_t)blockIdx.x * n_out;
  dec_store_first<CM>(dst, C, lane, acc);
  // W2: one value per lane after the wavefront's reduce-scatter
  bool store;
  const int slot = scatter_slot<2 * kDecHidden>(lane, store);
  const float w2sum = wave_reduce_scatter<2 * kDecHidden>(gw2);
  if (store) dst[nb1 + slot] = w2sum;
  dec_store_b2(dst, C, lane, gb0, gb1);
}

// weight gradients (+=) from the column sums of the workgroups' partials
struct MlpGradStore {
  SplatLidarMLPGrads g;
  int C;
  __device__ void operator()(int o, float s) const {
    const int nw1 = kDecHidden * (C + 3), nb1 = nw1 + kDecHidden, nw2 = nb1 + 2 * kDecHidden;
    if (o < nw1) { if (g.w1) g.w1[o] += s; }
    else if (o < nb1) { if (g.b1) g.b1[o - nw1] += s; }
    else if (o < nw2) { if (g.w2) g.w2[o - nb1] += s; }
    else if (g.b2) g.b2[o - nw2] += s;
  }
};

// Workgroups of the adjoint: at most kDecBwdMaxGrid (which sizes the partial sums), at most one
// per chunk of rays, and no more than the device holds at once (the grid is persistent).
constexpr int kDecBwdMaxGrid = 8192;

static int bwd_blocks(int64_t n) {
  int64_t b = div_up(n, kDecChunk);
  return (int)(b < kDecBwdMaxGrid ? (b < 1 ? 1 : b) : kDecBwdMaxGrid);
}

// returns the grid: the number of partial-sum rows written
template <typename Kernel>
static int launch_decode_bwd(Kernel kernel, int64_t n, const float* feat, const float* az, const float* el, const SplatLidarMLP& m,
                              const float* d_int, const float* d_drop, float* d_feat, float* partial, int n_out,
                              hipStream_t s) {
  int dev = 0, n_cu = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kDecChunk, 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  const int64_t resident = (int64_t)n_cu * per_cu;
  const int b = bwd_blocks(n), grid = (int)(b < resident ? b : resident);
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kDecChunk), 0, s, n, feat, az, el, m,
                     d_int, d_drop, d_feat, partial, n_out);
  return grid;
}

static bool mlp_ok(const SplatLidarMLP* m) {
  return m && m->n_feat >= 0 && m->n_feat <= kDecMaxC && m->w1 && m->b1 && m->w2 && m->b2;
}

}  // namespace splat

using namespace splat;

extern "C" {

int splat_lidar_decode(int64_t n_rays, const float* feat, const float* ray_az, const float* ray_el,
                       const SplatLidarMLP* mlp, float* intensity, float* drop_prob, void* stream) {
  if (n_rays < 0 || !mlp_ok(mlp)) return SPLAT_ERR_INVALID_ARG;
  if (n_rays == 0 || (!intensity && !drop_prob)) return SPLAT_OK;
  if ((mlp->n_feat > 0 && !feat) || !ray_az || !ray_el) return SPLAT_ERR_INVALID_ARG;
  int64_t blocks = div_up(n_rays, kDecBlock);
  if (blocks > 4096) blocks = 4096;
  const int C = mlp->n_feat;
  const int vec = ((C == 8 || C == 16 || C == 32) && ((uintptr_t)feat & 15) == 0) ? 1 : 0;
  const dim3 g((unsigned)blocks), blk(kDecBlock);
  hipStream_t s = (hipStream_t)stream;
#define DEC_LAUNCH(CM, VEC) \
  hipLaunchKernelGGL((k_lidar_decode<CM, VEC>), g, blk, 0, s, n_rays, feat, ray_az, ray_el, *mlp, intensity, drop_prob)
  if (vec && C == 8) DEC_LAUNCH(8, true);
  else if (vec && C == 16) DEC_LAUNCH(16, true);
  else if (vec && C == 32) DEC_LAUNCH(32, true);
  else if (C <= 8) DEC_LAUNCH(8, false);
  else if (C <= 16) DEC_LAUNCH(16, false);
  else DEC_LAUNCH(32, false);
#undef DEC_LAUNCH
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

size_t splat_lidar_decode_workspace_bytes(int64_t n_rays, int32_t n_feat) {
  if (n_rays < 0 || n_feat < 0 || n_feat > kDecMaxC) return 0;
  return (size_t)bwd_blocks(n_rays) * dec_outputs(n_feat) * sizeof(float);
}

int splat_lidar_decode_bwd(int64_t n_rays, const float* feat, const float* ray_az, const float* ray_el,
                           const SplatLidarMLP* mlp, const float* d_intensity, const float* d_drop_prob,
                           float* d_feat, const SplatLidarMLPGrads* d_mlp, void* ws, size_t ws_bytes, void* stream) {
  if (n_rays < 0 || !mlp_ok(mlp) || !d_mlp) return SPLAT_ERR_INVALID_ARG;
  if (n_rays == 0) return SPLAT_OK;
  if ((mlp->n_feat > 0 && !feat) || !ray_az || !ray_el) return SPLAT_ERR_INVALID_ARG;
  if (!ws || ws_bytes < splat_lidar_decode_workspace_bytes(n_rays, mlp->n_feat)) return SPLAT_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  const int C = mlp->n_feat, n_out = dec_outputs(C);
  float* partial = (float*)ws;
  // vec: the feature rows (and the gradient rows) are whole 16-byte aligned rows of the kernel's width
  const int cm = C <= 8 ? 8 : C <= 16 ? 16 : 32;
  const int vec = (C == cm && ((uintptr_t)feat & 15) == 0 && ((uintptr_t)d_feat & 15) == 0) ? 1 : 0;
  const float *di = d_intensity, *dd = d_drop_prob;
  const SplatLidarMLP& w = *mlp;
  int nb;
#define DEC_LAUNCH(...) \
  nb = launch_decode_bwd(__VA_ARGS__, n_rays, feat, ray_az, ray_el, w, di, dd, d_feat, partial, n_out, s)
  if (vec && C == 8) DEC_LAUNCH(k_lidar_decode_bwd_valu);
  else if (vec && C == 16) DEC_LAUNCH((k_lidar_decode_bwd<16, true>));
  else if (vec && C == 32) DEC_LAUNCH((k_lidar_decode_bwd<32, true>));
  else if (C <= 8) DEC_LAUNCH((k_lidar_decode_bwd<8, false>));
  else if (C <= 16) DEC_LAUNCH((k_lidar_decode_bwd<16, false>));
  else DEC_LAUNCH((k_lidar_decode_bwd<32, false>));
#undef DEC_LAUNCH
  launch_column_sums((const float*)partial, n_out, nb, n_out, MlpGradStore{*d_mlp, mlp->n_feat}, s);
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

}  // extern "C"
