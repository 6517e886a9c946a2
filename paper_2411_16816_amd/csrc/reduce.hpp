// reduce.hpp -- fixed-order column sums of per-workgroup partial sums (the weight gradients of
// the decoders are contractions over rays or pixels; each workgroup leaves one row of partials).
#pragma once

#include <hip/hip_runtime.h>

namespace splat {

constexpr int kColWaves = 16, kColWidth = 16;
constexpr int kColRows = kColWaves * (64 / kColWidth);   // rows that a workgroup reads at a time
constexpr int kColFlight = 8;

// Column sums of partial [n_rows, stride] for columns [0, n_cols): a 1024-thread workgroup takes 16
// consecutive columns (about one cache line of a row) and 64 rows at a time; a lane keeps 8 running
// sums with as many loads in flight, which are then added across the wavefront's 4 rows and over the
// 16 wavefronts.  It is a chain of load latencies, so it is split to shorten the chain: the sums of
// 3072 rows of 450 columns take 8 us; with 64 columns to a workgroup (8 workgroups) and 4 loads in
// flight they took 18, with 16 in flight 14 to 19.  The order of every addition is fixed, so the result
// does not depend on timing.  `st(col, sum)` stores it.
template <class Store>
__global__ __launch_bounds__(1024) void k_column_sums(const float* __restrict__ partial, int64_t stride, int n_rows,
                                                      int n_cols, Store st) {
  __shared__ float s[kColWaves][kColWidth];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane % kColWidth;
  const int o = blockIdx.x * kColWidth + col;
  const int r0 = w * (64 / kColWidth) + lane / kColWidth;
  float a[kColFlight];
#pragma unroll
  for (int u = 0; u < kColFlight; ++u) a[u] = 0.f;
  if (o < n_cols) {
    // rows past the end re-read the last one and add nothing
    for (int r = r0; r < n_rows; r += kColFlight * kColRows) {
      float v[kColFlight];
#pragma unroll
      for (int u = 0; u < kColFlight; ++u) {
        const int q = r + u * kColRows;
        v[u] = partial[(int64_t)(q < n_rows ? q : n_rows - 1) * stride + o];
      }
#pragma unroll
      for (int u = 0; u < kColFlight; ++u) a[u] += r + u * kColRows < n_rows ? v[u] : 0.f;
    }
  }
#pragma unroll
  for (int d = kColFlight / 2; d >= 1; d >>= 1)
#pragma unroll
    for (int u = 0; u < d; ++u) a[u] += a[u + d];
#pragma unroll
  for (int d = 32; d >= kColWidth; d >>= 1) a[0] += __shfl_xor(a[0], d);
  if (lane < kColWidth) s[w][col] = a[0];
  __syncthreads();
  if (threadIdx.x < kColWidth && o < n_cols) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kColWaves; ++k) t += s[k][col];
    st(o, t);
  }
}

template <class Store>
inline void launch_column_sums(const float* partial, int64_t stride, int n_rows, int n_cols, Store st, hipStream_t s) {
  if (n_cols <= 0) return;
  hipLaunchKernelGGL(k_column_sums<Store>, dim3((unsigned)((n_cols + kColWidth - 1) / kColWidth)),
                     dim3(64 * kColWaves), 0, s, partial, stride, n_rows, n_cols, st);
}

// dst[col] += sum (dst may be null: nothing stored)
struct AddTo {
  float* dst;
  __device__ void operator()(int o, float v) const {
    if (dst) dst[o] += v;
  }
};

}  // namespace splat
