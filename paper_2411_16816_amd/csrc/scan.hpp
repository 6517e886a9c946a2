// scan.hpp -- device-wide exclusive scans in two launches (block totals, then a down-sweep that hands
// every element with its prefix to a visitor), for binning and for the relocation of Gaussians.
#pragma once

#include "kernels.hpp"

namespace splat {

__device__ __forceinline__ int64_t shfl_up_i64(int64_t v, int d) {
  int lo = __shfl_up((int)(uint32_t)(uint64_t)v, d, 64);
  int hi = __shfl_up((int)(uint32_t)((uint64_t)v >> 32), d, 64);
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}
__device__ __forceinline__ uint32_t shfl_up_t(uint32_t v, int d) { return (uint32_t)__shfl_up((int)v, d, 64); }
__device__ __forceinline__ int64_t shfl_up_t(int64_t v, int d) { return shfl_up_i64(v, d); }

// Two int64 counters scanned together (trivially constructible, so it can live in LDS).
struct P64 {
  int64_t a, b;
  P64() = default;
  __device__ P64(int v) : a(v), b(v) {}
  __device__ P64(int64_t x, int64_t y) : a(x), b(y) {}
  __device__ P64& operator+=(const P64& o) {
    a += o.a;
    b += o.b;
    return *this;
  }
};
__device__ __forceinline__ P64 operator+(P64 x, const P64& y) { return x += y; }
__device__ __forceinline__ P64 operator-(P64 x, const P64& y) { return P64(x.a - y.a, x.b - y.b); }
__device__ __forceinline__ P64 shfl_up_t(P64 v, int d) { return P64(shfl_up_i64(v.a, d), shfl_up_i64(v.b, d)); }

// exclusive scan across a 256-thread block; `tmp` holds 4 entries
template <typename T>
__device__ T block_exclusive_scan(T v, T* tmp, T& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    T y = shfl_up_t(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) tmp[wid] = x;
  __syncthreads();
  T pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    T s = tmp[w];
    pre += (w < wid) ? s : (T)0;
    tot += s;
  }
  total = tot;
  __syncthreads();
  return pre + x - v;
}

// ------------------------------------------------------------------------------------------
// device-wide exclusive scan (reduce, scan of partials, downsweep); Load(i) gives element i
// ------------------------------------------------------------------------------------------
struct LoadI64 {
  const int64_t* p;
  __device__ int64_t operator()(int64_t i) const { return p[i]; }
};

// Elements scanned: the capacity n, or fewer when the count is only known on the device
// (n_dev non-null: min(n, *n_dev)).  Blocks wholly past that count do nothing, except that the
// block holding the last element (block 0 when there is none) closes the scan.
__device__ __forceinline__ int64_t scan_count(const int64_t* n_dev, int64_t n) {
  if (!n_dev) return n;
  const int64_t m = *n_dev;
  return m < 0 ? 0 : (m < n ? m : n);
}
// Elements per thread and per block of a scan over T: 16-byte elements take half as many, so
// that a block's LDS tile stays at 34 KB (four blocks per compute unit).
template <typename T>
constexpr int scan_items() { return sizeof(T) > 8 ? kScanItems / 2 : kScanItems; }
template <typename T>
constexpr int scan_tile() { return kScanThreads * scan_items<T>(); }

template <typename T>
__device__ __forceinline__ int64_t scan_last_block(int64_t n_eff) { return n_eff > 0 ? (n_eff - 1) / scan_tile<T>() : 0; }

template <typename T, typename Load>
__global__ __launch_bounds__(256) void k_scan_reduce(Load ld, int64_t n, const int64_t* n_dev, T* __restrict__ part) {
  __shared__ T tmp[4];
  const int64_t n_eff = scan_count(n_dev, n);
  constexpr int kItems = scan_items<T>();
  const int64_t base = (int64_t)blockIdx.x * scan_tile<T>();   // < n: the grid has div_up(n, tile) blocks
  if ((int64_t)blockIdx.x > scan_last_block<T>(n_eff)) {      // uniform: contributes nothing
    if (threadIdx.x == 0) part[blockIdx.x] = (T)0;
    return;
  }
  const int64_t hi = n_eff > 0 ? n_eff - 1 : 0;
  T acc = 0;
  // indices clamped into [0, n_eff): every load is issued unconditionally, back to back
#pragma unroll 4
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + (int64_t)r * kScanThreads + threadIdx.x;
    const T x = ld(i < hi ? i : hi);
    acc += i < n_eff ? x : (T)0;
  }
  T total;
  block_exclusive_scan<T>(acc, tmp, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Up to this many blocks every down-sweep block sums the block totals before it itself (one
// launch fewer); beyond it a single block scans the totals first.
constexpr int64_t kScanFusedBlocks = 4096;

// single block: exclusive scan of part[0..nb) in place, part[nb] = total
template <typename T>
__global__ __launch_bounds__(256) void k_scan_partials(T* __restrict__ part, int64_t nb) {
  __shared__ T tmp[4];
  T carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 256) {
    int64_t i = b0 + threadIdx.x;
    T v = i < nb ? part[i] : (T)0;
    T total;
    T ex = block_exclusive_scan<T>(v, tmp, total);
    if (i < nb) part[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) part[nb] = carry;
}

// Per-element work of a scan, in two phases so that the loads of several elements are issued
// before any of their stores: In load(i, value) reads what element i needs, then
// operator()(i, prefix, value, in) writes; finish(total) runs once with the grand total.
struct NoVisit {
  struct In {};
  template <typename T>
  __device__ In load(int64_t, T) const { return In{}; }
  template <typename T>
  __device__ void operator()(int64_t, T, T, In) const {}
  template <typename T>
  __device__ void finish(T) const {}
};

// Writes the grand total to *dst (no per-element work).
struct StoreTotal {
  int64_t* dst;
  struct In {};
  template <typename T>
  __device__ In load(int64_t, T) const { return In{}; }
  template <typename T>
  __device__ void operator()(int64_t, T, T, In) const {}
  __device__ void finish(int64_t total) const { *dst = total; }
};

// Block b: exclusive scan of its tile, offset by the total of the blocks before it: with
// `fused`, the sum of the block totals part[0..b) (read by the block itself; the closing block
// writes the grand total to part[nb]), otherwise part[b] as scanned by k_scan_partials.  Every
// element i is handed to the visitor with its prefix and its value; the closing block's first
// thread hands it the grand total (vis.finish).  `out` may be null (visitor only).
template <typename T, typename Load, typename Visit>
__global__ __launch_bounds__(256) void k_scan_down(Load ld, int64_t n, const int64_t* n_dev, T* __restrict__ part,
                                                   int64_t nb, bool fused, T* __restrict__ out, Visit vis) {
  // element li of the tile lives at pad(li) = li + li / 16: a thread's 16 consecutive
  // elements then start 17 apart, which spreads the per-thread pass over the LDS banks
  constexpr int kItems = scan_items<T>();
  constexpr int kTile = scan_tile<T>();
  __shared__ T tile[kTile + kTile / kItems];
  __shared__ T tmp[4];
  auto pad = [](int li) { return li + li / kItems; };
  const int64_t n_eff = scan_count(n_dev, n);
  const int64_t last = scan_last_block<T>(n_eff);
  if ((int64_t)blockIdx.x > last) return;   // uniform
  const int64_t hi = n_eff > 0 ? n_eff - 1 : 0;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  T xs[kItems];   // the tile's loads are issued first and stay in flight while the blocks
                  // before this one are summed
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + (int64_t)r * kScanThreads + threadIdx.x;
    xs[r] = ld(i < hi ? i : hi);
  }
  T before;
  if (fused) {
    T pb = 0;
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) pb += part[i];
    block_exclusive_scan<T>(pb, tmp, before);
  } else {
    before = part[blockIdx.x];
  }
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + (int64_t)r * kScanThreads + threadIdx.x;
    tile[pad(r * kScanThreads + threadIdx.x)] = i < n_eff ? xs[r] : (T)0;
  }
  __syncthreads();
  T loc[kItems];
  T acc = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    loc[k] = acc;
    acc += tile[pad(threadIdx.x * kItems + k)];
  }
  T total;
  T pre = block_exclusive_scan<T>(acc, tmp, total) + before;
  if ((int64_t)blockIdx.x == last && threadIdx.x == 0) {
    if (fused) part[nb] = before + total;
    vis.finish(before + total);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kItems; ++k) tile[pad(threadIdx.x * kItems + k)] = pre + loc[k];
  __syncthreads();
  const T end = before + total;   // exclusive prefix after the block
  constexpr int kBatch = 4;
#pragma unroll
  for (int r0 = 0; r0 < kItems; r0 += kBatch) {
    T p[kBatch], gap[kBatch];
    typename Visit::In in[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int li = (r0 + u) * kScanThreads + threadIdx.x;
      const int64_t i = base + li;
      p[u] = tile[pad(li)];
      gap[u] = (li + 1 < kTile ? tile[pad(li + 1)] : end) - p[u];   // element i's value
      if (i < n_eff) in[u] = vis.load(i, gap[u]);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int64_t i = base + (r0 + u) * kScanThreads + threadIdx.x;
      if (i < n_eff) {
        if (out) out[i] = p[u];
        vis(i, p[u], gap[u], in[u]);
      }
    }
  }
}

// the scan of no elements: total 0
template <typename T, typename Visit>
__global__ void k_scan_empty(T* part, Visit vis) {
  part[0] = (T)0;
  vis.finish((T)0);
}

// exclusive scan of n elements (fewer when n_dev is given, see scan_count) into out[0..n)
// (out may alias the loaded array: each block reads its tile before writing it; out may be
// null); part[nb] receives the total
template <typename T, typename Load, typename Visit = NoVisit>
hipError_t device_scan(Load ld, int64_t n, T* out, T* part, hipStream_t s, Visit vis = Visit(),
                       const int64_t* n_dev = nullptr) {
  int64_t nb = div_up(n, scan_tile<T>());
  if (nb == 0) {
    hipLaunchKernelGGL((k_scan_empty<T, Visit>), dim3(1), dim3(1), 0, s, part, vis);
    return hipGetLastError();
  }
  // one block needs no block totals (the fused down-sweep sums none before block 0)
  if (nb > 1)
    hipLaunchKernelGGL((k_scan_reduce<T, Load>), dim3((unsigned)nb), dim3(kScanThreads), 0, s, ld, n, n_dev, part);
  const bool fused = nb <= kScanFusedBlocks;
  if (!fused) hipLaunchKernelGGL((k_scan_partials<T>), dim3(1), dim3(256), 0, s, part, nb);
  hipLaunchKernelGGL((k_scan_down<T, Load, Visit>), dim3((unsigned)nb), dim3(kScanThreads), 0, s, ld, n, n_dev, part,
                     nb, fused, out, vis);
  return hipGetLastError();
}

}  // namespace splat
