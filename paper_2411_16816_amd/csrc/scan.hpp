// scan.hpp -- device-wide exclusive scans in two launches (block totals, then a down-sweep that hands
// every element with its prefix to a visitor), for binning and for the relocation of Gaussians.
#pragma once

#include "kernels.hpp"

namespace splat {

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

// What a wavefront scans in place of T: a pair whose first member counts elements (at most 2^15 to a
// block) and whose second stays below 2^47 over a block is one 64-bit sum, the count from bit 48 on.
__device__ __forceinline__ uint32_t scan_pack(uint32_t x) { return x; }
__device__ __forceinline__ int64_t scan_pack(int64_t x) { return x; }
__device__ __forceinline__ int64_t scan_pack(P64 x) { return (int64_t)(((uint64_t)x.a << 48) + (uint64_t)x.b); }
template <typename T>
struct ScanLocal {
  using type = T;
  static __device__ __forceinline__ T unpack(T x) { return x; }
};
template <>
struct ScanLocal<P64> {
  using type = int64_t;
  static __device__ __forceinline__ P64 unpack(int64_t x) {
    const int64_t b = (int64_t)((uint64_t)x << 16) >> 16;
    return P64((x - b) >> 48, b);
  }
};

// x of the lane that a DPP step names, zero where it names none
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_from(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t dpp_from(int64_t x) {
  const uint32_t lo = dpp_from<CTRL, ROWS>((uint32_t)(uint64_t)x);
  const uint32_t hi = dpp_from<CTRL, ROWS>((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ P64 dpp_from(P64 x) {
  return P64(dpp_from<CTRL, ROWS>(x.a), dpp_from<CTRL, ROWS>(x.b));
}

__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
__device__ __forceinline__ int64_t last_lane(int64_t x) {
  return (int64_t)(((uint64_t)last_lane((uint32_t)((uint64_t)x >> 32)) << 32) | last_lane((uint32_t)(uint64_t)x));
}
__device__ __forceinline__ P64 last_lane(P64 x) { return P64(last_lane(x.a), last_lane(x.b)); }

// Inclusive scan across the wavefront (every lane active): shifts by 1, 2, 4 and 8 inside the rows of 16
// lanes, then the last lane of a row added to the rows after it.  All on the vector units: shuffles
// through LDS are a chain of six LDS latencies.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
  x += dpp_from<0x111, 0xf>(x);
  x += dpp_from<0x112, 0xf>(x);
  x += dpp_from<0x114, 0xf>(x);
  x += dpp_from<0x118, 0xf>(x);
  x += dpp_from<0x142, 0xa>(x);
  x += dpp_from<0x143, 0xc>(x);
  return x;
}

// the sum of the WAVES entries of `sums`, and of those before entry w
template <int WAVES, typename T>
__device__ __forceinline__ T sum_before(const T* sums, int w, T& total) {
  T pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const T s = sums[k];
    pre += k < w ? s : (T)0;
    tot += s;
  }
  total = tot;
  return pre;
}

// exclusive scan across a block of WAVES wavefronts; `tmp` holds one entry per wavefront
template <typename T, int WAVES = 4>
__device__ T block_exclusive_scan(T v, T* tmp, T& total) {
  const int w = threadIdx.x >> 6;
  const T x = wave_inclusive_scan(v);
  if ((threadIdx.x & 63) == 63) tmp[w] = x;
  __syncthreads();
  T pre = sum_before<WAVES>(tmp, w, total);
  __syncthreads();
  pre += x;
  return pre - v;
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
// Elements per thread and per block of a scan over T.  Pairs take half as many: the visit of the visible
// records, which follows the scan of its block, is then split over twice the blocks (10.5M records: 112 us
// against 140).
template <typename T>
constexpr int scan_items() { return sizeof(T) > 8 ? kScanItems / 2 : kScanItems; }
template <typename T>
constexpr int scan_tile() { return kScanThreads * scan_items<T>(); }

// Element of a lane's r-th row: wavefront w of a block owns scan_items x 64 consecutive elements of the
// block's tile, row by row.
template <typename T>
__device__ __forceinline__ int64_t scan_element(int r) {
  return (int64_t)blockIdx.x * scan_tile<T>() + (int64_t)((threadIdx.x >> 6) * scan_items<T>() + r) * 64 +
         (threadIdx.x & 63);
}

template <typename T>
__device__ __forceinline__ int64_t scan_last_block(int64_t n_eff) { return n_eff > 0 ? (n_eff - 1) / scan_tile<T>() : 0; }

template <typename T, typename Load>
__global__ __launch_bounds__(256) void k_scan_reduce(Load ld, int64_t n, const int64_t* n_dev, T* __restrict__ part) {
  __shared__ T tmp[4];
  const int64_t n_eff = scan_count(n_dev, n);
  if ((int64_t)blockIdx.x > scan_last_block<T>(n_eff)) {   // uniform: contributes nothing
    if (threadIdx.x == 0) part[blockIdx.x] = (T)0;
    return;
  }
  const int64_t hi = n_eff > 0 ? n_eff - 1 : 0;
  T acc = 0;
  // indices clamped into [0, n_eff): every load is issued unconditionally, back to back
#pragma unroll
  for (int r = 0; r < scan_items<T>(); ++r) {
    const int64_t i = scan_element<T>(r);
    const T x = ld(i < hi ? i : hi);
    acc += i < n_eff ? x : (T)0;
  }
  acc = wave_inclusive_scan(acc);
  if ((threadIdx.x & 63) == 63) tmp[threadIdx.x >> 6] = acc;
  __syncthreads();
  T total;
  sum_before<4>(tmp, 0, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Up to this many blocks every down-sweep block sums the block totals before it itself (one
// launch fewer); beyond it a single block scans the totals first.
constexpr int64_t kScanFusedBlocks = 4096;

// single block: exclusive scan of part[0..nb) in place, part[nb] = total.  4096 entries at a time, each
// wavefront four consecutive rows of 64; a chain of load latencies (8160 sums in two steps 4.7 us, in 32
// steps of 256 entries 17).
constexpr int kPartialWaves = 16, kPartialRows = 4;

template <typename T>
__global__ __launch_bounds__(64 * kPartialWaves) void k_scan_partials(T* __restrict__ part, int64_t nb) {
  __shared__ T tmp[kPartialWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  T carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kPartialWaves * kPartialRows * 64) {
    const int64_t i0 = b0 + w * kPartialRows * 64 + lane;
    T v[kPartialRows], pre[kPartialRows];
#pragma unroll
    for (int r = 0; r < kPartialRows; ++r) {
      const int64_t i = i0 + r * 64;
      const T x = part[i < nb ? i : nb - 1];
      v[r] = i < nb ? x : (T)0;
    }
    T run = 0;
#pragma unroll
    for (int r = 0; r < kPartialRows; ++r) {
      const T x = wave_inclusive_scan(v[r]);
      pre[r] = run + x - v[r];
      run += last_lane(x);
    }
    if (lane == 0) tmp[w] = run;
    __syncthreads();
    T total;
    const T before = carry + sum_before<kPartialWaves>(tmp, w, total);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPartialRows; ++r)
      if (i0 + r * 64 < nb) part[i0 + r * 64] = before + pre[r];
    carry += total;
  }
  if (threadIdx.x == 0) part[nb] = carry;
}

// Per-element work of a scan, in two phases so that the loads of several elements are issued
// before any of their stores: In load(i, value) reads what element i needs (kBatch rows' at a time), then
// operator()(i, prefix, value, in) writes; finish(total) runs once with the grand total.
struct NoVisit {
  static constexpr int kBatch = 4;
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
  static constexpr int kBatch = 4;
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
  using L = typename ScanLocal<T>::type;
  __shared__ L s_sum[4];
  __shared__ T s_before[4];
  const int64_t n_eff = scan_count(n_dev, n);
  const int64_t last = scan_last_block<T>(n_eff);
  if ((int64_t)blockIdx.x > last) return;   // uniform
  const int64_t hi = n_eff > 0 ? n_eff - 1 : 0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  L xs[scan_items<T>()], pre[scan_items<T>()];   // the loads are issued first and stay in flight while the blocks
                               // before this one are summed
#pragma unroll
  for (int r = 0; r < scan_items<T>(); ++r) {
    const int64_t i = scan_element<T>(r);
    const T x = ld(i < hi ? i : hi);
    xs[r] = i < n_eff ? scan_pack(x) : (L)0;
  }
  T pb = 0;
  if (fused) {
    const int64_t nb_before = blockIdx.x;
    constexpr int kFlight = 4;
    for (int64_t i0 = threadIdx.x; i0 < nb_before; i0 += kFlight * kScanThreads) {
      T p[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int64_t i = i0 + u * kScanThreads;
        p[u] = part[i < nb_before ? i : 0];
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) pb += i0 + u * kScanThreads < nb_before ? p[u] : (T)0;
    }
    pb = wave_inclusive_scan(pb);
  }
  L run = 0;
#pragma unroll
  for (int r = 0; r < scan_items<T>(); ++r) {
    const L x = wave_inclusive_scan(xs[r]);
    pre[r] = run + x - xs[r];
    run += last_lane(x);
  }
  if (lane == 63) {
    s_sum[w] = run;
    s_before[w] = pb;
  }
  __syncthreads();
  L local;
  const L wave_base = sum_before<4>(s_sum, w, local);
  const T total = ScanLocal<T>::unpack(local);
  T before;
  if (fused) sum_before<4>(s_before, 0, before);
  else before = part[blockIdx.x];
  if ((int64_t)blockIdx.x == last && threadIdx.x == 0) {
    if (fused) part[nb] = before + total;
    vis.finish(before + total);
  }
  constexpr int kBatch = Visit::kBatch;
#pragma unroll
  for (int r0 = 0; r0 < scan_items<T>(); r0 += kBatch) {
    typename Visit::In in[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int64_t i = scan_element<T>(r0 + u);
      if (i < n_eff) in[u] = vis.load(i, ScanLocal<T>::unpack(xs[r0 + u]));
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int64_t i = scan_element<T>(r0 + u);
      if (i < n_eff) {
        const T p = before + ScanLocal<T>::unpack(wave_base + pre[r0 + u]);
        if (out) out[i] = p;
        vis(i, p, ScanLocal<T>::unpack(xs[r0 + u]), in[u]);
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
  if (!fused) hipLaunchKernelGGL((k_scan_partials<T>), dim3(1), dim3(64 * kPartialWaves), 0, s, part, nb);
  hipLaunchKernelGGL((k_scan_down<T, Load, Visit>), dim3((unsigned)nb), dim3(kScanThreads), 0, s, ld, n, n_dev, part,
                     nb, fused, out, vis);
  return hipGetLastError();
}

}  // namespace splat
