// mcmc.hip -- the MCMC regulariser of the training-details appendix (SplatAD, arXiv 2411.16816;
// the opacity and scale regularisation of the MCMC densification strategy the paper adopts):
//   L = lambda_o sum_i |o_i| + lambda_S sum_i sum_j |sqrt(eig_j(Sigma_i))|.
// With Sigma = R diag(exp(2 l)) R^T (Sec. 3.1) the eigenvalues are exp(2 l_j) for any rotation,
// so the scale term is lambda_S sum exp(l_j): no rotation enters, and dL/dl_j = lambda_S exp(l_j),
// dL/do = lambda_o sign(o).
//
// HBM-bound: per Gaussian it reads o and l (16 B) and read-modify-writes their gradients
// (32 B).  A grid-stride loop over groups of four Gaussians (16-byte accesses); L is summed per
// wavefront, then per workgroup through LDS, and added to the caller's scalar with one atomic per
// workgroup.
#include <cmath>

#include "kernels.hpp"
#include "scan.hpp"
#include "wave_ops.hpp"

namespace splat {

__device__ __forceinline__ float sgnf(float o) { return o > 0.f ? 1.f : (o < 0.f ? -1.f : 0.f); }

// Four Gaussians per thread with 16-byte accesses when every array is 16-byte aligned (their
// log-scale rows then span three float4), one per thread otherwise and for the tail.
__global__ __launch_bounds__(256) void k_mcmc_reg(int64_t n, const float* __restrict__ opac,
                                                  const float* __restrict__ log_scales, float lam_o, float lam_s,
                                                  float* __restrict__ value, float* __restrict__ d_opac,
                                                  float* __restrict__ d_ls, int vec) {
  __shared__ float s_part[4];
  float acc = 0.f;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t n4 = vec ? n / 4 : 0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n4; q += stride) {
    const float4 o = reinterpret_cast<const float4*>(opac)[q];
    const float4* lp = reinterpret_cast<const float4*>(log_scales) + 3 * q;
    const float4 l0 = lp[0], l1 = lp[1], l2 = lp[2];
    const float e[12] = {expf(l0.x), expf(l0.y), expf(l0.z), expf(l0.w), expf(l1.x), expf(l1.y),
                         expf(l1.z), expf(l1.w), expf(l2.x), expf(l2.y), expf(l2.z), expf(l2.w)};
    float se = 0.f;
#pragma unroll
    for (int k = 0; k < 12; ++k) se += e[k];
    acc += lam_o * (fabsf(o.x) + fabsf(o.y) + fabsf(o.z) + fabsf(o.w)) + lam_s * se;
    if (d_opac) {
      float4 g = reinterpret_cast<float4*>(d_opac)[q];
      g.x += lam_o * sgnf(o.x);
      g.y += lam_o * sgnf(o.y);
      g.z += lam_o * sgnf(o.z);
      g.w += lam_o * sgnf(o.w);
      reinterpret_cast<float4*>(d_opac)[q] = g;
    }
    if (d_ls) {
      float4* gp = reinterpret_cast<float4*>(d_ls) + 3 * q;
      float4 g0 = gp[0], g1 = gp[1], g2 = gp[2];
      g0.x += lam_s * e[0]; g0.y += lam_s * e[1]; g0.z += lam_s * e[2]; g0.w += lam_s * e[3];
      g1.x += lam_s * e[4]; g1.y += lam_s * e[5]; g1.z += lam_s * e[6]; g1.w += lam_s * e[7];
      g2.x += lam_s * e[8]; g2.y += lam_s * e[9]; g2.z += lam_s * e[10]; g2.w += lam_s * e[11];
      gp[0] = g0;
      gp[1] = g1;
      gp[2] = g2;
    }
  }
  for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const float o = opac[i];
    const float s0 = expf(log_scales[3 * i]), s1 = expf(log_scales[3 * i + 1]), s2 = expf(log_scales[3 * i + 2]);
    acc += lam_o * fabsf(o) + lam_s * (s0 + s1 + s2);
    if (d_opac) d_opac[i] += lam_o * sgnf(o);
    if (d_ls) {
      d_ls[3 * i] += lam_s * s0;
      d_ls[3 * i + 1] += lam_s * s1;
      d_ls[3 * i + 2] += lam_s * s2;
    }
  }
  if (!value) return;   // uniform
  float v[1] = {acc};
  acc = wave_reduce_scatter<1>(v);   // one value: every lane ends with the wavefront's sum
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(value, s_part[0] + s_part[1] + s_part[2] + s_part[3]);
}

}  // namespace splat

using namespace splat;

extern "C" {

int splat_mcmc_regularizer(const SplatGaussians* g, float lambda_o, float lambda_s, float* value,
                           const SplatGrads* grads, void* stream) {
  if (!g || g->n < 0 || !std::isfinite(lambda_o) || !std::isfinite(lambda_s)) return SPLAT_ERR_INVALID_ARG;
  if (g->n == 0) return SPLAT_OK;
  if (!g->opacities || !g->log_scales) return SPLAT_ERR_INVALID_ARG;
  float* d_o = grads ? grads->opacities : nullptr;
  float* d_l = grads ? grads->log_scales : nullptr;
  if (!value && !d_o && !d_l) return SPLAT_OK;
  const uintptr_t al = (uintptr_t)g->opacities | (uintptr_t)g->log_scales | (uintptr_t)d_o | (uintptr_t)d_l;
  const int vec = (al & 15) == 0;
  // few workgroups, each striding over many Gaussians: every workgroup adds its part of L with
  // one atomic on the same address, and those atomics serialise
  int64_t blocks = div_up(vec ? div_up(g->n, 4) : g->n, 256);
  if (blocks > 512) blocks = 512;
  hipLaunchKernelGGL(k_mcmc_reg, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, g->n, g->opacities,
                     g->log_scales, lambda_o, lambda_s, value, d_o, d_l, vec);
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Relocation of dead Gaussians (the MCMC densification strategy the paper adopts): a Gaussian
// with opacity <= the dead threshold takes the place of an alive one drawn with probability
// proportional to opacity; a target shared by N Gaussians gets o' = 1 - (1 - o)^(1/N) and its
// scales times o / sum_{k=1..N} C(N, k) (-1)^(k+1) o'^k / sqrt(k) (the N copies' composited
// profile integrates to the original's).  The draw is exact integer arithmetic: weights
// floor(o * 2^24) (alive only), their exclusive scan, r = floor(u * total / 2^32) from the
// caller's 32-bit random u, the target the first Gaussian whose inclusive sum exceeds r.
// Passes: one scan of the opacities (weights, and the list of the dead), then three over the list of
// the dead alone, with dense wavefronts: the draw, the new opacity and scales of each target (FP64),
// the copies.  2M Gaussians of 30 words, a tenth dead: 104 us (18 + 28 + 16 + 41) against 185 for passes
// over all Gaussians with a tenth of the lanes at work.
// ---------------------------------------------------------------------------------------------
namespace splat {

constexpr float kWeightOne = 16777216.f;   // 2^24
constexpr int kSampleLog = 12;             // the draw's first step searches up to 2^12 samples in LDS

// The scan stores the sum before every 8th Gaussian: between two of them the draw adds the weights up
// again, from the one or two cache lines that hold their opacities.
constexpr int kFineLog = 3;
inline int64_t reloc_fine(int64_t n) { return ((n - 1) >> kFineLog) + 1; }

// samples of the stored sums: every 2^s-th, the smallest s that leaves at most 2^kSampleLog
inline int reloc_sample_shift(int64_t n_fine) {
  int s = 0;
  while (((n_fine - 1) >> s) >= ((int64_t)1 << kSampleLog)) ++s;
  return s;
}

// weight of a Gaussian's opacity (none for the dead)
__device__ __forceinline__ int64_t reloc_weight(float o, float thr) {
  return o > thr ? (int64_t)fminf(floorf(o * kWeightOne), kWeightOne) : 0;
}

// (dead, weight) of Gaussian i
struct LoadReloc {
  const float* o;
  float thr;
  __device__ P64 operator()(int64_t i) const {
    const float oi = o[i];
    return P64((int64_t)(oi > thr ? 0 : 1), reloc_weight(oi, thr));
  }
};

// Stores the sums before every 8th Gaussian and their samples, lists the dead, and clears what the draw counts in;
// adds the number of Gaussians that will move (the dead, unless there is no weight to draw from).
struct RelocVisit {
  int64_t* fine;
  int64_t* sample;
  int shift;
  int32_t* dead;
  int32_t* target;
  int32_t* counts;
  unsigned long long* n_moved;
  static constexpr int kBatch = 4;
  struct In {};
  __device__ In load(int64_t, P64) const { return In{}; }
  __device__ void operator()(int64_t i, P64 p, P64 v, In) const {
    if ((i & ((1 << kFineLog) - 1)) == 0) {
      const int64_t f = i >> kFineLog;
      fine[f] = p.b;
      if ((f & (((int64_t)1 << shift) - 1)) == 0) sample[f >> shift] = p.b;
    }
    if (v.a) dead[p.a] = (int32_t)i;
    target[i] = -1;
    counts[i] = 0;
  }
  __device__ void finish(P64 total) const {
    if (n_moved && total.b > 0 && total.a > 0) atomicAdd(n_moved, (unsigned long long)total.a);
  }
};

constexpr uint32_t kFirstDraw = 0x80000000u;   // in a drawn target: the first draw of that target

// Grid-stride over the dead.  r's target is the first Gaussian whose inclusive sum exceeds r: a binary
// search over the samples, which a workgroup keeps in LDS, then 8-way steps, whose seven loads are in
// flight together, over the 2^shift stored sums between two of them (two steps at 2M Gaussians), then the
// eight weights after the last sum that does not exceed r.  Bound by the cache lines that a draw
// touches (about 7); with a stored sum for every Gaussian it was 17, and 36 us instead of 28 for
// 200k draws among 2M.
__global__ __launch_bounds__(256) void k_reloc_draw(const float* __restrict__ o, int64_t n, float thr,
                                                    const uint32_t* __restrict__ u, const int64_t* __restrict__ fine,
                                                    const int64_t* __restrict__ sample, int shift,
                                                    const P64* __restrict__ total, const int32_t* __restrict__ dead,
                                                    int32_t* __restrict__ counts, int32_t* __restrict__ target,
                                                    uint32_t* __restrict__ drawn) {
  __shared__ int64_t s_sample[1 << kSampleLog];
  const P64 tot = *total;
  if (tot.b <= 0 || (int64_t)blockIdx.x * blockDim.x >= tot.a) return;   // uniform
  const int64_t n_fine = ((n - 1) >> kFineLog) + 1;
  const int n_sample = (int)((n_fine - 1) >> shift) + 1;
  for (int k = threadIdx.x; k < n_sample; k += blockDim.x) s_sample[k] = sample[k];
  __syncthreads();
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < tot.a; j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = dead[j];
    const uint64_t T = (uint64_t)tot.b, ui = u[i];
    const int64_t r = (int64_t)((T >> 32) * ui + (((T & 0xffffffffull) * ui) >> 32));   // < total
    int lo = 0, hi = n_sample;   // sample[lo] <= r < sample[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_sample[mid] <= r) lo = mid;
      else hi = mid;
    }
    int64_t f = (int64_t)lo << shift, sum = s_sample[lo];
    for (int s = shift; s > 0;) {
      const int d = s < 3 ? s : 3;
      s -= d;
      int64_t e[7];
#pragma unroll
      for (int m = 0; m < 7; ++m) {
        const int64_t q = f + ((int64_t)(m + 1) << s);
        e[m] = fine[q < n_fine ? q : n_fine - 1];
      }
      int below = 0;   // the sums do not decrease
#pragma unroll
      for (int m = 0; m < 7; ++m)
        if (m + 1 < (1 << d) && f + ((int64_t)(m + 1) << s) < n_fine && e[m] <= r) {
          below = m + 1;
          sum = e[m];
        }
      f += (int64_t)below << s;
    }
    const int64_t t0 = f << kFineLog;
    float w[1 << kFineLog];
#pragma unroll
    for (int m = 0; m < (1 << kFineLog); ++m) w[m] = o[t0 + m < n ? t0 + m : n - 1];
    int t = 0;   // weights that leave the sum at r or below
#pragma unroll
    for (int m = 0; m < (1 << kFineLog) - 1; ++m) {
      sum += reloc_weight(w[m], thr);
      t += sum <= r && t0 + m + 1 < n;
    }
    const int64_t tg = t0 + t;
    target[i] = (int32_t)tg;
    drawn[j] = (uint32_t)tg | (atomicAdd(&counts[tg], 1) == 0 ? kFirstDraw : 0u);
  }
}

// The first to have drawn a target (one of the dead per target) writes its new opacity and scales
__global__ __launch_bounds__(256) void k_reloc_update(float* __restrict__ o, float* __restrict__ ls,
                                                      const P64* __restrict__ total, const uint32_t* __restrict__ drawn,
                                                      const int32_t* __restrict__ counts, int n_max) {
  const P64 tot = *total;
  if (tot.b <= 0) return;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < tot.a; j += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t t = drawn[j];
    if (!(t & kFirstDraw)) continue;
    const int64_t i = t & ~kFirstDraw;
    int N = counts[i] + 1;
    N = N < n_max ? N : n_max;
    const double od = o[i];
    const double on = 1.0 - pow(1.0 - od, 1.0 / N);
    double denom = 0.0, c = 1.0, p = 1.0;   // c = C(N, k), p = o'^k
    for (int k = 1; k <= N; ++k) {
      c = c * (double)(N - k + 1) / (double)k;
      p *= on;
      denom += ((k & 1) ? c : -c) * p / sqrt((double)k);
    }
    const double lf = log(od / denom);
    o[i] = (float)on;
    for (int d = 0; d < 3; ++d) ls[3 * i + d] = (float)((double)ls[3 * i + d] + lf);
  }
}

// Every dead Gaussian becomes a copy of its target (alive, so not written here): 16 lanes to one, of
// which 14 take a word of its geometry each, and all of them its features in turn.  200k rows of 30
// words among 2M: 41 us, 78 MB read (random lines) and 49 MB written; two rows in flight: 45.
constexpr int kCopyLanes = 16;

__global__ __launch_bounds__(256) void k_reloc_copy(SplatGaussianState g, const P64* __restrict__ total,
                                                    const int32_t* __restrict__ dead, const uint32_t* __restrict__ drawn) {
  const P64 tot = *total;
  if (tot.b <= 0) return;
  const int w = threadIdx.x % kCopyLanes;
  float* const base = w < 3 ? g.means : w < 7 ? g.quats : w < 8 ? g.opacities : w < 11 ? g.log_scales : w < 14 ? g.velocities : nullptr;
  const int64_t row = w < 3 ? 3 : w < 7 ? 4 : w < 8 ? 1 : 3;
  const int col = w < 3 ? w : w < 7 ? w - 3 : w < 8 ? 0 : w < 11 ? w - 8 : w - 11;
  const int64_t step = (int64_t)gridDim.x * (blockDim.x / kCopyLanes);
  for (int64_t j = (int64_t)blockIdx.x * (blockDim.x / kCopyLanes) + threadIdx.x / kCopyLanes; j < tot.a; j += step) {
    const int64_t i = dead[j], t = drawn[j] & ~kFirstDraw;
    if (base) base[i * row + col] = base[t * row + col];
    if (g.features)
      for (int d = w; d < g.c_total; d += kCopyLanes) g.features[i * g.c_total + d] = g.features[t * g.c_total + d];
  }
}

struct RelocWs {
  int64_t* fine;
  P64* part;
  int32_t* counts;
  int32_t* target;
  int32_t* dead;
  uint32_t* drawn;
  int64_t* sample;
  size_t bytes;
};

inline RelocWs carve_reloc(void* base, int64_t n) {
  RelocWs r;
  char* b = (char*)base;
  size_t off = 0;
  auto take = [&](size_t bytes) {   // base == nullptr: sizes only, pointers stay null
    char* p = b ? b + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  r.fine = (int64_t*)take(reloc_fine(n) * sizeof(int64_t));
  r.part = (P64*)take((div_up(n, scan_tile<P64>()) + 1) * sizeof(P64));
  r.counts = (int32_t*)take(n * sizeof(int32_t));
  r.target = (int32_t*)take(n * sizeof(int32_t));
  r.dead = (int32_t*)take(n * sizeof(int32_t));
  r.drawn = (uint32_t*)take(n * sizeof(uint32_t));
  r.sample = (int64_t*)take((((reloc_fine(n) - 1) >> reloc_sample_shift(reloc_fine(n))) + 1) * sizeof(int64_t));
  r.bytes = off;
  return r;
}

}  // namespace splat

extern "C" {

size_t splat_mcmc_relocate_workspace_bytes(int64_t n) {
  if (n < 0) return 0;
  return carve_reloc(nullptr, n > 0 ? n : 1).bytes;
}

int splat_mcmc_relocate(const SplatGaussianState* g, const uint32_t* u, float dead_opacity, int32_t n_max,
                        int32_t* target, unsigned long long* n_relocated, void* ws, size_t ws_bytes, void* stream) {
  if (!g || g->n < 0 || n_max < 1 || !std::isfinite(dead_opacity)) return SPLAT_ERR_INVALID_ARG;
  if (g->n == 0) return SPLAT_OK;
  if (g->n >= ((int64_t)1 << 31)) return SPLAT_ERR_UNSUPPORTED;
  if (!u || !g->means || !g->log_scales || !g->quats || !g->opacities || (g->c_total > 0 && !g->features) ||
      g->c_total < 0)
    return SPLAT_ERR_INVALID_ARG;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < splat_mcmc_relocate_workspace_bytes(g->n)) return SPLAT_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  RelocWs w = carve_reloc(ws, g->n);
  int32_t* tgt = target ? target : w.target;
  const int shift = reloc_sample_shift(reloc_fine(g->n));
  if (device_scan<P64>(LoadReloc{g->opacities, dead_opacity}, g->n, (P64*)nullptr, w.part, s,
                       RelocVisit{w.fine, w.sample, shift, w.dead, tgt, w.counts, n_relocated}) != hipSuccess)
    return SPLAT_ERR_DEVICE;
  const P64* total = w.part + div_up(g->n, scan_tile<P64>());
  // grids for any number of dead: workgroups past it leave at once
  const int64_t nb = div_up(g->n, 256), nc = div_up(g->n, 256 / kCopyLanes);
  hipLaunchKernelGGL(k_reloc_draw, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, s,
                     (const float*)g->opacities, g->n, dead_opacity, u, (const int64_t*)w.fine, (const int64_t*)w.sample,
                     shift, total, (const int32_t*)w.dead, w.counts, tgt, w.drawn);
  hipLaunchKernelGGL(k_reloc_update, dim3((unsigned)(nb < 2048 ? nb : 2048)), dim3(256), 0, s, g->opacities,
                     g->log_scales, total, (const uint32_t*)w.drawn, (const int32_t*)w.counts, (int)n_max);
  hipLaunchKernelGGL(k_reloc_copy, dim3((unsigned)(nc < 8192 ? nc : 8192)), dim3(256), 0, s, *g, total,
                     (const int32_t*)w.dead, (const uint32_t*)w.drawn);
  return hipGetLastError() == hipSuccess ? SPLAT_OK : SPLAT_ERR_DEVICE;
}

}  // extern "C"
