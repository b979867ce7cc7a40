// Applications and tooling around the smoother (Sec. 3.4, Sec. 4, Sec. 5):
//   * luminance-only colour mode: Y = 0.299 R + 0.587 G + 0.114 B, smooth Y,
//     add the change of Y back to every channel (a YUV round trip with U, V
//     unchanged);
//   * single- and multi-scale HDR tone mapping on the logarithm of the
//     luminance;
//   * the energy of Eq. (1) for the Charbonnier (Eq. (2)) and Welsch
//     (Eq. (18)) penalties, accumulated in double, for convergence studies.
// Elementwise kernels are grid-stride loops over the pixels of a plane, four
// to a thread; reductions over a plane leave per-block partials that the next
// kernel's blocks finish themselves (1080p: 10.3 + 4.6 -> 4.6 us for the
// extremes of the base).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <initializer_list>
#include <vector>

#include "../../include/ils.h"
#include "fft_reg.hpp"
#include "ils_desc.hpp"

namespace {

constexpr int kThreads = 256;
constexpr int kEnergyBlocks = 256;

// V consecutive values (V = 4: one 16-byte access; the launchers check the
// alignment of every plane).
template <int V>
struct Vec {
  float v[V];
};
template <int V>
__device__ __forceinline__ Vec<V> ld(const float* p) {
  Vec<V> r;
  if constexpr (V == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    r.v[0] = t.x, r.v[1] = t.y, r.v[2] = t.z, r.v[3] = t.w;
  } else {
    r.v[0] = *p;
  }
  return r;
}
template <int V>
__device__ __forceinline__ void st(float* p, const Vec<V>& a) {
  if constexpr (V == 4)
    *reinterpret_cast<float4*>(p) = make_float4(a.v[0], a.v[1], a.v[2], a.v[3]);
  else
    *p = a.v[0];
}

__device__ __forceinline__ float luma(float r, float g, float b) {
  return fmaf(0.114f, b, fmaf(0.587f, g, 0.299f * r));
}

template <int V>
__global__ void __launch_bounds__(kThreads) k_luma(const float* __restrict__ rgb, float* __restrict__ y, long long plane) {
  const long long stride = (long long)gridDim.x * kThreads * V;
  for (long long i = ((long long)blockIdx.x * kThreads + threadIdx.x) * V; i < plane; i += stride) {
    const Vec<V> r = ld<V>(rgb + i), g = ld<V>(rgb + i + plane), b = ld<V>(rgb + i + 2 * plane);
    Vec<V> o;
#pragma unroll
    for (int e = 0; e < V; ++e) o.v[e] = luma(r.v[e], g.v[e], b.v[e]);
    st<V>(y + i, o);
  }
}

// out_c = f_c + (v - Y) for c = 0, 1, 2 (out may be f)
template <int V>
__global__ void __launch_bounds__(kThreads) k_recombine(const float* f, const float* __restrict__ y,
                                                         const float* __restrict__ v, float* out, long long plane) {
  const long long stride = (long long)gridDim.x * kThreads * V;
  for (long long i = ((long long)blockIdx.x * kThreads + threadIdx.x) * V; i < plane; i += stride) {
    const Vec<V> vv = ld<V>(v + i), yy = ld<V>(y + i);
    Vec<V> c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] = ld<V>(f + i + k * plane);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
      for (int e = 0; e < V; ++e) c[k].v[e] += vv.v[e] - yy.v[e];
      st<V>(out + i + k * plane, c[k]);
    }
  }
}

// Sum / min / max over a block of kThreads, the same order in every block.
__device__ __forceinline__ float block_sum(float a) {
  __shared__ float red[kThreads / 64];
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  float s = red[0];
  for (int w = 1; w < kThreads / 64; ++w) s += red[w];
  return s;
}
__device__ __forceinline__ void block_minmax(float& lo, float& hi) {
  __shared__ float rl[kThreads / 64], rh[kThreads / 64];
  for (int o = 32; o > 0; o >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    rl[threadIdx.x >> 6] = lo;
    rh[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  lo = rl[0];
  hi = rh[0];
  for (int w = 1; w < kThreads / 64; ++w) {
    lo = fminf(lo, rl[w]);
    hi = fmaxf(hi, rh[w]);
  }
}

// Log of the luminance over 2^n, floored (HDR tone mapping works on log Y).
// n is the mean of log2 Y over kThreads samples: the smoother then works on
// values around zero, where its float32 error, which grows with their size
// (log Y of a radiance map is 6 to 9 on average), is a few times smaller,
// and the operators only need differences of the logarithm and one exact
// factor 2^-n.  Every block forms the same n; block 0 leaves 2^-n in *scale,
// and writes the work lists of the levels to smooth L to.
template <int V>
__global__ void __launch_bounds__(kThreads) k_loglum(const float* __restrict__ rgb, float* __restrict__ L,
                                                      long long plane, float floor_y, float* scale,
                                                      ilsk::LevelLists lists) {
  if (blockIdx.x == 0 && lists.ngroups > 0) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < ilsk::kMaxLevels; ++k)
      if (t == k && k < lists.first[lists.ngroups]) lists.descs[k] = lists.d[k];
#pragma unroll
    for (int g = 0; g < 2; ++g)
      if (g < lists.ngroups && t <= lists.first[g + 1] - lists.first[g]) {
        int* s = lists.starts + 2 * g * (ilsk::kMaxLevels + 1);
        s[t] = t * lists.bands[g];
        s[ilsk::kMaxLevels + 1 + t] = t * lists.tiles[g];
      }
  }
  const long long stride = (long long)gridDim.x * kThreads * V;
  long long i = ((long long)blockIdx.x * kThreads + threadIdx.x) * V;
  Vec<V> c[3];
  auto load = [&]() {
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q] = ld<V>(rgb + i + q * plane);
  };
  if (i < plane) load();  // in flight during the samples' reduction
  const long long at = (long long)threadIdx.x * plane / kThreads;
  const float ys = fmaxf(luma(rgb[at], rgb[at + plane], rgb[at + 2 * plane]), floor_y);
  const float mean = block_sum(log2f(ys)) * (1.0f / kThreads);
  const float n = rintf(fminf(fmaxf(mean, -20.0f), 40.0f));
  const float k = ldexpf(1.0f, -(int)n);
  if (blockIdx.x == 0 && threadIdx.x == 0) *scale = k;
  while (i < plane) {
    Vec<V> o;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const float y = fmaxf(luma(c[0].v[e], c[1].v[e], c[2].v[e]), floor_y), t = y * k;
      o.v[e] = t < INFINITY ? logf(t) : logf(y) - n * 0.69314718f;  // (y 2^-n beyond float32)
    }
    st<V>(L + i, o);
    i += stride;
    if (i < plane) load();
  }
}

// min and max of a plane: per-block partials (the operators' blocks finish)
constexpr int kMinMaxBlocks = kThreads;
template <int V>
__global__ void __launch_bounds__(kThreads) k_minmax_partial(const float* __restrict__ b, long long plane,
                                                              float* partial) {
  float lo = INFINITY, hi = -INFINITY;
  constexpr long long stride = (long long)kMinMaxBlocks * kThreads * V;
#pragma unroll 4
  for (long long i = ((long long)blockIdx.x * kThreads + threadIdx.x) * V; i < plane; i += stride) {
    const Vec<V> v = ld<V>(b + i);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      lo = fminf(lo, v.v[e]);
      hi = fmaxf(hi, v.v[e]);
    }
  }
  block_minmax(lo, hi);
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = lo;
    partial[2 * blockIdx.x + 1] = hi;
  }
}

// K smoothed levels B_1..B_K of L (increasing lambda; K = 1: single-scale),
// detail layers D_1 = L - B_1, D_i = B_{i-1} - B_i kept times w_i, base B_K
// compressed: out_c = f_c exp(L' - log Y), L' = (B_K - max B_K) s + sum w_i D_i,
// s = log(contrast) / (max B_K - min B_K); L = log(Y scale), so exp(-log Y) =
// scale exp(-L); where exp(L' - L) is near the ends of float32, scale joins
// the exponent, since their product need not be.  mm: the partial minima and maxima of B_K.  out may be f,
// and L and the levels may lie in out: every value at i is read first.
constexpr int kMaxScales = ILS_MAX_SCALES;
struct ToneArgs {
  const float* B[kMaxScales];
  float w[kMaxScales];
  int K;
};
template <int V>
__global__ void __launch_bounds__(kThreads) k_tonemap(const float* f, const float* L, ToneArgs a, const float* mm,
                                                       const float* scale, float log_contrast, float* out,
                                                       long long plane) {
  const long long stride = (long long)gridDim.x * kThreads * V;
  long long i = ((long long)blockIdx.x * kThreads + threadIdx.x) * V;
  Vec<V> l, b[kMaxScales], c[3];
  auto load = [&]() {
    l = ld<V>(L + i);
#pragma unroll
    for (int q = 0; q < kMaxScales; ++q)
      if (q < a.K) b[q] = ld<V>(a.B[q] + i);
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q] = ld<V>(f + i + q * plane);
  };
  if (i < plane) load();  // in flight during the reduction of the partials
  float bmin = mm[2 * threadIdx.x], bmax = mm[2 * threadIdx.x + 1];
  const float k = *scale, lk = logf(k);
  block_minmax(bmin, bmax);
  const float s = bmax > bmin ? log_contrast / (bmax - bmin) : 1.0f;
  while (i < plane) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      float prev = l.v[e], acc = 0.0f;
#pragma unroll
      for (int q = 0; q < kMaxScales; ++q)
        if (q < a.K) {
          acc = fmaf(a.w[q], prev - b[q].v[e], acc);
          prev = b[q].v[e];
        }
      const float x = fmaf(prev - bmax, s, acc) - l.v[e];
      const float g = fabsf(x) < 80.0f ? k * expf(x) : expf(x + lk);
#pragma unroll
      for (int q = 0; q < 3; ++q) c[q].v[e] *= g;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) st<V>(out + i + q * plane, c[q]);
    i += stride;
    if (i < plane) load();
  }
}

struct EnergyArgs {
  const float* f;
  const float* u;
  int H, W, C;
  int penalty;
  double lambda, half_p, eps, inv_2g2, two_g2;
};

__device__ __forceinline__ double phi(const EnergyArgs& a, double x) {
  if (a.penalty == ILS_PENALTY_WELSCH) return a.two_g2 * (1.0 - exp(-x * x * a.inv_2g2));  // Eq. (18)
  return pow(x * x + a.eps, a.half_p);                                                  // Eq. (2)
}

// Per-block partial sums of (u - f)^2 + lambda (phi(D_x u) + phi(D_y u)),
// periodic differences, in double.  Blocks stride over image rows (all
// channels), threads over the columns of a row.
__global__ void __launch_bounds__(kThreads) k_energy_partial(EnergyArgs a, double* partial) {
  const long long plane = (long long)a.H * a.W;
  double acc = 0.0;
  for (int row = blockIdx.x; row < a.C * a.H; row += kEnergyBlocks) {
    const int ch = row / a.H, y = row - ch * a.H;
    const int yd = y + 1 == a.H ? 0 : y + 1;
    const float* uc = a.u + (long long)ch * plane;
    const float* ur = uc + (long long)y * a.W;
    const float* ud = uc + (long long)yd * a.W;
    const float* fr = a.f + (long long)ch * plane + (long long)y * a.W;
    for (int x = threadIdx.x; x < a.W; x += kThreads) {
      const int xr = x + 1 == a.W ? 0 : x + 1;
      const double u0 = ur[x];
      const double d = u0 - (double)fr[x];
      acc += d * d + a.lambda * (phi(a, (double)ur[xr] - u0) + phi(a, (double)ud[x] - u0));
    }
  }
  __shared__ double red[kThreads];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(kEnergyBlocks) k_energy_final(const double* partial, double* energy) {
  __shared__ double red[kEnergyBlocks];
  red[threadIdx.x] = partial[threadIdx.x];
  __syncthreads();
  for (int s = kEnergyBlocks / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *energy = red[0];
}

// Blocks of a grid-stride loop over n values, V per thread.
int grid_for(long long n, int V) {
  const long long per = (long long)kThreads * V;
  long long g = (n + per - 1) / per;
  return (int)(g < 2048 ? (g < 1 ? 1 : g) : 2048);
}

// Whether planes of `plane` values can be read four at a time.
bool quads(long long plane, std::initializer_list<const void*> ptrs) {
  uintptr_t u = 0;
  for (const void* p : ptrs) u |= (uintptr_t)p;
  return plane % 4 == 0 && (u & 15) == 0;
}

}  // namespace

extern "C++" int ilsk_plan_scratch(ils_plan* plan, void** scratch, size_t* bytes, void** stream);

// Launchers used by the planner (same stream as the plan).  Four values per
// thread where plane size and pointers allow 16-byte accesses, else one.
hipError_t ilsk_launch_luma(const float* rgb, float* y, long long plane, hipStream_t st) {
  if (quads(plane, {rgb, y}))
    hipLaunchKernelGGL((k_luma<4>), dim3(grid_for(plane, 4)), dim3(kThreads), 0, st, rgb, y, plane);
  else
    hipLaunchKernelGGL((k_luma<1>), dim3(grid_for(plane, 1)), dim3(kThreads), 0, st, rgb, y, plane);
  return hipGetLastError();
}

hipError_t ilsk_launch_recombine(const float* f, const float* y, const float* v, float* out, long long plane,
                                 hipStream_t st) {
  if (quads(plane, {f, y, v, out}))
    hipLaunchKernelGGL((k_recombine<4>), dim3(grid_for(plane, 4)), dim3(kThreads), 0, st, f, y, v, out, plane);
  else
    hipLaunchKernelGGL((k_recombine<1>), dim3(grid_for(plane, 1)), dim3(kThreads), 0, st, f, y, v, out, plane);
  return hipGetLastError();
}

hipError_t ilsk_launch_loglum(const float* rgb, float* L, long long plane, float floor_y, float* scale,
                              const ilsk::LevelLists& lists, hipStream_t st) {
  if (quads(plane, {rgb, L}))
    hipLaunchKernelGGL((k_loglum<4>), dim3(grid_for(plane, 4)), dim3(kThreads), 0, st, rgb, L, plane, floor_y, scale,
                       lists);
  else
    hipLaunchKernelGGL((k_loglum<1>), dim3(grid_for(plane, 1)), dim3(kThreads), 0, st, rgb, L, plane, floor_y, scale,
                       lists);
  return hipGetLastError();
}

// out = the tone-mapped f from L, its K levels B with weights w and L's scale;
// scratch holds 2 * 256 floats of partials
hipError_t ilsk_launch_tonemap(const float* f, const float* L, const float* const* B, const float* w, int K,
                               float* scratch, const float* scale, float log_contrast, float* out, long long plane,
                               hipStream_t st) {
  if (K < 1 || K > kMaxScales) return hipErrorInvalidValue;
  ToneArgs a{};
  bool q = quads(plane, {f, L, out});
  for (int k = 0; k < K; ++k) {
    a.B[k] = B[k];
    a.w[k] = w[k];
    q = q && quads(plane, {B[k]});
  }
  a.K = K;
  if (q) {
    hipLaunchKernelGGL((k_minmax_partial<4>), dim3(kMinMaxBlocks), dim3(kThreads), 0, st, B[K - 1], plane, scratch);
    hipLaunchKernelGGL((k_tonemap<4>), dim3(grid_for(plane, 4)), dim3(kThreads), 0, st, f, L, a, scratch, scale,
                       log_contrast, out, plane);
  } else {
    hipLaunchKernelGGL((k_minmax_partial<1>), dim3(kMinMaxBlocks), dim3(kThreads), 0, st, B[K - 1], plane, scratch);
    hipLaunchKernelGGL((k_tonemap<1>), dim3(grid_for(plane, 1)), dim3(kThreads), 0, st, f, L, a, scratch, scale,
                       log_contrast, out, plane);
  }
  return hipGetLastError();
}

static int energy_impl(ils_plan* plan, const float* f, const float* u, int H, int W, int C, float lambda,
                       int penalty, float p, float eps, float gamma, double* energy) {
  if (!plan || !f || !u || !energy || H < 2 || W < 2 || C < 1) return ILS_ERR_INVALID_ARG;
  if (!std::isfinite(lambda) || lambda < 0.0f) return ILS_ERR_INVALID_ARG;
  EnergyArgs a{};
  a.f = f;
  a.u = u;
  a.H = H;
  a.W = W;
  a.C = C;
  a.penalty = penalty;
  a.lambda = lambda;
  if (penalty == ILS_PENALTY_WELSCH) {
    if (!std::isfinite(gamma) || !(gamma > 0.0f)) return ILS_ERR_INVALID_ARG;
    a.two_g2 = 2.0 * (double)gamma * (double)gamma;
    a.inv_2g2 = 1.0 / a.two_g2;
  } else {
    if (!std::isfinite(p) || !(p > 0.0f) || p > 2.0f || !std::isfinite(eps) || !(eps > 0.0f))
      return ILS_ERR_INVALID_ARG;
    a.half_p = (double)p / 2.0;
    a.eps = eps;
  }
  void* scratch = nullptr;
  size_t bytes = 0;
  void* stream = nullptr;
  if (ilsk_plan_scratch(plan, &scratch, &bytes, &stream) != ILS_OK) return ILS_ERR_INVALID_ARG;
  if (bytes < kEnergyBlocks * sizeof(double)) return ILS_ERR_WORKSPACE;
  double* partial = static_cast<double*>(scratch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_energy_partial, dim3(kEnergyBlocks), dim3(kThreads), 0, st, a, partial);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(kEnergyBlocks), 0, st, partial, energy);
    e = hipGetLastError();
  }
  return e == hipSuccess ? ILS_OK : ILS_ERR_HIP;
}

extern "C" int ils_energy(ils_plan* plan, const float* f, const float* u, int H, int W, int C, float lambda,
                          float p, float eps, double* energy) {
  return energy_impl(plan, f, u, H, W, C, lambda, ILS_PENALTY_CHARBONNIER, p, eps, 0.0f, energy);
}

extern "C" int ils_energy_welsch(ils_plan* plan, const float* f, const float* u, int H, int W, int C,
                                 float lambda, float gamma, double* energy) {
  return energy_impl(plan, f, u, H, W, C, lambda, ILS_PENALTY_WELSCH, 0.0f, 0.0f, gamma, energy);
}
