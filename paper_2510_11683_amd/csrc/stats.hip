// Statistics of repeated gradient estimates: per-element running mean and
// sum of squared deviations (Welford's update), and their summary over all
// elements (mean standard deviation across repeats, mean absolute deviation
// of the mean from a reference gradient), reduced in a fixed order.
#include <math.h>

#include <algorithm>

#include "../../include/bgpo.h"
#include "../../include/bgpo_stats.h"
#include "common.hpp"

namespace bgpo {

typedef float vec4 __attribute__((ext_vector_type(4)));

// Above this many elements the four arrays of a problem (16 bytes per element)
// are well past the 256 MB last-level cache: nothing that is read or written
// will be found there again, and streaming (non-temporal) accesses are faster
// (update and summary together: 518M elements 3234 us without, 2673 with; 33M
// 192 and 173).  Below it they would lose what the summary re-reads (16.8M: 82
// and 88 us).
constexpr int64_t kStreamElements = int64_t(24) << 20;

template <bool NT>
__device__ __forceinline__ vec4 load4(const float* p) {
  return NT ? __builtin_nontemporal_load(reinterpret_cast<const vec4*>(p))
            : *reinterpret_cast<const vec4*>(p);
}

__device__ __forceinline__ void welford(float g, float& mean, float& m2, float inv) {
  const float dl = g - mean;
  mean += dl * inv;
  m2 += dl * (g - mean);
}

// k = number of estimates already folded in: delta = g - mean,
// mean += delta / (k + 1), m2 += delta (g - mean_new).  Four elements per
// thread, one step per workgroup (up to kMaxUpdateBlocks of them; a loop over
// 4096 resident workgroups kept fewer loads in flight).  Bound by HBM, 20 bytes
// per element: 518M elements 2215 us (4.7 TB/s) in the loop, 1707 us (6.1
// TB/s) so, streaming.
//
// A launch takes fewer than 2^32 work-items; above 2^33 elements the workgroups
// take several steps each.
constexpr int64_t kMaxUpdateBlocks = int64_t(1) << 23;

template <bool NT>
__global__ __launch_bounds__(256) void k_moments_update(const float* __restrict__ g,
                                                        float* __restrict__ mean,
                                                        float* __restrict__ m2, int64_t n,
                                                        int k) {
  const float inv = 1.f / (float)(k + 1);
  const int64_t stride = (int64_t)gridDim.x * 256 * 4;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += stride) {
    if (i + 4 <= n) {
      const vec4 gv = load4<NT>(g + i);
      vec4 mv = load4<NT>(mean + i), sv = load4<NT>(m2 + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float m = mv[e], q = sv[e];
        welford(gv[e], m, q, inv);
        mv[e] = m;
        sv[e] = q;
      }
      if constexpr (NT) {
        __builtin_nontemporal_store(mv, reinterpret_cast<vec4*>(mean + i));
        __builtin_nontemporal_store(sv, reinterpret_cast<vec4*>(m2 + i));
      } else {
        *reinterpret_cast<vec4*>(mean + i) = mv;
        *reinterpret_cast<vec4*>(m2 + i) = sv;
      }
    } else {
      for (int64_t q = i; q < n; ++q) welford(g[q], mean[q], m2[q], inv);
    }
  }
}

constexpr int kSumBlocks = 1024;

// Per-workgroup partial sums of (std_i, |mean_i - ref_i|, |ref_i|) in float64,
// std_i = sqrt(m2_i / (count - 1)); U groups of 4 consecutive elements per
// thread and step, steps a whole grid apart, in a fixed order.  `vec`: the
// arrays are 16-byte aligned.  Bound by HBM, 12 bytes per element: 518M
// elements 1440 us with 4-byte loads, 956 us (6.5 TB/s) with U = 4, streaming.
template <int U, bool NT>
__global__ __launch_bounds__(256) void k_moments_partial(const float* __restrict__ mean,
                                                         const float* __restrict__ m2,
                                                         const float* __restrict__ ref, int64_t n,
                                                         int count, bool vec,
                                                         double* __restrict__ part) {
  __shared__ double red[3][4];
  const double dof = count > 1 ? 1.0 / (double)(count - 1) : 0.0;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  auto load = [&](const float* p, int64_t i) -> vec4 {
    vec4 v = (vec4){0.f, 0.f, 0.f, 0.f};
    if (!p || i >= n) return v;
    if (vec && i + 4 <= n) return load4<NT>(p + i);
    for (int e = 0; e < 4; ++e)
      if (i + e < n) v[e] = p[i + e];
    return v;
  };
  const int64_t step = (int64_t)U * 1024;
  for (int64_t b = blockIdx.x * step; b < n; b += gridDim.x * step) {
    vec4 a[U], c[U], r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = b + u * 1024 + threadIdx.x * 4;
      a[u] = load(m2, i);
      c[u] = ref ? load(mean, i) : a[u];   // (without a reference only the deviations count)
      r[u] = load(ref, i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 += sqrt((double)a[u][e] * dof);
        if (ref) {
          s1 += fabs((double)c[u][e] - (double)r[u][e]);
          s2 += fabs((double)r[u][e]);
        }
      }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off, 64);
    s1 += __shfl_xor(s1, off, 64);
    s2 += __shfl_xor(s2, off, 64);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wv] = s0;
    red[1][wv] = s1;
    red[2][wv] = s2;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int c = threadIdx.x;
    part[(int64_t)blockIdx.x * 3 + c] = red[c][0] + red[c][1] + red[c][2] + red[c][3];
  }
}

// One wave per sum: lane l adds partials l, l + 64, .. and the lanes are added
// in a fixed tree (one thread per sum took 22 us for its serial loads).
__global__ __launch_bounds__(192) void k_moments_final(const double* __restrict__ part, int64_t n,
                                                       double* __restrict__ out) {
  const int c = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double s = 0.0;
#pragma unroll
  for (int b = lane; b < kSumBlocks; b += 64) s += part[b * 3 + c];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) out[c] = s / (double)n;
}

}  // namespace bgpo

using namespace bgpo;

extern "C" {

int bgpo_moments_update(const float* g, float* mean, float* m2, int64_t n, int32_t count,
                        void* stream) {
  if (!g || !mean || !m2 || n < 0 || count < 0) return BGPO_ERR_INVALID_ARG;
  if (((uintptr_t)g | (uintptr_t)mean | (uintptr_t)m2) & 15) return BGPO_ERR_INVALID_ARG;
  if (n == 0) return BGPO_OK;
  const int64_t blocks = std::min<int64_t>((n - 1) / 1024 + 1, kMaxUpdateBlocks);
  const auto kernel = n >= kStreamElements ? k_moments_update<true> : k_moments_update<false>;
  kernel<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>(g, mean, m2, n, count);
  return hipGetLastError() == hipSuccess ? BGPO_OK : BGPO_ERR_HIP;
}

size_t bgpo_moments_workspace_size(void) { return (size_t)kSumBlocks * 3 * sizeof(double); }

int bgpo_moments_summary(const float* mean, const float* m2, const float* ref, int64_t n,
                         int32_t count, double* out, void* workspace, size_t ws_bytes,
                         void* stream) {
  if (!mean || !m2 || !out || n <= 0 || count < 1) return BGPO_ERR_INVALID_ARG;
  if (!workspace || ((uintptr_t)workspace & 7) || ws_bytes < bgpo_moments_workspace_size())
    return BGPO_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  double* part = static_cast<double*>(workspace);
  const bool vec = !(((uintptr_t)mean | (uintptr_t)m2 | (uintptr_t)ref) & 15);
  const auto kernel = n >= kStreamElements ? k_moments_partial<4, true> : k_moments_partial<1, false>;
  kernel<<<kSumBlocks, 256, 0, s>>>(mean, m2, ref, n, count, vec, part);
  if (hipGetLastError() != hipSuccess) return BGPO_ERR_HIP;
  k_moments_final<<<1, 192, 0, s>>>(part, n, out);
  return hipGetLastError() == hipSuccess ? BGPO_OK : BGPO_ERR_HIP;
}

}  // extern "C"
