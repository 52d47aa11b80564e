// Sum of per-chunk partials in a fixed order (reproducible): the last step of every reduction that
// is split over workgroups (the low-rank summary, the outer products and the gate's dW_g of the
// backward).
#pragma once

#include "common.h"

namespace rola {
namespace {

// out[o][e] = sum over b < B and c < n of part[((b * gridDim.y + o) * n + c) * stride + e], e < per.
// Elements e < split go to out0[o * split + e], the rest to out1[o * (per - split) + e - split] (out1
// may be NULL).
//
// Bound by latency, not bytes: with one thread per element walking all its rows, a reduction of few
// elements kept a handful of waves busy with one load in flight each (5 heads, r 32, 843 chunks: 200
// us for 69 MB; d_model 1536, 1024 chunks: 370 us for 6 MB). Here a workgroup takes 64 V elements and
// its S waves take a contiguous slice of the rows each, eight loads of V elements in flight per
// lane; the slices are then added in order through LDS. Both reductions above take under 20 us.
// V = 4 needs a stride that is a multiple of 4 and may read up to three elements past `per` (never
// past the row's stride).
template <int S, int V>
__global__ __launch_bounds__(64 * S) void chunk_reduce_kernel(int per, int split, long stride, int B,
                                                              int n, const float* __restrict__ part,
                                                              float* __restrict__ out0,
                                                              float* __restrict__ out1) {
  typedef float vec __attribute__((ext_vector_type(V)));
  __shared__ vec slice[S][64];
  const int lane = threadIdx.x % 64, w = wave_uniform(threadIdx.x / 64);
  const int e = (blockIdx.x * 64 + lane) * V;
  const long o = blockIdx.y;
  const int rows = B * n;
  const int m0 = (int)((long)rows * w / S), m1 = (int)((long)rows * (w + 1) / S);
  vec s = 0.f;
  if (e < per) {
    const auto row = [&](int m) {  // rows of one output: n consecutive ones per b
      const int b = B == 1 ? 0 : m / n;
      return *reinterpret_cast<const vec*>(
          part + (((long)b * gridDim.y + o) * n + (m - b * n)) * stride + e);
    };
    // whole batches, the last one re-reading the slice's last row without adding it
    constexpr int kBatch = 8;
    for (int m = m0; m < m1; m += kBatch) {
      vec v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v[u] = row(min(m + u, m1 - 1));
#pragma unroll
      for (int u = 0; u < kBatch; ++u) s = m + u < m1 ? s + v[u] : s;
    }
  }
  slice[w][lane] = s;
  __syncthreads();
  if (w != 0) return;
  s = slice[0][lane];
#pragma unroll
  for (int i = 1; i < S; ++i) s += slice[i][lane];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const int ek = e + k;
    if (ek < split) out0[o * split + ek] = s[k];
    else if (ek < per && out1) out1[o * (per - split) + (ek - split)] = s[k];
  }
}

// The same sums over few rows (B n), one element per thread: nothing to split, and the slices' meeting in
// LDS costs more than it saves (the reduction of 5 rows of 2064 elements 3.1 us with it, 2.2 here).
constexpr int kFewRows = 20;
__global__ __launch_bounds__(256) void few_rows_reduce_kernel(int per, int split, long stride, int B,
                                                              long b_stride, int n,
                                                              const float* __restrict__ part,
                                                              float* __restrict__ out0,
                                                              float* __restrict__ out1) {
  const long o = blockIdx.y;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= per) return;
  const float* src = part + o * n * stride + e;
  float s = 0.f;
  for (int b = 0; b < B; ++b, src += b_stride) {
    constexpr int kBatch = 8;
    for (int c0 = 0; c0 < n; c0 += kBatch) {
      float v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v[u] = src[min(c0 + u, n - 1) * stride];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) s = c0 + u < n ? s + v[u] : s;
    }
  }
  if (e < split) out0[o * split + e] = s;
  else if (out1) out1[o * (per - split) + (e - split)] = s;
}

// Four waves per workgroup up to 128 rows, sixteen beyond (26 rows of 8256 elements, 40 heads: with
// sixteen waves of one or two loads each the call is 13 us longer).
template <int V>
hipError_t launch_chunk_reduce_v(int per, int split, long stride, int B, int outputs, int n,
                                 const float* part, float* out0, float* out1, hipStream_t st) {
  const dim3 grid((per + 64 * V - 1) / (64 * V), (unsigned)outputs);
  if ((long)B * n <= 128)
    hipLaunchKernelGGL((chunk_reduce_kernel<4, V>), grid, dim3(256), 0, st, per, split, stride, B, n,
                       part, out0, out1);
  else
    hipLaunchKernelGGL((chunk_reduce_kernel<16, V>), grid, dim3(1024), 0, st, per, split, stride, B,
                       n, part, out0, out1);
  return hipGetLastError();
}

// part must be 16-byte aligned.
inline hipError_t launch_chunk_reduce(int per, int split, long stride, int B, int outputs, int n,
                                      const float* part, float* out0, float* out1, hipStream_t st) {
  if ((long)B * n <= kFewRows) {
    hipLaunchKernelGGL(few_rows_reduce_kernel, dim3((per + 255) / 256, (unsigned)outputs), dim3(256), 0, st,
                       per, split, stride, B, (long)outputs * n * stride, n, part, out0, out1);
    return hipGetLastError();
  }
  if (stride % 4 == 0 && (per + 3) / 4 * 4 <= stride)
    return launch_chunk_reduce_v<4>(per, split, stride, B, outputs, n, part, out0, out1, st);
  return launch_chunk_reduce_v<1>(per, split, stride, B, outputs, n, part, out0, out1, st);
}

}  // namespace
}  // namespace rola
