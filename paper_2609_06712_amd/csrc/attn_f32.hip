// Block-sparse (or dense) softmax attention of the fp32 path (d_h 64 or 128), on fp32 MFMA.
//
// A workgroup takes 16 queries of one query block and its four waves split their keys: wave w walks
// the 16-key sub-tiles w, w + 4, ... of the selected blocks with an online softmax of its own, and the
// four partial results are merged through LDS at the end. fp32 layers are small (the tiny layer has
// 256 tokens, two heads, 64 keys per query), so the time is one chain of latencies: 16 queries per
// workgroup instead of a whole block give four times the workgroups, and the key split shortens the
// chain. Per wave and sub-tile, on v_mfma_f32_16x16x4_f32 (A: row l%16, k = l/16; B: column l%16,
// k = l/16; D: column l%16, rows 4(l/16) + i):
//   S^T = K Q^T   contraction step s of lane group g = channel g d/4 + s, so that a lane reads its K row
//                 (and its Q row, once) as contiguous 16-byte pieces;
//   O^T = V^T P^T step i of group g = key 4g + i, which is where S^T leaves the probabilities; row
//                 l%16 of tile w = channel (l%16) d/16 + w, so V rows are read, and O rows written, as
//                 contiguous pieces too.
// One thread per query walking its keys from LDS took 143 us at the tiny layer, 4.7 us now (a whole layer
// of 2048 tokens, 8 heads, d 128: 1.69 ms to 0.15 ms).
#include "common.h"
#include "launch.h"

namespace rola {
namespace {

constexpr int kQ = 16;      // queries per workgroup
constexpr int kWaves = 4;   // key split

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D>
__global__ __launch_bounds__(64 * kWaves) void attn_f32_kernel(
    int N, int block, int nb, int keep, const int32_t* __restrict__ idx, float scale,
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    float* __restrict__ O) {
  constexpr int C4 = D / 16;  // 16-byte pieces of a lane's quarter row of Q or K
  constexpr int W = D / 16;   // channel tiles of O^T, and consecutive channels per lane and key of V
  __shared__ float os[kWaves][kQ][D + 4];
  __shared__ float ms[kWaves][kQ], ls[kWaves][kQ];
  const int lane = threadIdx.x % 64, wave = wave_uniform(threadIdx.x / 64);
  const int lr = lane % 16, g = lane / 16;
  const int tiles = block / kQ;  // query tiles per block; sub-tiles per key block
  const int I = blockIdx.x / tiles, q = I * block + (blockIdx.x % tiles) * kQ + lr;
  if (q - lr >= N) return;  // the whole tile is past the last token
  const long head = (long)blockIdx.z * gridDim.y + blockIdx.y;
  const float* Kh = K + head * (long)N * D;
  const float* Vh = V + head * (long)N * D;
  const int32_t* sel = idx ? idx + (head * nb + I) * (long)keep : nullptr;

  float4 qv[C4];
  {
    const float* row = Q + (head * N + min(q, N - 1)) * (long)D + g * (D / 4);
#pragma unroll
    for (int s = 0; s < C4; ++s) qv[s] = *reinterpret_cast<const float4*>(row + 4 * s);
  }
  f32x4 acc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) acc[w] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int T = keep * tiles;
  for (int t = wave; t < T; t += kWaves) {
    const int J = sel ? sel[t / tiles] : t / tiles;
    const int k0 = J * block + (t % tiles) * kQ;
    if ((unsigned)J >= (unsigned)nb || k0 >= N) continue;  // out-of-range entry, or past the last key
    float4 kv[C4], vv[4][W / 4];
    {
      const float* row = Kh + min(k0 + lr, N - 1) * (long)D + g * (D / 4);
#pragma unroll
      for (int s = 0; s < C4; ++s) kv[s] = *reinterpret_cast<const float4*>(row + 4 * s);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* row = Vh + min(k0 + 4 * g + i, N - 1) * (long)D + lr * W;
#pragma unroll
      for (int s = 0; s < W / 4; ++s) vv[i][s] = *reinterpret_cast<const float4*>(row + 4 * s);
    }
    f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};  // two chains
#pragma unroll
    for (int s = 0; s < C4; ++s) {
      sc[0] = mfma_f32(kv[s].x, qv[s].x, sc[0]);
      sc[1] = mfma_f32(kv[s].y, qv[s].y, sc[1]);
      sc[0] = mfma_f32(kv[s].z, qv[s].z, sc[0]);
      sc[1] = mfma_f32(kv[s].w, qv[s].w, sc[1]);
    }
    float p[4], mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // key k0 + 4g + i of this lane's query
      p[i] = k0 + 4 * g + i < N ? (sc[0][i] + sc[1][i]) * scale : -INFINITY;
      mt = fmaxf(mt, p[i]);
    }
    const float mx = fmaxf(m, rows_max(mt));  // finite: key k0 is valid
    const float alpha = expf(m - mx);
    m = mx;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = expf(p[i] - mx);
      sum += p[i];
    }
    l = l * alpha + sum;  // this lane's quarter of the keys
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] *= alpha;
    if (k0 + kQ > N) {  // ragged tail: V zero past the last key (P is zero there, and 0 x inf is not)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int s = 0; s < W / 4; ++s)
          vv[i][s] = k0 + 4 * g + i < N ? vv[i][s] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float4 v = vv[i][w / 4];
        const float a = w % 4 == 0 ? v.x : w % 4 == 1 ? v.y : w % 4 == 2 ? v.z : v.w;
        acc[w] = mfma_f32(a, p[i], acc[w]);
      }
  }
  // Merge the waves: acc[w][i] is channel (4g + i) W + w of query lr.
  l = rows_sum(l);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int s = 0; s < W / 4; ++s)
      *reinterpret_cast<float4*>(&os[wave][lr][(4 * g + i) * W + 4 * s]) =
          make_float4(acc[4 * s][i], acc[4 * s + 1][i], acc[4 * s + 2][i], acc[4 * s + 3][i]);
  if (g == 0) {
    ms[wave][lr] = m;
    ls[wave][lr] = l;
  }
  __syncthreads();
  const int qi = threadIdx.x / 16, c0 = (threadIdx.x % 16) * W;  // 16 threads per query
  const int qo = q - lr + qi;
  if (qo >= N) return;
  float mx = ms[0][qi];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, ms[w][qi]);
  float sum = 0.f, o[W];
#pragma unroll
  for (int c = 0; c < W; ++c) o[c] = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float a = expf(ms[w][qi] - mx);  // 0 for a wave without keys
    sum = fmaf(a, ls[w][qi], sum);
#pragma unroll
    for (int c = 0; c < W; ++c) o[c] = fmaf(a, os[w][qi][c0 + c], o[c]);
  }
  const float inv = 1.0f / sum;
  float* row = O + (head * N + qo) * (long)D + c0;
#pragma unroll
  for (int s = 0; s < W / 4; ++s)
    *reinterpret_cast<float4*>(row + 4 * s) =
        make_float4(o[4 * s] * inv, o[4 * s + 1] * inv, o[4 * s + 2] * inv, o[4 * s + 3] * inv);
}

}  // namespace

hipError_t launch_attn_f32(const Shape& s, const void* Qr, const void* Kr, const void* V, int block,
                           int keep, const int32_t* idx, float scale, void* Os, hipStream_t st) {
  const int nb = num_blocks(s.N, block);
  const dim3 grid(nb * (block / kQ), s.H, s.B);
  const auto kernel = s.d == 64 ? attn_f32_kernel<64> : attn_f32_kernel<128>;
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), 0, st, s.N, block, nb, keep, idx, scale,
                     (const float*)Qr, (const float*)Kr, (const float*)V, (float*)Os);
  return hipGetLastError();
}

}  // namespace rola
