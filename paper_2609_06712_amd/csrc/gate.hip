// Token gate logits of the gated fusion (Sec. 4.4; Algorithm step 8): logit[b, n] = X[b, n, :] . W_g
// + b_g over the attention block's input hidden states X [B, N, d_model]; the combine applies the
// sigmoid. A GEMV, bound by reading X once from HBM (d_model * elt bytes per token).
//
// One wave per token row (rows strided over the grid's waves), W_g staged once per workgroup in LDS
// as fp32; each lane reads 16-byte pieces of the row (8 bf16 or 4 fp32 values), accumulates in fp32,
// and the row sum is a cross-lane reduction. Two rows are in flight per wave so that each lane keeps
// two independent 16-byte loads outstanding per step.
#include "common.h"
#include "launch.h"
#include "reduce.h"

namespace rola {
namespace {

constexpr int kGateMaxModel = 16384;  // W_g in LDS as fp32: 64 KB

// One 16-byte piece of a row as fp32: 8 bf16 or 4 fp32 values.
__device__ __forceinline__ void load_piece(const bf16* p, float v[8]) { load8(p, v); }
__device__ __forceinline__ void load_piece(const float* p, float v[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}

__device__ __forceinline__ float wave_sum(float x) {
  x = rows_sum(x);  // lanes l, l^16, l^32, l^48
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

template <typename T>
__global__ __launch_bounds__(256) void gate_logits_kernel(long rows, int dm, const T* __restrict__ X,
                                                          const T* __restrict__ W, float bias,
                                                          float* __restrict__ logits) {
  extern __shared__ float w[];  // [dm]
  for (int i = threadIdx.x; i < dm; i += 256) w[i] = to_f32(W[i]);
  __syncthreads();
  constexpr int PER = 16 / sizeof(T);  // values per 16-byte piece
  const int lane = threadIdx.x % 64;
  const long wave = (long)blockIdx.x * 4 + threadIdx.x / 64, nwaves = (long)gridDim.x * 4;
  for (long r0 = 2 * wave; r0 < rows; r0 += 2 * nwaves) {
    const bool two = r0 + 1 < rows;
    const T* x0 = X + r0 * dm;
    const T* x1 = X + (two ? r0 + 1 : r0) * dm;
    float s0 = 0.f, s1 = 0.f;
    for (int c = lane * PER; c < dm; c += 64 * PER) {
      float a[8], b[8];
      load_piece(x0 + c, a);
      load_piece(x1 + c, b);
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        s0 = fmaf(a[k], w[c + k], s0);
        s1 = fmaf(b[k], w[c + k], s1);
      }
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if (lane == 0) {
      logits[r0] = s0 + bias;
      if (two) logits[r0 + 1] = s1 + bias;
    }
  }
}

// Backward of the gate logits: dX[row] = dlogit[row] W_g (fp32), and per chunk of rows the partial
// sums of dW_g = sum_row dlogit[row] X[row] and db_g = sum_row dlogit[row] (slot dm of the partial).
// Bound by reading X and writing dX. A workgroup is tx columns of eight channels by 256 / tx rows, so
// a wave reads and writes whole 16-byte pieces with four rows in flight per thread; the 512 chunks
// are two workgroups per CU. d_model 1536, 32760 rows: 158 us with one channel per thread and one
// row in flight, 1024 partials then added in 370 us; 55 + 12 us now (5.5 TB/s over X and dX).
constexpr int kGateBwdChunks = 512;
constexpr int kGateBwdBatch = 4;  // rows in flight per thread

template <typename T>
__global__ __launch_bounds__(256) void gate_bwd_kernel(long rows, int dm, int tx, long chunk,
                                                       const T* __restrict__ X,
                                                       const T* __restrict__ W,
                                                       const float* __restrict__ dlog,
                                                       float* __restrict__ dX,
                                                       float* __restrict__ part, long stride) {
  __shared__ float red[256 * 8];
  const int ty = 256 / tx, x = threadIdx.x % tx, y = threadIdx.x / tx;
  const long r0 = blockIdx.x * chunk, r1 = min(rows, r0 + chunk);
  float* out = part + blockIdx.x * stride;
  for (int c0 = 0; c0 < dm; c0 += 8 * tx) {
    const int c = c0 + 8 * x;
    float acc[8] = {};
    if (c < dm) {
      float w[8];
      load8(W + c, w);
      for (long r = r0 + y; r < r1; r += kGateBwdBatch * ty) {
        float v[kGateBwdBatch][8], g[kGateBwdBatch];
#pragma unroll
        for (int u = 0; u < kGateBwdBatch; ++u) {  // rows past the chunk re-read this one, with weight 0
          const long ru = r + u * ty < r1 ? r + u * ty : r;
          load8(X + ru * dm + c, v[u]);
          g[u] = dlog[ru];
        }
#pragma unroll
        for (int u = 0; u < kGateBwdBatch; ++u) {
          if (r + u * ty >= r1) break;
          float d[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            acc[k] = fmaf(g[u], v[u][k], acc[k]);
            d[k] = g[u] * w[k];
          }
          if (dX) store8(dX + (r + u * ty) * dm + c, d);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) red[threadIdx.x * 8 + k] = acc[k];
    __syncthreads();
    for (int e = threadIdx.x; e < 8 * tx && c0 + e < dm; e += 256) {  // rows of the tile, in order
      float s = 0.f;
      for (int j = 0; j < ty; ++j) s += red[j * 8 * tx + e];
      out[c0 + e] = s;
    }
  }
  // db_g: the chunk's logit gradients, by one wave
  if (threadIdx.x < 64) {
    float s = 0.f;
    for (long r = r0 + threadIdx.x; r < r1; r += 64) s += dlog[r];
    s = wave_sum(s);
    if (threadIdx.x == 0) out[dm] = s;
  }
}

// Columns (of eight channels) of the workgroup tile: the power of two that leaves the fewest idle
// threads in the last pass over d_model / 8 columns, the largest such (fewer row slices to add).
int gate_bwd_columns(int d_model) {
  const int cols = d_model / 8;
  int best = 256;
  for (int tx = 128; tx >= 16; tx /= 2)
    if ((cols + tx - 1) / tx * tx < (cols + best - 1) / best * best) best = tx;
  return best;
}

// Row length of the partials, whole 16-byte pieces.
long gate_bwd_stride(int d_model) { return d_model + 4; }

}  // namespace

size_t gate_backward_workspace_bytes(int d_model) {
  return (size_t)kGateBwdChunks * gate_bwd_stride(d_model) * sizeof(float);
}

hipError_t launch_gate_backward(const Shape& s, const void* X, int d_model, const void* Wg,
                                const float* dlogits, float* dX, float* dWg, float* dbg, void* ws,
                                hipStream_t st) {
  const long rows = (long)s.B * s.N;
  const long chunk = (rows + kGateBwdChunks - 1) / kGateBwdChunks;
  const int n = (int)((rows + chunk - 1) / chunk);
  const int tx = gate_bwd_columns(d_model);
  const long stride = gate_bwd_stride(d_model);
  float* part = (float*)ws;
  if (s.bf16)
    hipLaunchKernelGGL(gate_bwd_kernel<bf16>, dim3(n), dim3(256), 0, st, rows, d_model, tx, chunk,
                       (const bf16*)X, (const bf16*)Wg, dlogits, dX, part, stride);
  else
    hipLaunchKernelGGL(gate_bwd_kernel<float>, dim3(n), dim3(256), 0, st, rows, d_model, tx, chunk,
                       (const float*)X, (const float*)Wg, dlogits, dX, part, stride);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_chunk_reduce(d_model + 1, d_model, stride, 1, 1, n, part, dWg, dbg, st);
}

hipError_t launch_gate_logits(const Shape& s, const void* X, int d_model, const void* Wg, float bg,
                              float* logits, hipStream_t st) {
  const long rows = (long)s.B * s.N;
  const long want = (rows + 7) / 8;  // workgroups of 4 waves, 2 rows per wave per pass
  const dim3 grid((unsigned)(want < 2048 ? want : 2048));
  const size_t lds = (size_t)d_model * sizeof(float);
  if (s.bf16)
    hipLaunchKernelGGL(gate_logits_kernel<bf16>, grid, dim3(256), lds, st, rows, d_model,
                       (const bf16*)X, (const bf16*)Wg, bg, logits);
  else
    hipLaunchKernelGGL(gate_logits_kernel<float>, grid, dim3(256), lds, st, rows, d_model,
                       (const float*)X, (const float*)Wg, bg, logits);
  return hipGetLastError();
}

int gate_max_model() { return kGateMaxModel; }

}  // namespace rola
