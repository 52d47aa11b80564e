// 3D rotary schedule (Sec. 3, 3D RoPE; Sec. 4.2): the backbone's cos/sin tables and the main-path
// rotation Q^r = R(Q^n) (Algorithm step 3). Both are memory-bound elementwise kernels.
#include "common.h"
#include "launch.h"

namespace rola {
namespace {

// Tables of short sequences, one thread per (token, pair): one evaluation each, nothing to wait for. 320
// tokens 2.9 us against 4.3 of the shared evaluation below, whose three phases are a chain; 3549 4.8 and 6.0,
// 4410 5.5 and 5.4. Angles in fp64, so the fp32 tables are correctly rounded values of cos/sin of the exact
// angle.
constexpr int kTableFew = 4096 * 64;  // entries
__global__ void rope_tables_few_kernel(int N, int HsWs, int Ws, int half, int pt, int py, int dt,
                                       int dy, int dx, double base, int ot, int oy, int ox,
                                       float* __restrict__ cos_tab, float* __restrict__ sin_tab) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)N * half) return;
  const int n = (int)(i / half), j = (int)(i % half);
  const int t = n / HsWs, rem = n % HsWs, y = rem / Ws, x = rem % Ws;
  double pos;
  int loc, width;
  if (j < pt) { pos = t + ot; loc = j; width = dt; }
  else if (j < pt + py) { pos = y + oy; loc = j - pt; width = dy; }
  else { pos = x + ox; loc = j - pt - py; width = dx; }
  const double ang = pos * pow(base, -2.0 * loc / width);
  double s, c;
  sincos(ang, &s, &c);
  cos_tab[i] = (float)c;
  sin_tab[i] = (float)s;
}

// Tables of kTableRows grid rows (t, y) per workgroup. A pair's angle depends on one coordinate only, so the
// workgroup evaluates each (x, pair) and each of its rows' (t, pair), (y, pair) once into LDS and
// writes the rows from there: one fp64 pow and sincos per (token, pair) took 25 us at 32760 tokens and
// 50 at 67545; 15 and 22 now. Wide rows are split over workgroups (kTableX / pairs values of x each).
constexpr int kTableRows = 4;
constexpr int kTableX = 2048;
__global__ __launch_bounds__(256) void rope_tables_kernel(int rows, int Hs, int Ws, int half, int pt,
                                                          int py, int dt, int dy, int dx, double base,
                                                          int ot, int oy, int ox,
                                                          float* __restrict__ cos_tab,
                                                          float* __restrict__ sin_tab) {
  __shared__ double freq[64];                    // half <= 64
  __shared__ float2 yt[kTableRows][64];          // pairs of t and y, per row
  __shared__ float2 xs[kTableX];                 // [x][pair of x]
  const int tid = threadIdx.x, px = half - pt - py, pyt = pt + py;
  const int row0 = blockIdx.x * kTableRows, nrows = min(kTableRows, rows - row0);
  if (tid < half) {
    const int j = tid;
    const int loc = j < pt ? j : j < pyt ? j - pt : j - pyt, width = j < pt ? dt : j < pyt ? dy : dx;
    freq[j] = pow(base, -2.0 * loc / width);
  }
  __syncthreads();
  auto entry = [&](double pos, int j) {
    double s, c;
    sincos(pos * freq[j], &s, &c);
    return make_float2((float)c, (float)s);
  };
  for (int e = tid; e < nrows * pyt; e += 256) {
    const int r = e / pyt, j = e % pyt, t = (row0 + r) / Hs, y = (row0 + r) % Hs;
    yt[r][j] = entry(j < pt ? t + ot : y + oy, j);
  }
  const int xn = kTableX / px, x0 = blockIdx.y * xn, n = min(xn, Ws - x0);
  for (int e = tid; e < n * px; e += 256) xs[e] = entry(x0 + e / px + ox, pyt + e % px);
  __syncthreads();
  const int j = tid % half;
  for (int e = tid / half; e < nrows * n; e += 256 / half) {
    const int r = e / n, x = e % n;
    const float2 v = j < pyt ? yt[r][j] : xs[x * px + j - pyt];
    const long i = ((long)(row0 + r) * Ws + x0 + x) * half + j;
    cos_tab[i] = v.x;
    sin_tab[i] = v.y;
  }
}

// Xr = R(X): one thread per 4 pairs (8 elements) of a token, for `per` heads: the token's table entries
// (twice the bytes of a bf16 row) are read once for them, BATCH heads' rows are in flight at a time, and
// the indices are shifts (a 64-bit division per thread and a table read per head made the bf16
// rotation of 32760 tokens x 12 heads 50 us for 201 MB; 37 now).
template <typename T, int BATCH>
__global__ __launch_bounds__(256) void rope_apply_kernel(int heads, int per, int N, int shift, int ld,
                                                         const T* __restrict__ X,
                                                         const float* __restrict__ cos_tab,
                                                         const float* __restrict__ sin_tab,
                                                         T* __restrict__ Xr) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;  // (token, 8-element piece)
  const long pieces = (long)N << shift;
  if (i >= pieces) return;
  const long n = i >> shift;
  const int g = (int)(i & ((1 << shift) - 1));
  const float4 c = *reinterpret_cast<const float4*>(cos_tab + n * ld + g * 4);
  const float4 s = *reinterpret_cast<const float4*>(sin_tab + n * ld + g * 4);
  const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {s.x, s.y, s.z, s.w};
  const int h0 = blockIdx.y * per, h1 = min(heads, h0 + per);
  for (int h = h0; h < h1; h += BATCH) {
    float v[BATCH][8];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) load8(X + (min(h + u, h1 - 1) * pieces + i) * 8, v[u]);
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      if (h + u >= h1) break;
      float o[8];
#pragma unroll
      for (int p = 0; p < 4; ++p)
        rope_pair(v[u][2 * p], v[u][2 * p + 1], cc[p], ss[p], o[2 * p], o[2 * p + 1]);
      store8(Xr + ((h + u) * pieces + i) * 8, o);
    }
  }
}

// Backward of the rotation (fp32): dX += R(p)^T dY, pair (a, b) -> (a cos + b sin, b cos - a sin),
// or dX += dY without the rotation. One thread per 4 pairs of one row.
template <bool ROT>
__global__ void rope_grad_kernel(long rows, int N, int d, int ld, const float* __restrict__ dY,
                                 const float* __restrict__ cos_tab,
                                 const float* __restrict__ sin_tab, float* __restrict__ dX) {
  const int per_row = d / 8;
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * per_row) return;
  const long row = i / per_row;
  const int g = (int)(i % per_row);
  float v[8], o[8];
  load8(dY + row * d + g * 8, v);
  load8(dX + row * d + g * 8, o);
  if constexpr (ROT) {
    const int n = (int)(row % N);
    const float4 c = *reinterpret_cast<const float4*>(cos_tab + (long)n * ld + g * 4);
    const float4 sn = *reinterpret_cast<const float4*>(sin_tab + (long)n * ld + g * 4);
    const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      o[2 * p] += v[2 * p] * cc[p] + v[2 * p + 1] * ss[p];
      o[2 * p + 1] += v[2 * p + 1] * cc[p] - v[2 * p] * ss[p];
    }
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] += v[k];
  }
  store8(dX + row * d + g * 8, o);
}

}  // namespace

hipError_t launch_rope_grad(const Shape& s, const float* dY, const float* cos_tab,
                            const float* sin_tab, int ld, bool rotate, float* dX, hipStream_t st) {
  const long rows = (long)s.B * s.H * s.N;
  const long total = rows * (s.d / 8);
  const int threads = 256;
  const dim3 grid((unsigned)((total + threads - 1) / threads));
  if (rotate)
    hipLaunchKernelGGL(rope_grad_kernel<true>, grid, dim3(threads), 0, st, rows, s.N, s.d, ld, dY,
                       cos_tab, sin_tab, dX);
  else
    hipLaunchKernelGGL(rope_grad_kernel<false>, grid, dim3(threads), 0, st, rows, s.N, s.d, ld, dY,
                       cos_tab, sin_tab, dX);
  return hipGetLastError();
}

hipError_t launch_rope_tables(const Shape& s, int dt, int dy, int dx, double base, int ot, int oy,
                              int ox, float* cos_tab, float* sin_tab, hipStream_t st) {
  const int half = s.d / 2;
  if ((long)s.N * half <= kTableFew) {
    hipLaunchKernelGGL(rope_tables_few_kernel, dim3((s.N * half + 255) / 256), dim3(256), 0, st, s.N,
                       s.Hs * s.Ws, s.Ws, half, dt / 2, dy / 2, dt, dy, dx, base, ot, oy, ox, cos_tab,
                       sin_tab);
    return hipGetLastError();
  }
  const int rows = s.T * s.Hs, xn = kTableX / (dx / 2);
  hipLaunchKernelGGL(rope_tables_kernel,
                     dim3((unsigned)((rows + kTableRows - 1) / kTableRows), (unsigned)((s.Ws + xn - 1) / xn)),
                     dim3(256), 0, st, rows, s.Hs, s.Ws, half, dt / 2, dy / 2, dt, dy, dx, base, ot,
                     oy, ox, cos_tab, sin_tab);
  return hipGetLastError();
}

hipError_t launch_rope_apply(const Shape& s, const void* X, const float* cos_tab,
                             const float* sin_tab, int ld, void* Xr, hipStream_t st) {
  const int heads = s.B * s.H, shift = s.d == 128 ? 4 : 3;  // 16 or 8 pieces per row
  const unsigned gx = (unsigned)((((long)s.N << shift) + 255) / 256);
  // heads per thread: eight where that leaves four workgroups per CU, fewer in small problems
  int per = 8;
  while (per > 1 && (long)gx * ((heads + per - 1) / per) < 4 * kCus) per /= 2;
  const dim3 grid(gx, (unsigned)((heads + per - 1) / per));
  const auto launch = [&](auto zero) {
    using T = decltype(zero);
    const int most = heads < per ? heads : per;  // rows that a thread has to load
    const auto kernel = most == 1   ? rope_apply_kernel<T, 1>
                        : most == 2 ? rope_apply_kernel<T, 2>
                                    : rope_apply_kernel<T, 4>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, heads, per, s.N, shift, ld, (const T*)X, cos_tab,
                       sin_tab, (T*)Xr);
  };
  if (s.bf16)
    launch(bf16{});
  else
    launch(0.f);
  return hipGetLastError();
}

}  // namespace rola
