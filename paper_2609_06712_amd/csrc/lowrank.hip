// Rotary low-rank branch (eq. qklr, eq. ctx; Algorithm steps 5-7) and gated fusion (eq. gate,
// Algorithm steps 8-10).
//
// Features are the paper's even/odd split (Sec. 4.5, fused inference kernel): projecting with the
// even rows and the odd rows of P separately puts both members of every rotary pair in the same lane
// and register slot, so SiLU and the rotation R_r are in-register arithmetic between two MFMA
// results, no lane exchange.
//
// bf16 summary: per (b, h, token chunk) one workgroup of 4 waves, 32 tokens per wave per step.
//   Psi = K^n P^T      (even and odd P rows)  A = K^n rows straight from HBM (prefetched one step
//                      ahead), B = P fragments in registers; lane = pair j, 4 tokens per 16-token tile
//   k~ = R_r SiLU(Psi) in registers (fp32), rounded to bf16 as the B operand of
//   C^T += V^T k~      A = V^T from LDS (V transposed while staged), fp32 accumulators in registers.
// Waves are summed through LDS in a fixed order, chunks by a second kernel in a fixed order: C and z
// are bitwise reproducible (no float atomics).
//
// bf16 readout (+ combine): per wave 16-token tiles.
//   Phi = P Q^T        A = P fragments (registers), B = Q^n rows from HBM; lane = token, 4 pairs
//   q~ = R_r SiLU(Phi) in registers, rounded to bf16
//   u^T = C^T q~       A = C^T (bf16, registers, loaded once per workgroup)
//   RMSNorm over d_h (in-lane sums + 2 shuffles); fused: O = (O^s/r_s + g O^lr) r_s.
// Both kernels are HBM-bound; grids are ordered head-minor. The readout's is remapped so an XCD
// works on one token range for all heads, reading each rotary-table row once into its L2; the
// summary's is dealt round-robin (measured faster for it).
#include "common.h"
#include "launch.h"
#include "reduce.h"
#define MAP_FN __device__ __forceinline__
#define MAP_RCP __builtin_amdgcn_rcpf
#define MAP_EXP __expf
#include "feature_maps.h"

namespace rola {
namespace {

constexpr int kSummaryStep = 128;  // tokens per workgroup step (4 waves x 32)

__device__ __forceinline__ f32x4 mfma16x16x32(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Feature map of the low-rank branch. The paper's design is SiLU with the rotation applied outside
// it (eq. qklr); its ablations replace SiLU by Identity, Tanh, ReLU or GELU and move the rotation
// inside the activation or drop it (Sec. 5.1 RoPE placement, Prop. inside). feat = phi | order << 8
// with the ROLA_PHI_* / ROLA_ROPE_* values of the ABI. Every phi maps 0 to 0, so zero rows (padding
// tokens, padding pairs) keep zero features under every variant.
constexpr int kPhiSilu = 0, kPhiIdentity = 1, kPhiTanh = 2, kPhiRelu = 3, kPhiGelu = 4;
constexpr int kRopeOutside = 0, kRopeInside = 1;  // any other order: no rotation

__device__ __forceinline__ float feature_act(float x, int phi) {
  switch (phi) {
    case kPhiIdentity: return x;
    case kPhiTanh: return tanhf(x);
    case kPhiRelu: return fmaxf(x, 0.f);
    case kPhiGelu: return 0.5f * x * (1.f + erff(x * 0.70710678118654752f));  // exact (erf) GELU
    default: return silu(x);
  }
}

// Features of one rotary pair from its two projections (e, o) = (P_2j x, P_2j+1 x) at a position
// with rotation (c, s), feat at run time (the fp32 kernels).
__device__ __forceinline__ void feature_pair(float& e, float& o, float c, float s, int feat) {
  const int phi = feat & 0xFF, order = feat >> 8;
  if (order == kRopeInside) {
    const float a = e * c - o * s, b = e * s + o * c;
    e = a;
    o = b;
  }
  const float a = feature_act(e, phi), b = feature_act(o, phi);
  if (order == kRopeOutside) {
    e = a * c - b * s;
    o = a * s + b * c;
  } else {
    e = a;
    o = b;
  }
}

// The bf16 kernels' form of feature_pair: the N pairs a lane holds at once, phi a template argument
// (kPaper: SiLU with the rotation outside, compiled as the plain design; otherwise a ROLA_PHI_* value
// with the rotation order at run time), and branch-free maps. One uniform branch per phase instead of
// a switch and a divergent erff / tanhf per value lets the values of a tile overlap: readout at
// r 128 with GELU inside, 39689 tokens x 12 heads: 383 us with the per-value form, 132 now (with the longer chunks).
constexpr int kPaper = -1;

template <int PHI>
__device__ __forceinline__ float feature_map(float x) {
  if constexpr (PHI == kPhiIdentity) return x;
  if constexpr (PHI == kPhiTanh) return tanh_fast(x);
  if constexpr (PHI == kPhiRelu) return fmaxf(x, 0.f);
  if constexpr (PHI == kPhiGelu) return gelu_fast(x);
  return silu(x);
}

template <int PHI, int N>
__device__ __forceinline__ void feature_tile(float (&e)[N], float (&o)[N], const float (&c)[N],
                                             const float (&s)[N], int order) {
  const auto rotate = [&] {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float a = e[i], b = o[i];
      e[i] = a * c[i] - b * s[i];
      o[i] = a * s[i] + b * c[i];
    }
  };
  if (PHI != kPaper && order == kRopeInside) rotate();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    e[i] = feature_map<PHI>(e[i]);
    o[i] = feature_map<PHI>(o[i]);
  }
  if (PHI == kPaper || order == kRopeOutside) rotate();
}

// Tokens per summary workgroup: one per CU to a round, two for each chunk at r = 128; the bf16 kernel takes
// two steps per turn. (Least length: at the 14B shape, r = 64, 2048 workgroups took 420 us, 1024 388: fewer
// partials to write and reduce.) Calls that fit the chip with one step per workgroup take chunks of one step
// and the kernel's form without a turn of two, whose second step would mostly add zeros: 2 heads of 320
// tokens, r 16 10.0 -> 8.2 us, r 64 18.1 -> 14.7. Not past 96 partials to add (116, r 16: 12.1 against 11.5).
int summary_chunk_len(const Shape& s, int r) {
  if (!s.bf16) return chunk_tokens(s, 1024, 1024, kSummaryStep);
  const long slots = r <= 64 ? kCus : kCus / 2, steps = (s.N + kSummaryStep - 1) / kSummaryStep;
  if (steps <= 96 && s.B * s.H * steps <= slots) return kSummaryStep;
  return chunk_tokens(s, 1024, slots, 2 * kSummaryStep);
}

// ------------------------------------------------------------------------------------------------
// bf16 summary
// ------------------------------------------------------------------------------------------------
// split = 2: each (b, h, chunk) is served by two workgroups, one per half of the pair tiles (r = 128
// as two r = 64 halves: one workgroup holding all four tiles spills). The two sit eight launch
// slots apart, i.e. on the same XCD at about the same time, so the second reads K^n and V from L2.
// ONE: chunks of a single step.
template <int JT, int PHI, bool ONE>
__global__ __launch_bounds__(256, JT == 1 ? 2 : 1) void summary_mfma_kernel(
    int N, int H, int r, int chunk_len, int n_chunks, int total, int split, int ld, int order,
    const bf16* __restrict__ Kn, const bf16* __restrict__ V, const bf16* __restrict__ Pk,
    const float* __restrict__ cos_tab, const float* __restrict__ sin_tab,
    float* __restrict__ part) {
  constexpr int D = 128, TOK = kSummaryStep;
  constexpr int TILE = TOK * D * 2;  // one step's V tile: 32 KB, row-major, chunks swizzled
  // Two V stages filled by direct global-to-LDS loads, then reused for the cross-wave reduction.
  __shared__ __attribute__((aligned(1024))) char lds[2 * TILE];

  const int BH = total / n_chunks;
  // heads minor in launch order, dealt round-robin to the XCDs: 2.7 % faster at the 14B shape than
  // giving each XCD a contiguous token range of all heads (which shared the table rows in L2)
  int L = blockIdx.x, jt0 = 0;  // jt0: first pair tile of this workgroup
  if (split == 2) {
    L = (int)(blockIdx.x / 16) * 8 + blockIdx.x % 8;
    jt0 = JT * ((blockIdx.x / 8) % 2);
    if (L >= total) return;  // the grid is rounded up to whole groups of 16
  }
  const int head = L % BH, chunk = L / BH;
  const int h = head % H;
  const int tid = threadIdx.x, lane = tid % 64, lr = lane % 16, g = lane / 16;
  const int wave = wave_uniform(tid / 64);
  const int half = r / 2;
  const bf16* Kh = Kn + (long)head * N * D;
  const char* Vh = reinterpret_cast<const char*>(V + (long)head * N * D);
  const bf16* Ph = Pk + (long)h * r * D;

  // This lane's pair of tile jt is jb + jt: a token's table entries of its pairs are consecutive.
  const int jb = 16 * jt0 + JT * lr;
  bf16x8 pe[JT][4], po[JT][4];
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    const int j = jb + jt;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
      if (j < half) {
        pe[jt][kc] = *reinterpret_cast<const bf16x8*>(Ph + (long)(2 * j) * D + 32 * kc + 8 * g);
        po[jt][kc] = *reinterpret_cast<const bf16x8*>(Ph + (long)(2 * j + 1) * D + 32 * kc + 8 * g);
      } else {
        pe[jt][kc] = bf16x8{};
        po[jt][kc] = bf16x8{};
      }
    }
  }
  f32x4 ce[JT][8], co[JT][8];
  float ze[JT], zo[JT];
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    ze[jt] = zo[jt] = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) ce[jt][w] = co[jt][w] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int t0 = chunk * chunk_len, t1 = min(N, t0 + chunk_len);
  // V tile DMA: lane l of 1-KB slot q (8 slots per wave) fills row 4q + l/16, position l%16 with
  // source chunk position ^ 2(row%8). Rows past the chunk re-read its last one, as do K^n rows and
  // table entries: the features of those tokens are zeroed, and their V rows once they are in LDS.
  const int row0 = 32 * wave + lane / 16;
  uint32_t dvp[2];  // slot i's row is row0 + 4i; its swizzle depends only on i's parity
#pragma unroll
  for (int p = 0; p < 2; ++p)
    dvp[p] = (row0 + 4 * p) * D * 2 + (((lane % 16) ^ (((row0 + 4 * p) & 7) << 1)) << 4);
  const uint32_t lds0 = lds_address(lds);
  auto issue_v = [&](int base, int buf) {  // always 8 loads
    const uint32_t dst = lds0 + buf * TILE + wave * 8192;
    if (base + TOK <= t1) {
      const char* vb = Vh + (long)base * D * 2;
#pragma unroll
      for (int i = 0; i < 8; ++i) dma16(vb, dvp[i & 1] + (i >> 1) * 2048, dst + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = row0 + 4 * i, src = min(base + row, t1 - 1);
        dma16(Vh, (uint32_t)(src - row) * (D * 2) + dvp[i & 1] + (i >> 1) * 2048, dst + i * 1024);
      }
    }
  };
  // Transposing-read offsets of the V^T operand: lane (g, 4 s' + m') reads token row
  // wave*32 + 4g + s' (+16), channels 16w + 4m'.
  const int sp = lr >> 2, mp = lr & 3, vr = wave * 32 + 4 * g + sp;
  int vo[8];
#pragma unroll
  for (int w = 0; w < 8; ++w)
    vo[w] = vr * 256 + (((2 * w + (mp >> 1)) ^ ((vr & 7) << 1)) << 4) + ((mp & 1) << 3);

  // Pipeline, per wave (each wave fills and reads only its own 32 rows of a stage, so there is no
  // workgroup barrier): the V rows (LDS DMA) and K^n rows (registers) of step t+1 are issued before
  // step t is computed, the table entries of step t+2 in the middle of step t. No load is
  // conditional, so the compiler's waits for a step's K^n rows and table entries leave the later
  // loads in flight; with guarded loads it drained the whole queue at the top of each step, which
  // serialised loads and compute (r = 64, 32760 tokens x 40 heads: 210 us).
  // The V DMA is inline assembly, which the compiler does not track. What makes a step's V rows
  // complete before they are read: vector-memory loads retire in order, the K^n loads of a step are
  // issued after its V DMA (their address passes through an asm statement behind it), and the reads
  // of V stand behind an asm statement that takes a product of the last of those K^n rows.
  typedef float tvec __attribute__((ext_vector_type(JT)));
  struct KRows {
    bf16x8 k[2][4];
  };
  struct Tables {
    tvec c[2][4], s[2][4];
  };
  // Rows are addressed from a scalar base per step with 32-bit lane offsets (whole 64-bit addresses
  // per load cost the registers that the second sets need).
  auto issue_k = [&](int base, KRows& R) {
    uint32_t fence = 16 * g;
    asm volatile("" : "+v"(fence) : : "memory");
    const int first = min(base, t1 - 1), lim = t1 - 1 - first;
    const char* kb = reinterpret_cast<const char*>(Kh + (long)first * D);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const uint32_t off = (uint32_t)min(wave * 32 + tt * 16 + lr, lim) * (D * 2) + fence;
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) R.k[tt][kc] = *reinterpret_cast<const bf16x8*>(kb + off + 64 * kc);
    }
  };
  // pairs past r/2 re-read the last ones and meet zero rows of P
  const uint32_t joff = 4 * min(jb, half - JT), ldb = 4 * ld;  // ld <= 65536: 24-bit products
  auto load_tables = [&](int base, Tables& T) {
    const int first = min(base, t1 - 1), lim = t1 - 1 - first;
    const char* cb = reinterpret_cast<const char*>(cos_tab + (long)first * ld);
    const char* sb = reinterpret_cast<const char*>(sin_tab + (long)first * ld);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t off = __umul24(min(wave * 32 + tt * 16 + 4 * g + v, lim), ldb) + joff;
        T.c[tt][v] = *reinterpret_cast<const tvec*>(cb + off);
        T.s[tt][v] = *reinterpret_cast<const tvec*>(sb + off);
      }
  };
  auto step = [&](int base, int buf, const KRows& cur, KRows& nxt, Tables& T) {
    if constexpr (!ONE) {
      asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the reads of the stage V goes into are done
      issue_v(base + TOK, buf ^ 1);
      issue_k(base + TOK, nxt);
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8 be[JT], bo[JT];
    float last = 0.f;
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        f32x4 ye = {0.f, 0.f, 0.f, 0.f}, yo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
          ye = mfma16x16x32(cur.k[tt][kc], pe[jt][kc], ye);
          yo = mfma16x16x32(cur.k[tt][kc], po[jt][kc], yo);
        }
        last = yo[0];
        float ke[4] = {ye[0], ye[1], ye[2], ye[3]}, ko[4] = {yo[0], yo[1], yo[2], yo[3]};
        float cs[4], sn[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          cs[v] = T.c[tt][v][jt];
          sn[v] = T.s[tt][v][jt];
        }
        feature_tile<PHI>(ke, ko, cs, sn, order);
        if (base + TOK > t1) {  // (uniform) tokens past the chunk
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const bool ok = base + wave * 32 + tt * 16 + 4 * g + v < t1;
            ke[v] = ok ? ke[v] : 0.f;
            ko[v] = ok ? ko[v] : 0.f;
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          ze[jt] += ke[v];
          zo[jt] += ko[v];
          be[jt][4 * tt + v] = (bf16)ke[v];
          bo[jt][4 * tt + v] = (bf16)ko[v];
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!ONE) load_tables(base + 2 * TOK, T);
    asm volatile("" : "+v"(last) : : "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (base + TOK > t1) {  // (uniform) V past the chunk: zero as well, 0 x inf is not 0
      const int first = max(0, t1 - base - 32 * wave);  // of the wave's rows
      if constexpr (ONE) {
        if (first == 0) return;  // no token of this wave's in the step
        for (int row = first + lane / 16; row < 32; row += 4)
          *reinterpret_cast<uint4*>(lds + buf * TILE + wave * 8192 + row * (D * 2) + 16 * (lane % 16)) =
              make_uint4(0u, 0u, 0u, 0u);
      } else {
        int ln;  // (the lane index made here, and one register of zeros: what is more spills)
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
        float* rows = reinterpret_cast<float*>(lds + buf * TILE + wave * 8192) + ln;
#pragma unroll 1
        for (int row = first; row < 32; ++row) rows[row * (D / 2)] = 0.f;
      }
      asm volatile("" : : : "memory");
    }
    const char* Vs = lds + buf * TILE;
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(Vs + vo[w]));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(Vs + vo[w] + 16 * 256));
      const bf16x8 va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        ce[jt][w] = mfma16x16x32(va, be[jt], ce[jt][w]);
        co[jt][w] = mfma16x16x32(va, bo[jt], co[jt][w]);
      }
    }
  };

  KRows ra, rb;
  Tables ta, tb;
  load_tables(t0, ta);  // (in the loop's issue order: the waits at its head assume the worse of the two)
  issue_v(t0, 0);
  issue_k(t0, ra);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (ONE) {
    step(t0, 0, ra, rb, ta);
  } else {
    load_tables(t0 + TOK, tb);
    __builtin_amdgcn_sched_barrier(0);
    // two steps per turn without an exit between them (it costs 60 to 130 spilled registers): the second
    // of an odd count adds zeros to zeros
    for (int base = t0; base < t1; base += 2 * TOK) {
      step(base, 0, ra, rb, ta);
      step(base + TOK, 1, rb, ra, tb);
    }
  }
  // the last look-ahead has landed before the stages are reused below (barriers follow)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");

  // z: the four lane groups hold different tokens of the same pair j
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    ze[jt] = rows_sum(ze[jt]);
    zo[jt] = rows_sum(zo[jt]);
  }
  // Sum the four waves in a fixed order: wave 3 -> 2 -> 1 -> 0, one pair-tile at a time.
  constexpr int PER = 2 * 8 * 4 + 2;  // floats per lane per pair tile
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    for (int src = 3; src >= 1; --src) {
      __syncthreads();
      if (wave == src) {
#pragma unroll
        for (int w = 0; w < 8; ++w)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            red[((0 * 8 + w) * 4 + v) * 64 + lane] = ce[jt][w][v];
            red[((1 * 8 + w) * 4 + v) * 64 + lane] = co[jt][w][v];
          }
        red[(PER - 2) * 64 + lane] = ze[jt];
        red[(PER - 1) * 64 + lane] = zo[jt];
      }
      __syncthreads();
      if (wave == src - 1) {
#pragma unroll
        for (int w = 0; w < 8; ++w)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            ce[jt][w][v] += red[((0 * 8 + w) * 4 + v) * 64 + lane];
            co[jt][w][v] += red[((1 * 8 + w) * 4 + v) * 64 + lane];
          }
        ze[jt] += red[(PER - 2) * 64 + lane];
        zo[jt] += red[(PER - 1) * 64 + lane];
      }
    }
  }
  if (wave == 0) {
    float* P = part + ((long)head * n_chunks + chunk) * (long)(r * D + r);
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      const int j = jb + jt;
      if (j >= half) continue;
#pragma unroll
      for (int w = 0; w < 8; ++w)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int dim = 16 * w + 4 * g + v;
          P[(long)(2 * j) * D + dim] = ce[jt][w][v];
          P[(long)(2 * j + 1) * D + dim] = co[jt][w][v];
        }
      if (g == 0) {
        P[(long)r * D + 2 * j] = ze[jt];
        P[(long)r * D + 2 * j + 1] = zo[jt];
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// fp32 path, on v_mfma_f32_16x16x4_f32 (A: row l%16, k = l/16; B: column l%16, k = l/16; D: column l%16,
// rows 4(l/16) + i). fp32 layers are small, so a call is a chain of latencies: scalar dot products per
// (token, pair) took 32 us (summary) and 10 us (readout) at the tiny layer, 9 and 5 us now.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Features of pair tile jt (pairs 16 jt ..) for 16 tokens, lane = token l%16, pairs 16 jt + 4(l/16) + i:
// Y^T = P X^T with contraction step s of lane group g = channel g D/4 + s, so that x (the lane's quarter
// of its token row) and the rows of P are contiguous 16-byte pieces. Pairs past r/2 get zero features.
template <int D>
__device__ __forceinline__ void features_f32(const float* __restrict__ P, int r, int jt,
                                             const float4 (&x)[D / 16], const float* cos_row,
                                             const float* sin_row, int feat, int lane, float (&fe)[4],
                                             float (&fo)[4]) {
  const int lr = lane % 16, g = lane / 16, half = r / 2, j = 16 * jt + lr, jb = 16 * jt + 4 * g;
  const float* pe = P + (long)(2 * min(j, half - 1)) * D + g * (D / 4);
  f32x4 ye = {0.f, 0.f, 0.f, 0.f}, yo = {0.f, 0.f, 0.f, 0.f};
  float4 e[D / 16], o[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    e[s] = *reinterpret_cast<const float4*>(pe + 4 * s);
    o[s] = *reinterpret_cast<const float4*>(pe + D + 4 * s);
  }
  // the tables' rows are whole 16-byte pieces: a piece that starts below half can be read
  float4 c4 = make_float4(1.f, 1.f, 1.f, 1.f), s4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (jb < half) {
    c4 = *reinterpret_cast<const float4*>(cos_row + jb);
    s4 = *reinterpret_cast<const float4*>(sin_row + jb);
  }
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    ye = mfma_f32(e[s].x, x[s].x, ye);
    yo = mfma_f32(o[s].x, x[s].x, yo);
    ye = mfma_f32(e[s].y, x[s].y, ye);
    yo = mfma_f32(o[s].y, x[s].y, yo);
    ye = mfma_f32(e[s].z, x[s].z, ye);
    yo = mfma_f32(o[s].z, x[s].z, yo);
    ye = mfma_f32(e[s].w, x[s].w, ye);
    yo = mfma_f32(o[s].w, x[s].w, yo);
  }
  const float cc[4] = {c4.x, c4.y, c4.z, c4.w}, ss[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = ye[i], b = yo[i];
    feature_pair(a, b, cc[i], ss[i], feat);
    fe[i] = jb + i < half ? a : 0.f;
    fo[i] = jb + i < half ? b : 0.f;
  }
}

// Summary: per (b, h, token chunk) one workgroup, 64 tokens per step. Each wave computes the features of
// 16 tokens and leaves them in LDS ([token][coordinate]); after a barrier each wave contracts all 64
// tokens for its own quarter of the channels, C[coord][ch] += f[tok][coord] V[tok][ch], step s of lane
// group g = token 4s + g, column n of channel tile t = channel w D/4 + n CT + t (contiguous V pieces).
template <int D>
__global__ __launch_bounds__(256) void summary_f32_kernel(
    int N, int H, int r, int chunk_len, int n_chunks, int ld, int feat, const float* __restrict__ Kn,
    const float* __restrict__ V, const float* __restrict__ Pk, const float* __restrict__ cos_tab,
    const float* __restrict__ sin_tab, float* __restrict__ part) {
  constexpr int TT = 64, RP = 128 + 4, CT = D / 64;
  typedef float vvec __attribute__((ext_vector_type(CT)));
  __shared__ __attribute__((aligned(16))) float ft[TT][RP];
  __shared__ float zs[2][128];
  const int chunk = blockIdx.x, h = blockIdx.y;
  const long head = (long)blockIdx.z * gridDim.y + h;
  const int tid = threadIdx.x, lane = tid % 64, wave = wave_uniform(tid / 64);
  const int lr = lane % 16, g = lane / 16;
  const int JT = (r / 2 + 15) / 16, RT = (r + 15) / 16;
  const float* Kh = Kn + head * (long)N * D;
  const float* Vh = V + head * (long)N * D + wave * (D / 4) + lr * CT;
  const float* Ph = Pk + (long)h * r * D;
  const int t0 = chunk * chunk_len, t1 = min(N, t0 + chunk_len);
  f32x4 acc[8][CT];
#pragma unroll
  for (int rt = 0; rt < 8; ++rt)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float z = 0.f;  // thread: coordinate tid % 128, half the tokens of each step
  for (int b0 = t0; b0 < t1; b0 += TT) {
    // tokens past the chunk re-read its last one and get zero features and zero V (0 x inf is not 0)
    vvec v[TT / 4];
#pragma unroll
    for (int s = 0; s < TT / 4; ++s)
      v[s] = *reinterpret_cast<const vvec*>(Vh + (long)min(b0 + 4 * s + g, t1 - 1) * D);
    if (b0 + TT > t1) {
#pragma unroll
      for (int s = 0; s < TT / 4; ++s) v[s] = b0 + 4 * s + g < t1 ? v[s] : vvec(0.f);
    }
    const int tok = b0 + 16 * wave + lr, tk = min(tok, t1 - 1);
    float4 x[D / 16];
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      x[s] = *reinterpret_cast<const float4*>(Kh + (long)tk * D + g * (D / 4) + 4 * s);
    for (int jt = 0; jt < JT; ++jt) {
      float fe[4], fo[4];
      features_f32<D>(Ph, r, jt, x, cos_tab + (long)tk * ld, sin_tab + (long)tk * ld, feat, lane, fe, fo);
      if (tok >= t1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) fe[i] = fo[i] = 0.f;
      }
      float4* dst = reinterpret_cast<float4*>(&ft[16 * wave + lr][32 * jt + 8 * g]);
      dst[0] = make_float4(fe[0], fo[0], fe[1], fo[1]);
      dst[1] = make_float4(fe[2], fo[2], fe[3], fo[3]);
    }
    __syncthreads();
    if (tid % 128 < r) {
#pragma unroll 8
      for (int t = 0; t < TT / 2; ++t) z += ft[TT / 2 * (tid / 128) + t][tid % 128];
    }
#pragma unroll
    for (int rt = 0; rt < 8; ++rt) {
      if (rt >= RT) break;
#pragma unroll
      for (int s = 0; s < TT / 4; ++s) {
        const float a = ft[4 * s + g][16 * rt + lr];
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[rt][t] = mfma_f32(a, v[s][t], acc[rt][t]);
      }
    }
    __syncthreads();
  }
  zs[tid / 128][tid % 128] = z;
  __syncthreads();
  float* P = part + (head * n_chunks + chunk) * (long)(r * D + r);
#pragma unroll
  for (int rt = 0; rt < 8; ++rt) {
    if (rt >= RT) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int coord = 16 * rt + 4 * g + i;
      if (coord >= r) continue;
#pragma unroll
      for (int t = 0; t < CT; ++t) P[(long)coord * D + wave * (D / 4) + lr * CT + t] = acc[rt][t][i];
    }
  }
  if (tid < r) P[(long)r * D + tid] = zs[0][tid] + zs[1][tid];
}

// ------------------------------------------------------------------------------------------------
// bf16 readout, optionally fused with the gated combine
// ------------------------------------------------------------------------------------------------
// One workgroup per (b, h, chunk of tokens), 16 tokens per wave and step. P (fragments in registers, in
// LDS at r = 128) and C^T (fragments in LDS) are set up once per workgroup, so chunks are long: at most
// 1024 workgroups, in whole rounds. The next tile's Q^n and O^s rows, table entries and logit load while a tile is
// computed (tokens past the chunk re-read its last one and are not stored). r = 128 takes eight waves
// to a workgroup: with its fragments in LDS one workgroup fills a CU, and two waves per SIMD overlap
// one's products with the other's features.
// Against 256-token workgroups that waited for each pair of tiles (32760 tokens x 40 heads, with the
// combine): r 64 294 -> 228-257 us; r 128 with GELU inside, 39689 tokens x 12 heads: 383 -> 132 us.
constexpr int kReadoutWorkgroups = 1024;
template <int JT>
constexpr int readout_waves() { return JT == 4 ? 8 : 4; }

template <int JT, bool COMBINE, int PHI>
__global__ __launch_bounds__(64 * readout_waves<JT>(), 2) void readout_mfma_kernel(
    int N, int H, int r, int chunk_len, int n_chunks, int total, int ld, int order,
    const bf16* __restrict__ Qn, const bf16* __restrict__ Pq, const float* __restrict__ cos_tab,
    const float* __restrict__ sin_tab, const float* __restrict__ C, float eps_lr, const bf16* Os,
    const float* __restrict__ logits, float eps, bf16* Out) {
  constexpr int D = 128, NW = readout_waves<JT>(), THREADS = 64 * NW, STEP = 16 * NW;
  constexpr bool kPLds = JT == 4;
  const int BH = total / n_chunks;
  const int L = xcd_remap(blockIdx.x, total);
  const int head = L % BH, chunk = L / BH;
  const int h = head % H, b = head / H;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, lr = lane % 16, g = lane / 16;
  const int half = r / 2;
  const bf16* Ph = Pq + (long)h * r * D;
  const float* Ch = C + (long)head * r * D;

  struct Tile {
    bf16x8 q[4], o[COMBINE ? 4 : 1];
    float4 c[JT], s[JT];
    float lg;
  };
  const int t0 = chunk * chunk_len, t1 = min(N, t0 + chunk_len);
  const int tok0 = 16 * wave + lr;
  auto load_tile = [&](int base, Tile& t) {
    const int tok = min(base + tok0, t1 - 1);
    const long row = ((long)head * N + tok) * D + 8 * g;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) t.q[kc] = *reinterpret_cast<const bf16x8*>(Qn + row + 32 * kc);
    if constexpr (COMBINE) {
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) t.o[kc] = *reinterpret_cast<const bf16x8*>(Os + row + 32 * kc);
      t.lg = logits[(long)b * N + tok];
    }
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {  // pairs past r/2 re-read the last four and meet zero rows of P
      const int jb = min(16 * jt + 4 * g, half - 4);
      t.c[jt] = *reinterpret_cast<const float4*>(cos_tab + (long)tok * ld + jb);
      t.s[jt] = *reinterpret_cast<const float4*>(sin_tab + (long)tok * ld + jb);
    }
  };
  Tile nxt;
  load_tile(t0, nxt);

  // A operand of Phi = P Q^T: even / odd rows of P for pair j = 16 jt + lr.
  __shared__ bf16x8 pfrag[kPLds ? 2 * JT * 4 * 64 : 1];
  bf16x8 pe[kPLds ? 1 : JT][4], po[kPLds ? 1 : JT][4];
  auto p_row = [&](int jt, int par, int kc, int ln) {
    const int j = 16 * jt + ln % 16;
    return j < half ? *reinterpret_cast<const bf16x8*>(Ph + (long)(2 * j + par) * D + 32 * kc + 8 * (ln / 16))
                    : bf16x8{};
  };
  if constexpr (kPLds) {
    for (int e = tid; e < 2 * JT * 4 * 64; e += THREADS)
      pfrag[e] = p_row(e / 512, (e / 256) % 2, (e / 64) % 4, e % 64);
  } else {
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        pe[jt][kc] = p_row(jt, 0, kc, lane);
        po[jt][kc] = p_row(jt, 1, kc, lane);
      }
  }
  // A operand of u^T = C^T q~, staged once per workgroup in LDS in the order lanes read it.
  // Fragment (jt, w) row c holds channel 32(w/2) + 8(c/4) + 4(w%2) + c%4, so the output lane
  // (g, token) of tiles 2p and 2p+1 ends up with the 8 consecutive channels 32p + 8g .. +7 (16-byte
  // O^s loads and O stores). Slots 0-3 = even rows 2(16jt+4g+s), slots 4-7 = odd rows. C = hi + lo
  // (two bf16 terms) keeps the contraction accurate to ~2^-16 relative with fp32 accumulation.
  __shared__ bf16x8 cfrag[2][JT * 8 * 64];
  for (int e = tid; e < JT * 8 * 64; e += THREADS) {
    const int ln = e % 64, w = (e / 64) % 8, jt = e / 512;
    const int c = ln % 16, ch = 32 * (w >> 1) + 8 * (c >> 2) + 4 * (w & 1) + (c & 3), gg = ln / 16;
    bf16x8 hi, lo;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int jj = 16 * jt + 4 * gg + (s & 3);
      const float c = jj < half ? Ch[(long)(2 * jj + (s >> 2)) * D + ch] : 0.f;
      hi[s] = (bf16)c;
      lo[s] = (bf16)(c - (float)hi[s]);
    }
    cfrag[0][e] = hi;
    cfrag[1][e] = lo;
  }
  __syncthreads();

  for (int base = t0; base < t1; base += STEP) {
    const Tile t = nxt;
    load_tile(min(base + STEP, t1 - 1), nxt);
    const int tok = base + tok0;
    if (tok - lr >= t1) continue;  // whole tile past the end (uniform)
    const bool valid = tok < t1;
    f32x4 u[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) u[w] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      f32x4 ye = {0.f, 0.f, 0.f, 0.f}, yo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        ye = mfma16x16x32(kPLds ? pfrag[((2 * jt) * 4 + kc) * 64 + lane] : pe[kPLds ? 0 : jt][kc], t.q[kc], ye);
        yo = mfma16x16x32(kPLds ? pfrag[((2 * jt + 1) * 4 + kc) * 64 + lane] : po[kPLds ? 0 : jt][kc], t.q[kc], yo);
      }
      const float cc[4] = {t.c[jt].x, t.c[jt].y, t.c[jt].z, t.c[jt].w};
      const float ss[4] = {t.s[jt].x, t.s[jt].y, t.s[jt].z, t.s[jt].w};
      float qe[4] = {ye[0], ye[1], ye[2], ye[3]}, qo[4] = {yo[0], yo[1], yo[2], yo[3]};
      feature_tile<PHI>(qe, qo, cc, ss, order);
      bf16x8 bq, bl;  // q~ = hi + lo
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        bq[v] = (bf16)qe[v];
        bq[4 + v] = (bf16)qo[v];
        bl[v] = (bf16)(qe[v] - (float)bq[v]);
        bl[4 + v] = (bf16)(qo[v] - (float)bq[4 + v]);
      }
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const bf16x8 ch = cfrag[0][(jt * 8 + w) * 64 + lane];
        const bf16x8 cl = cfrag[1][(jt * 8 + w) * 64 + lane];
        u[w] = mfma16x16x32(ch, bq, u[w]);
        u[w] = mfma16x16x32(cl, bq, u[w]);
        u[w] = mfma16x16x32(ch, bl, u[w]);
      }
    }
    float ss_u = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w)
#pragma unroll
      for (int v = 0; v < 4; ++v) ss_u = fmaf(u[w][v], u[w][v], ss_u);
    const float inv_u = rsqrtf(rows_sum(ss_u) * (1.0f / D) + eps_lr);
    // Lane holds channels 32p + 8g + 4h + v in u[2p + h][v].
    float scale = inv_u;
    if constexpr (COMBINE) {
      float ss_s = 0.f;
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float x = (float)t.o[p][i];
          ss_s = fmaf(x, x, ss_s);
        }
      const float rs = sqrtf(rows_sum(ss_s) * (1.0f / D) + eps);
      // (O^s / r + g O^lr) r  ==  O^s + (g r / rms(u)) u
      scale = sigmoid(t.lg) * rs * inv_u;
    }
    if (!valid) continue;
    bf16* orow = Out + ((long)head * N + tok) * D + 8 * g;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      bf16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = u[2 * p + (i >> 2)][i & 3];
        o[i] = COMBINE ? (bf16)fmaf(scale, x, (float)t.o[COMBINE ? p : 0][i]) : (bf16)(x * scale);
      }
      *reinterpret_cast<bf16x8*>(orow + 32 * p) = o;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// fp32 readout (+ combine): one wave per 16 tokens. u^T = C^T q~ with contraction step i of lane group g
// = pair 4g + i of a pair tile (even, then odd coordinate), where features_f32 leaves q~; row l%16 of
// channel tile w = channel (l%16) W + w, so C rows are read, and O rows written, in contiguous pieces.
// ------------------------------------------------------------------------------------------------
template <int D, bool COMBINE>
__global__ __launch_bounds__(64) void readout_f32_kernel(
    int N, int H, int r, int ld, int feat, const float* __restrict__ Qn, const float* __restrict__ Pq,
    const float* __restrict__ cos_tab, const float* __restrict__ sin_tab,
    const float* __restrict__ C, float eps_lr, const float* Os, const float* __restrict__ logits,
    float eps, float* Out) {
  constexpr int W = D / 16;
  const int h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x, lr = lane % 16, g = lane / 16;
  const long head = (long)b * gridDim.y + h;
  const int tok = blockIdx.x * 16 + lr, tk = min(tok, N - 1);
  const int half = r / 2, JT = (half + 15) / 16;
  const float* Ch = C + head * (long)r * D + lr * W;
  const long row = (head * N + tk) * (long)D;
  float4 x[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    x[s] = *reinterpret_cast<const float4*>(Qn + row + g * (D / 4) + 4 * s);
  float os[4][W];  // O^s, channels (4g + i) W + w
  float lg = 0.f;
  if constexpr (COMBINE) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int s = 0; s < W / 4; ++s)
        *reinterpret_cast<float4*>(&os[i][4 * s]) =
            *reinterpret_cast<const float4*>(Os + row + (4 * g + i) * W + 4 * s);
    lg = logits[(long)b * N + tk];
  }
  f32x4 u[W];
#pragma unroll
  for (int w = 0; w < W; ++w) u[w] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int jt = 0; jt < JT; ++jt) {
    float4 cv[2][4][W / 4];  // C rows of the lane's pairs, zero past r/2
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* cr = Ch + (long)(2 * min(16 * jt + 4 * g + i, half - 1)) * D;
#pragma unroll
      for (int s = 0; s < W / 4; ++s) {
        cv[0][i][s] = *reinterpret_cast<const float4*>(cr + 4 * s);
        cv[1][i][s] = *reinterpret_cast<const float4*>(cr + D + 4 * s);
      }
    }
    if (16 * jt + 16 > half) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int s = 0; s < W / 4; ++s)
          if (16 * jt + 4 * g + i >= half)
            cv[0][i][s] = cv[1][i][s] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float f[2][4];
    features_f32<D>(Pq + (long)h * r * D, r, jt, x, cos_tab + (long)tk * ld, sin_tab + (long)tk * ld,
                    feat, lane, f[0], f[1]);
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const float4 v = cv[par][i][w / 4];
          const float a = w % 4 == 0 ? v.x : w % 4 == 1 ? v.y : w % 4 == 2 ? v.z : v.w;
          u[w] = mfma_f32(a, f[par][i], u[w]);
        }
  }
  float ss_u = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w)
#pragma unroll
    for (int i = 0; i < 4; ++i) ss_u = fmaf(u[w][i], u[w][i], ss_u);
  const float inv_u = 1.0f / sqrtf(rows_sum(ss_u) / D + eps_lr);
  float rs = 1.f, gate = 0.f;
  if constexpr (COMBINE) {
    float ss_s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int w = 0; w < W; ++w) ss_s = fmaf(os[i][w], os[i][w], ss_s);
    rs = sqrtf(rows_sum(ss_s) / D + eps);
    gate = 1.0f / (1.0f + expf(-lg));
  }
  if (tok >= N) return;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int s = 0; s < W / 4; ++s) {
      float4 o;
      float* op = &o.x;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float ol = u[4 * s + k][i] * inv_u;
        op[k] = COMBINE ? (os[i][4 * s + k] / rs + gate * ol) * rs : ol;
      }
      *reinterpret_cast<float4*>(Out + row + (4 * g + i) * W + 4 * s) = o;
    }
}

// ------------------------------------------------------------------------------------------------
// Gated combine alone: one row of d_h elements per d_h/8 lanes, 8 elements per lane.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void combine_kernel(long rows, int N, int H, int d,
                                                      const T* Os, const T* __restrict__ Olr,
                                                      const float* __restrict__ logits, float eps,
                                                      T* O) {
  const int G = d / 8;
  const long gidx = (long)blockIdx.x * 256 + threadIdx.x;
  const long row = gidx / G;
  const int sub = (int)(gidx % G);
  const bool valid = row < rows;
  float os[8] = {}, ol[8] = {};
  if (valid) {
    load8(Os + row * d + sub * 8, os);
    load8(Olr + row * d + sub * 8, ol);
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) ss = fmaf(os[i], os[i], ss);
  for (int m = 1; m < G; m <<= 1) ss += __shfl_xor(ss, m);
  if (!valid) return;
  const float rs = sqrtf(ss / d + eps);
  const long b = row / ((long)H * N);
  const int n = (int)(row % N);
  const float gate = 1.0f / (1.0f + expf(-logits[b * N + n]));
  float o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (os[i] / rs + gate * ol[i]) * rs;
  store8(O + row * d + sub * 8, o);
}

// ------------------------------------------------------------------------------------------------
// Features q~ (or k~) of every token, fp32 [B, H, N, r], pairs interleaved: one thread per (token,
// pair), fp32 projection, then feature_pair. Not on the module's path: it exposes the features for
// checks and for the positional metrics of the RoPE-placement study (Sec. 5.1).
// ------------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ __launch_bounds__(256) void features_kernel(long total, int N, int H, int r, int ld,
                                                       int feat, const T* __restrict__ X,
                                                       const T* __restrict__ P,
                                                       const float* __restrict__ cos_tab,
                                                       const float* __restrict__ sin_tab,
                                                       float* __restrict__ F) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int half = r / 2;
  const int j = (int)(i % half);
  const long row = i / half;  // (b, h, token)
  const int tok = (int)(row % N), h = (int)((row / N) % H);
  const T* x = X + row * D;
  const T* pe = P + ((long)h * r + 2 * j) * D;
  const T* po = pe + D;
  float e = 0.f, o = 0.f;
  for (int c = 0; c < D; ++c) {
    const float xc = to_f32(x[c]);
    e = fmaf(to_f32(pe[c]), xc, e);
    o = fmaf(to_f32(po[c]), xc, o);
  }
  feature_pair(e, o, cos_tab[(long)tok * ld + j], sin_tab[(long)tok * ld + j], feat);
  F[row * r + 2 * j] = e;
  F[row * r + 2 * j + 1] = o;
}

template <int JT, int PHI>
hipError_t summary_mfma(const Shape& s, const void* Kn, const void* V, const void* Pk, int r,
                        const float* ct, const float* st_, int ld, int order, float* part,
                        int chunk_len, int n_chunks, hipStream_t st) {
  const int total = s.B * s.H * n_chunks;
  const int split = r > 32 * JT ? 2 : 1;  // r = 128 on the two-tile kernel
  const unsigned grid = split == 2 ? (unsigned)((total + 7) / 8 * 16) : (unsigned)total;
  const auto kernel = chunk_len == kSummaryStep ? summary_mfma_kernel<JT, PHI, true>
                                                : summary_mfma_kernel<JT, PHI, false>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, s.N, s.H, r,
                     chunk_len, n_chunks, total, split, ld, order, (const bf16*)Kn, (const bf16*)V,
                     (const bf16*)Pk, ct, st_, part);
  return hipGetLastError();
}

template <int JT>
hipError_t summary_mfma_feat(const Shape& s, const void* Kn, const void* V, const void* Pk, int r,
                             const float* ct, const float* st_, int ld, int feat, float* part,
                             int chunk_len, int n_chunks, hipStream_t st) {
  const auto launch = feat == 0                         ? summary_mfma<JT, kPaper>
                      : (feat & 0xFF) == kPhiIdentity ? summary_mfma<JT, kPhiIdentity>
                      : (feat & 0xFF) == kPhiTanh     ? summary_mfma<JT, kPhiTanh>
                      : (feat & 0xFF) == kPhiRelu     ? summary_mfma<JT, kPhiRelu>
                      : (feat & 0xFF) == kPhiGelu     ? summary_mfma<JT, kPhiGelu>
                                                      : summary_mfma<JT, kPhiSilu>;
  return launch(s, Kn, V, Pk, r, ct, st_, ld, feat >> 8, part, chunk_len, n_chunks, st);
}

template <int JT, bool COMBINE, int PHI>
hipError_t readout_mfma(const Shape& s, const void* Qn, const void* Pq, int r, const float* ct,
                        const float* st_, int ld, int order, const float* C, float eps_lr,
                        const void* Os, const float* logits, float eps, void* Out, hipStream_t st) {
  constexpr int threads = 64 * readout_waves<JT>();
  // workgroups per CU by registers (LDS at r = 128), and what four waves alone cost (40 heads of 15876
  // tokens, r 32: 113 us in 240 workgroups, 105 in 1000; r 64 125 in 240, 116 in 480; 6 of 39732, r 64: 46.7
  // in 750, 43.4 in 468)
  constexpr int per_cu = JT == 1 ? 3 : JT == 2 ? 2 : 1, alone = JT == 1 ? 17 : 19;
  const int chunk_len = chunk_tokens(s, kReadoutWorkgroups, kCus, threads / 4, per_cu, alone);
  const int n_chunks = (s.N + chunk_len - 1) / chunk_len;
  const int total = s.B * s.H * n_chunks;
  hipLaunchKernelGGL((readout_mfma_kernel<JT, COMBINE, PHI>), dim3(total), dim3(threads), 0, st, s.N,
                     s.H, r, chunk_len, n_chunks, total, ld, order, (const bf16*)Qn, (const bf16*)Pq,
                     ct, st_, C, eps_lr, (const bf16*)Os, logits, eps, (bf16*)Out);
  return hipGetLastError();
}

template <int JT, bool COMBINE>
hipError_t readout_mfma_feat(const Shape& s, const void* Qn, const void* Pq, int r,
                             const float* ct, const float* st_, int ld, int feat, const float* C,
                             float eps_lr, const void* Os, const float* logits, float eps,
                             void* Out, hipStream_t st) {
  const auto launch = feat == 0                         ? readout_mfma<JT, COMBINE, kPaper>
                      : (feat & 0xFF) == kPhiIdentity ? readout_mfma<JT, COMBINE, kPhiIdentity>
                      : (feat & 0xFF) == kPhiTanh     ? readout_mfma<JT, COMBINE, kPhiTanh>
                      : (feat & 0xFF) == kPhiRelu     ? readout_mfma<JT, COMBINE, kPhiRelu>
                      : (feat & 0xFF) == kPhiGelu     ? readout_mfma<JT, COMBINE, kPhiGelu>
                                                      : readout_mfma<JT, COMBINE, kPhiSilu>;
  return launch(s, Qn, Pq, r, ct, st_, ld, feat >> 8, C, eps_lr, Os, logits, eps, Out, st);
}

template <bool COMBINE>
hipError_t readout_dispatch(const Shape& s, const void* Qn, const void* Pq, int r, const float* ct,
                            const float* st_, int ld, int feat, const float* C, float eps_lr,
                            const void* Os, const float* logits, float eps, void* Out,
                            hipStream_t st) {
  if (s.bf16) {
    if (r <= 32)
      return readout_mfma_feat<1, COMBINE>(s, Qn, Pq, r, ct, st_, ld, feat, C, eps_lr, Os, logits,
                                           eps, Out, st);
    if (r <= 64)
      return readout_mfma_feat<2, COMBINE>(s, Qn, Pq, r, ct, st_, ld, feat, C, eps_lr, Os, logits,
                                           eps, Out, st);
    return readout_mfma_feat<4, COMBINE>(s, Qn, Pq, r, ct, st_, ld, feat, C, eps_lr, Os, logits,
                                         eps, Out, st);
  }
  const auto kernel = s.d == 64 ? readout_f32_kernel<64, COMBINE> : readout_f32_kernel<128, COMBINE>;
  hipLaunchKernelGGL(kernel, dim3((s.N + 15) / 16, s.H, s.B), dim3(64), 0, st, s.N, s.H, r, ld, feat,
                     (const float*)Qn, (const float*)Pq, ct, st_, C, eps_lr, (const float*)Os, logits,
                     eps, (float*)Out);
  return hipGetLastError();
}

}  // namespace

int summary_chunks(const Shape& s, int r) {
  const int len = summary_chunk_len(s, r);
  return (s.N + len - 1) / len;
}

size_t summary_workspace_bytes(const Shape& s, int r) {
  return (size_t)s.B * s.H * summary_chunks(s, r) * (size_t)(r * s.d + r) * sizeof(float);
}

hipError_t launch_lowrank_summary(const Shape& s, const void* Kn, const void* V, const void* Pk,
                                  int r, const float* cos_tab, const float* sin_tab, int ld,
                                  int feat, float* C, float* z, void* ws, hipStream_t st) {
  const int chunk_len = summary_chunk_len(s, r);
  const int n_chunks = (s.N + chunk_len - 1) / chunk_len;
  float* part = (float*)ws;
  hipError_t e;
  if (s.bf16) {
    if (r <= 32)
      e = summary_mfma_feat<1>(s, Kn, V, Pk, r, cos_tab, sin_tab, ld, feat, part, chunk_len,
                               n_chunks, st);
    else if (r <= 64)
      e = summary_mfma_feat<2>(s, Kn, V, Pk, r, cos_tab, sin_tab, ld, feat, part, chunk_len,
                               n_chunks, st);
    else  // r = 128: two workgroups of two pair tiles each per chunk
      e = summary_mfma_feat<2>(s, Kn, V, Pk, r, cos_tab, sin_tab, ld, feat, part, chunk_len,
                               n_chunks, st);
  } else {
    const auto kernel = s.d == 64 ? summary_f32_kernel<64> : summary_f32_kernel<128>;
    hipLaunchKernelGGL(kernel, dim3(n_chunks, s.H, s.B), dim3(256), 0, st, s.N, s.H, r, chunk_len,
                       n_chunks, ld, feat, (const float*)Kn, (const float*)V, (const float*)Pk, cos_tab,
                       sin_tab, part);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  const int per = r * s.d + r;
  return launch_chunk_reduce(per, r * s.d, per, 1, s.B * s.H, n_chunks, part, C, z, st);
}

hipError_t launch_lowrank_readout(const Shape& s, const void* Qn, const void* Pq, int r,
                                  const float* cos_tab, const float* sin_tab, int ld, int feat,
                                  const float* C, float eps_lr, const void* Os,
                                  const float* logits, float eps, void* Out, hipStream_t st) {
  if (Os)
    return readout_dispatch<true>(s, Qn, Pq, r, cos_tab, sin_tab, ld, feat, C, eps_lr, Os, logits,
                                  eps, Out, st);
  return readout_dispatch<false>(s, Qn, Pq, r, cos_tab, sin_tab, ld, feat, C, eps_lr, nullptr,
                                 nullptr, 0.f, Out, st);
}

hipError_t launch_lowrank_features(const Shape& s, const void* X, const void* P, int r,
                                   const float* cos_tab, const float* sin_tab, int ld, int feat,
                                   float* F, hipStream_t st) {
  const long total = (long)s.B * s.H * s.N * (r / 2);
  const dim3 grid((unsigned)((total + 255) / 256));
  if (s.bf16) {
    if (s.d == 64)
      hipLaunchKernelGGL((features_kernel<bf16, 64>), grid, dim3(256), 0, st, total, s.N, s.H, r,
                         ld, feat, (const bf16*)X, (const bf16*)P, cos_tab, sin_tab, F);
    else
      hipLaunchKernelGGL((features_kernel<bf16, 128>), grid, dim3(256), 0, st, total, s.N, s.H, r,
                         ld, feat, (const bf16*)X, (const bf16*)P, cos_tab, sin_tab, F);
  } else {
    if (s.d == 64)
      hipLaunchKernelGGL((features_kernel<float, 64>), grid, dim3(256), 0, st, total, s.N, s.H, r,
                         ld, feat, (const float*)X, (const float*)P, cos_tab, sin_tab, F);
    else
      hipLaunchKernelGGL((features_kernel<float, 128>), grid, dim3(256), 0, st, total, s.N, s.H, r,
                         ld, feat, (const float*)X, (const float*)P, cos_tab, sin_tab, F);
  }
  return hipGetLastError();
}

hipError_t launch_combine(const Shape& s, const void* Os, const void* Olr, const float* logits,
                          float eps, void* O, hipStream_t st) {
  const long rows = (long)s.B * s.H * s.N;
  const long threads = rows * (s.d / 8);
  const dim3 grid((unsigned)((threads + 255) / 256));
  if (s.bf16)
    hipLaunchKernelGGL(combine_kernel<bf16>, grid, dim3(256), 0, st, rows, s.N, s.H, s.d,
                       (const bf16*)Os, (const bf16*)Olr, logits, eps, (bf16*)O);
  else
    hipLaunchKernelGGL(combine_kernel<float>, grid, dim3(256), 0, st, rows, s.N, s.H, s.d,
                       (const float*)Os, (const float*)Olr, logits, eps, (float*)O);
  return hipGetLastError();
}

}  // namespace rola
