// Backward pass of the block-sparse attention (the sparse branch's part of fine-tuning, Sec. 4.5):
// from dO^s, the saved O^s and the forward's log-sum-exp, the gradients dQ^r, dK^r, dV of
// O^s = softmax(Q^r K^r^T * scale) V restricted to the selected key blocks (Algorithm step 4). The
// block lists are constant (the selection is piecewise constant in Q^r, K^r).
//
// With P = exp(S*scale - lse) and D_q = sum_c dO^s_qc O^s_qc:  dP = dO V^T,  dS = P (dP - D),
// dQ = scale dS K,  dK = scale dS^T Q,  dV = P^T dO.  Two passes, each recomputing S and P:
//   dQ                 the forward's attention kernel in its dQ mode, per query block (or pair) over its
//                      own list (a kernel of its own, which handed dS to the transposed product through
//                      LDS, took 0.93 ms where this takes 0.88: 5 heads, 67545 tokens, blocks of 128);
//   sparse_dkv_kernel  per key block, walking the query blocks that selected it (lists transposed by
//                      bwd_reverse_kernel) in 32-query steps: one role of waves holds the keys' K
//                      (S, P, dV), the other their V (dP, dS, dK) and takes P from the first one
//                      step later; Q and dO rows (and the queries' lse and D) through four LDS
//                      stages: one read back (role 1), one current, one ahead, one in flight.
// Products on v_mfma_f32_32x32x16_bf16. S and dP come out with one lane per key and the 32 queries
// in its registers; the products that contract over queries (dK, dV) take their other operand through
// the transposing LDS read ds_read_b64_tr_b16, in the order the registers hold the contracted index (as
// the forward's P V). Tiles are stored with a swizzle that keeps both the row reads and the transposing
// reads free of bank conflicts. Gradients are fp32.
#include "common.h"
#include "launch.h"

namespace rola {
namespace {

constexpr int kBSub = 32;     // queries per sub-tile
constexpr int kLsePad = 128;  // zero entries after the packed lse/D array: a sub-tile of the last
                              // query block reads up to block - 1 entries past the last query
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma32(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}


// D_q = sum_c dO_qc O_qc and the forward's lse, packed per query: lseD[q] = {lse_q, D_q}. 16 lanes
// per query row, 8 channels each. The array is padded by kLsePad zero entries (read past the end).
__global__ __launch_bounds__(256) void bwd_rowdot_kernel(long rows, const bf16* __restrict__ O,
                                                         const bf16* __restrict__ dO,
                                                         const float* __restrict__ lse,
                                                         float2* __restrict__ lseD) {
  const long row = ((long)blockIdx.x * 256 + threadIdx.x) / 16;
  const int part = threadIdx.x % 16;
  float s = 0.f;
  if (row < rows) {
    float a[8], b[8];
    load8(O + row * 128 + part * 8, a);
    load8(dO + row * 128 + part * 8, b);
#pragma unroll
    for (int i = 0; i < 8; ++i) s = fmaf(a[i], b[i], s);
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off, 16);
  if (part == 0) {
    if (row < rows) lseD[row] = make_float2(lse[row], s);
    else if (row < rows + kLsePad) lseD[row] = make_float2(0.f, 0.f);
  }
}

// Membership bitmaps of the block lists: bits[head][I][J / 32] bit J % 32. Each row is built in
// LDS (words * 4 bytes of dynamic shared memory) and written whole, so no clearing pass is needed.
__global__ __launch_bounds__(64) void bwd_bits_kernel(int nb, int keep, int words,
                                                      const int32_t* __restrict__ idx,
                                                      uint32_t* __restrict__ bits) {
  extern __shared__ uint32_t row_bits[];
  const long row = blockIdx.x;  // head * nb + I
  for (int w = threadIdx.x; w < words; w += 64) row_bits[w] = 0u;
  __syncthreads();
  for (int k = threadIdx.x; k < keep; k += 64) {
    const int J = idx[row * keep + k];
    if ((unsigned)J < (unsigned)nb) atomicOr(&row_bits[J >> 5], 1u << (J & 31));
  }
  __syncthreads();
  for (int w = threadIdx.x; w < words; w += 64) bits[row * words + w] = row_bits[w];
}

// Walk order of the transposed lists: query blocks by increasing bit-reversed index over the smallest
// power of two >= nb, a low-discrepancy order in which every list's entries spread evenly. Key
// blocks whose lists are about equally long then sit on about the same query blocks after the same
// number of steps, and bwd_order_kernel has the dK/dV workgroups that run at once take key blocks
// of about equal list length: concurrent workgroups share Q and dO rows in L2.
__host__ __device__ inline int rev_walk_bits(int nb) {
  int k = 1;
  while ((1 << k) < nb) ++k;
  return k;
}

// Transposed lists: rev[head][J] = count, then the query blocks I that selected J in walk order.
// One workgroup per (head, 32 key blocks): the bitmap column of the 32 key blocks goes to LDS in walk
// order ([1 << kb] words), then each wave collects a key block at a time, 64 walk positions per step
// (ballot and prefix count). With one lane per key block walking all positions the serial chain took
// 47 us at 12 heads of 512 blocks and 55 at 5 of 528; 12 and 20 now.
__global__ __launch_bounds__(256) void bwd_reverse_kernel(int nb, int words, int kb,
                                                          const uint32_t* __restrict__ bits,
                                                          int32_t* __restrict__ rev) {
  extern __shared__ uint32_t col[];  // [1 << kb]: bit j of col[p] = query block brev(p) selected 32w + j
  const long head = blockIdx.x / words;
  const int w = (int)(blockIdx.x % words), tid = threadIdx.x, lane = tid % 64;
  const int np = 1 << kb;
  auto block_at = [&](int p) { return (int)(__brev((unsigned)p) >> (32 - kb)); };  // an involution
  for (int I = tid; I < np; I += 256)
    col[block_at(I)] = I < nb ? bits[(head * nb + I) * words + w] : 0u;
  __syncthreads();
  for (int j = wave_uniform(tid / 64); j < 32; j += 4) {
    const int J = 32 * w + j;
    if (J >= nb) break;
    int32_t* out = rev + (head * nb + J) * (long)(nb + 1);
    int cnt = 0;
    for (int p0 = 0; p0 < np; p0 += 64) {
      const int p = p0 + lane;
      const bool has = p < np && ((col[p] >> j) & 1u);
      const uint64_t m = __ballot(has);
      if (has) out[1 + cnt + __popcll(m & ((1ull << lane) - 1))] = block_at(p);
      cnt += __popcll(m);
    }
    if (lane == 0) out[0] = cnt;
  }
}

// Order of the key blocks for the dK/dV workgroups: longer lists first (equal lengths by ascending
// J), order[head][rank] = J. One workgroup per (head, 64 key blocks): every list length of the head
// goes to LDS, and four threads rank one key block against a quarter of them each.
constexpr int kOrderBlocks = 64;
__global__ __launch_bounds__(4 * kOrderBlocks) void bwd_order_kernel(int nb, int chunks,
                                                                     const int32_t* __restrict__ rev,
                                                                     int32_t* __restrict__ order) {
  extern __shared__ int32_t len[];  // [nb]
  __shared__ int32_t part[4][kOrderBlocks];
  const long head = blockIdx.x / chunks;
  const int tid = threadIdx.x, jl = tid % kOrderBlocks, quarter = wave_uniform(tid / kOrderBlocks);
  const int J = (int)(blockIdx.x % chunks) * kOrderBlocks + jl;
  for (int K = tid; K < nb; K += 4 * kOrderBlocks) len[K] = rev[(head * nb + K) * (long)(nb + 1)];
  __syncthreads();
  const int e = len[min(J, nb - 1)];
  const int per = (nb + 3) / 4, k1 = min(nb, (quarter + 1) * per);
  int rank = 0;
#pragma unroll 8
  for (int K = quarter * per; K < k1; ++K) rank += len[K] > e || (len[K] == e && K < J);
  part[quarter][jl] = rank;
  __syncthreads();
  if (quarter == 0 && J < nb)
    order[head * nb + part[0][jl] + part[1][jl] + part[2][jl] + part[3][jl]] = J;
}

// ---- dK, dV: one workgroup per (b, h, key block) ------------------------------------------------
// Two roles of BLK/32 waves each over the same 32-key column tiles. Role 0 holds the keys' K and
// computes S, P = exp2(S scale log2e - lse) and dV += dO^T P; role 1 holds their V and computes
// dP = dO V^T, dS = P (dP - D) and dK += Q^T dS, taking P from role 0 through LDS one step later
// (double-buffered, so one barrier per step serves the tile stages and the hand-over). A wave then
// needs one B operand set and one accumulator set (a wave doing both needs twice that, more than
// half the register file, and the compiler then moves accumulators between the two register files
// every step), so two waves run per SIMD. A step takes 32 queries. P goes over as fp16: it lies
// in [0, 1], where fp16's relative error (2^-11; absolute 2^-25 below 2^-14) is an eighth of the
// bf16 rounding dS takes next.
//
// What bounds it: per step a wave reads 16 KB of operands from LDS for 16 products, so the LDS and the
// matrix cores have about the same work (140 and 128 cycles per wave and step), and all waves of a
// workgroup leave the barrier together. Operands are therefore read a product ahead: the row operand of
// the next step while this step's second product runs, the transposed one while the first does, and
// the second half's softmax (or dS) between the first half's products. Read at the head of their own
// step instead, the eight waves of a CU waited for 128 KB of LDS reads while the matrix cores idled: 12
// heads of 512 blocks of 64 1.73 -> 1.46 ms, 5 of 528 blocks of 128 1.79 -> 1.37 (matrix cores busy 29 %
// -> 40 %).
//
// Workgroups take a head's key blocks longest list first
// (bwd_order_kernel) and walk each list in the bit-reversed order, so that workgroups running at
// the same time sit on about the same query blocks and share their Q and dO rows in L2.
//
// Which XCD takes which key block (workgroups are dealt to the XCDs round-robin): each XCD takes
// heads / 8 whole heads, and the key blocks of the heads that are left are dealt over all XCDs. With
// contiguous eighths of everything instead, an XCD of a few-headed problem got the long lists of a head
// and its neighbour the short ones (5 heads, 528 blocks of 128: 2.10 ms; 12 heads, 512 blocks of 64:
// 1.73 ms).
// LDS stages of sparse_dkv_kernel: 32 Q rows, 32 dO rows, lse/D (17 KB). A fifth, which 128-token blocks
// have room for, cost 1 % (5 heads of 67545 tokens).
constexpr int kDkvNbuf = 4;
// Workgroups of the grid, and the place (head * nb + rank) workgroup wg takes, -1 for none.
__host__ __device__ inline int dkv_grid(int heads, int nb) {
  return kNumXcd * (heads / kNumXcd * nb + (heads % kNumXcd * nb + kNumXcd - 1) / kNumXcd);
}
__host__ __device__ inline int dkv_place(int wg, int heads, int nb) {
  const int xcd = wg % kNumXcd, i = wg / kNumXcd, whole = heads / kNumXcd * nb;
  if (i < whole) return xcd * whole + i;
  const int d = (i - whole) * kNumXcd + xcd;
  return d < heads % kNumXcd * nb ? kNumXcd * whole + d : -1;
}

template <int BLK>
__global__ __launch_bounds__(BLK * 4) __attribute__((amdgpu_waves_per_eu(2, 2)))
void sparse_dkv_kernel(
    int N, int nb, int heads, const int32_t* __restrict__ rev, float scale_log2, float scale,
    const bf16* __restrict__ Q, const bf16* __restrict__ K, const bf16* __restrict__ V,
    const bf16* __restrict__ dO, const float2* __restrict__ lseD, const int32_t* __restrict__ order,
    GradTables acc_tab, float* __restrict__ dK, float* __restrict__ dV) {
  constexpr int D = 128, NKW = BLK / 32, NW = 2 * NKW;
  constexpr int TILE = kBSub * D * 2;          // 32 rows of 256 bytes
  constexpr int STAGE = 2 * TILE + 1024;       // Q, dO, then lse/D of the 32 queries (256 B used)
  constexpr int DPW = 2 * (TILE / 1024) / NW;  // 1 KB tile loads per wave and step
  constexpr int SUBS = BLK / kBSub;            // steps per query block
  constexpr int PBUF = NKW * 2048;             // P of a step, fp16: per key tile 16 values a lane
  constexpr int NBUF = kDkvNbuf;
  constexpr int AHEAD = NBUF - 3;              // stages in flight: three are read (one back, one on)
  static_assert(DPW >= 1 && 2 * (TILE / 1024) % NW == 0, "64- or 128-key blocks");
  static_assert(AHEAD == 1, "every load in flight is the next step's: the waits below are for all of them");
  __shared__ __attribute__((aligned(1024))) char lds[NBUF * STAGE + 2 * PBUF];

  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  const int L = dkv_place(blockIdx.x, heads, nb);
  if (L < 0) return;
  const long head = L / nb;
  const int J = ((const_i32)order)[L];  // key blocks of one head, longer lists first
  const int tid = threadIdx.x, lane = tid % 64, hh = lane / 32;
  const int wave = wave_uniform(tid / 64);
  const int role = wave / NKW, kw = wave % NKW;
  const int key = J * BLK + kw * 32 + lane % 32;  // B-operand column of this lane
  const bool kvalid = key < N;
  const long hoff = head * (long)N * D;
  const char* Qh = reinterpret_cast<const char*>(Q + hoff);
  const char* dOh = reinterpret_cast<const char*>(dO + hoff);
  const const_i32 rl = (const_i32)(rev + (head * nb + J) * (long)(nb + 1));
  const int E = rl[0];
  const int T = E * SUBS;

  const bf16* bsrc = (role ? V : K) + hoff + (long)key * D + 8 * hh;
  bf16x8 bf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
    bf[s] = kvalid ? *reinterpret_cast<const bf16x8*>(bsrc + 16 * s) : bf16x8{};
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0)

  f32x16 acc[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) acc[w] = f32x16{};

  // Tile loads: load g = wave * DPW + i moves rows 4(g % 8) .. +3 of Q (g < 8) or dO (g >= 8).
  uint32_t dsrc[DPW];
#pragma unroll
  for (int i = 0; i < DPW; ++i) {
    const int g = wave * DPW + i, row = 4 * (g % 8) + lane / 16, pos = lane % 16;
    dsrc[i] = row * D * 2 + ((pos ^ bw_swizzle(row)) << 4);
  }
  const uint32_t lds0 = lds_address(lds);
  const char* lsebase = reinterpret_cast<const char*>(lseD + head * (long)N);
  auto query0 = [&](int t) {  // t >= 0
    return rl[1 + (unsigned)t / SUBS] * BLK + (int)((unsigned)t % SUBS) * kBSub;
  };
  auto issue = [&](int q0, int buf) {  // DPW loads per wave, and wave 0 one more (lse/D)
    const uint32_t dst = lds0 + buf * STAGE;
    if (q0 + kBSub <= N) {  // every row of the tile exists: one scalar base per tensor
      const uint32_t base = (uint32_t)q0 * (D * 2);
#pragma unroll
      for (int i = 0; i < DPW; ++i) {
        const int g = wave * DPW + i;
        dma16((g < 8 ? Qh : dOh) + base, dsrc[i], dst + (g / 8) * TILE + (g % 8) * 1024);
      }
    } else {
#pragma unroll
      for (int i = 0; i < DPW; ++i) {
        const int g = wave * DPW + i, r = 4 * (g % 8) + lane / 16;
        const uint32_t rowoff = (uint32_t)(min(q0 + r, N - 1) - r) * (D * 2);  // rows past N: N-1
        dma16(g < 8 ? Qh : dOh, rowoff + dsrc[i], dst + (g / 8) * TILE + (g % 8) * 1024);
      }
    }
    // lse, D of the 32 queries (256 bytes; lanes 16-63 repeat lanes 0-15): the array is padded by
    // kLsePad entries, and rows past N are masked below
    if (wave == 0) dma16(lsebase, (uint32_t)(q0 * 8 + (lane % 16) * 16), dst + 2 * TILE);
  };

  char* pbase = lds + NBUF * STAGE + kw * 2048 + lane * 16;  // + buffer * PBUF + u * 1024
  int issued = 0;
#pragma unroll
  for (int j = 0; j <= AHEAD; ++j)
    if (j < T) issue(query0(j), j), ++issued;
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0)
  __syncthreads();
  // Iteration t: role 0 takes step t, role 1 step t - 1. Each role has a loop of its own (its stage
  // offsets are then constants), of whole turns of NBUF iterations (an exit between them costs
  // registers); both meet the same barriers.
  auto walk = [&](auto role_tag) {
    constexpr int ROLE = decltype(role_tag)::value;
    // Row operands (Q for role 0, dO for role 1) of the wave's next step.
    bf16x8 fa[8];
    auto row_operands = [&](int stage) {
#pragma unroll
      for (int s = 0; s < 8; ++s) fa[s] = row_frag(lds + stage * STAGE + ROLE * TILE, lane % 32, s, hh);
    };
    if (ROLE == 0) row_operands(0);
    for (int t = 0; t <= T;) {
#pragma unroll
      for (int b = 0; b < NBUF; ++b, ++t) {
        // The first query of this step's tile and of the tile whose loads it issues, read from the
        // list before the wait and the barrier (indices clamped into the list; pinned in SGPRs, or
        // the compiler sinks the scalar loads behind the barrier).
        int qcur = query0(max(0, min(t, T - 1))), qiss = query0(max(0, min(issued, T - 1)));
        asm volatile("" : "+s"(qcur), "+s"(qiss));
        __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt(0): stage t + 1 has landed
        __syncthreads();
        if (issued < T) issue(qiss, (b + 1 + AHEAD) % NBUF), ++issued;
        const int step = t - ROLE;
        if (step >= 0 && step < T) {
          const char* stage = lds + (ROLE ? (b + NBUF - 1) % NBUF : b) * STAGE;
          const float* lt = reinterpret_cast<const float*>(stage + 2 * TILE) + ROLE;
          char* pb = pbase + ((b + ROLE) % 2) * PBUF;  // role 0 writes step t's, role 1 reads t - 1's
          // The transposed operand of the second product and the step's other LDS values are read
          // while the first product runs, the next step's row operand while the second does.
          bf16x8 fb[8];
#pragma unroll
          for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int u = 0; u < 2; ++u) fb[2 * w + u] = tr_frag(stage + (1 - ROLE) * TILE, w, u, lane);
          float lv[16];  // lse (role 0) or D (role 1) of the step's queries
#pragma unroll
          for (int k = 0; k < 16; ++k) lv[k] = lt[2 * (8 * (k / 4) + 4 * hh + k % 4)];
          // S (role 0) or dP (role 1): one lane per key; rows 8j + 4(l/32) + i are the step's queries
          f32x16 X = f32x16{};
#pragma unroll
          for (int s = 0; s < 8; ++s) X = mfma32(fa[s], bf[s], X);
          f16x8 ph[2];
          if constexpr (ROLE == 1) {
            ph[0] = *reinterpret_cast<const f16x8*>(pb);
            ph[1] = *reinterpret_cast<const f16x8*>(pb + 1024);
          }
          __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          row_operands(ROLE ? b : (b + 1) % NBUF);
          if (ROLE == 0 && qcur + kBSub > N) {  // ragged last query block (uniform): P = 0 past N
#pragma unroll
            for (int k = 0; k < 16; ++k)
              lv[k] = qcur + 8 * (k / 4) + 4 * hh + k % 4 < N ? lv[k] : __builtin_inff();
          }
          __builtin_amdgcn_sched_barrier(0);
          // dV^T += dO^T P (role 0) or dK^T += Q^T dS (role 1), the transposed operand in the order
          // the registers hold the queries, in two halves: the second half's P or dS is computed
          // between the first half's products.
          bf16x8 b2[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              if constexpr (ROLE == 0) {
                const float p = __builtin_amdgcn_exp2f(fmaf(X[8 * u + k], scale_log2, -lv[8 * u + k]));
                b2[u][k] = (bf16)p;
                ph[u][k] = (_Float16)p;
              } else {
                b2[u][k] = (bf16)((float)ph[u][k] * (X[8 * u + k] - lv[8 * u + k]));
              }
            }
            if constexpr (ROLE == 0) *reinterpret_cast<f16x8*>(pb + 1024 * u) = ph[u];
#pragma unroll
            for (int w = 0; w < 4; ++w) acc[w] = mfma32(fb[2 * w + u], b2[u], acc[w]);
          }
          __builtin_amdgcn_sched_group_barrier(0x402, 28, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x402, 7, 0);
          }
        } else if (step < 0) {
          row_operands(0);
        }
      }
    }
  };
  if (role)
    walk(std::integral_constant<int, 1>{});
  else
    walk(std::integral_constant<int, 0>{});
  if (kvalid) {  // dV^T (role 0), dK^T (role 1): lane = key, rows = channels 32w + 8j + 4(l/32) + i
    float* out = (role ? dK : dV) + hoff + (long)key * D;
    const float f = role ? scale : 1.f;
    if (acc_tab.cos_tab) {  // dK^n += R(p)^T dK^r, dV += dV
      const uint32_t off = (uint32_t)key * (uint32_t)acc_tab.ld;
      store_grad_row<true>(out, acc, f, hh, role ? acc_tab.cos_tab + off : nullptr,
                           role ? acc_tab.sin_tab + off : nullptr);
    } else {
      store_grad_row<false>(out, acc, f, hh, nullptr, nullptr);
    }
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace: [lse, D per query][bitmaps][transposed lists][key-block order][the attention
// workspace of the dQ pass (pairs, merged lists, queue counters; none with 128-token blocks)].
struct BwdWs {
  size_t lsed, bits, rev, order, dq;
};
BwdWs bwd_layout(const Shape& s, int block, int keep) {
  const size_t heads = (size_t)s.B * s.H, nb = num_blocks(s.N, block), words = (nb + 31) / 32;
  return {align256((heads * s.N + kLsePad) * sizeof(float2)), align256(heads * nb * words * 4),
          align256(heads * nb * (nb + 1) * 4), align256(heads * nb * 4),
          align256(sparse_workspace_bytes(s, block, keep))};
}

static_assert(kMaxBlocks * sizeof(int32_t) <= 32768, "one LDS word per block of a head, beside the kernels' own");

template <int BLK>
hipError_t launch_bwd(const Shape& s, const void* Qr, const void* Kr, const void* V, int keep,
                      const int32_t* idx, float scale, const void* Os, const float* lse,
                      const void* dOs, const GradTables& acc, float* dQ, float* dK, float* dV, void* ws,
                      hipStream_t st) {
  const int nb = num_blocks(s.N, BLK), words = (nb + 31) / 32;
  const long heads = (long)s.B * s.H, rows = heads * s.N;
  const BwdWs lay = bwd_layout(s, BLK, keep);
  float2* lseD = (float2*)ws;
  uint32_t* bits = (uint32_t*)((char*)ws + lay.lsed);
  int32_t* rev = (int32_t*)((char*)ws + lay.lsed + lay.bits);
  int32_t* order = (int32_t*)((char*)ws + lay.lsed + lay.bits + lay.rev);
  const long rd_threads = (rows + kLsePad) * 16;
  hipLaunchKernelGGL(bwd_rowdot_kernel, dim3((unsigned)((rd_threads + 255) / 256)), dim3(256), 0,
                     st, rows, (const bf16*)Os, (const bf16*)dOs, lse, lseD);
  hipLaunchKernelGGL(bwd_bits_kernel, dim3((unsigned)(heads * nb)), dim3(64), words * sizeof(uint32_t),
                     st, nb, keep, words, idx, bits);
  const int kb = rev_walk_bits(nb);
  hipLaunchKernelGGL(bwd_reverse_kernel, dim3((unsigned)(heads * words)), dim3(256),
                     sizeof(uint32_t) << kb, st, nb, words, kb, (const uint32_t*)bits, rev);
  const int ochunks = (nb + kOrderBlocks - 1) / kOrderBlocks;
  hipLaunchKernelGGL(bwd_order_kernel, dim3((unsigned)(heads * ochunks)), dim3(4 * kOrderBlocks),
                     nb * sizeof(int32_t), st, nb, ochunks, (const int32_t*)rev, order);
  const float sl = scale * 1.4426950408889634f;
  // dQ on the attention kernel (block 64: paired, queued)
  const hipError_t e2 = launch_sparse_dq(s, Qr, Kr, V, BLK, keep, idx, scale, dOs, lseD, acc, dQ,
                                         (char*)ws + lay.lsed + lay.bits + lay.rev + lay.order, st);
  if (e2 != hipSuccess) return e2;
  hipLaunchKernelGGL(sparse_dkv_kernel<BLK>, dim3(dkv_grid((int)heads, nb)), dim3(BLK * 4), 0,
                     st, s.N, nb, (int)heads,
                     (const int32_t*)rev, sl, scale, (const bf16*)Qr, (const bf16*)Kr,
                     (const bf16*)V, (const bf16*)dOs, (const float2*)lseD, (const int32_t*)order,
                     acc, dK, dV);
  return hipGetLastError();
}

}  // namespace

size_t sparse_backward_workspace_bytes(const Shape& s, int block, int keep) {
  if (!s.bf16 || s.d != 128 || (block != 64 && block != 128)) return 0;
  const BwdWs w = bwd_layout(s, block, keep);
  return w.lsed + w.bits + w.rev + w.order + w.dq;
}

hipError_t launch_sparse_backward(const Shape& s, const void* Qr, const void* Kr, const void* V,
                                  int block, int keep, const int32_t* idx, float scale,
                                  const void* Os, const float* lse, const void* dOs,
                                  const GradTables& acc, float* dQ, float* dK, float* dV, void* ws,
                                  hipStream_t st) {
  if (block == 64)
    return launch_bwd<64>(s, Qr, Kr, V, keep, idx, scale, Os, lse, dOs, acc, dQ, dK, dV, ws, st);
  return launch_bwd<128>(s, Qr, Kr, V, keep, idx, scale, Os, lse, dOs, acc, dQ, dK, dV, ws, st);
}

}  // namespace rola
