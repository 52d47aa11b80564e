// Internal launcher interface between the C ABI (rola_api.cpp) and the kernels (*.hip).
// Launchers assume their arguments were validated by the ABI layer; they only enqueue work.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rola {

struct Shape {
  int B, H, N, d;      // activations [B, H, N, d]
  int T, Hs, Ws;       // latent grid, N == T*Hs*Ws
  bool bf16;           // element type: bf16 (true) or fp32
};

inline int num_blocks(int N, int block) { return (N + block - 1) / block; }

constexpr int kMaxBlocks = 8192;  // blocks per head that the calls with a block size take

// Tokens per workgroup of the low-rank kernels, which give each (b, h) to several workgroups of
// consecutive tokens: a multiple of `step`, at least what about `workgroups` workgroups give (and no
// more of them than that), chosen so that whole rounds of `slots` workgroups cost least, a round lasting
// as long as its chunk plus its set-up (about `step` tokens). A round is one workgroup per CU, also where a
// CU holds two or three: they share its bandwidth and its SIMDs, so what counts is the CU with the most of
// them (summary, r 32, 36 heads of 2079 tokens: 324 workgroups 20.4 us, 180 of twice the length 16.4; readout,
// r 16, 12 heads of 8400: 528 22.3, 396 19.9, 228 18.9; 40 heads of 32760, r 64: the branch 425 us with the
// summary in 4.1 rounds, 383 in one). `alone`: what a token costs, in sixteenths, in a round that a CU which
// could hold `per_cu` workgroups has to itself, with nothing to hide its latencies.
constexpr int kCus = 256;
inline int chunk_tokens(const Shape& s, long workgroups, long slots, int step, int per_cu = 1,
                        int alone = 16) {
  const long heads = (long)s.B * s.H;
  const long want = heads < workgroups ? workgroups / heads : 1;
  const long least = ((s.N + want - 1) / want + step - 1) / step * step;
  long best = least, best_cost = -1;
  // of the lengths that give the same number of chunks the shortest costs least: one turn per number, up
  // to one chunk or 8 times the least length (a turn per multiple of `step` came to a thousand 64-bit
  // divisions per call with 1024 heads)
  for (long len = least; len <= 8 * least;) {
    const long chunks = (s.N + len - 1) / len, rounds = (heads * chunks + slots - 1) / slots;
    const long cost = (len + step) * (16 * rounds + (per_cu > 1 && rounds % per_cu == 1 ? alone - 16 : 0));
    if (best_cost < 0 || cost < best_cost) {
      best = len;
      best_cost = cost;
    }
    if (chunks == 1) break;
    len = ((s.N + chunks - 2) / (chunks - 1) + step - 1) / step * step;
  }
  return (int)best;
}

// rope.hip
hipError_t launch_rope_tables(const Shape& s, int dt, int dy, int dx, double base, int ot, int oy,
                              int ox, float* cos_tab, float* sin_tab, hipStream_t st);
hipError_t launch_rope_apply(const Shape& s, const void* X, const float* cos_tab,
                             const float* sin_tab, int ld, void* Xr, hipStream_t st);
// fp32 [B, H, N, d]: dX += R(p)^T dY (rotate) or dX += dY.
hipError_t launch_rope_grad(const Shape& s, const float* dY, const float* cos_tab,
                            const float* sin_tab, int ld, bool rotate, float* dX, hipStream_t st);

// select.hip
size_t select_workspace_bytes(const Shape& s, int block);
hipError_t launch_block_select(const Shape& s, const void* Qr, const void* Kr, int block, int keep,
                               int32_t* idx, void* ws, hipStream_t st);
// Means of the rotated rows per block from Q^n or K^n and the tables (fp32 [B, H, nb, d]); the
// rotated rows also go to Xr unless it is null. Built for d = 128 (rope_pool_supported). nmax, if
// not null: per block the largest fp32 norm of its (rotated, rounded) rows, [B, H, nb].
bool rope_pool_supported(const Shape& s, int block);
// Block means of an already rotated X (the pooling of launch_block_select alone).
hipError_t launch_block_pool(const Shape& s, const void* X, int block, float* means, float* nmax,
                             hipStream_t st);
hipError_t launch_rope_pool(const Shape& s, const void* X, const float* cos_tab,
                            const float* sin_tab, int ld, int block, void* Xr, float* means,
                            float* nmax, hipStream_t st);
// Scores and top-k from given means; ws: select_pooled_workspace_bytes(s, block).
size_t select_pooled_workspace_bytes(const Shape& s, int block);
hipError_t launch_select_pooled(const Shape& s, const float* qbar, const float* kbar, int block,
                                int keep, int32_t* idx, void* ws, hipStream_t st);

// sparse_attn.hip  (idx == nullptr: dense, every key block in order; keep must equal n_blocks)
// ws: sparse_workspace_bytes(s, block, keep) bytes, or nullptr (then no K/V loads are shared
// between query blocks).
size_t sparse_workspace_bytes(const Shape& s, int block, int keep);
// The low-rank readout and gated combine fused into the attention epilogue (bf16, d 128, r 16-64):
// Os then receives O = combine(O^s, RMSNorm(q~^T C), logits). fuse_ws: fuse_workspace_bytes(s, r).
struct LowrankFuse {
  const void* Qn;
  const void* Pq;
  int r;
  const float* cos_tab;
  const float* sin_tab;
  int ld;
  const float* C;
  float eps_lr;
  const float* logits;
  float eps;
  const float* knorm;  // optional: per key block the largest key norm, [B, H, nb] (score bound)
};
bool fuse_supported(const Shape& s, int r);
size_t fuse_workspace_bytes(const Shape& s, int r);
// lse (optional, bf16 path): [B, H, N] fp32, log2 of each query's softmax denominator of the
// log2e-scaled scores, i.e. P = exp2(S * scale * log2e - lse).
// planned: ws already holds the groups of these lists (launch_sparse_plan with the same r), so the
// pairing and list merge are not launched again.
hipError_t launch_sparse_attn(const Shape& s, const void* Qr, const void* Kr, const void* V,
                              int block, int keep, const int32_t* idx, float scale, void* Os,
                              void* ws, hipStream_t st, const LowrankFuse* lf = nullptr,
                              void* fuse_ws = nullptr, float* lse = nullptr, bool planned = false);
// attn_f32.hip: the fp32 path of launch_sparse_attn (idx == nullptr: dense, keep == n_blocks).
hipError_t launch_attn_f32(const Shape& s, const void* Qr, const void* Kr, const void* V, int block,
                           int keep, const int32_t* idx, float scale, void* Os, hipStream_t st);
// Whether the path of (s, block) uses a plan (pairs, merged lists, queue counters in ws).
bool plan_used(const Shape& s, int block);
// The pairing and list merge of the 64-token bf16 path into ws (sparse_workspace_bytes), for the
// walk period of the kernel variant with fused rank r (0: plain attention). No-op elsewhere.
hipError_t launch_sparse_plan(const Shape& s, int keep, const int32_t* idx, int r, void* ws,
                              hipStream_t st);
// The per-device static scratch of the allocation-free entry point: its size, and its address on
// the current device (asked once per device, then cached).
size_t static_scratch_bytes();
hipError_t static_scratch(void** ptr);

// lowrank_bwd.hip: gradients of the low-rank branch and the gated fusion (bf16, d 128, r <= 64, SiLU
// with the rotation outside). dOs bf16; the other gradients fp32; dP_q, dP_k summed over the batch,
// dlogits over the heads. ws: lowrank_backward_workspace_bytes(s, r).
size_t lowrank_backward_workspace_bytes(const Shape& s, int r);
hipError_t launch_lowrank_backward(const Shape& s, const void* Qn, const void* Kn, const void* V,
                                   const void* Pq, const void* Pk, int r, const float* cos_tab,
                                   const float* sin_tab, int ld, const float* C, const void* Os,
                                   const float* logits, float eps_lr, float eps, const void* dO,
                                   void* dOs, float* dQn, float* dKn, float* dV, float* dPq,
                                   float* dPk, float* dlogits, void* ws, hipStream_t st);

// Rotary tables of the accumulating form of the sparse backward: with cos_tab set, the gradients of Q^r
// and K^r are rotated back (R(p)^T) and added to the outputs, dV is added; otherwise they are stored.
struct GradTables {
  const float* cos_tab = nullptr;
  const float* sin_tab = nullptr;
  int ld = 0;
};
// sparse_attn.hip: dQ^r of the block-sparse attention on the attention kernel (bf16, d 128, block 64:
// paired and queued, or 128); lseD: per query {log-sum-exp (log2), D = dO^s . O^s}; ws:
// sparse_workspace_bytes(s, block, keep).
hipError_t launch_sparse_dq(const Shape& s, const void* Qr, const void* Kr, const void* V, int block,
                            int keep, const int32_t* idx, float scale, const void* dO,
                            const void* lseD, const GradTables& acc, float* dQ, void* ws,
                            hipStream_t st);

// sparse_bwd.hip: gradients of the block-sparse attention (bf16, d 128, block 64 or 128; the transposed
// lists are built through one LDS word per block of a head); fp32 outputs; ws:
// sparse_backward_workspace_bytes(s, block, keep), 0 when unsupported.
size_t sparse_backward_workspace_bytes(const Shape& s, int block, int keep);
hipError_t launch_sparse_backward(const Shape& s, const void* Qr, const void* Kr, const void* V,
                                  int block, int keep, const int32_t* idx, float scale,
                                  const void* Os, const float* lse, const void* dOs,
                                  const GradTables& acc, float* dQ, float* dK, float* dV, void* ws,
                                  hipStream_t st);

// lowrank.hip
int summary_chunks(const Shape& s, int r);
size_t summary_workspace_bytes(const Shape& s, int r);
// feat: feature map phi | rotation order << 8 (the ROLA_PHI_* / ROLA_ROPE_* values; 0 = SiLU with
// the rotation outside, the paper's design).
hipError_t launch_lowrank_summary(const Shape& s, const void* Kn, const void* V, const void* Pk,
                                  int r, const float* cos_tab, const float* sin_tab, int ld,
                                  int feat, float* C, float* z, void* ws, hipStream_t st);
// Os == nullptr: plain readout into Out; otherwise readout fused with the gated combine.
hipError_t launch_lowrank_readout(const Shape& s, const void* Qn, const void* Pq, int r,
                                  const float* cos_tab, const float* sin_tab, int ld, int feat,
                                  const float* C, float eps_lr, const void* Os,
                                  const float* logits, float eps, void* Out, hipStream_t st);
// Features of every token, fp32 [B, H, N, r].
hipError_t launch_lowrank_features(const Shape& s, const void* X, const void* P, int r,
                                   const float* cos_tab, const float* sin_tab, int ld, int feat,
                                   float* F, hipStream_t st);
hipError_t launch_combine(const Shape& s, const void* Os, const void* Olr, const float* logits,
                          float eps, void* O, hipStream_t st);

// gate.hip: logits [B, N] = X [B, N, d_model] . Wg + bg (d_model % 8 == 0, <= gate_max_model()).
hipError_t launch_gate_logits(const Shape& s, const void* X, int d_model, const void* Wg, float bg,
                              float* logits, hipStream_t st);
int gate_max_model();
// Backward of the gate logits: dX (optional, fp32 [B, N, d_model]) = dlogits W_g; dWg (fp32 [d_model])
// = sum dlogits X; dbg (fp32 scalar) = sum dlogits. ws: gate_backward_workspace_bytes(d_model).
size_t gate_backward_workspace_bytes(int d_model);
hipError_t launch_gate_backward(const Shape& s, const void* X, int d_model, const void* Wg,
                                const float* dlogits, float* dX, float* dWg, float* dbg, void* ws,
                                hipStream_t st);

}  // namespace rola
