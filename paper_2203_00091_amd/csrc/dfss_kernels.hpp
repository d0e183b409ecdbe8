// Host-side launchers of the DFSS kernels (internal to the library; the public
// interface is include/dfss.h).  Every launcher assumes validated arguments.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace dfss {

// A scale that is a power of two can be folded into Q without a rounding.
inline bool is_pow2(float x) {
    int e;
    return frexpf(x, &e) == 0.5f;
}

// Whether the workgroups of a launch keep level on their compute units (Pace in dfss_device.hpp).  per_cu: how many a compute
// unit holds; keys: how many each of them walks.
// They do where all of them are resident at once, more than one to a compute unit, and where long ones, of `from` keys on, fill every
// round, the last one to `eighths` / 8 or more: who is level ends together, and what is left then starts late, on a chip filled in part.
// us, without and with --
//   all at once: 24 heads x 4096 x 4096, one kernel, 104 and 97
//   one to a compute unit: 1 - 3 % slower
//   a last round up to half full: stage 1, 1024 workgroups, 768 at a time, 8 x 4096 x 4096 37.0 and 40.5; with key lengths, 64 x 2048 x
//     2048 61.3 and 71.4; dQ and dK, dV at d = 128, 768 of 512, 192 x 512 x 512 82.5 and 91.8
//   two thirds full (80 x 2048 x 2048): one kernel 85.5 and 82.7, stage 1 90.6 and 94.3, backward pass 264 and 271; more (88 x 2048 x
//     2048): 99.2 and 95.0, 99.5 and 98.6, 295 and 286
//   whole rounds: one kernel, d = 128, two of them, 64 x 2048 x 2048 117 and 114; 512 keys: 256 x 512 x 512 37.5 and 38.1; 256 keys: 512 x
//     256 x 256 26.6 and 27.7
inline bool keep_level(unsigned grid, unsigned per_cu, int keys, unsigned eighths = 6, int from = 1024) {
    const unsigned resident = 256 * per_cu, last = grid % resident;
    return grid > 256 && (grid <= resident || (keys >= from && (last == 0 || 8 * last >= eighths * resident)));
}

// key_bias (where present): fp32 [BH / H][Lk] added to the scaled scores before the selection, or
// nullptr for none (then H is ignored).
// LqR, LkR (where present): the real lengths of the caller's arrays (Q, K, V, key_bias, O) when they differ from the
// layout lengths Lq (a multiple of 64) and Lk (of 128) of the compressed arrays; else equal to Lq, Lk.
// Stage 1 (Sec. 3.4, App. A.1.2): scores + N:M pruning epilogue.  mode: 0 = 2:4, 1 = 1:2.
hipError_t launch_sddmm_prune(const void *Q, const void *K, const float *key_bias, int H, int causal, int BH, int Lq, int Lk,
                              int LqR, int LkR, int d, int mode, float scale, void *vals, void *meta, hipStream_t st);
// Dense scores S = scale * Q K^T stored as bfloat16 [BH, Lq, Lk] (Eq. 1), same mainloop.
hipError_t launch_dense_scores(const void *Q, const void *K, const float *key_bias, int H, int causal, int BH, int Lq, int Lk,
                               int LqR, int LkR, int d, float scale, void *S, hipStream_t st);
// The same two with an additive mask fp32 [LqR][LkR] shared by all heads (added like the key bias; -inf hides a key
// from a query) in the place of the per-key bias.
hipError_t launch_sddmm_prune_mask(const void *Q, const void *K, const float *mask, int BH, int Lq, int Lk, int LqR,
                                   int LkR, int d, int mode, float scale, void *vals, void *meta, hipStream_t st);
hipError_t launch_dense_scores_mask(const void *Q, const void *K, const float *mask, int BH, int Lq, int Lk, int LqR,
                                    int LkR, int d, float scale, void *S, hipStream_t st);
// Row softmax in place over bfloat16 rows (App. A.1.3); rows of `cols` elements.
hipError_t launch_row_softmax(void *x, long rows, int cols, hipStream_t st);
// Stage 3 (Sec. 3.1): O = A_sparse V from compressed weights + metadata.
hipError_t launch_spmm(const void *vals, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d,
                       void *O, hipStream_t st);
// The same product on the kept SCORES of stage 1, with the softmax over them applied on the way.
hipError_t launch_softmax_spmm(const void *scores, const void *meta, const void *V, int BH, int Lq, int Lk, int LqR,
                               int LkR, int d, void *O, hipStream_t st);
// Dense O = P V with P bfloat16 [BH, Lq, Lk].
hipError_t launch_dense_av(const void *P, const void *V, int BH, int Lq, int Lk, int LqR, int LkR, int d, void *O,
                           hipStream_t st);
// Whole forward pass in one kernel.  mode: 0 = 2:4, 1 = 1:2, 2 = dense (full attention, Eq. 1).
// block_mask: uint8 [Lq/64][Lk/64] shared by all heads (zero = block not part of the attention), or nullptr.
// variant: a DFSS_VARIANT_* tiling (dfss_internal.h), 0 = chosen from the shape.
// The same for a padded batch given by its lengths: key_len int32 [BH / H] on the device (keys key_len[b] .. Lk - 1 of batch
// element b are padding); Lq a multiple of 64, Lk of 64; mode 0 or 1.
hipError_t launch_fused_attention_varlen(const void *Q, const void *K, const void *V, const int *key_len, int H, int BH,
                                         int Lq, int Lk, int d, int mode, float scale, void *O, hipStream_t st);
// The same with an additive mask fp32 [Lq][Lk] shared by all heads (any Lq; Lk a multiple of 4); mode 2 = full attention.
hipError_t launch_fused_attention_mask(const void *Q, const void *K, const void *V, const float *mask, int BH, int Lq,
                                       int Lk, int d, int mode, float scale, void *O, hipStream_t st);
hipError_t launch_fused_attention(const void *Q, const void *K, const void *V, const float *key_bias, int H,
                                  const uint8_t *block_mask, int causal, int BH, int Lq, int Lk, int d, int mode, float scale,
                                  void *O, int variant, hipStream_t st);
// Calls whose few query tiles take the kernel of few_queries.hip, shared between several workgroups each: bytes of the
// workspace (0: not such a call, or nothing to gain), and the call with it (no key bias).
size_t few_queries_workspace_bytes(int BH, int Lq, int Lk, int d);
hipError_t launch_fused_attention_few_split(const void *Q, const void *K, const void *V, int BH, int Lq, int Lk, int d, int mode,
                                            float scale, void *O, void *part, hipStream_t st);
// The same with a block pattern (block_mask not null) and a workspace of fused_attention_split_workspace_bytes: row
// blocks that visit many blocks are shared between several workgroups and merged by a second kernel.
size_t fused_attention_split_workspace_bytes(int BH, int Lq, int d);
hipError_t launch_fused_attention_split_rows(const void *Q, const void *K, const void *V, const float *key_bias, int H,
                                             const uint8_t *block_mask, int BH, int Lq, int Lk, int d, int mode,
                                             float scale, void *O, void *part, hipStream_t st);
// Transposed sparse product out[BH, Lk, d] = A^T X for compressed A (vals + metadata) and X bf16 [BH, Lq, d]:
// dV = P^T dO and dK = dS^T Q of the backward pass.
hipError_t launch_spmm_t(const void *vals, const void *meta, const void *X, int BH, int Lq, int Lk, int LqR, int LkR,
                         int d, void *out, hipStream_t st);
// Backward pass through the fixed selection (P, meta as kept from the forward pass).  ws: backward_workspace_least or more,
// 256-byte aligned; with backward_workspace_bytes workgroups may share keys and queries.
size_t backward_workspace_least(int BH, int Lq);
size_t backward_workspace_bytes(int BH, int Lq, int Lk, int LqR, int LkR, int d);
hipError_t launch_backward(const void *dO, const void *Q, const void *K, const void *V, const void *O, const void *P,
                           const void *meta, int BH, int Lq, int Lk, int LqR, int LkR, int d, float scale, void *ws,
                           size_t ws_bytes, void *dQ, void *dK, void *dV, hipStream_t st);
// The 4-byte mode (Sec. 2.3: float data, 1:2): fp32 Q, K, V, kept scores, weights and O; metadata = one
// 4-bit code per kept float, 32-bit words in the blocked order [BH, Lq/16, Lk/64, 16, 4].
hipError_t launch_sddmm_prune_f32(const void *Q, const void *K, const float *key_bias, int H, int BH, int Lq, int Lk,
                                  int d, float scale, void *vals, void *meta, hipStream_t st);
hipError_t launch_dense_scores_f32(const void *Q, const void *K, const float *key_bias, int H, int BH, int Lq, int Lk,
                                   int d, float scale, void *S, hipStream_t st);
hipError_t launch_row_softmax_f32(void *x, long rows, int cols, hipStream_t st);
hipError_t launch_spmm_f32(const void *vals, const void *meta, const void *V, int BH, int Lq, int Lk, int d, void *O,
                           hipStream_t st);
hipError_t launch_dense_av_f32(const void *P, const void *V, int BH, int Lq, int Lk, int d, void *O, hipStream_t st);
// The same four operations with every fp32 product formed from bfloat16 pieces on the bf16 matrix pipe
// (x = hi + lo; a.b ~ a_hi b_hi + a_hi b_lo + a_lo b_hi, fp32 accumulation); same layouts.
hipError_t launch_sddmm_prune_split(const void *Q, const void *K, const float *key_bias, int H, int BH, int Lq, int Lk,
                                    int d, float scale, void *vals, void *meta, hipStream_t st);
hipError_t launch_dense_scores_split(const void *Q, const void *K, const float *key_bias, int H, int BH, int Lq,
                                     int Lk, int d, float scale, void *S, hipStream_t st);
hipError_t launch_spmm_split(const void *vals, const void *meta, const void *V, int BH, int Lq, int Lk, int d,
                             void *O, hipStream_t st);
hipError_t launch_dense_av_split(const void *P, const void *V, int BH, int Lq, int Lk, int d, void *O,
                                 hipStream_t st);
// dS' = scale * P .* (dO V^T - delta) at the kept positions of the 4-byte mode (split products), compressed like P.
hipError_t launch_masked_sddmm_ds_split(const void *dO, const void *V, const void *O, const void *P, const void *meta,
                                        int BH, int Lq, int Lk, int d, float scale, void *dS, hipStream_t st);
// out[BH, Lk, d] = A^T X for A in the compressed form of the 4-byte mode, X fp32 [BH, Lq, d] (split products).
hipError_t launch_spmm_t_split(const void *vals, const void *meta, const void *X, int BH, int Lq, int Lk, int d,
                               void *out, hipStream_t st);
// Whole forward pass of the 4-byte mode in one kernel (split products).  prune = false: full attention.
// key_bias and block_mask (both may be null) as in launch_fused_attention.
hipError_t launch_fused_attention_split(const void *Q, const void *K, const void *V, const float *key_bias, int H,
                                        const uint8_t *block_mask, int BH, int Lq, int Lk, int d, bool prune,
                                        float scale, void *O, hipStream_t st);
// Metadata word order: library <-> canonical.  W = 32-bit words per row; permute: the 2-byte modes' order of
// the four words of a (row, block), false for the 4-byte mode.
hipError_t launch_meta_reorder(const void *src, void *dst, int BH, int Lq, int W, bool to_canonical, bool permute,
                               hipStream_t st);

}  // namespace dfss
