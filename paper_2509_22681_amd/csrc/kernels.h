// Launch interface between the host API and the gfx950 kernels.  All pointers are device
// pointers unless stated; every launcher only enqueues work on `s`.
#pragma once
#include <atomic>

#include <hip/hip_runtime.h>

#include "plan.h"

namespace flame {

// Shapes every launcher needs.
struct Shape {
  int d, H, dh, n_layers, n_buckets, D;
  float eps, alpha;
  int64_t ws_rows;  // rows of every workspace matrix (plane stride = ws_rows * d)
  int softmax;      // attention weights: 0 = pointwise SiLU, 1 = softmax with a temperature per layer and head
  int latency;      // MFMA attention: 0 = throughput configuration, 1 = latency configuration (four wavefronts split the keys of a query tile)
};

// ---- shared small kernels (misc.hip) --------------------------------------------------------
// Prologue of a pass (one launch; misc.hip): any of its parts may be absent.
struct Prologue {
  // plan tables, host (pinned) -> device; n_table_words % 4 == 0, both on 16 bytes
  const void *tables_src = nullptr;
  void *tables_dst = nullptr;
  int n_table_words = 0;
  // rows of blocks <- embeddings: fp32 X in the fp32 path, the k-tile blocked fp16 word Xh in the MFMA path (whose residual is
  // the pair Xh = fp16(X), Xl = fp16(X - Xh); embeddings are exact in Xh and Xl is not written); padding rows zeroed.
  // The n_blk blocks are list[0..n_blk) if list is given, else the first n_blk (blocks and list: pinned host or device memory).
  int dtype = 0, d = 0, n_blk = 0;
  const RowBlock *blocks = nullptr;
  const int32_t *list = nullptr;
  const void *hist = nullptr, *cand = nullptr;
  float *X = nullptr;
  void *Xh = nullptr;
  // what is derived from the weights (w1 == nullptr: nothing): the projection matrices packed by fragments as fp16 (W1h, and W2p for the fused K3, else W2h), or
  // (fp32 path, if Ws) split into bf16 parts; bias[lh][distance] = bias_scale * rab[lh][bucket_tab[distance]] for all layers and heads (scale = 1/2 in the MFMA path, whose
  // attention kernel works on halved logits; 1 in the fp32 path); tscale[i] = logit_factor / temperature[i] (softmax)
  const void *w1 = nullptr, *w2 = nullptr;
  void *W1h = nullptr, *W2h = nullptr, *W2p = nullptr, *Ws = nullptr;
  const float *rab = nullptr, *temperature = nullptr;
  const int32_t *bucket_tab = nullptr;
  float *bias = nullptr, *tscale = nullptr;
  int n_layers = 0, H = 0, n_buckets = 0, D = 0;
  float bias_scale = 1.f, logit_factor = 1.f;
};
void launch_prologue(const Prologue &p, hipStream_t s);
// G = (LayerNorm(O) * gamma + beta) * U, one row at a time (MFMA path, for widths whose output projection is not fused with it);
// padding rows of a block get G = 0 so that they stay finite through the layers.
void launch_ln_gate(const void *O, const void *U, const void *gamma, const void *beta,
                    void *G, const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, int d,
                    float eps, hipStream_t s);
// scores[src_row + i] = <X[row], w_s> + b_s for the valid rows of every candidate block (MFMA path: X = Xh + Xl).
void launch_scores(int dtype, const float *X, const void *Xh, const void *Xl, const void *w_s, float b_s, const RowBlock *blocks,
                   const int32_t *cand_blocks, int n_cblk, float *scores, int d, hipStream_t s);
// hidden[(src_row + i) * d ..] = X[row] for the valid rows of every candidate block (fp32).
// (Xh given: the residual is the pair Xh, Xl of the MFMA path; else fp32 X)
void launch_gather_hidden(const float *X, const void *Xh, const void *Xl, const RowBlock *blocks, const int32_t *cand_blocks, int n_cblk,
                          float *hidden, int d, hipStream_t s);
// out[row][k] = Xh + Xl as fp32 for rows [row_begin, row_end) (debug capture of the MFMA path's residual)
void launch_residual_to_f32(const void *Xh, const void *Xl, float *out, int64_t row_begin, int64_t row_end, int d, hipStream_t s);
// bucket(delta) for delta in [0, D), computed on the device (the integers of plan.h's bucket_of)
void launch_bucket_table(int n_buckets, int D, int32_t *out, hipStream_t s);
// Host words -> device memory without a copy engine or staging buffer: the words travel as kernel arguments
// (UploadWords::kWords per launch; bytes % 4 == 0).  For small tables on paths that may not allocate or copy.
struct UploadWords {
  static constexpr int kWords = 960;
  uint32_t w[kWords];
};
void launch_upload_words(const void *host_src, size_t bytes, void *dst, hipStream_t s);
// rows [row0, row0 + n) of the row-major K plane and of the feature-major V plane (d features) <- 0
void launch_clear_spare(void *K, void *Vt, int d, int64_t ws_rows, int64_t row0, int n, hipStream_t s);
// mask / bucket of one request evaluated with the device predicate (debug export).
void launch_debug_mask(int L, int M, const int32_t *bucket_tab, int D, uint8_t *mask, int32_t *bucket,
                       hipStream_t s);

// ---- fp32 path (kernels_f32.hip): projections on split bf16 operands, attention on the fp32 matrix instruction ----------------------------------
// The projection matrices of all layers split into bf16 parts for the two products below (kernels_f32.hip), packed by fragments: matrix m of the copy, W1's planes layer after layer
// and then W2's, starts at m * split_w_bytes(d, 1) / 5.  The products take the packed matrix of the layer (packed), or the matrix itself.
int64_t split_w_bytes(int d, int n_layers);
// planes[p][row][n] = silu(X W1^T + b1), p = U,V,Q,K; rows = the listed 64-row blocks (blk_list == nullptr: [blk_first, blk_first+n_blk));
// plane_mask: all planes (0xF), U and Q (0x5) or V and K (0xA); uq_list (n_uq blocks, with V and K): their U and Q with it
void launch_uvqk_f32(const float *X, const void *W1, bool packed, const float *b1, float *planes, const int32_t *blk_list, int n_blk, int blk_first,
                     int plane_mask, const int32_t *uq_list, int n_uq, const Shape &sh, hipStream_t s);
// tscale_h (softmax only): per head, the factor from the logit the kernel forms to the exponent it feeds to
// its exponential: 1 / tau here (natural exponential of the full logit).
void launch_attn_f32(const float *planes, const float *bias_lh, const float *tscale_h, float *O, const AttnItem *items,
                     int n_items, const Shape &sh, hipStream_t s);
// X[row] += ((LayerNorm(O[row]) * gamma + beta) * U[row]) W2^T + b2 for the rows of the listed blocks (blk_list == nullptr:
// contiguous); padding rows of a block get the bias only, so that they stay finite through the layers.
// scores (where outproj_scores_f32 allows it): the rows' scores instead of the rows.
bool outproj_scores_f32(const float *gamma, const float *beta, const void *W2, bool packed, const Shape &sh);
void launch_outproj_f32(const float *O, const float *U, const float *gamma, const float *beta, const void *W2, bool packed, const float *b2, float *X,
                        const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, const float *w_s, float b_s, float *scores, const Shape &sh, hipStream_t s);

// The four activation planes of a layer (MFMA path), each [ws_rows][d] fp16 (V feature-major [d][ws_rows]).  The
// one-pass forward keeps them in one allocation; the two-stage path points v and k at the layer's cache.
struct PlanePtrs { void *u, *v, *q, *k; };

// ---- bf16-storage path (gemm_mfma.hip, attn_mfma.hip): fp16 MFMA kernels, fp32 accumulation --------
// Activations (Xh, planes, O, G) and the converted matrices W1h/W2h are fp16; biases stay bf16.
// Xh is k-tile blocked (device_common.h: blocked_index), W1h and W2h are packed by fragments (device_common.h); planes, O and G are row-major.
// U, Q, K planes row-major [row][d]; the V plane is written transposed, Vt[n][row] (row stride ws_rows).
// plane_mask bit p set = compute plane p (U=1, V=2, Q=4, K=8); uq_list (n_uq blocks, with the mask of V and K): their U and Q with it, in the same
// launch where the small tiles run.
void launch_uvqk_bf16(const void *Xh, const void *W1h, const void *b1, PlanePtrs planes, const int32_t *blk_list,
                      int n_blk, int blk_first, int plane_mask, const int32_t *uq_list, int n_uq, const Shape &sh, hipStream_t s);
// tscale_h (softmax only): 2 log2(e) / tau per head (the kernel holds halved logits and uses the base-2 exponential).
// n_cand: candidate tiles among the items; q_tile, longest: query rows per item and the longest history of this plan.
void launch_attn_bf16(PlanePtrs planes, const float *bias_lh, const float *tscale_h, void *O, const AttnItem *items,
                      int n_items, int n_cand, int q_tile, int longest, const Shape &sh, hipStream_t s);
// Whether a pointwise launch of a throughput handle (grid = items x heads) takes the key-ordered split.
bool attn_key_ordered(int grid, int n_items, int n_cand, int longest);
// Raises the dynamic LDS limit of a kernel on the current device.  The limit is a property of the kernel on one device, so `done`, the kernel's own, holds a bit per
// device; a failure is not kept.  Safe from several threads.
hipError_t raise_lds_limit(const void *kernel, int bytes, std::atomic<uint64_t> &done);
// Prepares the configurations of the attention kernel that split the keys, for this shape (raises their LDS limit); once per handle, on its device.
hipError_t attn_setup(const Shape &sh);
// X[row] += G W2h^T + b2 on the residual pair (Xh, Xl); lo_is_zero: Xl is not read (first layer)
void launch_outproj_bf16(const void *G, const void *W2h, const void *b2, void *Xh, void *Xl, bool lo_is_zero,
                         const int32_t *blk_list, int n_blk, int blk_first, const Shape &sh, hipStream_t s);

// K3 fused (k3_mfma.hip): LayerNorm * U gate + output projection + residual in one kernel, for
// d in {128, 192, 256, 384, 512}; W2p is the fragment-major packed fp16 copy of W2 written by the prologue.
bool k3_fused_supported(int d);
// (residual pair Xh, Xl as above; lo_is_zero: Xl is not read)
void launch_k3_fused(const void *O, const void *U, const void *gamma, const void *beta, const void *W2p_layer, const void *b2,
                     void *Xh, void *Xl, bool lo_is_zero, const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first,
                     const Shape &sh, hipStream_t s);

// K3 of a layer and K1 of the next in one kernel (layer_mfma.hip), for the widths that layer_fused names: the rows' planes of the next layer are made from the new
// residual rows; all_hist, all_cand: all four planes for history (candidate) blocks, or V and K only.  layer_setup: once per handle (raises the LDS limit).
// U may be the plane planes.u: a workgroup has read its rows of the one before it writes them to the other.
bool layer_fused(int d);
hipError_t layer_setup(int d);
void launch_layer(const void *O, const void *U, const void *gamma, const void *beta, const void *W2p_layer, const void *b2, void *Xh, void *Xl, bool lo_is_zero,
                  const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, const void *W1h_next, const void *b1_next, PlanePtrs planes, bool all_hist, bool all_cand,
                  const Shape &sh, hipStream_t s);

// Launches of up to this many 64-row blocks run K3 on half blocks: with the features cut in four (d = 512), in two, uncut with a compute unit for each
// (d = 384, 512), uncut (both sides of each are at launch_k3).
constexpr int kK3CutInFour = 22, kK3CutInTwo = 64, kK3OneEach = 128, kK3HalfBlocks = 384;

// A launch whose rows make a plane (rows x d fp16) larger than this writes and reads what is consumed once past the caches (nontemporal): what streams
// through would push the operands that are read many times out of them.  The line is where the two measured level, per forward, ordinary
// against nontemporal: 3 MB per plane (one request, d = 512) 1033 against 1078 us, 10 MB (32 x 640 rows, d = 256) 289 against 308 us; 27 MB equal;
// 100 MB 5.15 against 4.98 ms, 500 MB 65.4 against 63.7 ms.  (At the line the eight arrays of a layer are 128 MB, half of the cache behind the L2s.)
// K1's large tile and K3 count the rows of the launch, K2 128 rows per tile.  K1's small tile has a line of its own (kSmallStreamBytes) and none for
// d >= 256, which it leaves at 23 to 39 MB: d = 256, 32 MB, 4 layers of 512 x (64 + 64) 615 us, with the large tile 625.  The
// kernels of widths without a fused K3 (ln_gate, output projection) store through the caches at any size.
constexpr int64_t kStreamBytes = 16 << 20;

}  // namespace flame
