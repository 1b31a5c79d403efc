// Host-side plan of one forward: tile shapes, grid sizes and the layout of the caller's workspace.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/hybrid_attn.h"

namespace ha {

struct Plan {
  // problem
  int B, H, N, D, HD, F, R, NS, NL, P, act_q, act_k;
  int G;                 // granularity of the token split (1: per token, Sec. 3.2)
  int CC, n_cc, nsub;    // chunk-causal variant: chunk length in tokens (0: off), number of chunks, state-pass
                         // workgroups per chunk.  Local-window variant: CC = the query tile, one state per tile
  int LW;                // local-window variant: window in tokens on either side of the query's tile (0: off)
  int DM;   // width of the second hidden layer of a three-layer feature map, 0 for two layers
  bool f32;
  int64_t sb, sh, sn;
  float scale;
  // softmax part: KT = block_size (the key fragments are padded to whole multiples of it), 32-key blocks
  int KT, n_ktiles, n_kblocks;
  // state pass: CH linear tokens per workgroup, partial tiles per chunk
  int CH, n_chunks, n_state_tiles;
  // workspace byte offsets (all multiples of 256)
  size_t off_w1q, off_w2q, off_w1k, off_w2k, off_ks, off_vs, off_part, off_S, off_z, off_sthi, off_stlo, total;
  // 128 -> 256 -> 256 maps, plain operator, and small problems with the 128-wide maps: the linear part of the query side is a
  // pass of its own (ha_linear256.hip, ha_linear.hip), whose results (n_tb 32-query blocks per (batch, head)) the query
  // kernel adds; lin_rows queries of every head at a time
  bool split_linear;
  int n_tb, lin_rows;
  size_t off_lin, off_e;
  // key ranges the softmax loop is split into (1: one workgroup walks all keys of its tile), with the partial sums of every
  // range (see SplitArgs): blocks of 32 queries per (batch, head), images, maxima and sums
  int n_split, n_tb_split;
  size_t off_po, off_pm, off_pl;
  // bytes by which the key fragments are larger than with block_size 64, and smaller than with 128
  size_t key_pad_64, key_pad_128;
};

// Partial sums of the softmax loop over one of n_split key ranges, per (range, batch, head): the accumulators as fp32 register
// images, and per query the exact maximum of its raw logits over the range (which the accumulators are expressed
// against) and the sum of weights.  n_split <= 1: none.
struct SplitArgs {
  float *po;                  // [n_split][B*H][n_tb][d/32][4][64][4]
  float *pm, *pl;             // [n_split][B*H][32 n_tb]
  int n_split, n_tb, BH;
  float scale_log2e;
};
static inline SplitArgs split_args(const Plan &pl, void *ws) {
  char *w = static_cast<char *>(ws);
  return SplitArgs{reinterpret_cast<float *>(w + pl.off_po), reinterpret_cast<float *>(w + pl.off_pm), reinterpret_cast<float *>(w + pl.off_pl),
                   pl.n_split, pl.n_tb_split, pl.B * pl.H, pl.scale * 1.4426950408889634f};
}

// Workspace of the value-distillation gradient beyond the forward's: operand fragments of W2^T, S and dS, the
// per-row factors, the sign tensor and the partial tiles of the two gradient passes.
struct GradPlan {
  int CHq, n_chunks_q, CHk, n_chunks_k, tiles_per_set;
  size_t off_w2tq, off_w2tk, off_shi, off_slo, off_dS, off_dz, off_dshi, off_dslo, off_gsign, off_rs, off_wp, off_part, total;
};

// Workspace of the layer-by-layer path for feature maps beyond the fused kernels' widths (beyond the forward's):
// hidden activations (hi + lo where another layer reads them), fp32 pre-activations, and for the queries n = phi_q S and
// e = phi_q . z.
struct WidePlan {
  int n_tb_q, n_tb_k;      // 32-token blocks of the query tokens / the linear key tokens
  size_t off_w1, off_wm, off_w2;   // weight fragments of the map being evaluated (key side, then query side)
  size_t off_hhi, off_h2hi, off_h2lo, off_u, off_stat, off_phi, off_lin, off_e, total;
};

// Number of softmax tokens among the first t tokens: the first G of every R G tokens (Sec. 3.2 with G = 1).
static __host__ __device__ inline int softmax_before(int t, int R, int G) {
  if (R == 0) return 0;
  const int grp = R * G, rem = t % grp;
  return (t / grp) * G + (rem < G ? rem : G);
}

// Workspace of the value-distillation gradient of maps that take the layer-by-layer path (beyond WidePlan's).
struct WideGradPlan {
  int CHq, n_chunks_q, CHk, n_chunks_k;
  size_t off_wt, off_wtm, off_dpre2, off_shi, off_slo, off_dS, off_dz, off_dshi, off_dslo, off_gsign, off_rs, off_wp, off_tdt, off_pdot, off_du,
      off_dpre, off_part, total;
};

// Workspace of the value-distillation gradient of the maps 128 -> 256 -> 256 (ha_grad256.hip), [0] query side, [1] key side: fragments of the
// weights, of W2^T and of S or dS, the bf16 images of 32-token blocks that the passes leave to the products over the tokens, and those
// products' partial tiles over nc[side][product] ranges of blocks.
struct Grad256Plan {
  int n_tb[2], nc[2][3];
  size_t off_w1[2], off_w2[2], off_w2t[2], off_mhi[2], off_mlo[2], off_dz, off_gsign, off_rs, off_wp, off_h, off_du, off_dpre, off_phi,
      off_x, off_part, total;
};

// Which state passes read the feature map's weights straight from the caller's tensors (no preparation needed): the 128-wide
// maps' in bf16; that of the 64-wide heads but for the chunk-causal variant with softmax keys, whose compaction is a launch of its own
// and prepares the weights as well.  (There its many short chunks pay for fetching them row by row: raw / as fragments, whole calls, us:
// B = 2, H = 6, N = 5583, R = 4, chunks of 256, bf16  67.1 / 66.4; H = 12, N = 20000  260.6 / 259.9; without softmax keys, H = 8, N = 4000,
// chunks of 128, fp32, where the preparation is one launch more  41.7 / 44.0.  Local window, H = 8, N = 4000  51.3 / 51.9.)
static inline bool state_uses_pipelined_kernel(const Plan &pl) { return pl.D == 128 && pl.HD == 128 && pl.F == 128; }
static inline bool state_reads_raw_weights(const Plan &pl) {
  if (pl.D == 64) return pl.CC == 0 || pl.LW > 0 || pl.NS == 0;
  return state_uses_pipelined_kernel(pl) && !pl.f32;
}
// ... and compacts the softmax keys on the way (no compact_kernel launch): bf16 or d = 64, the plain operator with both kinds of tokens
static inline bool state_compacts_softmax_keys(const Plan &pl) {
  return state_reads_raw_weights(pl) && pl.CC == 0 && pl.LW == 0 && pl.NS > 0 && pl.NL > 0 && pl.n_chunks > 0;
}

// Purely linear attention with the 128-wide maps has a query-side kernel of its own (ha_linear.hip).
static inline bool query_side_is_linear(const Plan &pl) {
  return pl.NS == 0 && pl.CC == 0 && pl.LW == 0 && pl.DM == 0 && state_uses_pipelined_kernel(pl);
}

// Fills `pl` from a validated problem.  Pure host arithmetic.  limit: size of a workspace that cannot grow; where the
// results of the 256-wide maps' linear pass (516 bytes per query and head) do not fit it, they take the place of the state
// partials, which are spent by then, as many queries at a time as that holds.
constexpr size_t kStaticScratchBytes = (size_t)HA_STATIC_SCRATCH_MIB << 20;
// Whether a plan of `base` bytes may take a route that needs `extra` more.  A call has the same bits with a workspace of any
// size and with the static one, and with either block_size, so the answer must be the same in all four: a problem that fits
// the static array with one of the block sizes has to fit it with both, the extra included.
static inline bool route_has_room(const Plan &pl, size_t base, size_t extra) {
  return base - pl.key_pad_64 > kStaticScratchBytes || base + pl.key_pad_128 + extra <= kStaticScratchBytes;
}
void make_plan(const ha_problem &p, const ha_feature_map *phi_q, const ha_feature_map *phi_k, Plan &pl, size_t limit = SIZE_MAX);

// Kernel launchers (ha_kernels.hip).  Each enqueues on `st` and returns the launch status.
hipError_t launch_weight_prep(const Plan &pl, const ha_feature_map &fm, bool is_query, void *ws, hipStream_t st);
// prep_k (optional): the key-side map, whose weights are re-ordered in the same launch
hipError_t launch_compact(const Plan &pl, const void *k, const void *v, void *ws, hipStream_t st, const ha_feature_map *prep_k);
hipError_t launch_state(const Plan &pl, const void *k, const void *v, const ha_feature_map &phi_k, void *ws,
                        hipStream_t st);
hipError_t launch_state256(const Plan &pl, const void *k, const void *v, const ha_feature_map &phi_k, void *ws,
                           hipStream_t st);   // ha_state256.hip: 128 -> 256 -> 256
hipError_t launch_state_pipelined(const Plan &pl, const void *k, const void *v, const ha_feature_map &phi_k, void *ws,
                                  hipStream_t st);
hipError_t launch_state_pipelined_weighted(const Plan &pl, const void *q, const void *gsign, const float *rs, const float *wp,
                                           const ha_feature_map &fm, const void *w1f, const void *w2f, float *part, int CH,
                                           int n_chunks, hipStream_t st);   // ha_state.hip: the d -> d -> d maps
hipError_t launch_weighted_state(const Plan &pl, const void *q, const void *gsign, const float *rs, const float *wp,
                                 const ha_feature_map &fm, const void *w1f, const void *w2f, float *part, int CH,
                                 int n_chunks, hipStream_t st);
hipError_t launch_state_reduce(const Plan &pl, void *ws, hipStream_t st);
// the plain reduction (no prefix / window states) together with the re-ordering of phi_q's weights, one launch
hipError_t launch_state_reduce_with_prep(const Plan &pl, const ha_feature_map &phi_q, void *ws, hipStream_t st);
hipError_t launch_query(const Plan &pl, const void *q, const ha_feature_map *phi_q, void *out, float *row_den, void *ws,
                        hipStream_t st, const WidePlan *wide = nullptr);
// Teacher (rate 1) and student of one problem whose query kernels take the same tiling: both in one launch, each with a workspace of its own
bool query_pair_fits(const Plan &teacher, const Plan &student);
hipError_t launch_query_pair(const Plan &teacher, const Plan &student, const void *q, const ha_feature_map &phi_q, void *y_teacher,
                             void *y_student, float *row_den, void *ws_teacher, void *ws_student, hipStream_t st);
// ha_linear.hip: the query side where there is no softmax token at all; with pl.split_linear its n = phi_q(q) S and e only
hipError_t launch_linear_query(const Plan &pl, const void *q, const ha_feature_map &phi_q, void *out, float *row_den, void *ws,
                               hipStream_t st);
// ha_linear256.hip: n = phi_q(q) S and e = phi_q(q) . z of the 128 -> 256 -> 256 maps
hipError_t launch_linear256(const Plan &pl, const void *q, const ha_feature_map &phi_q, void *ws, hipStream_t st);
// ha_wide.hip
// backward: with the images only a backward pass reads (first hidden layer, phi)
void make_wide_plan(const Plan &pl, size_t base_off, WidePlan &wp, bool backward);
hipError_t launch_wide_key_side(const Plan &pl, const WidePlan &wp, const void *k, const void *v, const ha_feature_map &phi_k,
                                void *ws, hipStream_t st);
hipError_t launch_wide_query_side(const Plan &pl, const WidePlan &wp, const void *q, const ha_feature_map &phi_q, void *ws,
                                  hipStream_t st);
size_t l1_partial_bytes(const Plan &pl);
hipError_t launch_l1_distance(const Plan &pl, const void *ya, const void *yb, double *partial, double *loss,
                              hipStream_t st);
constexpr int64_t kMemorySideCache = 256 << 20;   // bytes, in front of HBM
constexpr int kMaxGridRows = 65535;               // blocks along a grid's second and third dimension: B H may be as many, B H + H more
constexpr int kL1Parts = 64;   // partial sums of the loss per (batch, head)
hipError_t launch_l1_final(const Plan &pl, const double *partial, double *loss, hipStream_t st);
// ha_grad.hip
void make_grad_plan(const Plan &pl, size_t base_off, GradPlan &gp);
hipError_t launch_fill_zero(float *p, size_t n, hipStream_t st);
hipError_t launch_value_distill_backward(const Plan &pl, const GradPlan &gp, const void *q, const void *k, const void *v,
                                         const ha_feature_map &phi_q, const ha_feature_map &phi_k, const void *y_teacher,
                                         const void *y_student, const float *row_den, const ha_feature_map_grad &gq,
                                         const ha_feature_map_grad &gk, void *ws, hipStream_t st, double *l1_partial = nullptr,
                                         double *loss = nullptr);
// l1_partial / loss given (bf16 io only): the pass over the two outputs also forms the loss (the partial sums of
// l1_partial_kernel, bit for bit), and the final sum is launched behind it
hipError_t launch_vd_rows(const Plan &pl, const void *y_teacher, const void *y_student, const float *row_den, void *gsign,
                          float *rs, float *wp, hipStream_t st, double *l1_partial = nullptr, double *loss = nullptr);
hipError_t launch_natural_frags(const float *M, void *hi, void *lo, int rows, int cols, int n_mat, hipStream_t st);
// ha_wide_mlp.hip: one layer of a map that goes layer by layer.  x given: the input is the first hidden layer
// relu(W1 x + b1), formed on the way (its bf16 image is left in h_hi if that is given); otherwise the images in_hi, in_lo.
// out_u, out_stat given: the last layer; otherwise out_hi, out_lo.
struct WideMlpLayer {
  const void *x, *in_hi, *in_lo, *w1f, *wf;
  const float *b1, *bias;
  void *h_hi, *out_hi, *out_lo, *out_u;
  float *out_stat;
  int K, NOUT, n_tok, R;
  bool channel_lanes;      // last layer: a channel per lane and the tokens in the registers (what the state pass reads)
};
hipError_t launch_wide_mlp(const Plan &pl, const WideMlpLayer &l, hipStream_t st);
// ha_wide.hip / ha_wide_grad.hip.  keep_hidden: leave the first hidden layer's image in the workspace (a backward pass
// reads it).
hipError_t launch_wide_map(const Plan &pl, const WidePlan &wp, const void *x, const ha_feature_map &fm, bool is_query, void *ws,
                           hipStream_t st, bool keep_hidden);
void make_wide_grad_plan(const Plan &pl, const WidePlan &wp, size_t base_off, WideGradPlan &gp);
hipError_t launch_wide_value_distill_backward(const Plan &pl, const WidePlan &wp, const WideGradPlan &gp, const void *q,
                                              const void *k, const void *v, const ha_feature_map &phi_q,
                                              const ha_feature_map &phi_k, const void *y_teacher, const void *y_student,
                                              const float *row_den, const ha_feature_map_grad &gq, const ha_feature_map_grad &gk,
                                              void *ws, hipStream_t st, double *l1_partial = nullptr, double *loss = nullptr);
// ha_grad256.hip: the same for the maps 128 -> 256 -> 256
void make_grad256_plan(const Plan &pl, size_t base_off, Grad256Plan &gp);
hipError_t launch_value_distill_backward256(const Plan &pl, const Grad256Plan &gp, const void *q, const void *k, const void *v,
                                            const ha_feature_map &phi_q, const ha_feature_map &phi_k, const void *y_teacher,
                                            const void *y_student, const float *row_den, const ha_feature_map_grad &gq,
                                            const ha_feature_map_grad &gk, void *ws, hipStream_t st, double *l1_partial = nullptr,
                                            double *loss = nullptr);
hipError_t launch_mfma_probe(float *sink, int workgroups, int iters, int random_operands, hipStream_t st);

}  // namespace ha
