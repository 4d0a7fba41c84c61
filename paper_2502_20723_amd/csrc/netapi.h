// Host-visible argument blocks and launchers of the network kernels.
#pragma once

#include "common.h"

namespace tdo {

struct FwdArgs {
  const void* wpack;            // this layer's packed weights (BF16 or FP32 fragments)
  const float* b1;              // [M] (padded)
  const float* b2;              // [D] (padded)
  const float* table;           // first layer: embedding table [64][D]
  const uint64_t* ecfg;         // first layer: configurations [E][2]
  const int64_t* n_entries_dev; // E on the device, or NULL to use n_entries
  int64_t n_entries;            // their number, or an upper bound when n_entries_dev gives it
  const float* x_in;            // residual in, [blocks][D/32] tiles (load_tile) (not first layer)
  float* x_out;                 // residual out (not last layer)
  void* save_x;                 // optional: layer input saved for the backward pass
  void* save_mid;               // optional: input of the feed-forward sub-layer
  float* save_lse;              // optional (BF16): [blocks][32 rows][D/DH heads] log2 of
                                // each attention row's softmax normaliser (+inf for a row with no key)
  void* save_last;              // optional (last layer): output x_L
  const float* head_w;          // last layer: [d][2]
  const float* head_b;          // last layer: [2]
  float* z;                     // last layer: [E][2 passes][2]
  int n, cpb, d_real, M;
  float score_scale;            // log2(e) / sqrt(d/heads)
  int first, last, masked, blocks_per_cu;
  int waves;                    // waves per workgroup (8 or 4) of the BF16 kernel
};

// The whole forward in one launch (net_stack.hip), n <= 32.  mode 0: lr of the E configurations ecfg;
// 1: `steps` proposals of the E chains on (alpha, beta); 2: of the diagonal chains; 3: z (and lr, unless
// NULL) of the configurations, with the activations kept for the backward pass.
struct StackArgs {
  const void* wpack;
  const float *b1, *b2, *table, *head_w, *head_b;
  const uint64_t* ecfg;
  int64_t E, layer_elems;
  float* lr;         // [E][2]
  const int64_t* n_entries_dev;  // mode 3: the number of entries on the device (E an upper bound), or NULL
  float* z;                      // mode 3: [E][2 passes][2]
  void *save_x, *save_mid, *save_last;
  float* save_lse;
  size_t layer_bytes, lse_layer;
  uint64_t* state;   // chains: [E][2] (mode 2: [E]), their log rho, and the states after the last proposal
  float* state_lr;
  uint64_t* record;
  uint64_t t0, seed, pair_thr;
  int steps, n, cpb, d_real, M, layers;
  int pairs;  // pairs of waves that compute, per workgroup (set by the launcher)
  float score_scale;
};
bool stack_supported(bool bf16, int D, int M, int layers, bool span);
int32_t launch_fwd_stack(const StackArgs& a, bool bf16, int D, int DH, bool masked, int mode, int num_cus, hipStream_t st);

int32_t launch_fwd_layer(const FwdArgs& a, bool bf16, int D, int DH, bool span, int num_cus, hipStream_t st);
int32_t launch_symmetrise(const int64_t* E_dev, int64_t E_host, const float* z, float* lr, hipStream_t st);

// Packing of the flat parameter vector into per-layer MFMA fragments.
struct PackPlan {
  int d, D, heads, layers, mlp, M;
  int64_t off_conv1, off_conv2_b, off_layer0, layer_stride, off_head_w, off_head_b;
  int64_t nparams;
  int64_t layer_elems;  // packed elements per layer (forward fragments)
};
int32_t make_pack_plan(const tdo_arch_t* arch, PackPlan* pp);
// Writes L layers of forward fragments (elem = bf16 if bf16 else f32), padded biases b1 [L][M] and
// b2 [L][D], the embedding table [64][D], and, if wb is not NULL, L layers of transposed fragments:
// Wq^T, Wk^T, Wv^T, Wo^T [D][D], then W2^T [D][M], W1^T [M][D].
int32_t launch_pack(const PackPlan& pp, const float* params, bool bf16, void* wf, void* wb, float* b1, float* b2,
                    float* table, hipStream_t st);

}  // namespace tdo

namespace tdo {

struct BwdArgs {
  const void* wf;               // this layer's forward fragments
  const void* wb;               // this layer's transposed fragments
  const float* b1;              // [M]
  const float* w1;              // this layer's W1 [d][mlp] and W2 [mlp][d] in the flat FP32 parameters
  const float* w2;
  const void* save_x;           // layer input
  const void* save_mid;         // feed-forward input
  const float* lse;             // attention row normalisers saved by the forward (or NULL)
  const float* g_in;            // incoming gradient [blocks][D/32] tiles (load_tile) (NULL: from seeds)
  const float* seeds;           // last layer: per configuration-pass (dF0, dF1), [E][2][2]
  const float* head_w;          // [d][2]
  float* g_out;                 // outgoing gradient
  float* partial;               // per-workgroup FP32 weight-gradient accumulators
  const int64_t* n_entries_dev;
  int64_t n_entries;
  int n, cpb, span, masked, d_real, M;
  float score_scale, inv_sqrt_dh;
  int blocks_per_wg;            // generic kernels: workgroup w takes these many blocks from w * blocks_per_wg (0: tiles in turn)
  int mlp_waves;                // BF16 feed-forward backward at mlp 256: 8 or 4 waves per workgroup
};

// Whether the generic feed-forward backward has a split for this width (padded) and mlp.
bool bwd_mlp_takes(int D, int M);
// Feed-forward backward with BF16 operands and per-wave register gradients (width 64).
bool bwd_mlp_bf16_supported(int d, int D, int M);
int32_t launch_bwd_mlp_bf16(const BwdArgs& a, int blocks, hipStream_t st);
// Attention backward with BF16 operands and per-wave register gradients (width 64, n <= 32).
bool bwd_attn_bf16_supported(int d, int D, int DH, bool span);
// Each of `grid` workgroups writes one weight-gradient partial [4 D^2].
int32_t launch_bwd_attn_bf16(const BwdArgs& a, int DH, int grid, hipStream_t st);
// workgroups that fill the chip with one per CU in `blocks`
int bwd_attn_bf16_parts(int blocks, bool span);
int32_t launch_bwd_mlp(const BwdArgs& a, bool bf16, int D, int blocks, hipStream_t st);
int32_t launch_bwd_attn(const BwdArgs& a, bool bf16, int D, int DH, int blocks, hipStream_t st);
// part: FP64 scratch of HEAD_BLOCKS * (2 d_real + 2) values (one slot per workgroup).
constexpr int HEAD_BLOCKS = 1024;
// workgroups for nblk blocks taken `per` at a time, at most cap
inline int grid_for(int cap, int64_t nblk, int per) {
  const int64_t g = (nblk + per - 1) / per;
  return g < 1 ? 1 : (g < cap ? (int)g : cap);
}
int32_t launch_bwd_head(bool bf16, int D, const void* save_last, const float* seeds, const int64_t* E_dev,
                        int64_t E_host, int n, int cpb, int span, int d_real, double* gw, double* gb, double* part,
                        hipStream_t st);
// One partial [64][D] per wave, blocks * waves of them.
int32_t launch_embed_scatter(int D, const float* dx0, const uint64_t* ecfg, const int64_t* E_dev, int64_t E_host,
                             int n, int cpb, int span, float* partial, int blocks, hipStream_t st, int waves = 4);
// part: FP64 scratch of 64 * (6 d + 2 d^2) values (one slot per window code).
int32_t launch_embed_params(const float* params, const double* dT, int d, int D, double* grad, double* part,
                            hipStream_t st);
// Rows of the Jacobian (jacobian.hip), for E configurations of bpc blocks each; row e of a part is
// jac + e * stride.  mpart: slots consecutive partials [2 D M + M + D] per configuration, apart: one
// [4 D^2]; they become the layer's rows at jac.
int32_t launch_jac_layer(const float* mpart, int slots, const float* apart, const PackPlan& pp, int64_t E, double* jac,
                         int64_t stride, hipStream_t st);
// head weights and bias, at jac; save_last and seeds as launch_bwd_head
int32_t launch_jac_head(bool bf16, int D, const void* save_last, const float* seeds, int64_t E, int n, int span,
                        int d_real, double* jac, int64_t stride, hipStream_t st);
// tables of the embedding's chain rule (FP64, jac_tables(d) values), once per call
inline size_t jac_tables(int d) { return (size_t)(2 * 16 + 64) * d; }
int32_t launch_jac_tables(const float* params, int d, double* tab, hipStream_t st);
// convolution parameters, at jac; part: bpc consecutive wave partials [64][D] per configuration
int32_t launch_jac_embed(const float* params, const double* tab, const float* part, int bpc, int d, int D, int64_t E,
                         double* jac, int64_t stride, hipStream_t st);
// out[i] += sum over the partials, in FP64: of whole vectors; of the feed-forward or attention
// partials of a layer into its part of the flat gradient g
int32_t launch_reduce_partials(const float* part, int nparts, int64_t len, double* out, hipStream_t st);
int32_t launch_reduce_mlp(const float* part, int nparts, const PackPlan& pp, double* g, hipStream_t st);
int32_t launch_reduce_attn(const float* part, int nparts, const PackPlan& pp, double* g, hipStream_t st);

}  // namespace tdo
