// Packing of the flat parameter vector (layout of tdo_num_params) into the
// per-layer MFMA fragment order of net.h, zero-padded to width D = max(32, d).
#include <algorithm>

#include "common.h"
#include "net.h"
#include "netapi.h"

namespace tdo {

int32_t make_pack_plan(const tdo_arch_t* arch, PackPlan* pp) {
  TDO_CHECK(arch != nullptr, TDO_EINVAL, "arch is NULL");
  const int d = arch->d, H = arch->heads, L = arch->layers, m = arch->mlp;
  TDO_CHECK(d == 16 || d == 32 || d == 64, TDO_EUNSUPPORTED, "width d=%d not in {16, 32, 64}", d);
  TDO_CHECK(H >= 1 && d % H == 0, TDO_EINVAL, "heads=%d does not divide d=%d", H, d);
  TDO_CHECK(d / H == 8 || d / H == 16, TDO_EUNSUPPORTED, "head width d/heads=%d not in {8, 16}", d / H);
  TDO_CHECK(m >= 32 && m % 32 == 0 && m <= 512, TDO_EUNSUPPORTED, "mlp=%d must be a multiple of 32 in [32, 512]", m);
  TDO_CHECK(L >= 1 && L <= 16, TDO_EUNSUPPORTED, "layers=%d not in [1, 16]", L);
  TDO_CHECK(arch->c1 == 0 || arch->c1 == d, TDO_EUNSUPPORTED,
            "conv-1 width c1=%d: the kernels implement c1 = d (0 selects it)", arch->c1);
  TDO_CHECK(arch->act == TDO_ACT_RELU_FFN, TDO_EUNSUPPORTED,
            "activation set %d: the kernels implement TDO_ACT_RELU_FFN (0) only", arch->act);
  PackPlan p{};
  p.d = d;
  p.D = d < 32 ? 32 : d;
  p.heads = H;
  p.layers = L;
  p.mlp = m;
  p.M = m;
  p.off_conv1 = 0;
  p.off_conv2_b = 5LL * d + 2LL * d * d;
  p.off_layer0 = 6LL * d + 2LL * d * d;
  p.layer_stride = 4LL * d * d + 2LL * d * m + m + d;
  p.off_head_w = p.off_layer0 + (int64_t)L * p.layer_stride;
  p.off_head_b = p.off_head_w + 2LL * d;
  p.nparams = p.off_head_b + 2;
  p.layer_elems = 4LL * p.D * p.D + 2LL * p.D * p.M;
  *pp = p;
  return TDO_OK;
}

// Embedding table of one window code: T[code][o] = act(b2 + e(t0,t1) W2[0] + e(t1,t2) W2[1]),
// e(ta,tb) = act(b1 + s(ta) W1[0] + s(tb) W1[1]), act = exact GELU (Eq. circ-conv); one workgroup.
__device__ void embed_table_row(const float* __restrict__ params, int d, int D, int code, float* __restrict__ table) {
  __shared__ float e0[64], e1[64];
  const int t0 = code & 3, t1 = (code >> 2) & 3, t2 = (code >> 4) & 3;
  const float* w1 = params;            // [2 taps][2 ch][d]
  const float* b1 = params + 4 * d;    // [d]
  const float* w2 = b1 + d;            // [2 taps][d][d]
  const float* b2 = w2 + 2 * d * d;    // [d]
  auto spin = [](int t, int ch) { return 1.0f - 2.0f * (float)((t >> ch) & 1); };
  auto gelu = [](float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); };
  const int c = threadIdx.x;
  if (c < d) {
    float a = b1[c] + spin(t0, 0) * w1[0 * d + c] + spin(t0, 1) * w1[1 * d + c] + spin(t1, 0) * w1[2 * d + c] +
              spin(t1, 1) * w1[3 * d + c];
    float b = b1[c] + spin(t1, 0) * w1[0 * d + c] + spin(t1, 1) * w1[1 * d + c] + spin(t2, 0) * w1[2 * d + c] +
              spin(t2, 1) * w1[3 * d + c];
    e0[c] = gelu(a);
    e1[c] = gelu(b);
  }
  __syncthreads();
  if (c < D) {
    float v = 0.f;
    if (c < d) {
      float acc = b2[c];
#pragma unroll 16
      for (int k = 0; k < d; ++k) acc += e0[k] * w2[k * d + c] + e1[k] * w2[d * d + k * d + c];
      v = gelu(acc);
    }
    table[code * D + c] = v;
  }
}

// One element of the packed layer matrices (bwd = false): Wq, Wk, Wv, Wo [D][D], W1 [D][M], W2 [M][D];
// or of their transposes (bwd = true), used by the backward pass: Wq^T, Wk^T, Wv^T, Wo^T [D][D],
// W2^T [D][M], W1^T [M][D].
template <int KPL>
__device__ __forceinline__ float packed_weight(const float* __restrict__ params, const PackPlan& pp, bool bwd, int64_t e) {
  constexpr int ST = 32 / (2 * KPL);
  const int D = pp.D, M = pp.M, d = pp.d;
  const int l = (int)(e / pp.layer_elems);
  int k = (int)(e % pp.layer_elems);
  const float* lp = params + pp.off_layer0 + l * pp.layer_stride;
  // Packed matrix A[in][out], in < in_p (padded).  Forward: A = W, W[rows][cols]
  // row-major with rows = in, cols = out.  Backward: A = W^T, A[in][out] = W[out][in].
  const float* src;
  int in_p, wrows, wcols;
  if (k < 4 * D * D) {
    const int mt = k / (D * D);
    k -= mt * D * D;
    src = lp + mt * d * d;
    in_p = D; wrows = d; wcols = d;
  } else if (k < 4 * D * D + D * M) {
    k -= 4 * D * D;
    if (!bwd) { src = lp + 4 * d * d; in_p = D; wrows = d; wcols = M; }                   // W1 [d][M]
    else { src = lp + 4 * d * d + d * M + M; in_p = D; wrows = M; wcols = d; }            // W2^T, W2 [M][d]
  } else {
    k -= 4 * D * D + D * M;
    if (!bwd) { src = lp + 4 * d * d + d * M + M; in_p = M; wrows = M; wcols = d; }       // W2 [M][d]
    else { src = lp + 4 * d * d; in_p = M; wrows = d; wcols = M; }                        // W1^T, W1 [d][M]
  }
  const int frag = k / (64 * KPL);
  const int rem = k % (64 * KPL);
  const int lane = rem / KPL, t = rem % KPL;
  const int s = frag % ST;
  const int ib = (frag / ST) % (in_p / 32);
  const int ob = frag / (ST * (in_p / 32));
  const int in = 32 * ib + tile_idx(s * KPL + t, lane >> 5);
  const int o = 32 * ob + (lane & 31);
  if (!bwd) return in < wrows && o < wcols ? src[in * wcols + o] : 0.f;
  return o < wrows && in < wcols ? src[o * wcols + in] : 0.f;
}

// Everything that depends on the parameters alone, in one launch (it had been three, 15 us at
// width 64): workgroups 0..63 form the embedding table, the others pack the forward fragments, the
// transposed ones (wb, or NULL) and the padded biases b1 [L][M], b2 [L][D].
template <int KPL, class T>
__global__ void __launch_bounds__(256) k_pack(const float* __restrict__ params, PackPlan pp, T* __restrict__ wf, T* __restrict__ wb,
                                              float* __restrict__ b1o, float* __restrict__ b2o, float* __restrict__ table) {
  if (blockIdx.x < 64) {
    embed_table_row(params, pp.d, pp.D, blockIdx.x, table);
    return;
  }
  const int D = pp.D, M = pp.M, d = pp.d;
  const int64_t total = pp.layer_elems * pp.layers, both = wb ? 2 * total : total, end = both + (int64_t)pp.layers * (M + D);
  for (int64_t e = (int64_t)(blockIdx.x - 64) * 256 + threadIdx.x; e < end; e += (int64_t)(gridDim.x - 64) * 256) {
    if (e < total) wf[e] = (T)packed_weight<KPL>(params, pp, false, e);
    else if (e < both) wb[e - total] = (T)packed_weight<KPL>(params, pp, true, e - total);
    else {
      const int q = (int)(e - both), l = q / (M + D), k = q % (M + D);
      const float* lp = params + pp.off_layer0 + (int64_t)l * pp.layer_stride + 4LL * d * d + (int64_t)d * M;
      if (k < M) b1o[l * M + k] = lp[k];
      else b2o[l * D + k - M] = k - M < d ? lp[(int64_t)M + (int64_t)d * M + k - M] : 0.0f;
    }
  }
}

int32_t launch_pack(const PackPlan& pp, const float* params, bool bf16, void* wf, void* wb, float* b1, float* b2,
                    float* table, hipStream_t st) {
  const int64_t total = pp.layer_elems * pp.layers * (wb ? 2 : 1) + pp.layers * (pp.M + pp.D);
  const int blocks = 64 + (int)std::min<int64_t>(ceil_div(total, 256), 4096);
  if (bf16) hipLaunchKernelGGL((k_pack<8, __bf16>), dim3(blocks), dim3(256), 0, st, params, pp, (__bf16*)wf, (__bf16*)wb, b1, b2, table);
  else hipLaunchKernelGGL((k_pack<4, float>), dim3(blocks), dim3(256), 0, st, params, pp, (float*)wf, (float*)wb, b1, b2, table);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

}  // namespace tdo
