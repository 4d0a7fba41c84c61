// Rows of the Jacobian O_k(x_b) = d log rho(x_b) / d theta_k (App. C, metric tensor of
// stochastic reconfiguration) from per-configuration results of the backward kernels: the
// layer kernels run with one workgroup per configuration, so each weight-gradient partial
// belongs to one configuration, and the kernels here write it out as FP64 rows.
#include "common.h"
#include "net.h"
#include "netapi.h"

namespace tdo {

// Layer part of E rows: the padded FP32 partials of configuration blockIdx.y, summed in FP64 over
// its slots, in the parameter layout.  Bound by the FP64 rows written (8 bytes a parameter; the
// partials, 4 bytes, come from the caches): one value per thread, consecutive in the row.
__global__ void __launch_bounds__(256) k_jac_layer(const float* __restrict__ mpart, int slots, const float* __restrict__ apart,
                                                   int d, int D, int M, double* __restrict__ jac, int64_t stride) {
  const int64_t e = blockIdx.y;
  const int mlen = 2 * D * M + M + D, tot = 4 * d * d + 2 * d * M + M + d;
  const float* ap = apart + e * 4 * D * D;
  const float* mp = mpart + e * slots * mlen;
  double* row = jac + e * stride;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < tot; i += gridDim.x * 256) {
    double v = 0.0;
    if (i < 4 * d * d) {
      const int mt = i / (d * d), rem = i % (d * d), r = rem / d, c = rem % d;
      v = (double)ap[mt * D * D + r * D + c];
    } else {
      int k = i - 4 * d * d;  // [W1 d x M][b1 M][W2 M x d][b2 d]
      if (k >= d * M) {  // W1 has the same layout padded
        if ((k -= d * M) < M) k += 2 * D * M;
        else if ((k -= M) < d * M) k = D * M + (k / d) * D + k % d;
        else k += 2 * D * M + M - d * M;
      }
      for (int s = 0; s < slots; ++s) v += (double)mp[(int64_t)s * mlen + k];
    }
    row[i] = v;
  }
}

// Head part of E rows: dW_head[f][k] = sum over the configuration's passes of (mean over its rows of
// x_L[f]) dF_k, db_head[k] = sum of dF_k / n over its rows (FP64 sums of FP32 products, as in the
// reverse-mode pass).  One workgroup per configuration, one wave per block.
template <class P, int D>
__global__ void __launch_bounds__(256) k_jac_head(const void* __restrict__ save_last, const float* __restrict__ seeds,
                                                  int n, int span, int d_real, double* __restrict__ jac, int64_t stride) {
  using save_t = typename P::save_t;
  constexpr int NB = D / 32;
  __shared__ double red[4][2 * D + 2];
  const int64_t e = blockIdx.x;
  const int bpc = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int pass = span ? wave >> 1 : wave, row = (span ? (wave & 1) * 32 : 0) + lr;
  const float inv_n = 1.0f / (float)n;
  float s0 = 0.f, s1 = 0.f;
  if (row < n) {
    s0 = seeds[(e * 2 + pass) * 2] * inv_n;
    s1 = seeds[(e * 2 + pass) * 2 + 1] * inv_n;
  }
  const save_t* xs = reinterpret_cast<const save_t*>(save_last) + (e * bpc + wave) * NB * 64 * 16;
  auto sum32 = [](double v) {
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
#pragma unroll
  for (int ob = 0; ob < NB; ++ob) {
    const f32x16 v = load_tile(xs + ob * 1024, lane);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double u0 = sum32((double)(v[r] * s0)), u1 = sum32((double)(v[r] * s1));
      const int f = 32 * ob + tile_idx(r, h);
      if (lr == 0) {
        red[wave][2 * f] = u0;
        red[wave][2 * f + 1] = u1;
      }
    }
  }
  const double c0 = sum32(h == 0 ? (double)s0 : 0.0), c1 = sum32(h == 0 ? (double)s1 : 0.0);
  if (lane == 0) {
    red[wave][2 * D] = c0;
    red[wave][2 * D + 1] = c1;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * d_real + 2; i += blockDim.x) {
    const int k = i < 2 * d_real ? i : 2 * D + (i - 2 * d_real);
    double v = red[0][k];
    for (int w = 1; w < bpc; ++w) v += red[w][k];
    jac[e * stride + i] = v;
  }
}

// Tables of the embedding's chain rule, in FP64 and the same for every configuration:
// tab = [e(q)[c] for the 16 codes q = t_a + 4 t_b of two sites][e'(q)[c]][phi'(pre(code))[o] for the
// 64 window codes], e = phi(b1 + ...) the first convolution (phi = GELU), pre the second's pre-activation.
__global__ void __launch_bounds__(64) k_jac_tables(const float* __restrict__ params, int d, double* __restrict__ tab) {
  __shared__ double ea[64], eb[64];
  const float *w1 = params, *b1 = params + 4 * d, *w2 = b1 + d, *b2 = w2 + 2 * d * d;
  auto spin = [](int t, int ch) { return 1.0 - 2.0 * (double)((t >> ch) & 1); };
  auto phi = [](double u) { return 0.5 * u * (1.0 + erf(u * 0.7071067811865476)); };
  auto dphi = [](double u) { return 0.5 * (1.0 + erf(u * 0.7071067811865476)) + u * 0.3989422804014327 * exp(-0.5 * u * u); };
  const int t = threadIdx.x, code = blockIdx.x;
  const int t0 = code & 3, t1 = (code >> 2) & 3, t2 = (code >> 4) & 3;
  auto pre = [&](int ta, int tb) {
    return b1[t] + spin(ta, 0) * w1[t] + spin(ta, 1) * w1[d + t] + spin(tb, 0) * w1[2 * d + t] + spin(tb, 1) * w1[3 * d + t];
  };
  if (t < d) {
    const double pa = pre(t0, t1);
    ea[t] = phi(pa);
    eb[t] = phi(pre(t1, t2));
    if (code < 16) {
      tab[code * d + t] = ea[t];
      tab[(16 + code) * d + t] = dphi(pa);
    }
  }
  __syncthreads();
  if (t < d) {
    double acc = b2[t];
    for (int c = 0; c < d; ++c) acc += ea[c] * w2[c * d + t] + eb[c] * w2[d * d + c * d + t];
    tab[(32 + code) * d + t] = dphi(acc);
  }
}

// Convolution part of E rows from the per-wave table gradients, in FP64: per window code the contribution
// that k_embed_params forms, operation for operation, and their sum in code order, so that a row has the
// bits of tdo_log_rho_vjp of its configuration alone.  (Summing over the site that a tap does not see first takes
// a quarter of the products, but rounds otherwise, by 1e-17 of the row, and a stopped SR solve on these
// rows amplifies that to 1e-8 and more of its update.)  One workgroup per configuration.  With G[code][o] =
// dT[code][o] phi'(pre) in LDS, a thread takes 8 weights (or the input gradients of 8 codes) at a time.
// Bound: FP64 on the vector ALU, 1.6 M operations a row at width 64 (51 us for 256 rows).
__global__ void __launch_bounds__(512) k_jac_embed(const float* __restrict__ params, const double* __restrict__ tab,
                                                   const float* __restrict__ part, int bpc, int d, int D,
                                                   double* __restrict__ jac, int64_t stride) {
#pragma clang fp contract(off)
  __shared__ double G[64][64 + 1], A[64][64], B[64][64], eq[16][64];
  const int t = threadIdx.x;
  const int64_t e = blockIdx.x;
  const float* pe = part + e * bpc * 64 * D;
  const float* w2 = params + 5 * d;
  const double *deq = tab + 16 * d, *dp = tab + 32 * d;
  double* row = jac + e * stride;  // [w1 4d][b1 d][w2 2 d^2][b2 d]
  for (int i = t; i < 64 * d; i += 512) {
    const int code = i / d, o = i % d;
    double v = 0.0;
    for (int w = 0; w < bpc; ++w) v += (double)pe[(w * 64 + code) * D + o];
    G[code][o] = v * dp[i];
  }
  for (int i = t; i < 16 * d; i += 512) eq[i / d][i % d] = tab[i];
  __syncthreads();
  // code = t0 + 4 t1 + 16 t2: tap 0 sees the sites of code mod 16, tap 1 those of code / 4
  for (int i = t; i < 2 * (d / 8) * d; i += 512) {
    const int o = i % d, c0 = i / d % (d / 8) * 8, tap = i / (d * (d / 8));
    double v[8] = {};
    for (int code = 0; code < 64; ++code) {
      const double g = G[code][o];
      const double* q = eq[tap ? code >> 2 : code & 15] + c0;
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] += q[k] * g;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) row[5 * d + (tap * d + c0 + k) * d + o] = v[k];
  }
  if (t < d) {
    double v = 0.0;
    for (int code = 0; code < 64; ++code) v += G[code][t];
    row[5 * d + 2 * d * d + t] = v;
  }
  // gradients with respect to the first convolution's outputs at the two sites: A, B[code][c] = sum_o w2[tap][c][o] G
  for (int i = t; i < 2 * 8 * d; i += 512) {
    const int c = i % d, k0 = i / d % 8 * 8, tap = i / (8 * d);
    const float* wr = w2 + (tap * d + c) * d;
    double v[8] = {};
    for (int o = 0; o < d; ++o) {
      const double w = (double)wr[o];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = __builtin_fma(w, G[k0 + k][o], v[k]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) (tap ? B : A)[k0 + k][c] = v[k];
  }
  __syncthreads();
  for (int i = t; i < 5 * d; i += 512) {
    const int k = i / d, c = i % d;  // k < 4: w1[site k / 2][channel k % 2]; 4: bias
    double v = 0.0;
    for (int code = 0; code < 64; ++code) {
      const double da = deq[(code & 15) * d + c], gb = B[code][c] * deq[(code >> 2) * d + c];
      if (k == 4) {
        v += __builtin_fma(A[code][c], da, gb);
      } else {
        const int ta = (code >> (k / 2 * 2)) & 3, tb = (code >> (k / 2 * 2 + 2)) & 3;
        const double ga = A[code][c] * da;
        v += (((ta >> (k & 1)) & 1) ? -ga : ga) + (((tb >> (k & 1)) & 1) ? -gb : gb);
      }
    }
    row[i] = v;
  }
}

int32_t launch_jac_layer(const float* mpart, int slots, const float* apart, const PackPlan& pp, int64_t E, double* jac,
                         int64_t stride, hipStream_t st) {
  const int tot = 4 * pp.d * pp.d + 2 * pp.d * pp.M + pp.M + pp.d;
  hipLaunchKernelGGL(k_jac_layer, dim3((unsigned)ceil_div(tot, 1024), (unsigned)E), dim3(256), 0, st, mpart, slots, apart,
                     pp.d, pp.D, pp.M, jac, stride);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_jac_head(bool bf16, int D, const void* save_last, const float* seeds, int64_t E, int n, int span,
                        int d_real, double* jac, int64_t stride, hipStream_t st) {
  const dim3 g((unsigned)E), t(span ? 256 : 128);
  if (D == 32) {
    if (bf16) hipLaunchKernelGGL((k_jac_head<PBF16, 32>), g, t, 0, st, save_last, seeds, n, span, d_real, jac, stride);
    else hipLaunchKernelGGL((k_jac_head<PF32, 32>), g, t, 0, st, save_last, seeds, n, span, d_real, jac, stride);
  } else {
    if (bf16) hipLaunchKernelGGL((k_jac_head<PBF16, 64>), g, t, 0, st, save_last, seeds, n, span, d_real, jac, stride);
    else hipLaunchKernelGGL((k_jac_head<PF32, 64>), g, t, 0, st, save_last, seeds, n, span, d_real, jac, stride);
  }
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_jac_tables(const float* params, int d, double* tab, hipStream_t st) {
  hipLaunchKernelGGL(k_jac_tables, dim3(64), dim3(64), 0, st, params, d, tab);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_jac_embed(const float* params, const double* tab, const float* part, int bpc, int d, int D, int64_t E,
                         double* jac, int64_t stride, hipStream_t st) {
  hipLaunchKernelGGL(k_jac_embed, dim3((unsigned)E), dim3(512), 0, st, params, tab, part, bpc, d, D, jac, stride);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

}  // namespace tdo
