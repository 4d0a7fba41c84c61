// Forward-mode derivative of log rho along a parameter direction (App. C, metric tensor of
// stochastic reconfiguration: S p = Re sum_b w_b conj(dO_b) (dO_b . p) needs O_b . p, the
// Jacobian-vector product), in FP32, and the matrix-free SR solve built on it.
//
// The network (main text "Transformer density operator ansatz"; App. B) is evaluated
// together with its tangent t(.) = d(.)/d eps at theta + eps p, layer by layer over a chunk
// of configurations, in the 32-row blocks of the forward:
//   embedding:  T and t(T) for the 64 window codes (two circular convolutions, GELU each);
//   per layer:  Q = X Wq, t(Q) = t(X) Wq + X t(Wq) (and K, V);
//               per head  S = Q K^T / sqrt(dh), t(S) = (t(Q) K^T + Q t(K)^T) / sqrt(dh),
//               P = softmax(S), t(P) = P (t(S) - rowsum(P t(S))), O = P V, t(O) = t(P) V + P t(V);
//               Y = X + O Wo, t(Y) = t(X) + t(O) Wo + O t(Wo);
//               H = max(0, Y W1 + b1), t(H) = [H > 0] (t(Y) W1 + Y t(W1) + t(b1));
//               X' = Y + H W2 + b2, t(X') = t(Y) + t(H) W2 + H t(W2) + t(b2);
//   head:       f = mean_i X_i Wh + bh, t(f) = mean_i (t(X_i) Wh + X_i t(Wh)) + t(bh), z = f0 + i f1;
//   log rho = log(e^{z1} + conj e^{z2}):  t(log rho) = (e^{z1} t(z1) + conj(e^{z2} t(z2))) / (e^{z1} + conj e^{z2}).
// A layer is one kernel on the FP32 matrix cores (k_jvp_layer), value and tangent together.
// Every sum is taken in ascending order (features, keys, hidden units), so that no value depends on the
// split into tiles.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "net.h"
#include "netapi.h"
#include "train.h"

namespace tdo {

namespace {

__device__ __forceinline__ float gelu_f(float u) { return 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)); }
// d/du [u Phi(u)] = Phi(u) + u phi(u)
__device__ __forceinline__ float gelu_d(float u) {
  return 0.5f * (1.0f + erff(u * 0.70710678118654752f)) + u * 0.39894228040143268f * expf(-0.5f * u * u);
}

}  // namespace

// Order of the activations and weights here.  Value r of lane half h of a 32-feature tile is
// feature 2 r + h, and lane m holds row asc(m) of its 32-row block: the products take operand pairs
// (2 i, 2 i + 1) in turn, so features, keys and hidden units all come in ascending order.  A tile
// in memory holds its 16 values per lane in that order (load_tile); pos(f) is feature f's position in a row.
__device__ __forceinline__ int asc(int m) { return 8 * (m >> 3) + 2 * (m & 3) + ((m >> 2) & 1); }
__host__ __device__ inline int pos(int f) { return (f & ~31) + 16 * (f & 1) + ((f & 31) >> 1); }
// Feature f's position in a row of d values of the embedding tables: a tile's values of each lane half together.
__device__ inline int table_pos(int f, int d) { return d == 16 ? 8 * (f & 1) + (f >> 1) : pos(f); }

// Embedding table of the 64 window codes and its tangent (as the forward's): rows of d values in the order
// of table_pos.
__global__ void k_embed_table_jvp(const float* __restrict__ params, const double* __restrict__ tan, int d,
                                  float* __restrict__ T, float* __restrict__ Td) {
  __shared__ float e0[64], e1[64], e0d[64], e1d[64];
  const int code = blockIdx.x;
  const int t0 = code & 3, t1 = (code >> 2) & 3, t2 = (code >> 4) & 3;
  const float *w1 = params, *b1 = params + 4 * d, *w2 = b1 + d, *b2 = w2 + 2 * d * d;
  const double *w1d = tan, *b1d = tan + 4 * d, *w2d = b1d + d, *b2d = w2d + 2 * d * d;
  auto spin = [](int t, int ch) { return 1.0f - 2.0f * (float)((t >> ch) & 1); };
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    const float sa0 = spin(t0, 0), sa1 = spin(t0, 1), sb0 = spin(t1, 0), sb1 = spin(t1, 1), sc0 = spin(t2, 0),
                sc1 = spin(t2, 1);
    const float d0 = (float)w1d[c], d1 = (float)w1d[d + c], d2 = (float)w1d[2 * d + c], d3 = (float)w1d[3 * d + c], db = (float)b1d[c];
    const float a = b1[c] + sa0 * w1[c] + sa1 * w1[d + c] + sb0 * w1[2 * d + c] + sb1 * w1[3 * d + c];
    const float ad = db + sa0 * d0 + sa1 * d1 + sb0 * d2 + sb1 * d3;
    const float b = b1[c] + sb0 * w1[c] + sb1 * w1[d + c] + sc0 * w1[2 * d + c] + sc1 * w1[3 * d + c];
    const float bd = db + sb0 * d0 + sb1 * d1 + sc0 * d2 + sc1 * d3;
    e0[c] = gelu_f(a);
    e0d[c] = gelu_d(a) * ad;
    e1[c] = gelu_f(b);
    e1d[c] = gelu_d(b) * bd;
  }
  __syncthreads();
  for (int o = threadIdx.x; o < d; o += blockDim.x) {
    float acc = b2[o], accd = (float)b2d[o];
    for (int c = 0; c < d; ++c) {
      acc += e0[c] * w2[c * d + o] + e1[c] * w2[d * d + c * d + o];
      accd += e0d[c] * w2[c * d + o] + e0[c] * (float)w2d[c * d + o] + e1d[c] * w2[d * d + c * d + o] +
              e1[c] * (float)w2d[d * d + c * d + o];
    }
    T[code * d + table_pos(o, d)] = gelu_f(acc);
    Td[code * d + table_pos(o, d)] = gelu_d(acc) * accd;
  }
}

// Embedding of every block: lane (row, half) copies its 16 values of each feature block from the
// tables; zero past d and where the row belongs to no configuration.
__global__ void __launch_bounds__(256) k_jvp_embed(const uint64_t* __restrict__ cfg, int64_t E, int n, int cpb, int span,
                                                   int d, int D, const float* __restrict__ T, const float* __restrict__ Td,
                                                   float* __restrict__ X, float* __restrict__ Xd) {
  const RowMap rm{n, cpb, span != 0};
  const int64_t nblk = span ? 4 * E : 2 * ((E + cpb - 1) / cpb);
  const int lane = threadIdx.x & 63, h = lane >> 5, NB = D / 32;
  for (int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); g < nblk; g += (int64_t)gridDim.x * 4) {
    int64_t e; int pass, i; bool valid;
    rm.at(g, asc(lane & 31), E, e, pass, i, valid);
    int code = 0;
    if (valid) {
      const uint64_t a = cfg[2 * e], b = cfg[2 * e + 1], c0 = pass ? b : a, c1 = pass ? a : b;
      for (int k = 0; k < 3; ++k) {
        int s = i + k;
        s = s >= n ? s - n : s;
        code += ((int)((c0 >> s) & 1ull) + 2 * (int)((c1 >> s) & 1ull)) << (2 * k);
      }
    }
    for (int ib = 0; ib < NB; ++ib) {
      const int64_t o = (g * NB + ib) * 1024;
      const int half = d == 16 ? 8 : 16;  // values of a lane
      const float4* t = reinterpret_cast<const float4*>(T + code * d + 32 * ib + half * h);
      const float4* td = reinterpret_cast<const float4*>(Td + code * d + 32 * ib + half * h);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = valid && 4 * q < half;
        reinterpret_cast<float4*>(X + o)[64 * q + lane] = in ? t[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        reinterpret_cast<float4*>(Xd + o)[64 * q + lane] = in ? td[q] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
}

// Weights and tangents of nl layers from l0 on, as 16-byte fragments in the order above: matrices Wq,
// Wk, Wv, Wo, W1, W2 padded to [in][out]; fragment (ob, ib, s) of a matrix, lane l, value t holds
// in = 32 ib + 2 (4 s + t) + l / 32, out = 32 ob + asc(l % 32).  Then b1 (M) and b2 (D) at pos.
__global__ void k_jvp_pack(const float* __restrict__ params, const double* __restrict__ tan, PackPlan pp, int l0, int nl,
                           float* __restrict__ out, float* __restrict__ outd) {
  const int D = pp.D, M = pp.M, d = pp.d, DD = D * D, DM = D * M;
  const int64_t len = pp.layer_elems + M + D;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nl * len; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t lp = pp.off_layer0 + (l0 + e / len) * pp.layer_stride;
    int k = (int)(e % len), in_p = D, rows = d, cols = d;
    int64_t src = lp;
    bool ok = true;
    if (k < pp.layer_elems) {
      if (k < 4 * DD) { src += (int64_t)(k / DD) * d * d; k %= DD; }
      else if ((k -= 4 * DD) < DM) { src += 4 * d * d; cols = M; }
      else { k -= DM; src += 4 * d * d + d * M + M; in_p = M; rows = M; }
      const int frag = k / 256, lane = (k >> 2) & 63, t = k & 3, s = frag & 3, ib = (frag >> 2) % (in_p / 32), ob = (frag >> 2) / (in_p / 32);
      const int in = 32 * ib + 2 * (4 * s + t) + (lane >> 5), o = 32 * ob + asc(lane & 31);
      ok = in < rows && o < cols;
      src += (int64_t)in * cols + o;
    } else {  // position k of a bias holds feature f, pos(f) = k
      k -= (int)pp.layer_elems;
      const bool first = k < M;
      if (!first) k -= M;
      const int f = (k & ~31) + 2 * (k & 15) + ((k >> 4) & 1);
      src += first ? 4 * d * d + d * M + f : 4 * d * d + 2 * d * M + M + f;
      ok = first || f < d;
    }
    out[e] = ok ? params[src] : 0.f;
    outd[e] = ok ? (float)tan[src] : 0.f;
  }
}

struct JvpArgs {
  const float *w, *wd;    // packed layer and its tangent (k_jvp_pack), or
  const float* params;    // the layer as it lies in the parameter vector
  const double* tan;      // and in the tangent
  float *x, *xd;          // residual stream and its tangent, [blocks][D/32] tiles (load_tile), in place
  int64_t E;
  int n, cpb, d, heads, M;
  float scale;
};

// One layer with its tangent.  A wave takes a 32-row block (in turn, 8 waves a workgroup) and holds
// the residual update of the block in registers; keys and values of a head block go through LDS,
// where a spanning pass's other wave reads them too.
//
// The order of every sum is part of the result.  J p is one factor of the operator that the SR solve
// iterates with, and a solve stopped after a few iterations on an ill-conditioned system carries a change
// of rounding here into its update (a changed order of the tangent's sums moved updates of the benchmark
// network by 1e-5, of one drawn system by 2e-4).  So: value sums in ascending order of their index; a tangent
// t(A) B + A t(B) of a matrix product as the ascending sum over t(A) B, then that over A t(B); in the
// attention, per key and feature, as one rounded term fma(t(a), b, a t(b)) added in ascending order.  The
// projections and the feed-forward part run on the FP32 matrix cores, which add their products one after the
// other; the second sum of a tangent repeats the hidden units (u is formed twice, a sixth of the
// feed-forward products).  The attention's tangents and its products with V, which the matrix cores would
// have to sum differently, run on the vector ALU, beside the other wave's products.  A row meets the keys of
// its own configuration only, also where a product with 0 would do: what is not finite in one configuration (an
// overflow, an infinite tangent of a hidden unit that is active there) stays out of the others.
//
// Bound: the FP32 matrix cores (157 TFLOP/s) and the latency of the weight fragments, which come through the
// caches: two waves per SIMD cover part of it (loaded ahead in registers, as the forward does, they spill).
// 16384 configurations at n = 32, benchmark network: 15.8 ms; 32768 at n = 16, 4 heads, 2 layers 8.2 ms; 4096 at
// n = 64, 2 layers 4.9 ms (with the sums in the order that suits the matrix cores 13.8, 6.6 and 4.6 ms; the same sums
// as separate products on the vector ALU between activations in memory 75.1, 28.1 and 31.2 ms).
// PACKED: weights from the packed fragments; otherwise, in a workspace too small for a packed layer, from the
// parameter vector element by element (16384 configurations at n = 32 in 380 KB, a few at a time: 2.7 s).
template <int D, int DH, bool SPAN, bool MASKED, bool PACKED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) k_jvp_layer(JvpArgs a) {
#pragma clang fp contract(off)
  constexpr int NB = D / 32, HPB = 32 / DH, VPH = DH / 2, NKB = SPAN ? 2 : 1, LS = 36, TILE = 32 * LS;
  using P = PF32;
  __shared__ __align__(16) float sm[8][4][TILE];  // per wave: k, t(k), v, t(v) [row][pos]
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = a.n, cpb = a.cpb, M = a.M, MB = M / 32, d = a.d;
  const int64_t nblk = SPAN ? 4 * a.E : 2 * ((a.E + cpb - 1) / cpb);
  // fragment (ob, ib, s) of matrix m (Wq, Wk, Wv, Wo, W1, W2) or of its tangent
  auto frag = [&](int m, int ob, int ib, int s, bool tangent) -> f32x4 {
    const int nib = m == 5 ? MB : NB;
    if constexpr (PACKED) {
      const float* w = (tangent ? a.wd : a.w) + (m < 4 ? m * D * D : 4 * D * D + (m - 4) * D * M);
      return ld_frag<P>(w, (ob * nib + ib) * 4 + s, lane);
    } else {
      const int rows = m == 5 ? M : d, cols = m == 4 ? M : d;
      const int o = m < 4 ? m * d * d : m == 4 ? 4 * d * d : 4 * d * d + d * M + M;
      const int out = 32 * ob + asc(lr);
      f32x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int in = 32 * ib + 2 * (4 * s + t) + h, i = o + in * cols + out;
        const bool ok = in < rows && out < cols;
        v[t] = !ok ? 0.f : tangent ? (float)a.tan[i] : a.params[i];
      }
      return v;
    }
  };
  // 16 values of a bias (b1 or b2) or of its tangent, features 32 c + 2 r + h
  auto bias = [&](bool second, int c, bool tangent) {
    f32x16 v;
    if constexpr (PACKED) {
      const float* p = (tangent ? a.wd : a.w) + 4 * D * D + 2 * D * M + (second ? M : 0) + 32 * c + 16 * h;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 t = reinterpret_cast<const float4*>(p)[q];
        v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
      }
    } else {
      const int o = 4 * d * d + d * M + (second ? M + d * M : 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f = 32 * c + 2 * r + h;
        v[r] = second && f >= d ? 0.f : tangent ? (float)a.tan[o + f] : a.params[o + f];
      }
    }
    return v;
  };
  // keys of this lane's query row asc(lr): bit k of keys[kb] is row k of key block kb
  uint32_t keys[NKB];
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    keys[kb] = SPAN ? (uint32_t)low_mask(n - 32 * kb < 32 ? n - 32 * kb : 32) : ~0u;
    if constexpr (MASKED && !SPAN) keys[kb] = asc(lr) / n < cpb ? (uint32_t)low_mask(n) << (asc(lr) / n * n) : 0u;
  }
  const int kw = SPAN ? wave & ~1 : wave;  // wave that holds key block 0, the next one key block 1
  auto store16 = [](float* p, const f32x16& v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) reinterpret_cast<float4*>(p)[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  };
  auto lds_sync = [] {
    if constexpr (SPAN) barrier_lds();
    else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    }
  };
  // both halves' value of a lane: lower half first
  auto halves = [](float v, float& lo, float& hi) {
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    lo = __uint_as_float(b[0]);
    hi = __uint_as_float(b[1]);
  };

  for (int64_t base = (int64_t)blockIdx.x * 8; base < nblk; base += (int64_t)gridDim.x * 8) {
    const bool live = base + wave < nblk;
    if (!SPAN && !live) continue;
    const int64_t g = live ? base + wave : base + (wave & 1);  // a spanning pass's waves all meet at the barriers
    float *xb = a.x + g * NB * 1024, *xdb = a.xd + g * NB * 1024;  // feature block ib at 1024 ib
    f32x16 o[NB], od[NB];
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) o[ob] = od[ob] = f32x16{};
#pragma unroll 1
    for (int hb = 0; hb < NB; ++hb) {
      // value and tangent of a projection's head block: c = W^T x, cd = W^T t(x), then + t(W)^T x
      auto project = [&](int m, f32x16& c, f32x16& cd) {
        c = cd = f32x16{};
        auto xo = [&](const float* x, int ib, int s) { return *reinterpret_cast<const f32x4*>(x + 1024 * ib + 256 * s + 4 * lane); };
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const f32x4 w = frag(m, hb, ib, s, false);
            c = P::mma(w, xo(xb, ib, s), c);
            cd = P::mma(w, xo(xdb, ib, s), cd);
          }
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int s = 0; s < 4; ++s) cd = P::mma(frag(m, hb, ib, s, true), xo(xb, ib, s), cd);
      };
      f32x16 q, qd;
      project(1, q, qd);
      store16(sm[wave][0] + lr * LS + 16 * h, q);
      store16(sm[wave][1] + lr * LS + 16 * h, qd);
      project(2, q, qd);
      store16(sm[wave][2] + lr * LS + 16 * h, q);
      store16(sm[wave][3] + lr * LS + 16 * h, qd);
      project(0, q, qd);
      lds_sync();
      f32x16 oh = f32x16{}, ohd = f32x16{};
      // One head at a time: its features of q and qd are the first VPH values, the registers are moved down by
      // VPH after each head, and its VPH output values enter at the top of oh, ohd.
#pragma unroll 1
      for (int j = 0; j < HPB; ++j) {
        float oj[VPH], odj[VPH];
#pragma unroll
        for (int t = 0; t < VPH; ++t) oj[t] = odj[t] = 0.f;
        if (hb * HPB + j < a.heads) {  // else padding features
          const float* kv = sm[kw][0] + VPH * j;  // block kb's k, t(k), v, t(v) at (4 kb + 0..3) TILE
          f32x16 p[NKB], pd[NKB];
          float qf[DH], qdf[DH];  // the query row's features of this head
#pragma unroll
          for (int t = 0; t < VPH; ++t) {
            halves(q[t], qf[2 * t], qf[2 * t + 1]);
            halves(qd[t], qdf[2 * t], qdf[2 * t + 1]);
          }
          float mx = -INFINITY;
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb) {
            p[kb] = f32x16{};
            const float* kp = kv + 4 * kb * TILE;
#pragma unroll
            for (int t = 0; t < VPH; ++t) p[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(kp[lr * LS + 16 * h + t], q[t], p[kb], 0, 0, 0);
            // tangents, key 2 r + h (at position tile_idx(r, h)) in turn; [k even, k odd, t(k) even, t(k) odd] one key ahead
            f32x4 w[2][VPH];
            auto fetch = [&](int r) {
              const float* k = kp + tile_idx(r, h) * LS;
#pragma unroll
              for (int t0 = 0; t0 < VPH; t0 += 4)
#pragma unroll
                for (int i = 0; i < 4; ++i) w[r & 1][t0 + i] = *reinterpret_cast<const f32x4*>(k + (i >> 1) * TILE + (i & 1) * 16 + t0);
            };
            fetch(0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              if (r < 15) fetch(r + 1);
              float s = 0.f;
#pragma unroll
              for (int f = 0; f < DH; ++f) {
                const int t0 = f / 8 * 4, t = f / 2 % 4;
                s = s + __builtin_fmaf(qdf[f], w[r & 1][t0 + (f & 1)][t], qf[f] * w[r & 1][t0 + 2 + (f & 1)][t]);
              }
              const bool ok = (keys[kb] >> (2 * r + h)) & 1u;
              p[kb][r] = ok ? p[kb][r] * a.scale : -INFINITY;
              pd[kb][r] = ok ? s * a.scale : 0.f;
              mx = fmaxf(mx, p[kb][r]);
              __builtin_amdgcn_sched_barrier(0);  // one key at a time: the registers
            }
          }
          mx = xor32_max(mx);
          const bool any = keys[0] != 0;  // a padding row has no key: P = 0
          const float mm = any ? mx : 0.f;
          float l = 0.f;
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {  // keys 2 r (lower half of the wave), then 2 r + 1
              p[kb][r] = expf(p[kb][r] - mm);
              float e0, e1;
              halves(p[kb][r], e0, e1);
              l += e0;
              l += e1;
            }
          const float inv = any ? 1.0f / l : 0.f;
          float dot = 0.f;
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              p[kb][r] *= inv;
              float e0, e1, d0, d1;
              halves(p[kb][r], e0, e1);
              halves(pd[kb][r], d0, d1);
              dot = __builtin_fmaf(e0, d0, dot);
              dot = __builtin_fmaf(e1, d1, dot);
            }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int kb = 0; kb < NKB; ++kb) {
            f32x4 w[2][VPH / 2];  // [v, t(v)] of the next key
            auto fetch = [&](int k) {
              const float* v = kv + (4 * kb + 2) * TILE + tile_idx(k >> 1, k & 1) * LS + 16 * h;
#pragma unroll
              for (int t0 = 0; t0 < VPH; t0 += 4)
#pragma unroll
                for (int i = 0; i < 2; ++i) w[k & 1][t0 / 2 + i] = *reinterpret_cast<const f32x4*>(v + i * TILE + t0);
            };
            fetch(0);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              pd[kb][r] = p[kb][r] * (pd[kb][r] - dot);
              float e[2], ed[2];
              halves(p[kb][r], e[0], e[1]);
              halves(pd[kb][r], ed[0], ed[1]);
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                const int k = 2 * r + i;
                if (k < 31) fetch(k + 1);
                const bool ok = (keys[kb] >> k) & 1u;
#pragma unroll
                for (int t = 0; t < VPH; ++t) {
                  float v = w[i][t / 4 * 2][t % 4], vd = w[i][t / 4 * 2 + 1][t % 4];
                  if (MASKED && (!SPAN || kb == 1)) { v = ok ? v : 0.f; vd = ok ? vd : 0.f; }
                  oj[t] = __builtin_fmaf(e[i], v, oj[t]);
                  odj[t] = odj[t] + __builtin_fmaf(ed[i], v, e[i] * vd);
                }
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          q[r] = r + VPH < 16 ? q[(r + VPH) & 15] : 0.f;
          qd[r] = r + VPH < 16 ? qd[(r + VPH) & 15] : 0.f;
          oh[r] = r + VPH < 16 ? oh[(r + VPH) & 15] : oj[(r + VPH) & (VPH - 1)];
          ohd[r] = r + VPH < 16 ? ohd[(r + VPH) & 15] : odj[(r + VPH) & (VPH - 1)];
        }
      }
      if (NB == 1 || hb == 0) { o[0] = oh; od[0] = ohd; }
      else { o[NB - 1] = oh; od[NB - 1] = ohd; }
      lds_sync();  // keys and values read before the next head block's (or block's) are written
    }
    f32x16 y[NB], yd[NB];
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      y[ob] = yd[ob] = f32x16{};
#pragma unroll
      for (int i = 0; i < 4 * NB; ++i) {
        const f32x4 w = frag(3, ob, i / 4, i % 4, false);
        y[ob] = P::mma(w, P::op(o[i / 4], i % 4), y[ob]);
        yd[ob] = P::mma(w, P::op(od[i / 4], i % 4), yd[ob]);
      }
#pragma unroll
      for (int i = 0; i < 4 * NB; ++i) yd[ob] = P::mma(frag(3, ob, i / 4, i % 4, true), P::op(o[i / 4], i % 4), yd[ob]);
    }
    f32x16 z[NB], zd[NB];
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      const f32x16 x = load_tile(xb + 1024 * ob, lane), xd = load_tile(xdb + 1024 * ob, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) { y[ob][r] += x[r]; yd[ob][r] += xd[r]; }
      z[ob] = zd[ob] = f32x16{};
    }
    // ---- feed-forward: hidden units in chunks of 32; first W2 with u and t(u), then t(W2) with u
#pragma unroll 1
    for (int c = 0; c < MB; ++c) {
      f32x16 u = f32x16{}, ud = f32x16{};
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f32x4 w = frag(4, c, ib, s, false);
          u = P::mma(w, P::op(y[ib], s), u);
          ud = P::mma(w, P::op(yd[ib], s), ud);
        }
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int s = 0; s < 4; ++s) ud = P::mma(frag(4, c, ib, s, true), P::op(y[ib], s), ud);
      const f32x16 b = bias(false, c, false), bd = bias(false, c, true);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        u[r] = fmaxf(u[r] + b[r], 0.f);
        ud[r] = u[r] > 0.f ? ud[r] + bd[r] : 0.f;
      }
#pragma unroll
      for (int ob = 0; ob < NB; ++ob)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f32x4 w = frag(5, ob, c, s, false);
          z[ob] = P::mma(w, P::op(u, s), z[ob]);
          zd[ob] = P::mma(w, P::op(ud, s), zd[ob]);
        }
    }
#pragma unroll 1
    for (int c = 0; c < MB; ++c) {
      f32x16 u = f32x16{};
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int s = 0; s < 4; ++s) u = P::mma(frag(4, c, ib, s, false), P::op(y[ib], s), u);
      const f32x16 b = bias(false, c, false);
#pragma unroll
      for (int r = 0; r < 16; ++r) u[r] = fmaxf(u[r] + b[r], 0.f);
#pragma unroll
      for (int ob = 0; ob < NB; ++ob)
#pragma unroll
        for (int s = 0; s < 4; ++s) zd[ob] = P::mma(frag(5, ob, c, s, true), P::op(u, s), zd[ob]);
    }
    if (live)
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        const f32x16 b = bias(true, ob, false), bd = bias(true, ob, true);
#pragma unroll
        for (int r = 0; r < 16; ++r) { z[ob][r] = (z[ob][r] + b[r]) + y[ob][r]; zd[ob][r] = (zd[ob][r] + bd[r]) + yd[ob][r]; }
        store_tile(xb + 1024 * ob, lane, z[ob]);
        store_tile(xdb + 1024 * ob, lane, zd[ob]);
      }
  }
}

// Mean pooling and head, one wave per configuration-pass: z = (f0, f1), t(z).  Lane l adds the elements
// l, l + 64, .. of the pass's n x d activations in order, then the lanes are summed.
__global__ void __launch_bounds__(256) k_jvp_head(int64_t E, int n, int cpb, int span, int d, int D, const float* __restrict__ X,
                                                  const float* __restrict__ Xd, const float* __restrict__ hw,
                                                  const double* __restrict__ hwd, float* __restrict__ z, float* __restrict__ zd) {
  const float* hb = hw + 2 * d;
  const double* hbd = hwd + 2 * d;
  const int lane = threadIdx.x & 63, NB = D / 32;
  const int f = lane % d, ib = f >> 5, r = (f & 31) >> 1, h = f & 1;  // feature f: value r of lane half h of tile ib
  const int in_tile = 256 * (r >> 2) + 128 * h + (r & 3);
  const float w0 = hw[2 * f], w1 = hw[2 * f + 1], wd0 = (float)hwd[2 * f], wd1 = (float)hwd[2 * f + 1];
  for (int64_t ep = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); ep < 2 * E; ep += (int64_t)gridDim.x * 4) {
    const int64_t e = ep >> 1, g = span ? 2 * ep : 2 * (e / cpb) + (ep & 1);
    const int row0 = span ? 0 : (int)(e % cpb) * n;
    float f0 = 0.f, f1 = 0.f, g0 = 0.f, g1 = 0.f;
    for (int i = lane / d; i < n; i += 64 / d) {
      const int row = row0 + i, m = (row & 24) + ((row >> 1) & 3) + 4 * (row & 1);  // asc(m) = row mod 32
      const int64_t at = ((g + (row >> 5)) * NB + ib) * 1024 + in_tile + 4 * m;
      const float x = X[at], xd = Xd[at];
      f0 = __builtin_fmaf(x, w0, f0);
      f1 = __builtin_fmaf(x, w1, f1);
      g0 = g0 + __builtin_fmaf(xd, w0, x * wd0);
      g1 = g1 + __builtin_fmaf(xd, w1, x * wd1);
    }
    f0 = wave_sum(f0);
    f1 = wave_sum(f1);
    g0 = wave_sum(g0);
    g1 = wave_sum(g1);
    if (lane == 0) {
      const float inv = 1.0f / (float)n;
      z[2 * ep] = __builtin_fmaf(f0, inv, hb[0]);
      z[2 * ep + 1] = __builtin_fmaf(f1, inv, hb[1]);
      zd[2 * ep] = __builtin_fmaf(g0, inv, (float)hbd[0]);
      zd[2 * ep + 1] = __builtin_fmaf(g1, inv, (float)hbd[1]);
    }
  }
}

// t(log rho) per configuration from z, t(z) of its two passes.
__global__ void k_jvp_combine(int64_t E, const float* __restrict__ z, const float* __restrict__ zd,
                              float* __restrict__ out) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E; e += (int64_t)gridDim.x * blockDim.x) {
    const float a0 = z[4 * e], a1 = z[4 * e + 1], b0 = z[4 * e + 2], b1 = z[4 * e + 3];
    const float mx = fmaxf(a0, b0);
    float s, c;
    const float ea = expf(a0 - mx), eb = expf(b0 - mx);
    sincosf(a1, &s, &c);
    const float w1r = ea * c, w1i = ea * s;   // e^{z1}
    sincosf(-b1, &s, &c);
    const float w2r = eb * c, w2i = eb * s;   // e^{conj z2}
    const float t1r = zd[4 * e], t1i = zd[4 * e + 1], t2r = zd[4 * e + 2], t2i = -zd[4 * e + 3];  // t(z1), conj t(z2)
    const float nr = w1r * t1r - w1i * t1i + w2r * t2r - w2i * t2i;
    const float ni = w1r * t1i + w1i * t1r + w2r * t2i + w2i * t2r;
    const float Sr = w1r + w2r, Si = w1i + w2i, nn = Sr * Sr + Si * Si;
    out[2 * e] = nn > 0.f ? (nr * Sr + ni * Si) / nn : 0.f;
    out[2 * e + 1] = nn > 0.f ? (ni * Sr - nr * Si) / nn : 0.f;
  }
}

}  // namespace tdo

namespace tdo {

namespace {

template <int D, int DH, bool SPAN>
int32_t launch_jvp_span(const JvpArgs& a, bool masked, bool packed, int num_cus, hipStream_t st) {
  const int64_t nblk = SPAN ? 4 * a.E : 2 * ((a.E + a.cpb - 1) / a.cpb);
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((nblk + 7) / 8, num_cus));
  auto k = !packed ? k_jvp_layer<D, DH, SPAN, true, false> : masked ? k_jvp_layer<D, DH, SPAN, true, true> : k_jvp_layer<D, DH, SPAN, false, true>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(512), 0, st, a);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

template <int D, int DH>
int32_t launch_jvp_layer(const JvpArgs& a, bool span, bool masked, bool packed, int num_cus, hipStream_t st) {
  return span ? launch_jvp_span<D, DH, true>(a, masked, packed, num_cus, st) : launch_jvp_span<D, DH, false>(a, masked, packed, num_cus, st);
}

// floats of one packed layer (weights, b1, b2)
int64_t jvp_layer_len(const PackPlan& pp) { return pp.layer_elems + pp.M + pp.D; }

}  // namespace

// Bytes that plan_jvp needs at least: the tables, one block's configurations (z and t(z) among them) and the
// roundings of eight buffers.
static size_t jvp_small(const NetPlan& np) { return 128 * (size_t)np.pp.d * 4 + 8 * 256; }
static size_t jvp_unit(const NetPlan& np) { return (np.span ? 4 : 2) * (32 * (size_t)np.D * 4 * 2) + np.cpb * 32; }
size_t jvp_min_bytes(const NetPlan& np) { return jvp_small(np) + jvp_unit(np); }

// Lay out the forward-mode buffers from ar.used on, for at most B configurations and
// within max_bytes.
int32_t plan_jvp(const NetPlan& np, int64_t B, size_t max_bytes, Arena& ar, JvpWs* j) {
  const PackPlan& pp = np.pp;
  const size_t unit = jvp_unit(np);
  const size_t layer = 2 * (size_t)jvp_layer_len(pp) * 4;
  TDO_CHECK(max_bytes >= jvp_min_bytes(np), TDO_ENOMEM,
            "workspace cannot hold the forward-mode buffers of one configuration (%zu bytes)", jvp_min_bytes(np));
  // every layer's weights packed once per call; in a small workspace one layer's at a time; or none
  j->layers = jvp_min_bytes(np) + pp.layers * layer <= max_bytes / 2 ? pp.layers : jvp_min_bytes(np) + layer <= max_bytes ? 1 : 0;
  const size_t fixed = jvp_small(np) + j->layers * layer;
  const int64_t units = std::max<int64_t>(1, std::min<int64_t>((B + np.cpb - 1) / np.cpb, (int64_t)((max_bytes - fixed) / unit)));
  j->ec = units * np.cpb;
  j->T = ar.take<float>(64 * (size_t)pp.d);
  j->Td = ar.take<float>(64 * (size_t)pp.d);
  j->w = ar.take<float>(j->layers * (size_t)jvp_layer_len(pp));
  j->wd = ar.take<float>(j->layers * (size_t)jvp_layer_len(pp));
  j->X = ar.take<float>((size_t)blocks_for(np, j->ec) * 32 * np.D);
  j->Xd = ar.take<float>((size_t)blocks_for(np, j->ec) * 32 * np.D);
  j->z = ar.take<float>(4 * (size_t)j->ec);
  j->zd = ar.take<float>(4 * (size_t)j->ec);
  return TDO_OK;
}

// Tables and packed weights (once per tangent), then per chunk the network and its tangent;
// out[e] = t(log rho(cfg[e])) as (re, im).
int32_t run_jvp(const NetPlan& np, void* ws, const JvpWs& j, const float* params, const double* tan, const uint64_t* cfg,
                int64_t B, float* out, hipStream_t st) {
  const PackPlan& pp = np.pp;
  const int64_t len = jvp_layer_len(pp);
  float *T = at<float>(ws, j.T), *Td = at<float>(ws, j.Td), *w = at<float>(ws, j.w), *wd = at<float>(ws, j.wd);
  float *X = at<float>(ws, j.X), *Xd = at<float>(ws, j.Xd), *z = at<float>(ws, j.z), *zd = at<float>(ws, j.zd);
  auto pack = [&](int l0) {
    hipLaunchKernelGGL(k_jvp_pack, dim3((unsigned)std::min<int64_t>(ceil_div(j.layers * len, 256), 4096)), dim3(256), 0, st,
                       params, tan, pp, l0, j.layers, w, wd);
  };
  hipLaunchKernelGGL(k_embed_table_jvp, dim3(64), dim3(64), 0, st, params, tan, pp.d, T, Td);
  const bool all = j.layers == pp.layers;
  if (all) pack(0);
  TDO_HIP(hipGetLastError());
  for (int64_t e0 = 0; e0 < B; e0 += j.ec) {
    const int64_t E = std::min(j.ec, B - e0), nblk = blocks_for(np, E);
    const unsigned grid = (unsigned)std::min<int64_t>(ceil_div(nblk, 4), 8192), grid2 = (unsigned)std::min<int64_t>(ceil_div(2 * E, 4), 8192);
    hipLaunchKernelGGL(k_jvp_embed, dim3(grid), dim3(256), 0, st, cfg + 2 * e0, E, np.n, np.cpb, (int)np.span, pp.d, np.D, T, Td, X, Xd);
    TDO_HIP(hipGetLastError());
    for (int l = 0; l < pp.layers; ++l) {
      if (j.layers && !all) pack(l);
      JvpArgs a{};
      const int64_t o = all ? l * len : 0;
      a.w = w + o;
      a.wd = wd + o;
      a.params = params + pp.off_layer0 + l * pp.layer_stride;
      a.tan = tan + pp.off_layer0 + l * pp.layer_stride;
      a.d = pp.d;
      a.x = X;
      a.xd = Xd;
      a.E = E;
      a.n = np.n;
      a.cpb = np.cpb;
      a.heads = pp.heads;
      a.M = pp.M;
      a.scale = (float)(1.0 / std::sqrt((double)np.DH));
      if (np.D == 32) TDO_TRY(np.DH == 8 ? (launch_jvp_layer<32, 8>(a, np.span, np.masked, j.layers > 0, np.num_cus, st)) : (launch_jvp_layer<32, 16>(a, np.span, np.masked, j.layers > 0, np.num_cus, st)));
      else TDO_TRY(np.DH == 8 ? (launch_jvp_layer<64, 8>(a, np.span, np.masked, j.layers > 0, np.num_cus, st)) : (launch_jvp_layer<64, 16>(a, np.span, np.masked, j.layers > 0, np.num_cus, st)));
    }
    hipLaunchKernelGGL(k_jvp_head, dim3(grid2), dim3(256), 0, st, E, np.n, np.cpb, (int)np.span, pp.d, np.D, X, Xd,
                       params + pp.off_head_w, tan + pp.off_head_w, z, zd);
    hipLaunchKernelGGL(k_jvp_combine, dim3((unsigned)std::min<int64_t>(ceil_div(E, 256), 4096)), dim3(256), 0, st, E,
                       z, zd, out + 2 * e0);
    TDO_HIP(hipGetLastError());
  }
  return TDO_OK;
}

int32_t jvp_check(const Context& c, const tdo_arch_t* arch, int32_t n, int64_t B, NetPlan* np) {
  TDO_TRY(net_plan(&c, arch, n, false, np));
  TDO_CHECK(B >= 0, TDO_EINVAL, "B=%lld < 0", (long long)B);
  return TDO_OK;
}

}  // namespace tdo

using namespace tdo;

extern "C" int32_t tdo_log_rho_jvp(tdo_ctx_t* ctx, const tdo_arch_t* arch, const float* params, int32_t n,
                                   const uint64_t* cfg, int64_t B, const double* tangent, float* jvp,
                                   hipStream_t stream) {
  clear_error();
  TDO_CHECK(ctx != nullptr, TDO_EINVAL, "ctx is NULL");
  NetPlan np;
  TDO_TRY(jvp_check(ctx->c, arch, n, B, &np));
  if (B == 0) return TDO_OK;
  TDO_CHECK(params && cfg && tangent && jvp, TDO_EINVAL, "NULL buffer");
  TDO_HIP(hipSetDevice(ctx->c.device));
  Context& c = ctx->c;
  WsOrder order;
  TDO_TRY(order.begin(&c, stream));
  TDO_TRY(check_params_finite(&c, params, np.pp.nparams, stream));
  Arena ar;
  JvpWs j;
  TDO_CHECK(c.budget > 4096, TDO_ENOMEM, "workspace budget %zu too small", c.budget);
  TDO_TRY(plan_jvp(np, B, c.budget, ar, &j));
  TDO_TRY(ensure_workspace(&c, ar.used));
  return run_jvp(np, c.ws, j, params, tangent, cfg, B, jvp, stream);
}
