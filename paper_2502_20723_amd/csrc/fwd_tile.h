// One tile of the forward pass in a wave's registers: the embedding code of a row, the attention and
// feed-forward sub-layers, the pooled head and the Hermitian symmetrisation.  Shared by the
// layer-by-layer kernel and the kernel that takes a tile through the whole network, so that both
// give the same bits.
#pragma once

#include "net.h"

namespace tdo {

template <int D>
struct EmbedRow {
  // Window code of the two width-2 circular convolutions: x_i depends on
  // sites i, i+1, i+2; code = t_i + 4 t_{i+1} + 16 t_{i+2},
  // t = bit(channel 0) + 2 bit(channel 1).
  __device__ static __forceinline__ int code(uint64_t c0, uint64_t c1, int i, int n) {
    int cd = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      int s = i + k;
      s = s >= n ? s - n : s;
      const int t = (int)((c0 >> s) & 1ull) + 2 * (int)((c1 >> s) & 1ull);
      cd += t << (2 * k);
    }
    return cd;
  }
};

// FP32 weights come through the caches, and a load left to the compiler sits right before its use,
// where the wave waits for L2.  Here the fragments of the next group of STEPS products are loaded
// before the current group's are issued, into the other of two register buffers.  Groups of STEPS:
// with groups of a whole matrix the buffers spill (one layer of 32768 FP32 configurations, width 64,
// n = 16: 1.23 ms without, 1.15 with whole matrices, 1.00 so; n = 32: 2.65, 2.22, 2.11).  Sixteen-wide
// heads keep the plain loads in the attention part: their accumulators leave too few registers
// (1.03 ms with, though 16 configurations take 96 us without and 86 with).  Two row blocks per wave
// use a fragment twice and have registers to spare with one wave per SIMD only (WAVES = 4), where they
// need it most.  BF16 weights are in LDS.
template <class P, int NBR, int WAVES>
constexpr bool frags_ahead() {
  return P::KPL == 4 && (NBR == 1 || WAVES == 4);
}
template <class P>
struct Frags {
  typename P::op_t w[P::STEPS];
  __device__ __forceinline__ void load(const typename P::elem_t* W, int f0, int lane) {
#pragma unroll
    for (int s = 0; s < P::STEPS; ++s) w[s] = ld_frag<P>(W, f0 + s, lane);
    __builtin_amdgcn_sched_barrier(0);  // issued here, not at the use
  }
};

// Attention sub-layer: x += W_O concat_j softmax(Q_j K_j^T / sqrt(dh)) V_j.  okbits[qb][kb]: the valid
// (query row qb*32+lr, key row kb*32+tile_idx(r, h)) pairs as bit r; sc = log2(e)/sqrt(dh);
// put_lse(hb, lsev): the log2 softmax normalisers of head block hb, per row block and head.
template <class P, int D, int DH, int NBR, bool MASKED, int WAVES = 8, class Lse>
__device__ __forceinline__ void tile_attention(f32x16 (&x)[NBR][D / 32], const typename P::elem_t* Wq, const typename P::elem_t* Wk,
                                               const typename P::elem_t* Wv, const typename P::elem_t* Wo,
                                               const uint32_t (&okbits)[NBR][NBR], float sc, int lane, Lse&& put_lse) {
  constexpr int NB = D / 32, ST = P::STEPS, HPB = 32 / DH;
  constexpr bool AHEAD = (DH == 8 || WAVES == 4) && frags_ahead<P, NBR, WAVES>();
  using op_t = typename P::op_t;
  // operands of x taken before the residual is updated
  op_t xo[NBR][NB][ST];
#pragma unroll
  for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int s = 0; s < ST; ++s) xo[rb][ib][s] = P::op(x[rb][ib], s);

  Frags<P> w[2];
  if constexpr (AHEAD) w[0].load(Wq, 0, lane);
#pragma unroll 1
  for (int hb = 0; hb < NB; ++hb) {
    f32x16 q[NBR], k[NBR], v[NBR];
#pragma unroll
    for (int rb = 0; rb < NBR; ++rb) q[rb] = k[rb] = v[rb] = f32x16{};
    if constexpr (AHEAD) {
      // groups of ST fragments, alternating between the two halves of w
#pragma unroll
      for (int g = 0; g < 3 * NB; ++g) {
        const int mtx = g / NB, ib = g % NB, nx = g + 1;
        if (nx < 3 * NB)
          w[nx & 1].load(nx / NB == 0 ? Wq : nx / NB == 1 ? Wk : Wv, (hb * NB + nx % NB) * ST, lane);
        else
          w[nx & 1].load(Wo, hb * ST, lane);
#pragma unroll
        for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
          for (int s = 0; s < ST; ++s) {
            if (mtx == 0) q[rb] = P::mma(w[g & 1].w[s], xo[rb][ib][s], q[rb]);
            if (mtx == 1) k[rb] = P::mma(w[g & 1].w[s], xo[rb][ib][s], k[rb]);
            if (mtx == 2) v[rb] = P::mma(xo[rb][ib][s], w[g & 1].w[s], v[rb]);
          }
      }
    } else {
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int s = 0; s < ST; ++s) {
            const int f = (hb * NB + ib) * ST + s;
            q[rb] = P::mma(ld_frag<P>(Wq, f, lane), xo[rb][ib][s], q[rb]);
            k[rb] = P::mma(ld_frag<P>(Wk, f, lane), xo[rb][ib][s], k[rb]);
            v[rb] = P::mma(xo[rb][ib][s], ld_frag<P>(Wv, f, lane), v[rb]);  // (row x feature)
          }
    }
    // score scale folded into q; per-head score operands of q and k packed once per head
    // block; V as operands (lane -> feature)
    using sop = typename P::template SOp<DH>;
    sop qp[NBR][HPB], kp[NBR][HPB];
#pragma unroll
    for (int rb = 0; rb < NBR; ++rb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) q[rb][r] *= sc;
#pragma unroll
      for (int j = 0; j < HPB; ++j) {
        qp[rb][j] = P::template pack_head<DH>(q[rb], j);
        kp[rb][j] = P::template pack_head<DH>(k[rb], j);
      }
    }
    op_t vop[NBR][ST];
#pragma unroll
    for (int kb = 0; kb < NBR; ++kb)
#pragma unroll
      for (int s = 0; s < ST; ++s) vop[kb][s] = P::op(v[kb], s);
    // o = P V per head, row-major (lane -> row, values -> features).  Each head's product goes
    // into a fresh accumulator with the unmasked V operand (lane -> feature): only values
    // [VPH j, VPH (j + 1)) of each lane (the features of head j, see tile_idx) are head j's
    // output and are kept, normalised; the other values are dropped.
    constexpr int VPH = DH / 2;
    f32x16 o[NBR];
    float lsev[NBR][HPB];  // log2 softmax normalisers of this lane's row in each row block
#pragma unroll
    for (int j = 0; j < HPB; ++j) {
#pragma unroll
      for (int qb = 0; qb < NBR; ++qb) {
        f32x16 st[NBR];
        float m = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < NBR; ++kb) {
          st[kb] = P::template scores_packed<DH>(kp[kb][j], qp[qb][j], f32x16{});
          if constexpr (MASKED) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (!((okbits[qb][kb] >> r) & 1u)) st[kb][r] = -INFINITY;
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) m = fmaxf(m, st[kb][r]);
        }
        m = xor32_max(m);
        const float mm = (m == -INFINITY) ? 0.f : m;  // a row with no key keeps P = 0
#pragma unroll
        for (int kb = 0; kb < NBR; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) st[kb][r] = __builtin_amdgcn_exp2f(st[kb][r] - mm);
        // row sum as a pairwise tree (short dependency chains)
        float part[NBR * 8];
#pragma unroll
        for (int kb = 0; kb < NBR; ++kb)
#pragma unroll
          for (int i = 0; i < 8; ++i) part[8 * kb + i] = st[kb][2 * i] + st[kb][2 * i + 1];
#pragma unroll
        for (int w = NBR * 4; w >= 1; w /= 2)
#pragma unroll
          for (int i = 0; i < w; ++i) part[i] += part[i + w];
        const float l = xor32_sum(part[0]);
        // l >= 1 when the row has a key (its maximum contributes exp2(0)): the hardware
        // reciprocal (1 ulp) replaces the division sequence
        const float invl = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
        // for the backward: P = exp2(s - lse) (+inf for a row with no key, so that P = 0)
        lsev[qb][j] = l > 0.f ? mm + __builtin_amdgcn_logf(l) : INFINITY;
        f32x16 to = {};
#pragma unroll
        for (int kb = 0; kb < NBR; ++kb)
#pragma unroll
          for (int s = 0; s < ST; ++s) to = P::mma(vop[kb][s], P::op(st[kb], s), to);
#pragma unroll
        for (int r = VPH * j; r < VPH * (j + 1); ++r) o[qb][r] = to[r] * invl;
      }
    }
    put_lse(hb, lsev);
    // W_O into the residual
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      if constexpr (AHEAD) {
        if (ob + 1 < NB)
          w[(NB + ob + 1) & 1].load(Wo, ((ob + 1) * NB + hb) * ST, lane);
        else
          w[0].load(Wq, (hb + 1 < NB ? hb + 1 : hb) * NB * ST, lane);
      }
#pragma unroll
      for (int qb = 0; qb < NBR; ++qb)
#pragma unroll
        for (int s = 0; s < ST; ++s)
          x[qb][ob] = P::mma(AHEAD ? w[(NB + ob) & 1].w[s] : ld_frag<P>(Wo, (ob * NB + hb) * ST + s, lane), P::op(o[qb], s), x[qb][ob]);
    }
  }
}

// Feed-forward sub-layer: x += relu(x W1 + b1) W2 + b2, MB chunks of 32 hidden units.
template <class P, int D, int NBR, int WAVES = 8>
__device__ __forceinline__ void tile_ffn(f32x16 (&x)[NBR][D / 32], const typename P::elem_t* W1, const typename P::elem_t* W2,
                                         const float* b1s, const float* b2s, int MB, int lane) {
  constexpr int NB = D / 32, ST = P::STEPS;
  constexpr bool SPAN = NBR == 2;
  using op_t = typename P::op_t;
  const int h = lane >> 5;
  op_t xo[NBR][NB][ST];
#pragma unroll
  for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int s = 0; s < ST; ++s) xo[rb][ib][s] = P::op(x[rb][ib], s);
  // pre-activations of 32-unit chunk c: the products accumulate onto b1 (values
  // r = 4q .. 4q+3 hold 4 consecutive hidden units)
  auto ffn_pre = [&](int c, int rb) {
    f32x16 u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = *reinterpret_cast<const float4*>(b1s + 32 * c + 8 * q + 4 * h);
      u[4 * q] = b.x; u[4 * q + 1] = b.y; u[4 * q + 2] = b.z; u[4 * q + 3] = b.w;
    }
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int s = 0; s < ST; ++s) u = P::mma(ld_frag<P>(W1, (c * NB + ib) * ST + s, lane), xo[rb][ib][s], u);
    return u;
  };
  // One row block: software-pipelined over the chunks, chunk c+1's pre-activation products
  // issued before chunk c's ReLU and conversions, which then overlap them on the vector ALU
  // (two row blocks: chunk by chunk, a second chunk in flight would not fit in the
  // registers).  Each accumulator of x takes the chunks in order either way.
  if constexpr (frags_ahead<P, NBR, WAVES>()) {
    Frags<P> w[2];
    w[0].load(W1, 0, lane);
#pragma unroll 1
    for (int c = 0; c < MB; ++c) {
      f32x16 u[NBR];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 b = *reinterpret_cast<const float4*>(b1s + 32 * c + 8 * q + 4 * h);
#pragma unroll
        for (int rb = 0; rb < NBR; ++rb) { u[rb][4 * q] = b.x; u[rb][4 * q + 1] = b.y; u[rb][4 * q + 2] = b.z; u[rb][4 * q + 3] = b.w; }
      }
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) {
        if (ib + 1 < NB)
          w[(ib + 1) & 1].load(W1, (c * NB + ib + 1) * ST, lane);
        else
          w[NB & 1].load(W2, c * ST, lane);
#pragma unroll
        for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
          for (int s = 0; s < ST; ++s) u[rb] = P::mma(w[ib & 1].w[s], xo[rb][ib][s], u[rb]);
      }
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        if (ob + 1 < NB)
          w[(NB + ob + 1) & 1].load(W2, ((ob + 1) * MB + c) * ST, lane);
        else
          w[0].load(W1, (c + 1 < MB ? c + 1 : c) * NB * ST, lane);
#pragma unroll
        for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
          for (int s = 0; s < ST; ++s) x[rb][ob] = P::mma(w[(NB + ob) & 1].w[s], P::relu_op(u[rb], s), x[rb][ob]);
      }
    }
  } else if constexpr (SPAN) {
#pragma unroll
    for (int c = 0; c < MB; ++c)
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb) {
        const f32x16 u = ffn_pre(c, rb);
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
          for (int s = 0; s < ST; ++s)
            x[rb][ob] = P::mma(ld_frag<P>(W2, (ob * MB + c) * ST + s, lane), P::relu_op(u, s), x[rb][ob]);
      }
  } else {
    constexpr int rb = 0;
    f32x16 un = ffn_pre(0, rb);
#pragma unroll
    for (int c = 0; c < MB; ++c) {
      const f32x16 u = un;
      if (c + 1 < MB) un = ffn_pre(c + 1, rb);
      op_t uo[ST];
#pragma unroll
      for (int s = 0; s < ST; ++s) uo[s] = P::relu_op(u, s);
#pragma unroll
      for (int ob = 0; ob < NB; ++ob)
#pragma unroll
        for (int s = 0; s < ST; ++s)
          x[rb][ob] = P::mma(ld_frag<P>(W2, (ob * MB + c) * ST + s, lane), uo[s], x[rb][ob]);
    }
  }
#pragma unroll
  for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
    for (int ob = 0; ob < NB; ++ob)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[rb][ob][r] += b2s[32 * ob + tile_idx(r, h)];

}

// Head of the last layer: F = x_L W_h per row, summed over the rows up to and including this lane's
// in its configuration (pos = row within the configuration); the configuration's last row holds its sum.
template <int NBR, int NB>
__device__ __forceinline__ void tile_head(const f32x16 (&x)[NBR][NB], const float2* hws, const bool (&rvalid)[NBR], int pos, int h,
                                          float& v0, float& v1) {
  // per row: F = x_L W_h (features past d hold zero weights), summed over both lane halves
  float f0[NBR], f1[NBR];
#pragma unroll
  for (int rb = 0; rb < NBR; ++rb) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int ob = 0; ob < NB; ++ob)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float2 hw = hws[32 * ob + tile_idx(r, h)];
        s0 += x[rb][ob][r] * hw.x;
        s1 += x[rb][ob][r] * hw.y;
      }
    f0[rb] = xor32_sum(s0);
    f1[rb] = xor32_sum(s1);
  }
  // mean over the n sites of each configuration: a segmented inclusive scan over the 32 row
  // lanes (segment = the configuration's rows; rows past the last configuration add nothing),
  // a fixed order of additions; the last row of each segment then holds its sum
  v0 = v1 = 0.f;
#pragma unroll
  for (int rb = 0; rb < NBR; ++rb)
    if (rvalid[rb]) { v0 += f0[rb]; v1 += f1[rb]; }
#pragma unroll
  for (int dd = 1; dd < 32; dd <<= 1) {
    const float t0 = __shfl_up(v0, dd, 32), t1 = __shfl_up(v1, dd, 32);
    if (pos >= dd) { v0 += t0; v1 += t1; }
  }
}

// log rho = log(e^{z1} + conj(e^{z2})) on the principal branch (Eq. log_sum_exp_conjugate) from
// z1 = a0 + i a1 = z(alpha, beta) and z2 = b0 + i b1 = z(beta, alpha): (re, im).
__device__ __forceinline__ float2 symmetrise(float a0, float a1, float b0, float b1) {
  const float mx = fmaxf(a0, b0);
  const float ea = expf(a0 - mx), eb = expf(b0 - mx);
  float sa, ca, sb, cb;
  sincosf(a1, &sa, &ca);
  sincosf(b1, &sb, &cb);
  const float sr = ea * ca + eb * cb, si = ea * sa - eb * sb;
  return make_float2(mx + 0.5f * logf(sr * sr + si * si), atan2f(si, sr));
}

}  // namespace tdo
