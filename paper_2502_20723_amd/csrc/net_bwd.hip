// Backward pass of the transformer density operator: vector-Jacobian products
// of log rho with respect to every parameter, for per-pass seeds (dF0, dF1) on
// the head outputs z = F0 + i F1.
//
// Per layer two kernels run in reverse order, each recomputing the layer's
// internals from the activations saved by the forward pass:
//   MLP:       u = b1 + x W1, dh = g W2^T, du = dh [u > 0], dx = g + du W1^T,
//              dW1 += x^T du, dW2 += relu(u)^T g, db1 += sum du, db2 += sum g;
//   attention: q, k, v, P = softmax(q k^T / sqrt(dh)) per head, O = P v;
//              dO = dx W_O^T, dP = dO v^T, dS = P (dP - rowsum(P dP)) / sqrt(dh),
//              dq = dS k, dk = dS^T q, dv = P^T dO, dx += dq Wq^T + dk Wk^T + dv Wv^T,
//              dW_O += O^T dx, dWq += x^T dq, dWk += x^T dk, dWv += x^T dv.
// Contractions over features chain in registers exactly as in the forward;
// contractions over rows (attention over keys/queries and all weight
// gradients) take operands whose lanes enumerate features, obtained by
// computing the product in the (row x feature) orientation or read as columns
// of a tile in LDS.  Every wave keeps its share of the layer's weight gradients
// in registers over the whole launch; at the end each workgroup writes its
// gradients to a private partial buffer, and the partials are summed in FP64 in
// a fixed order, so results do not depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "net.h"
#include "netapi.h"

namespace tdo {

constexpr int TS = 36;  // row stride (floats) of the transpose scratch

// Row index of value i of lane half h in an operand built by transpose_tile: 8 consecutive rows
// per lane half (BF16), or rows in ascending order over the FP32 products (two rows each).
template <class P>
__device__ __forceinline__ int nat_idx(int i, int h) {
  if constexpr (P::KPL == 8) return (i / 8) * 16 + h * 8 + (i % 8);
  else return 2 * i + h;
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Input: a 32x32 tile in MFMA result layout (element (m, n) = value r of lane
// n + 32h with m = tile_idx(r, h)).  Output: the same tile with lane -> m and
// value i -> n = nat_idx(i, h), i.e. an operand for a contraction over n.
template <class P>
__device__ __forceinline__ f32x16 transpose_tile(const f32x16& v, float* sc, int lane) {
  const int h = lane >> 5, n = lane & 31;
#pragma unroll
  for (int r = 0; r < 16; ++r) sc[tile_idx(r, h) * TS + n] = v[r];
  wave_lds_sync();
  f32x16 o;
  const float* row = sc + n * TS;
  if constexpr (P::KPL == 8) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 t = *reinterpret_cast<const float4*>(row + 16 * (q >> 1) + 8 * h + 4 * (q & 1));
      o[4 * q] = t.x; o[4 * q + 1] = t.y; o[4 * q + 2] = t.z; o[4 * q + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = row[nat_idx<P>(i, h)];
  }
  wave_lds_sync();
  return o;
}

// ------------------------------------------------------------------ MLP backward
// Row of a 32-row block that lane m takes as the row operand of (row x hidden) products, so that
// value r of lane half h of the result is row nat_idx(r, h): the products over rows then take the
// result registers as operands in the natural row order.
template <class P>
__device__ __forceinline__ int nat_row(int m) {
  if constexpr (P::KPL == 8) return 16 * (m >> 4) + 8 * ((m >> 2) & 1) + 4 * ((m >> 3) & 1) + (m & 3);
  else return 8 * (m >> 3) + 2 * (m & 3) + ((m >> 2) & 1);
}

// LDS of the feed-forward backward: x and g of NBK blocks, row-major (and, BF16, transposed), and
// du of all hidden units.  Row paddings of 16 bytes keep the accesses on distinct banks.
template <class P, int D, int NBK>
struct MlpLds {
  static constexpr int R = 32 * NBK, FS = D + 4, BS = D + 8, TSB = R + 8;
  static constexpr bool BF = P::KPL == 8;
  static constexpr size_t x = 0;
  static constexpr size_t g32 = x + (BF ? (size_t)R * BS * 2 : (size_t)R * FS * 4);  // g in FP32 [R][FS]
  static constexpr size_t xt = g32 + (size_t)R * FS * 4;                             // BF16: x^T [D][TSB]
  static constexpr size_t g = xt + (BF ? (size_t)D * TSB * 2 : 0);                   // BF16: g [R][BS], g^T [D][TSB]
  static constexpr size_t gt = g + (BF ? (size_t)R * BS * 2 : 0);
  static constexpr size_t hw = gt + (BF ? (size_t)D * TSB * 2 : 0);                  // head weight pairs [D]
  static constexpr size_t du = hw + (size_t)D * 8;
  static size_t bytes(int M) { return du + (BF ? (size_t)R * (M + 8) * 2 : (size_t)NBK * M * TS * 4); }
};

// The FP32 kernel at every width, and the BF16 kernel where the width-64 ones do not apply.
// Workgroups of 8 waves (two per SIMD) walk tiles of NBK blocks.  Wave (rg, cw) owns the CPW
// chunks cw + CW i of 32 hidden units for the blocks of row group rg: their weight operands and
// weight gradients stay in registers for the whole launch, and x, g and du pass between the waves
// through LDS.  u and dh are formed as (row x hidden) tiles, whose registers are the operands of
// the products over rows; du goes through LDS once for dx = g + du W1^T, one wave per 32 x 32
// tile of dx.  Each block's gradient is formed in a fresh accumulator and then added.
// Bound: the FP32 matrix cores (8 n d m operations a pass, and 2 n d m for u, of 157 TFLOP/s).  It
// replaces per-block gradient tiles added into LDS by atomics, one wave per SIMD and weight operands
// reread from the caches for every block: 16384 configurations at n = 32, width 64, mlp 256 6.05 ->
// 1.48 ms (93 TFLOP/s, 116 with u); BF16, 65536 at n = 8, width 32, mlp 128 1.39 -> 0.154 ms.
template <class P, int D, int CW, int CPW, bool SEEDS>
__global__ void __launch_bounds__(512) k_bwd_mlp(BwdArgs a) {
  constexpr int NB = D / 32, ST = P::STEPS, RG = 8 / CW, BPG = CPW == 1 ? 2 : 1, NBK = RG * BPG;
  constexpr int JOBS = 2 * NBK * NB, JPW = (JOBS + 7) / 8;
  constexpr bool BF = P::KPL == 8;
  using L = MlpLds<P, D, NBK>;
  using elem_t = typename P::elem_t;
  using save_t = typename P::save_t;
  using op_t = typename P::op_t;
  extern __shared__ __align__(16) char smem[];
  elem_t* xs = reinterpret_cast<elem_t*>(smem + L::x);
  float* gf = reinterpret_cast<float*>(smem + L::g32);
  __bf16* xt = reinterpret_cast<__bf16*>(smem + L::xt);
  __bf16* gb = reinterpret_cast<__bf16*>(smem + L::g);
  __bf16* gt = reinterpret_cast<__bf16*>(smem + L::gt);
  float2* hws = reinterpret_cast<float2*>(smem + L::hw);
  elem_t* dus = reinterpret_cast<elem_t*>(smem + L::du);
  const int M = a.M, MB = M / 32, DUS = M + 8;

  const elem_t* W1f = reinterpret_cast<const elem_t*>(a.wf) + 4 * D * D;          // [MB][NB][ST]
  const elem_t* W2T = reinterpret_cast<const elem_t*>(a.wb) + 4 * D * D;          // [MB][NB][ST]
  const elem_t* W1T = reinterpret_cast<const elem_t*>(a.wb) + 4 * D * D + D * M;  // [NB][MB][ST]
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cw = wave % CW, rg = wave / CW;
  const int64_t E = a.n_entries_dev ? *a.n_entries_dev : a.n_entries;
  const RowMap rm{a.n, a.cpb, a.span != 0};
  int64_t nblk = a.span ? 4 * E : 2 * ((E + a.cpb - 1) / a.cpb);
  // blocks_per_wg: the workgroup's own consecutive blocks (one configuration), else tiles in turn
  int64_t blk0 = (int64_t)blockIdx.x * NBK, step = (int64_t)gridDim.x * NBK;
  if (a.blocks_per_wg) {
    blk0 = (int64_t)blockIdx.x * a.blocks_per_wg;
    nblk = blk0 + a.blocks_per_wg < nblk ? blk0 + a.blocks_per_wg : nblk;
    step = NBK;
  }

  if constexpr (SEEDS)
    for (int i = threadIdx.x; i < D; i += 512) hws[i] = i < a.d_real ? make_float2(a.head_w[2 * i], a.head_w[2 * i + 1]) : make_float2(0.f, 0.f);

  op_t w1[CPW][NB][ST], w2[CPW][NB][ST];
  float bias[CPW], db1[CPW], db2[NB];
  f32x16 dW1[CPW][NB], dW2[CPW][NB];
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int c = cw + CW * i;
    const bool own = c < MB;
    bias[i] = own ? a.b1[32 * c + lr] : 0.f;
    db1[i] = 0.f;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) {
      dW1[i][ib] = dW2[i][ib] = f32x16{};
#pragma unroll
      for (int s = 0; s < ST; ++s) {
        w1[i][ib][s] = own ? ld_frag<P>(W1f, (c * NB + ib) * ST + s, lane) : op_t{};
        w2[i][ib][s] = own ? ld_frag<P>(W2T, (c * NB + ib) * ST + s, lane) : op_t{};
      }
    }
  }
#pragma unroll
  for (int ib = 0; ib < NB; ++ib) db2[ib] = 0.f;

  // staging jobs of this wave: x tiles (block, feature block), then g tiles; loaded one tile ahead
  float4 pre[JPW][4];
  auto fetch = [&](int64_t b0) {
#pragma unroll
    for (int q = 0; q < JPW; ++q) {
      const int j = wave + 8 * q, jj = j < NBK * NB ? j : j - NBK * NB;
      const int64_t g = b0 + jj / NB;
      const bool ok = j < JOBS && g < nblk;
      if (j < NBK * NB) {
        const auto r = rsrc(reinterpret_cast<const save_t*>(a.save_mid) + (g * NB + jj % NB) * 64 * 16, ok ? 64 * 16 * sizeof(save_t) : 0);
#pragma unroll
        for (int k = 0; k < (BF ? 2 : 4); ++k) pre[q][k] = rld4(r, lane * 16 + 1024 * k);
      } else if constexpr (!SEEDS) {
        const auto r = rsrc(a.g_in + (g * NB + jj % NB) * 64 * 16, ok ? 64 * 16 * 4 : 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) pre[q][k] = rld4(r, lane * 16 + 1024 * k);
      } else {
        float s0 = 0.f, s1 = 0.f;
        if (ok) {
          int64_t e; int pass, ric; bool valid;
          rm.at(g, lr, E, e, pass, ric, valid);
          if (valid) { s0 = a.seeds[(e * 2 + pass) * 2] / (float)a.n; s1 = a.seeds[(e * 2 + pass) * 2 + 1] / (float)a.n; }
        }
        pre[q][0] = make_float4(s0, s1, 0.f, 0.f);
      }
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int q = 0; q < JPW; ++q) {
      const int j = wave + 8 * q;
      if (j >= JOBS) continue;
      const int jj = j < NBK * NB ? j : j - NBK * NB, blk = jj / NB, ob = jj % NB, row = 32 * blk + lr;
      if (j < NBK * NB) {
        if constexpr (BF) {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const bf16x8 v = __builtin_bit_cast(bf16x8, pre[q][s]);
            *reinterpret_cast<bf16x8*>(xs + row * L::BS + 32 * ob + 16 * s + 8 * h) = v;
#pragma unroll
            for (int t = 0; t < 8; ++t) xt[(32 * ob + tile_idx(8 * s + t, h)) * L::TSB + row] = v[t];
          }
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) *reinterpret_cast<float4*>(reinterpret_cast<float*>(xs) + row * L::FS + 32 * ob + 8 * k + 4 * h) = pre[q][k];
        }
      } else {
        f32x16 v;
        if constexpr (SEEDS) {
          const float s0 = pre[q][0].x, s1 = pre[q][0].y;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float2 hw = hws[32 * ob + tile_idx(r, h)];
            v[r] = s0 * hw.x + s1 * hw.y;
          }
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) { v[4 * k] = pre[q][k].x; v[4 * k + 1] = pre[q][k].y; v[4 * k + 2] = pre[q][k].z; v[4 * k + 3] = pre[q][k].w; }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          *reinterpret_cast<float4*>(gf + row * L::FS + 32 * ob + 8 * k + 4 * h) = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
        if constexpr (BF) {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const bf16x8 o = cvt8(v, s);
            *reinterpret_cast<bf16x8*>(gb + row * L::BS + 32 * ob + 16 * s + 8 * h) = o;
#pragma unroll
            for (int t = 0; t < 8; ++t) gt[(32 * ob + tile_idx(8 * s + t, h)) * L::TSB + row] = o[t];
          }
        }
      }
    }
  };
  // operand s of feature block ib for row `row` (lane -> row), and for the rows of block blk (lane -> feature)
  auto row_x = [&](int row, int ib, int s) -> op_t {
    if constexpr (BF) return *reinterpret_cast<const bf16x8*>(xs + row * L::BS + 32 * ib + 16 * s + 8 * h);
    else return *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(xs) + row * L::FS + 32 * ib + 8 * s + 4 * h);
  };
  auto row_g = [&](int row, int ib, int s) -> op_t {
    if constexpr (BF) return *reinterpret_cast<const bf16x8*>(gb + row * L::BS + 32 * ib + 16 * s + 8 * h);
    else return *reinterpret_cast<const f32x4*>(gf + row * L::FS + 32 * ib + 8 * s + 4 * h);
  };
  auto col = [&](const __bf16* tb, const float* tf, int blk, int ib, int s) -> op_t {
    if constexpr (BF) return *reinterpret_cast<const bf16x8*>(tb + (32 * ib + lr) * L::TSB + 32 * blk + 16 * s + 8 * h);
    else {
      const float* p = tf + (32 * blk + 8 * s + h) * L::FS + 32 * ib + lr;  // rows nat_idx(4 s + t, h)
      return op_t{p[0], p[2 * L::FS], p[4 * L::FS], p[6 * L::FS]};
    }
  };

  if (blk0 < nblk) fetch(blk0);
  if constexpr (SEEDS) __syncthreads();  // head weights staged
  for (int64_t b0 = blk0; b0 < nblk; b0 += step) {
    stage();
    barrier_lds();
    if (b0 + step < nblk) fetch(b0 + step);
    // ---- hidden units of this wave: u, dh, du; their weight gradients; du to LDS
#pragma unroll 1
    for (int bi = 0; bi < BPG; ++bi) {
      const int blk = rg * BPG + bi, row = 32 * blk + nat_row<P>(lr);
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        const int c = cw + CW * i;
        if (c >= MB) continue;
        f32x16 u, dh = f32x16{};
#pragma unroll
        for (int r = 0; r < 16; ++r) u[r] = bias[i];
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int s = 0; s < ST; ++s) {
            u = P::mma(row_x(row, ib, s), w1[i][ib][s], u);
            dh = P::mma(row_g(row, ib, s), w2[i][ib][s], dh);
          }
        float t = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float uu = u[r];
          u[r] = relu(uu);
          dh[r] = uu > 0.f ? dh[r] : 0.f;
          t += dh[r];
        }
        db1[i] += t + __shfl_xor(t, 32, 64);
        if constexpr (BF) {
#pragma unroll
          for (int r = 0; r < 16; ++r) dus[(32 * blk + nat_idx<P>(r, h)) * DUS + 32 * c + nat_row<P>(lr)] = (__bf16)dh[r];
        } else {
          float* dp = reinterpret_cast<float*>(dus) + ((blk * MB + c) * 32 + lr) * TS + 16 * h;
#pragma unroll
          for (int k = 0; k < 4; ++k) *reinterpret_cast<float4*>(dp + 4 * k) = make_float4(dh[4 * k], dh[4 * k + 1], dh[4 * k + 2], dh[4 * k + 3]);
        }
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {
          f32x16 acc = f32x16{};
#pragma unroll
          for (int s = 0; s < ST; ++s) acc = P::mma(col(xt, reinterpret_cast<const float*>(xs), blk, ib, s), P::op(dh, s), acc);
#pragma unroll
          for (int r = 0; r < 16; ++r) dW1[i][ib][r] += acc[r];
          if constexpr (!BF) __builtin_amdgcn_sched_barrier(0);  // FP32: one accumulator at a time, or registers spill
          acc = f32x16{};
#pragma unroll
          for (int s = 0; s < ST; ++s) acc = P::mma(P::op(u, s), col(gt, gf, blk, ib, s), acc);
#pragma unroll
          for (int r = 0; r < 16; ++r) dW2[i][ib][r] += acc[r];
          if constexpr (!BF) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (cw == 0)
#pragma unroll
        for (int ib = 0; ib < NB; ++ib) {  // db2 += sum over rows of g
          const float* p = gf + (32 * blk + (BF ? 8 : 1) * h) * L::FS + 32 * ib + lr;
          float t = 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) t += p[nat_idx<P>(i, 0) * L::FS];
          db2[ib] += t + __shfl_xor(t, 32, 64);
        }
    }
    barrier_lds();
    // ---- dx = g + du W1^T, a 32 x 32 tile per wave
    for (int j = wave; j < NBK * NB; j += 8) {
      const int blk = j / NB, ob = j % NB;
      if (b0 + blk >= nblk) continue;
      f32x16 acc;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 v = *reinterpret_cast<const float4*>(gf + (32 * blk + lr) * L::FS + 32 * ob + 8 * k + 4 * h);
        acc[4 * k] = v.x; acc[4 * k + 1] = v.y; acc[4 * k + 2] = v.z; acc[4 * k + 3] = v.w;
      }
#pragma unroll 2
      for (int c = 0; c < MB; ++c)
#pragma unroll
        for (int s = 0; s < ST; ++s) {
          op_t d;
          if constexpr (BF) d = *reinterpret_cast<const bf16x8*>(dus + (32 * blk + lr) * DUS + 32 * c + 16 * s + 8 * h);
          else {
            const float* dp = reinterpret_cast<const float*>(dus) + ((blk * MB + c) * 32 + 8 * s + 4 * h) * TS + 16 * (lr & 1) + (lr >> 1);
            d = op_t{dp[0], dp[TS], dp[2 * TS], dp[3 * TS]};
          }
          acc = P::mma(ld_frag<P>(W1T, (ob * MB + c) * ST + s, lane), d, acc);
        }
      store_tile(a.g_out + ((b0 + blk) * NB + ob) * 1024, lane, acc);
    }
    barrier_lds();
  }

  // ---- row groups summed in order, then this workgroup's gradients: dW1 [D][M], dW2 [M][D], db1 [M], db2 [D]
  float* red = reinterpret_cast<float*>(smem);
  constexpr int T = 2 * CPW * NB;  // 32 x 32 tiles of a wave
#pragma unroll
  for (int g = 1; g < RG; ++g) {
    __syncthreads();
    float* mine = red + cw * (T * 1024 + 64 * (CPW + NB)) + lane;
    if (rg == g) {
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        mine[T * 1024 + 64 * i] = db1[i];
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            mine[((i * NB + ib) * 2 * 16 + r) * 64] = dW1[i][ib][r];
            mine[(((i * NB + ib) * 2 + 1) * 16 + r) * 64] = dW2[i][ib][r];
          }
      }
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) mine[T * 1024 + 64 * (CPW + ib)] = db2[ib];
    }
    __syncthreads();
    if (rg == 0) {
#pragma unroll
      for (int i = 0; i < CPW; ++i) {
        db1[i] += mine[T * 1024 + 64 * i];
#pragma unroll
        for (int ib = 0; ib < NB; ++ib)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            dW1[i][ib][r] += mine[((i * NB + ib) * 2 * 16 + r) * 64];
            dW2[i][ib][r] += mine[(((i * NB + ib) * 2 + 1) * 16 + r) * 64];
          }
      }
#pragma unroll
      for (int ib = 0; ib < NB; ++ib) db2[ib] += mine[T * 1024 + 64 * (CPW + ib)];
    }
  }
  if (rg != 0) return;
  float* part = a.partial + (int64_t)blockIdx.x * (2 * D * M + M + D);
#pragma unroll
  for (int i = 0; i < CPW; ++i) {
    const int c = cw + CW * i;
    if (c >= MB) continue;
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        part[(32 * ib + tile_idx(r, h)) * M + 32 * c + lr] = dW1[i][ib][r];
        part[D * M + (32 * c + tile_idx(r, h)) * D + 32 * ib + lr] = dW2[i][ib][r];
      }
    if (h == 0) part[2 * D * M + 32 * c + lr] = db1[i];
  }
  if (cw == 0 && h == 0)
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) part[2 * D * M + M + 32 * ib + lr] = db2[ib];
}

// ------------------------------------------------------------------ attention backward
// The FP32 kernel at every width, and the BF16 kernel where the width-64 ones do not apply.
// Workgroups of 8 waves (two per SIMD) walk tiles of 4 (block, 32-feature head block) jobs, i.e. 2
// blocks at width 64 and 4 at width 32, two waves per job:
//  1. x and the incoming gradient g of the tile are staged in LDS, row-major;
//  2. a job's waves project q, k and v, dO (feature x row tiles) into the job's four LDS slots,
//     from which rows are score operands and columns operands of the products over rows;
//  3. each wave takes half of the job's heads: P, dS, and the head's features of O, dQ, dK, dV
//     (each in a fresh accumulator of which only those are kept).  In a spanning pass with 8-wide heads a
//     wave takes one head of both query blocks, and its dK and dV go on from the first block to the
//     second in one accumulator (BF16 rounds dx in the next kernel, and a sum of the two blocks' shares
//     rounds otherwise: 3e-6 of a log-derivative at n = 64; reverse mode of 2048 configurations at n = 64,
//     width 32: BF16 0.80 -> 0.79 ms, FP32 1.76 -> 1.80);
//  4. O, dQ, dK, dV replace dO, q, k, v in the slots (with 16-wide heads, FP32 only, a spanning pass first
//     adds the two query blocks' shares of dK and dV);
//  5. every wave adds the tile's rows to the weight-gradient tiles it keeps in registers for the
//     whole launch (a fresh accumulator per block, then added), and waves 0..3 form dx.
// Bound: the FP32 matrix cores, of which 8-wide heads use a quarter in the products of step 3.  The
// former kernel kept everything of a block in the registers of one wave per SIMD (478, or spills in
// a spanning pass), added every block's gradient tiles into LDS by atomics and formed k and v twice.
// FP32, width 64: 16384 configurations at n = 32, 8 heads 4.16 -> 1.66 ms; 32768 at n = 16, 4 heads
// 3.58 -> 1.38 ms; 8192 at n = 37 4.40 -> 1.89 ms; width 32, 65536 at n = 8 1.29 -> 0.64 ms (BF16
// 0.87 -> 0.27 ms).
template <class P, int D, int DH, bool SPAN>
__global__ void __launch_bounds__(512) k_bwd_attn(BwdArgs a) {
  constexpr int NB = D / 32, ST = P::STEPS, HPB = 32 / DH, VPH = DH / 2, HPS = HPB / 2;
  constexpr int NBK = 4 / NB, XS = D + 4, R = 32 * NBK, NKB = SPAN ? 2 : 1, SLOT = 32 * TS;
  constexpr bool WHOLE = SPAN && DH == 8;     // step 3: a wave takes one head of both query blocks of a pass
  constexpr int UN = WHOLE ? 2 : HPS;         // (query block, head) pairs of a wave in step 3
  constexpr bool BF = P::KPL == 8;
  using elem_t = typename P::elem_t;
  using save_t = typename P::save_t;
  using op_t = typename P::op_t;
  extern __shared__ __align__(16) float sm[];
  float* xs = sm;                  // [R][XS]
  float* gs = xs + R * XS;         // [R][XS]
  float* slots = gs + R * XS;      // [4 jobs][q -> dQ, k -> dK, v -> dV, dO -> O][32 rows][TS]
  float* scr = slots + 16 * SLOT;  // [8 waves][32][TS]

  const elem_t* Wf = reinterpret_cast<const elem_t*>(a.wf);  // Wq, Wk, Wv
  const elem_t* Wb = reinterpret_cast<const elem_t*>(a.wb);  // Wq^T, Wk^T, Wv^T, Wo^T
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int job = wave >> 1, sub = wave & 1, jblk = job / NB, hb = job % NB;
  const int own = SPAN ? jblk & 1 : 0;
  // step 3: its head block, first key block and pairs
  const int hb3 = WHOLE ? (NB == 2 ? wave >> 2 : 0) : hb, kbase = WHOLE ? (NB == 2 ? 0 : 2 * (wave >> 2)) : jblk - own;
  auto unit_head = [&](int u) { return WHOLE ? wave & 3 : sub * HPS + u; };
  auto unit_job = [&](int u) { return WHOLE ? (kbase + u) * NB + hb3 : job; };
  float* sc = scr + wave * SLOT;
  const int64_t E = a.n_entries_dev ? *a.n_entries_dev : a.n_entries;
  const int n = a.n, cpb = a.cpb;
  int64_t nblk = SPAN ? 4 * E : 2 * ((E + cpb - 1) / cpb);
  int64_t blk0 = (int64_t)blockIdx.x * NBK, step = (int64_t)gridDim.x * NBK;
  if (a.blocks_per_wg) {  // the workgroup's own consecutive blocks (one configuration)
    blk0 = (int64_t)blockIdx.x * a.blocks_per_wg;
    nblk = blk0 + a.blocks_per_wg < nblk ? blk0 + a.blocks_per_wg : nblk;
    step = NBK;
  }
  const float sc2 = a.score_scale, isd = a.inv_sqrt_dh;

  // valid keys (value r of the score tile with key block kb) of this lane's query row
  uint32_t okbits[NKB];
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    okbits[kb] = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = kb * 32 + tile_idx(r, h);
      const bool ok = SPAN ? key < n : (a.masked ? ((key / n) == (lr / n) && (key / n) < cpb) : true);
      okbits[kb] |= ok ? 1u << r : 0u;
    }
  }

  auto slot = [&](int jb, int m) { return slots + (jb * 4 + m) * SLOT; };
  // operand s of row `row`, features f0 + (result order)
  auto rowop = [&](const float* base, int stride, int row, int f0, int s) -> op_t {
    const float* p = base + row * stride + f0 + 2 * P::KPL * s + 4 * h;
    if constexpr (BF) {
      const float4 u = *reinterpret_cast<const float4*>(p), v = *reinterpret_cast<const float4*>(p + 8);
      const float t[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
      return cvt8(t, 0);
    } else return *reinterpret_cast<const f32x4*>(p);
  };
  // operand s of column `col` (lane -> feature): rows in natural (nat) or result order
  auto colop = [&](const float* base, int stride, int col, int s, bool nat) -> op_t {
    float t[P::KPL];
#pragma unroll
    for (int k = 0; k < P::KPL; ++k) t[k] = base[(nat ? nat_idx<P>(P::KPL * s + k, h) : tile_idx(P::KPL * s + k, h)) * stride + col];
    if constexpr (BF) return cvt8(t, 0);
    else return P::op(t, 0);
  };
  // score operand of one head: its features of this lane's row
  using sop = typename P::template SOp<DH>;
  auto headop = [&](const float* s, int j) -> sop {
    f32x16 t{};
#pragma unroll
    for (int k = 0; k < VPH / 4; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(s + lr * TS + DH * j + 8 * k + 4 * h);
      t[4 * k] = v.x; t[4 * k + 1] = v.y; t[4 * k + 2] = v.z; t[4 * k + 3] = v.w;
    }
    return P::template pack_head<DH>(t, 0);
  };
  auto put_head = [&](float* s, int j, const float* v) {  // the same places
#pragma unroll
    for (int k = 0; k < VPH / 4; ++k)
      *reinterpret_cast<float4*>(s + lr * TS + DH * j + 8 * k + 4 * h) = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
  };
  auto get_head = [&](const float* s, int j, float* v) {
#pragma unroll
    for (int k = 0; k < VPH / 4; ++k) {
      const float4 u = *reinterpret_cast<const float4*>(s + lr * TS + DH * j + 8 * k + 4 * h);
      v[4 * k] = u.x; v[4 * k + 1] = u.y; v[4 * k + 2] = u.z; v[4 * k + 3] = u.w;
    }
  };

  // staging job of this wave: an x or g tile (block, feature block), loaded one tile ahead
  const int sj = wave & 3, sblk = sj / NB, sob = sj % NB;
  float4 pre[4];
  auto fetch = [&](int64_t b0) {
    const int64_t g = b0 + sblk;
    if (wave < 4) {
      const auto r = rsrc(reinterpret_cast<const save_t*>(a.save_x) + (g * NB + sob) * 64 * 16, g < nblk ? 64 * 16 * sizeof(save_t) : 0);
#pragma unroll
      for (int k = 0; k < (BF ? 2 : 4); ++k) pre[k] = rld4(r, lane * 16 + 1024 * k);
    } else {
      const auto r = rsrc(a.g_in + (g * NB + sob) * 64 * 16, g < nblk ? 64 * 16 * 4 : 0);
#pragma unroll
      for (int k = 0; k < 4; ++k) pre[k] = rld4(r, lane * 16 + 1024 * k);
    }
  };
  auto stage = [&]() {
    float4 v[4];
    if (BF && wave < 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bf16x8 t = __builtin_bit_cast(bf16x8, pre[k >> 1]);
        v[k] = make_float4((float)t[4 * (k & 1)], (float)t[4 * (k & 1) + 1], (float)t[4 * (k & 1) + 2], (float)t[4 * (k & 1) + 3]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = pre[k];
    }
    float* d = (wave < 4 ? xs : gs) + (32 * sblk + lr) * XS + 32 * sob + 4 * h;
#pragma unroll
    for (int k = 0; k < 4; ++k) *reinterpret_cast<float4*>(d + 8 * k) = v[k];
  };

  // weight-gradient tiles of this wave: width 64: matrix wave / 2, first index wave % 2, both second
  // indices, all blocks; width 32: matrix wave % 4, the blocks of half wave / 4
  const int mt = NB == 2 ? wave >> 1 : wave & 3, mi = NB == 2 ? wave & 1 : 0;
  const int mb0 = NB == 2 ? 0 : 2 * (wave >> 2);
  f32x16 dW[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) dW[i] = f32x16{};

  if (blk0 < nblk) fetch(blk0);
  for (int64_t b0 = blk0; b0 < nblk; b0 += step) {
    // ---- 1. stage
    stage();
    barrier_lds();
    if (b0 + step < nblk) fetch(b0 + step);
    // ---- 2. projections of this wave: (q, k) or (v, dO)
    {
      const elem_t* W0 = sub ? Wf + 2 * D * D : Wf;
      const elem_t* W1 = sub ? Wb + 3 * D * D : Wf + D * D;
      const float* src1 = sub ? gs : xs;
      f32x16 t0 = f32x16{}, t1 = f32x16{};
#pragma unroll
      for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int s = 0; s < ST; ++s) {
          const int f = (hb * NB + ib) * ST + s;
          t0 = P::mma(ld_frag<P>(W0, f, lane), rowop(xs, XS, 32 * jblk + lr, 32 * ib, s), t0);
          t1 = P::mma(ld_frag<P>(W1, f, lane), rowop(src1, XS, 32 * jblk + lr, 32 * ib, s), t1);
        }
      float *s0 = slot(job, 2 * sub) + lr * TS + 4 * h, *s1 = slot(job, 2 * sub + 1) + lr * TS + 4 * h;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        *reinterpret_cast<float4*>(s0 + 8 * k) = make_float4(t0[4 * k], t0[4 * k + 1], t0[4 * k + 2], t0[4 * k + 3]);
        *reinterpret_cast<float4*>(s1 + 8 * k) = make_float4(t1[4 * k], t1[4 * k + 1], t1[4 * k + 2], t1[4 * k + 3]);
      }
    }
    barrier_lds();
    // ---- 3. heads of this wave
    constexpr int KU = WHOLE ? 1 : UN;  // dK, dV per pair, or of both together
    float ho[UN][VPH], hq[UN][VPH], hk[KU][NKB][VPH], hv[KU][NKB][VPH];
    f32x16 tk[WHOLE ? NKB : 1], tv[WHOLE ? NKB : 1];  // of both pairs
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int j = unit_head(u), jb = unit_job(u);
      // the head's values of a result tile whose features are the head block's
      auto keep = [&](const f32x16& t, float* v) {
#pragma unroll
        for (int r = 0; r < VPH; ++r) {
          if constexpr (WHOLE) v[r] = j < 2 ? (j ? t[VPH + r] : t[r]) : (j == 2 ? t[2 * VPH + r] : t[(3 * VPH + r) & 15]);
          else v[r] = sub ? t[VPH * (HPS + u) + r] : t[VPH * u + r];
        }
      };
      f32x16 p[NKB], dp[NKB];
      float m = -INFINITY;
      {
        const sop qo = headop(slot(jb, 0), j);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          p[kb] = P::template scores_packed<DH>(headop(slot((kbase + kb) * NB + hb3, 1), j), qo, f32x16{});
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            p[kb][r] = (okbits[kb] >> r) & 1u ? p[kb][r] * sc2 : -INFINITY;
            m = fmaxf(m, p[kb][r]);
          }
        }
      }
      m = xor32_max(m);
      float l = 0.f;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float e = (m == -INFINITY) ? 0.f : exp2f(p[kb][r] - m);
          p[kb][r] = e;
          l += e;
        }
      l = xor32_sum(l);
      const float il = l > 0.f ? 1.0f / l : 0.f;
      // dP^T (keys x queries) = V_j dO_j^T; Delta = sum_k P dP
      float delta = 0.f;
      {
        const sop oo = headop(slot(jb, 3), j);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          dp[kb] = P::template scores_packed<DH>(headop(slot((kbase + kb) * NB + hb3, 2), j), oo, f32x16{});
#pragma unroll
          for (int r = 0; r < 16; ++r) delta += p[kb][r] * dp[kb][r];
        }
      }
      delta = xor32_sum(delta);
      delta *= il;
      // O (unnormalised, scaled by 1/l at the end), dS, dQ: keys in result order on both sides
      f32x16 to = f32x16{}, tq = f32x16{};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const int kj = (kbase + kb) * NB + hb3;
#pragma unroll
        for (int s = 0; s < ST; ++s) to = P::mma(colop(slot(kj, 2), TS, lr, s, false), P::op(p[kb], s), to);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          p[kb][r] *= il;
          dp[kb][r] = p[kb][r] * (dp[kb][r] - delta) * isd;
        }
#pragma unroll
        for (int s = 0; s < ST; ++s) tq = P::mma(colop(slot(kj, 1), TS, lr, s, false), P::op(dp[kb], s), tq);
      }
      keep(to, ho[u]);
      keep(tq, hq[u]);
#pragma unroll
      for (int r = 0; r < VPH; ++r) ho[u][r] *= il;
      // dK += dS^T Q, dV += P^T dO: queries in natural order on both sides
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        auto add = [&](const f32x16& w, int slot_m, f32x16 t) {
          const f32x16 wT = transpose_tile<P>(w, sc, lane);
#pragma unroll
          for (int s = 0; s < ST; ++s) t = P::mma(colop(slot(jb, slot_m), TS, lr, s, true), P::op(wT, s), t);
          return t;
        };
        if constexpr (WHOLE) {
          tk[kb] = add(dp[kb], 0, u ? tk[kb] : f32x16{});
          tv[kb] = add(p[kb], 3, u ? tv[kb] : f32x16{});
          if (u == UN - 1) {
            keep(tk[kb], hk[0][kb]);
            keep(tv[kb], hv[0][kb]);
          }
        } else {
          keep(add(dp[kb], 0, f32x16{}), hk[u][kb]);
          keep(add(p[kb], 3, f32x16{}), hv[u][kb]);
        }
      }
    }
    barrier_lds();
    // ---- 4. O, dQ, dK, dV of this wave's heads into the slots
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int j = unit_head(u), jb = unit_job(u);
      put_head(slot(jb, 0), j, hq[u]);
      put_head(slot(jb, 3), j, ho[u]);
      if constexpr (WHOLE) {  // key block u
        put_head(slot(jb, 1), j, hk[0][u]);
        put_head(slot(jb, 2), j, hv[0][u]);
      } else if constexpr (!SPAN) {
        put_head(slot(jb, 1), j, hk[u][0]);
        put_head(slot(jb, 2), j, hv[u][0]);
      } else {  // this query block's share of the other key block
        const int oj = (kbase + 1 - own) * NB + hb;
        float k[VPH], v[VPH];
#pragma unroll
        for (int r = 0; r < VPH; ++r) { k[r] = own ? hk[u][0][r] : hk[u][NKB - 1][r]; v[r] = own ? hv[u][0][r] : hv[u][NKB - 1][r]; }
        put_head(slot(oj, 1), j, k);
        put_head(slot(oj, 2), j, v);
      }
    }
    barrier_lds();
    if constexpr (SPAN && !WHOLE) {
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int j = unit_head(u);
        float k[VPH], v[VPH];
        get_head(slot(job, 1), j, k);
        get_head(slot(job, 2), j, v);
#pragma unroll
        for (int r = 0; r < VPH; ++r) { k[r] += own ? hk[u][NKB - 1][r] : hk[u][0][r]; v[r] += own ? hv[u][NKB - 1][r] : hv[u][0][r]; }
        put_head(slot(job, 1), j, k);
        put_head(slot(job, 2), j, v);
      }
      barrier_lds();
    }
    // ---- 5. weight gradients: dW{q,k,v}[D-in][attn] += x^T d{q,k,v}, dW_O[attn][D-out] += O^T g
#pragma unroll 1
    for (int b = mb0; b < mb0 + 2; ++b)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const float *A = xs + 32 * b * XS + 32 * mi, *B = slot(b * NB + i, mt);
        int as = XS, bs = TS;
        if (mt == 3) { A = slot(b * NB + mi, 3); B = gs + 32 * b * XS + 32 * i; as = TS; bs = XS; }
        f32x16 acc = f32x16{};
#pragma unroll
        for (int s = 0; s < ST; ++s) acc = P::mma(colop(A, as, lr, s, true), colop(B, bs, lr, s, true), acc);
#pragma unroll
        for (int r = 0; r < 16; ++r) dW[i][r] += acc[r];
      }
    // dx = g + dQ Wq^T + dK Wk^T + dV Wv^T
    if (wave < 4 && b0 + sblk < nblk) {
      f32x16 acc;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 v = *reinterpret_cast<const float4*>(gs + (32 * sblk + lr) * XS + 32 * sob + 8 * k + 4 * h);
        acc[4 * k] = v.x; acc[4 * k + 1] = v.y; acc[4 * k + 2] = v.z; acc[4 * k + 3] = v.w;
      }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int jb = sblk * NB + i;
#pragma unroll
        for (int s = 0; s < ST; ++s) {
          const int f = (sob * NB + i) * ST + s;
          acc = P::mma3(ld_frag<P>(Wb, f, lane), rowop(slot(jb, 0), TS, lr, 0, s), ld_frag<P>(Wb + D * D, f, lane),
                        rowop(slot(jb, 1), TS, lr, 0, s), ld_frag<P>(Wb + 2 * D * D, f, lane), rowop(slot(jb, 2), TS, lr, 0, s), acc);
        }
      }
      store_tile(a.g_out + ((b0 + sblk) * NB + sob) * 1024, lane, acc);
    }
    barrier_lds();
  }

  // ---- this workgroup's gradients [dWq][dWk][dWv][dWo]; width 32: the two halves of the blocks summed
  float* part = a.partial + (int64_t)blockIdx.x * 4 * D * D + mt * D * D;
  if constexpr (NB == 1) {
    __syncthreads();
    float* red = sm + mt * 1024 + lane;
    if (wave >= 4)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[64 * r] = dW[0][r];
    __syncthreads();
    if (wave >= 4) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) dW[0][r] += red[64 * r];
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[(32 * mi + tile_idx(r, h)) * D + 32 * i + lr] = dW[i][r];
}

// ------------------------------------------------------------------ head and embedding
// dW_head[f][k] += sum over configuration-passes of (mean over its rows of x_L[f]) dF_k,
// db_head[k] += dF_k.  One wave per block of the saved x_L (lane -> row, values ->
// features): each lane adds x_L[row][f] dF_k / n for its row into FP64
// accumulators; once per launch the lanes and the waves of a workgroup are summed in a
// fixed order into the workgroup's slot, and k_reduce_head adds the slots to the gradient.
template <class P, int D>
__global__ void __launch_bounds__(256) k_bwd_head(const void* __restrict__ save_last, const float* __restrict__ seeds,
                                                  const int64_t* E_dev, int64_t E_host, int n, int cpb, int span,
                                                  int d_real, double* __restrict__ part) {
  using save_t = typename P::save_t;
  constexpr int NB = D / 32;
  const int64_t E = E_dev ? *E_dev : E_host;
  const RowMap rm{n, cpb, span != 0};
  const int64_t nblk = span ? 4 * E : 2 * ((E + cpb - 1) / cpb);
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31, wave = threadIdx.x >> 6;
  const save_t* xs = reinterpret_cast<const save_t*>(save_last);
  const float inv_n = 1.0f / (float)n;
  double a0[NB][16], a1[NB][16], c0 = 0.0, c1 = 0.0;
#pragma unroll
  for (int ob = 0; ob < NB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) a0[ob][r] = a1[ob][r] = 0.0;
  // no early exit for padding rows (their seeds are taken as 0: the forward wrote finite values
  // for them, which then add exactly 0), so that two blocks' loads can be in flight at once
#pragma unroll 2
  for (int64_t g = (int64_t)blockIdx.x * 4 + wave; g < nblk; g += (int64_t)gridDim.x * 4) {
    int64_t e; int pass, ric; bool valid;
    rm.at(g, lr, E, e, pass, ric, valid);
    float s0 = 0.f, s1 = 0.f;
    if (valid) {
      s0 = seeds[(e * 2 + pass) * 2] * inv_n;
      s1 = seeds[(e * 2 + pass) * 2 + 1] * inv_n;
    }
    if (h == 0) { c0 += s0; c1 += s1; }
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
      const f32x16 v = load_tile(xs + (g * NB + ob) * 1024, lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        a0[ob][r] += (double)(v[r] * s0);
        a1[ob][r] += (double)(v[r] * s1);
      }
    }
  }
  // sum over the 32 rows (lanes of one half) and then over the 4 waves, in a fixed order, into
  // this workgroup's slot part[block][2 d_real + 2] ([feature][2] head weights, then the bias)
  __shared__ double red[4][2 * D + 2];
#pragma unroll
  for (int ob = 0; ob < NB; ++ob)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      double u0 = a0[ob][r], u1 = a1[ob][r];
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) { u0 += __shfl_xor(u0, o, 64); u1 += __shfl_xor(u1, o, 64); }
      const int f = 32 * ob + tile_idx(r, h);
      if (lr == 0) {
        red[wave][2 * f] = u0;
        red[wave][2 * f + 1] = u1;
      }
    }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) { c0 += __shfl_xor(c0, o, 64); c1 += __shfl_xor(c1, o, 64); }
  if (lane == 0) {
    red[wave][2 * D] = c0;
    red[wave][2 * D + 1] = c1;
  }
  __syncthreads();
  const int len = 2 * d_real + 2;
  for (int i = threadIdx.x; i < len; i += 256) {
    const int k = i < 2 * d_real ? i : 2 * D + (i - 2 * d_real);
    part[(int64_t)blockIdx.x * len + i] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
  }
}

// Sum of the head kernel's workgroup slots, one workgroup per entry in a fixed order:
// gw[i] (i < 2 d_real) or gb[i - 2 d_real] += sum over the nparts slots.
__global__ void __launch_bounds__(256) k_reduce_head(const double* __restrict__ part, int nparts, int d_real,
                                                     double* __restrict__ gw, double* __restrict__ gb) {
  __shared__ double sh[256];
  const int len = 2 * d_real + 2, i = blockIdx.x, t = threadIdx.x;
  double s = 0.0;
  for (int p = t; p < nparts; p += 256) s += part[(int64_t)p * len + i];
  sh[t] = s;
  __syncthreads();
#pragma unroll
  for (int w = 128; w >= 1; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  if (t == 0) {
    if (i < 2 * d_real) gw[i] += sh[0];
    else gb[i - 2 * d_real] += sh[0];
  }
}

// dT[code][f] += sum over rows with that window code of dx_0[row][f], as a contraction
// over the rows of each block: C[f][code] = sum_row dx_0[row][f] onehot[row][code].  It runs
// on the BF16 matrix cores without losing FP32 accuracy: every FP32 value of dx_0 is split
// exactly into three BF16 terms (hi + mid + lo = x, each term the next 8 significant bits),
// the terms are transposed on the matrix cores (lane -> feature, values -> rows), and each is
// multiplied by the 0/1 operand: every product is exact and the sums accumulate in FP32 as
// in an FP32 contraction.  Accumulated in registers by every wave over its blocks and
// written to the wave's partial slot [64][D] once per launch.
template <int D>
__global__ void __launch_bounds__(256) k_embed_onehot(const float* __restrict__ dx0, const uint64_t* __restrict__ ecfg,
                                                      const int64_t* E_dev, int64_t E_host, int n, int cpb, int span,
                                                      float* __restrict__ partial) {
  constexpr int NB = D / 32;
  __shared__ uint32_t codes_s[4][8];  // per wave: window code of each of the 32 rows (byte r), 255 for padding
  const int64_t E = E_dev ? *E_dev : E_host;
  const RowMap rm{n, cpb, span != 0};
  const int64_t nblk = span ? 4 * E : 2 * ((E + cpb - 1) / cpb);
  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint8_t* cb = reinterpret_cast<uint8_t*>(codes_s[wave]);
  bf16x8 eye[2];  // permutation operands of the transposes: eye[s][t] = [tile_idx(8 s + t, h) == lr]
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
    for (int t2 = 0; t2 < 8; ++t2) eye[s2][t2] = (__bf16)(tile_idx(8 * s2 + t2, h) == lr ? 1.0f : 0.0f);
  auto mfma16 = [](const bf16x8& a, const bf16x8& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  };
  f32x16 acc[NB][2];
#pragma unroll
  for (int ft = 0; ft < NB; ++ft) acc[ft][0] = acc[ft][1] = f32x16{};
  const int wpg = blockDim.x >> 6;
  for (int64_t g = (int64_t)blockIdx.x * wpg + wave; g < nblk; g += (int64_t)gridDim.x * wpg) {
    // window code of this lane's row (255 if the row is padding), shared through LDS
    {
      int64_t e; int pass, ric; bool valid;
      rm.at(g, lr, E, e, pass, ric, valid);
      int code = 255;
      if (valid) {
        const uint64_t al = ecfg[2 * e], be = ecfg[2 * e + 1];
        const uint64_t c0 = pass ? be : al, c1 = pass ? al : be;
        code = 0;
        for (int k = 0; k < 3; ++k) {
          int s = ric + k;
          s = s >= n ? s - n : s;
          code += ((int)((c0 >> s) & 1ull) + 2 * (int)((c1 >> s) & 1ull)) << (2 * k);
        }
      }
      if (h == 0) cb[lr] = (uint8_t)code;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    // one-hot operands: lane (code 32 ct + lr, half h), value t of k-step s -> row tile_idx(8 s + t, h)
    bf16x8 oh[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint32_t w0 = codes_s[wave][4 * s + h], w1 = codes_s[wave][4 * s + 2 + h];  // rows 16s+4h.., 16s+8+4h..
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const uint32_t c = ((t < 4 ? w0 : w1) >> (8 * (t & 3))) & 255u;
          oh[ct][s][t] = (__bf16)(c == (uint32_t)(32 * ct + lr) ? 1.0f : 0.0f);
        }
    }
    __builtin_amdgcn_wave_barrier();  // codes read before the next block's codes are written
#pragma unroll
    for (int ft = 0; ft < NB; ++ft) {
      const f32x16 x = load_tile(dx0 + (g * NB + ft) * 1024, lane);
      bf16x8 tm[3][2];  // hi, mid, lo: R layout (lane -> row, values -> features tile_idx(r, h))
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const __bf16 hi = (__bf16)x[r];
        const float r1 = x[r] - (float)hi;
        const __bf16 mid = (__bf16)r1;
        const __bf16 lo = (__bf16)(r1 - (float)mid);
        tm[0][r >> 3][r & 7] = hi;
        tm[1][r >> 3][r & 7] = mid;
        tm[2][r >> 3][r & 7] = lo;
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        // transposed term: lane -> feature 32 ft + lr, value r -> row tile_idx(r, h) (exact)
        const f32x16 tt = mfma16(tm[k][1], eye[1], mfma16(tm[k][0], eye[0], f32x16{}));
        bf16x8 ta[2];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int t = 0; t < 8; ++t) ta[s][t] = (__bf16)tt[8 * s + t];
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int s = 0; s < 2; ++s) acc[ft][ct] = mfma16(ta[s], oh[ct][s], acc[ft][ct]);
      }
    }
  }
  float* part = partial + ((int64_t)blockIdx.x * wpg + wave) * 64 * D;
#pragma unroll
  for (int ft = 0; ft < NB; ++ft)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[(32 * ct + lr) * D + 32 * ft + tile_idx(r, h)] = acc[ft][ct][r];
}

// Chain rule from the table gradient dT[64][D] (FP64) into the convolution parameters, in FP64
// (recomputes the table's pre-activations).  One workgroup per window code: the code's
// contribution to every parameter gradient goes to its slot part[code][4d + d + 2d^2 + d] (the
// gradient's layout); k_embed_params_sum adds the slots in code order.
__global__ void __launch_bounds__(64) k_embed_params(const float* __restrict__ params, const double* __restrict__ dT,
                                                     int d, int D, double* __restrict__ part) {
  // grad layout: conv1_w [2][2][d], conv1_b [d], conv2_w [2][d][d], conv2_b [d]
  __shared__ double ea[64], eb[64], gpre[64];
  const float* w1 = params;
  const float* b1 = params + 4 * d;
  const float* w2 = b1 + d;
  const float* b2 = w2 + 2 * d * d;
  const int64_t len = 6LL * d + 2LL * d * d;
  double* p = part + (int64_t)blockIdx.x * len;
  double* p_w1 = p;
  double* p_b1 = p + 4 * d;
  double* p_w2 = p_b1 + d;
  double* p_b2 = p_w2 + 2 * d * d;
  auto spin = [](int t, int ch) { return 1.0 - 2.0 * (double)((t >> ch) & 1); };
  auto phi = [](double u) { return 0.5 * u * (1.0 + erf(u * 0.7071067811865476)); };
  auto dphi = [](double u) { return 0.5 * (1.0 + erf(u * 0.7071067811865476)) + u * 0.3989422804014327 * exp(-0.5 * u * u); };
  const int t = threadIdx.x, code = blockIdx.x;
  const int t0 = code & 3, t1 = (code >> 2) & 3, t2 = (code >> 4) & 3;
  double pa = 0, pb = 0;
  if (t < d) {
    pa = b1[t] + spin(t0, 0) * w1[t] + spin(t0, 1) * w1[d + t] + spin(t1, 0) * w1[2 * d + t] + spin(t1, 1) * w1[3 * d + t];
    pb = b1[t] + spin(t1, 0) * w1[t] + spin(t1, 1) * w1[d + t] + spin(t2, 0) * w1[2 * d + t] + spin(t2, 1) * w1[3 * d + t];
    ea[t] = phi(pa);
    eb[t] = phi(pb);
  }
  __syncthreads();
  if (t < d) {  // output feature o = t: pre-activation and its gradient
    double acc = b2[t];
    for (int c = 0; c < d; ++c) acc += ea[c] * w2[c * d + t] + eb[c] * w2[d * d + c * d + t];
    gpre[t] = dT[code * D + t] * dphi(acc);
  }
  __syncthreads();
  if (t < d) {
    p_b2[t] = gpre[t];
    for (int c = 0; c < d; ++c) {  // thread t = output channel o (coalesced rows)
      p_w2[c * d + t] = ea[c] * gpre[t];
      p_w2[d * d + c * d + t] = eb[c] * gpre[t];
    }
    double da = 0, db = 0;  // thread t = input channel c
    for (int o = 0; o < d; ++o) { da += w2[t * d + o] * gpre[o]; db += w2[d * d + t * d + o] * gpre[o]; }
    const double ga = da * dphi(pa), gb = db * dphi(pb);
    p_b1[t] = ga + gb;
    p_w1[t] = spin(t0, 0) * ga + spin(t1, 0) * gb;
    p_w1[d + t] = spin(t0, 1) * ga + spin(t1, 1) * gb;
    p_w1[2 * d + t] = spin(t1, 0) * ga + spin(t2, 0) * gb;
    p_w1[3 * d + t] = spin(t1, 1) * ga + spin(t2, 1) * gb;
  }
}

// grad[i] += sum over the 64 codes, in code order, of part[code][i].
__global__ void k_embed_params_sum(const double* __restrict__ part, int64_t len, double* __restrict__ grad) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (int64_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int c = 0; c < 64; ++c) s += part[c * len + i];
    grad[i] += s;
  }
}

// Where element i of a flat vector lies in a partial: the whole vector, or the feed-forward
// ([W1 d x M][b1 M][W2 M x d][b2 d] from dW1 [D][M], dW2 [M][D], db1 [M], db2 [D]) or attention (four
// d x d from D x D) part of a layer's parameters.
struct WholeMap {
  __device__ int64_t at(int64_t i) const { return i; }
};
struct MlpMap {
  int d, D, M;
  __device__ int at(int i) const {
    if (i < d * M) return i;
    if ((i -= d * M) < M) return 2 * D * M + i;
    if ((i -= M) < d * M) return D * M + (i / d) * D + i % d;
    return 2 * D * M + M + (i - d * M);
  }
};
struct AttnMap {
  int d, D;
  __device__ int at(int i) const {
    const int mt = i / (d * d), r = i % (d * d);
    return mt * D * D + (r / d) * D + r % d;
  }
};

// out[i] += sum of nparts FP32 partials (plen apart) in FP64, in a fixed order.  A workgroup of 256
// threads sums EPB consecutive elements over all partials: G = 256 / EPB groups of threads each
// take every G-th partial, and the group sums are added in a fixed order (deterministic), so that
// enough loads are in flight per element.
template <int EPB, class Map>
__global__ void __launch_bounds__(256) k_reduce_partials(const float* __restrict__ part, int nparts, int64_t plen, Map map,
                                                         int64_t len, double* __restrict__ out) {
  constexpr int G = 256 / EPB;
  __shared__ double sh[G][EPB];
  const int j = threadIdx.x % EPB, g = threadIdx.x / EPB;
  const int64_t i = (int64_t)blockIdx.x * EPB + j;
  double s = 0.0;
  if (i < len) {
    const float* q = part + map.at(i);
#pragma unroll 8
    for (int p = g; p < nparts; p += G) s += (double)q[(int64_t)p * plen];
  }
  sh[g][j] = s;
  __syncthreads();
  if (g == 0 && i < len) {
    double t = sh[0][j];
#pragma unroll
    for (int q = 1; q < G; ++q) t += sh[q][j];
    out[i] += t;
  }
}

// ------------------------------------------------------------------ launchers
// Split of the feed-forward backward over hidden units: CW waves, as many as there are chunks of 32 (2, 4 or
// 8), the others over rows; more than 8 chunks (width 32 only) take CPW = 2 per wave.  f(CW, CPW).
template <int D, class F>
static auto mlp_split(int M, F&& f) {
  const int MB = M / 32;
  if constexpr (D == 32) {
    if (MB <= 2) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
    if (MB > 8) return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
  }
  return MB <= 4 ? f(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{})
                 : f(std::integral_constant<int, 8>{}, std::integral_constant<int, 1>{});
}

// LDS of a workgroup: the tiles, and at the end the row groups' gradients.
template <class P, int D, int CW, int CPW>
static size_t mlp_lds(int M) {
  constexpr int RG = 8 / CW, NBK = RG * (CPW == 1 ? 2 : 1);
  const size_t red = RG > 1 ? (size_t)CW * (2 * CPW * (D / 32) * 1024 + 64 * (CPW + D / 32)) * 4 : 0;
  return std::max(MlpLds<P, D, NBK>::bytes(M), red);
}

template <class P, int D>
static bool mlp_takes(int M) {
  return mlp_split<D>(M, [&](auto cw, auto cpw) { return M / 32 <= cw * cpw && mlp_lds<P, D, cw, cpw>(M) <= 160 * 1024; });
}

bool bwd_mlp_takes(int D, int M) {
  return D == 32 ? mlp_takes<PBF16, 32>(M) && mlp_takes<PF32, 32>(M) : mlp_takes<PBF16, 64>(M) && mlp_takes<PF32, 64>(M);
}

template <class P, int D>
static int32_t mlp_t(const BwdArgs& a, int blocks, hipStream_t st) {
  TDO_CHECK((mlp_takes<P, D>(a.M)), TDO_EUNSUPPORTED, "feed-forward backward: width %d, mlp %d", D, a.M);
  return mlp_split<D>(a.M, [&](auto cw, auto cpw) -> int32_t {
    auto k = a.g_in ? k_bwd_mlp<P, D, cw, cpw, false> : k_bwd_mlp<P, D, cw, cpw, true>;
    TDO_TRY(allow_full_lds((const void*)k));
    hipLaunchKernelGGL(k, dim3(blocks), dim3(512), (mlp_lds<P, D, cw, cpw>(a.M)), st, a);
    TDO_HIP(hipGetLastError());
    return TDO_OK;
  });
}

template <class P, int D, int DH, bool SPAN>
static int32_t attn_t(const BwdArgs& a, int blocks, hipStream_t st) {
  const size_t lds = (size_t)(2 * 32 * (128 / D) * (D + 4) + 24 * 32 * TS) * 4;
  auto k = k_bwd_attn<P, D, DH, SPAN>;
  TDO_TRY(allow_full_lds((const void*)k));
  hipLaunchKernelGGL(k, dim3(blocks), dim3(512), lds, st, a);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_bwd_mlp(const BwdArgs& a, bool bf16, int D, int blocks, hipStream_t st) {
  if (D == 32) return bf16 ? mlp_t<PBF16, 32>(a, blocks, st) : mlp_t<PF32, 32>(a, blocks, st);
  if (D == 64) return bf16 ? mlp_t<PBF16, 64>(a, blocks, st) : mlp_t<PF32, 64>(a, blocks, st);
  return set_error(TDO_EUNSUPPORTED, "no MLP backward kernel for width %d", D);
}

template <class P>
static int32_t attn_p(const BwdArgs& a, int D, int DH, int blocks, hipStream_t st) {
  const bool sp = a.span != 0;
  if (D == 32 && DH == 8) return sp ? attn_t<P, 32, 8, true>(a, blocks, st) : attn_t<P, 32, 8, false>(a, blocks, st);
  if (D == 64 && DH == 8) return sp ? attn_t<P, 64, 8, true>(a, blocks, st) : attn_t<P, 64, 8, false>(a, blocks, st);
  if (D == 64 && DH == 16) return sp ? attn_t<P, 64, 16, true>(a, blocks, st) : attn_t<P, 64, 16, false>(a, blocks, st);
  return set_error(TDO_EUNSUPPORTED, "no attention backward kernel for width %d, head width %d", D, DH);
}

int32_t launch_bwd_attn(const BwdArgs& a, bool bf16, int D, int DH, int blocks, hipStream_t st) {
  return bf16 ? attn_p<PBF16>(a, D, DH, blocks, st) : attn_p<PF32>(a, D, DH, blocks, st);
}

int32_t launch_bwd_head(bool bf16, int D, const void* save_last, const float* seeds, const int64_t* E_dev,
                        int64_t E_host, int n, int cpb, int span, int d_real, double* gw, double* gb, double* part,
                        hipStream_t st) {
  const int G = grid_for(HEAD_BLOCKS, span ? 4 * E_host : 2 * ((E_host + cpb - 1) / cpb), 4);
  if (D == 32) {
    if (bf16) hipLaunchKernelGGL((k_bwd_head<PBF16, 32>), dim3(G), dim3(256), 0, st, save_last, seeds, E_dev, E_host, n, cpb, span, d_real, part);
    else hipLaunchKernelGGL((k_bwd_head<PF32, 32>), dim3(G), dim3(256), 0, st, save_last, seeds, E_dev, E_host, n, cpb, span, d_real, part);
  } else {
    if (bf16) hipLaunchKernelGGL((k_bwd_head<PBF16, 64>), dim3(G), dim3(256), 0, st, save_last, seeds, E_dev, E_host, n, cpb, span, d_real, part);
    else hipLaunchKernelGGL((k_bwd_head<PF32, 64>), dim3(G), dim3(256), 0, st, save_last, seeds, E_dev, E_host, n, cpb, span, d_real, part);
  }
  TDO_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_reduce_head, dim3(2 * d_real + 2), dim3(256), 0, st, part, G, d_real, gw, gb);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_embed_scatter(int D, const float* dx0, const uint64_t* ecfg, const int64_t* E_dev, int64_t E_host,
                             int n, int cpb, int span, float* partial, int blocks, hipStream_t st, int waves) {
  const dim3 g(blocks), t(64 * waves);
  if (D == 32) hipLaunchKernelGGL(k_embed_onehot<32>, g, t, 0, st, dx0, ecfg, E_dev, E_host, n, cpb, span, partial);
  else hipLaunchKernelGGL(k_embed_onehot<64>, g, t, 0, st, dx0, ecfg, E_dev, E_host, n, cpb, span, partial);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_embed_params(const float* params, const double* dT, int d, int D, double* grad, double* part,
                            hipStream_t st) {
  TDO_CHECK(d <= 64, TDO_EUNSUPPORTED, "embedding chain rule: width %d > 64", d);
  const int64_t len = 6LL * d + 2LL * d * d;
  hipLaunchKernelGGL(k_embed_params, dim3(64), dim3(64), 0, st, params, dT, d, D, part);
  TDO_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_embed_params_sum, dim3((unsigned)ceil_div(len, 256)), dim3(256), 0, st, part, len, grad);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

template <class Map>
static int32_t reduce(const float* part, int nparts, int64_t plen, Map map, int64_t len, double* out, hipStream_t st) {
  if (len <= 0) return TDO_OK;
  if (ceil_div(len, 64) >= 256) {  // enough workgroups with 4 groups of partials
    hipLaunchKernelGGL((k_reduce_partials<64, Map>), dim3((unsigned)ceil_div(len, 64)), dim3(256), 0, st, part, nparts, plen, map, len, out);
  } else {
    hipLaunchKernelGGL((k_reduce_partials<16, Map>), dim3((unsigned)ceil_div(len, 16)), dim3(256), 0, st, part, nparts, plen, map, len, out);
  }
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

int32_t launch_reduce_partials(const float* part, int nparts, int64_t len, double* out, hipStream_t st) {
  return reduce(part, nparts, len, WholeMap{}, len, out, st);
}

int32_t launch_reduce_mlp(const float* part, int nparts, const PackPlan& pp, double* g, hipStream_t st) {
  const int64_t d = pp.d, D = pp.D, M = pp.M;
  return reduce(part, nparts, 2 * D * M + M + D, MlpMap{pp.d, pp.D, pp.M}, 2 * d * M + M + d, g + 4 * d * d, st);
}

int32_t launch_reduce_attn(const float* part, int nparts, const PackPlan& pp, double* g, hipStream_t st) {
  return reduce(part, nparts, 4LL * pp.D * pp.D, AttnMap{pp.d, pp.D}, 4LL * pp.d * pp.d, g, st);
}

}  // namespace tdo
