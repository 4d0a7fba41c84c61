// Forward pass and Metropolis sweeps in one launch (which networks and batches: stack_takes): a workgroup
// takes its tiles through every layer, so that the residual stream never leaves the registers and nothing but the
// weights moves between layers.  The tile functions are those of the layer-by-layer kernel
// (fwd_tile.h), so the results are the same bits.
#include <algorithm>

#include "common.h"
#include "fwd_tile.h"
#include "metropolis.h"
#include "net.h"
#include "netapi.h"

namespace tdo {

constexpr int STACK_WAVES = 8;
// Floats after a row of the embedding table in LDS.  Without them every row starts at the same bank, and the
// lanes of a tile read up to 32 rows (a sweep of 1024 chains at n = 32: 2.21 -> 2.17 ms, log rho of 65536
// configurations 1.965 -> 1.936 ms).
constexpr int TABLE_PAD = 4;
constexpr int STACK_FF_BYTES = 64 * 1024;  // a layer's feed-forward weights (BF16), at most

// MODE 0: log rho of E configurations; 1, 2: `steps` proposals of every chain (doubled space,
// diagonal); 3: z (and log rho, if lr is given) of E configurations, with the activations that the
// backward pass needs.  A tile is one pass of cpb = 32 / n configurations, a pair both passes; a
// workgroup has `pairs` of them: 4, or fewer in a batch that leaves CUs idle (a wave alone on its SIMD
// is faster).  TW: tiles per wave.
//   TW = 1: waves 2p and 2p + 1 hold the tiles of pair p, p < pairs.
//   TW = 2 (BF16, large batches): wave p < pairs <= 8 holds both tiles of pair p.  A BF16 weight fragment is 1 KB of LDS for one product of 32 cycles, so four
//     SIMDs with one tile per wave ask for the 128 bytes per cycle that LDS delivers, and the bias
//     comes on top; in the feed-forward part a fragment now serves two tiles.  In the attention part the
//     tiles take turns: together they spill 17 to 110 registers.  65536 configurations, 4 layers,
//     n = 32: 2.17 -> 1.96 ms; width 32, n = 8: 175 -> 143 us; with the activations saved, 2 layers of
//     16384 at n = 32 430 -> 388 us.
// BF16: a layer's weights are staged in two LDS buffers, attention and feed-forward; each is
// copied from memory to LDS directly while the other is computed with, two barriers a layer.
// FP32: weight fragments come through the caches, no staging.
// Bound: latency in a small batch (one tile's chain of products through all layers), the products, the
// softmax on the vector ALU and LDS together in a large one.  Layer by layer, a proposal of 1024 chains
// at n = 32 took 77 us, about half of it launches, staging and the round trip of the residual stream;
// here 39 us, and 23 us for 16 chains (40 before).
template <class P, int D, int DH, int MBC, bool MASKED, int MODE, int TW>
__global__ void __launch_bounds__(512) k_fwd_stack(StackArgs a) {
  constexpr int NB = D / 32, HPB = 32 / DH, PAIRS = 4 * TW;
  constexpr bool WLDS = P::KPL == 8;
  using elem_t = typename P::elem_t;
  using save_t = typename P::save_t;
  extern __shared__ __align__(16) char smem[];
  __shared__ float2 zsh[PAIRS][10][2];
  __shared__ uint64_t cfg_s[PAIRS][10][2];
  const int M = MBC ? 32 * MBC : a.M, MB = M / 32, L = a.layers;
  // LDS: [attention weights][feed-forward weights] (BF16), [b1 M, b2 D] per layer, table [64][D + pad], head weights [64]
  elem_t* wa = reinterpret_cast<elem_t*>(smem);
  elem_t* wm = wa + 4 * D * D;
  float* bias = reinterpret_cast<float*>(smem + (WLDS ? (size_t)(4 * D * D + 2 * D * M) * sizeof(elem_t) : 0));
  float* tabs = bias + L * (M + D);
  float2* hws = reinterpret_cast<float2*>(tabs + 64 * (D + TABLE_PAD));
  const elem_t* wg = reinterpret_cast<const elem_t*>(a.wpack);
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), pair = TW == 2 ? wave : wave >> 1, pass0 = TW == 2 ? 0 : wave & 1;
  const int64_t E = MODE == 3 && a.n_entries_dev ? *a.n_entries_dev : a.E;
  const int n = a.n, cpb = a.cpb, G = a.pairs * cpb;
  const bool busy = pair < a.pairs;  // the other waves only stage weights

  for (int i = tid; i < L * (M + D); i += 512) {
    const int l = i / (M + D), k = i % (M + D);
    bias[i] = k < M ? a.b1[l * M + k] : a.b2[l * D + k - M];
  }
  for (int i = tid; i < 64 * D; i += 512) tabs[i / D * (D + TABLE_PAD) + i % D] = a.table[i];
  if (tid < 64) hws[tid] = tid < a.d_real ? make_float2(a.head_w[2 * tid], a.head_w[2 * tid + 1]) : make_float2(0.f, 0.f);

  // copies 16-byte pieces of a layer's weights (a multiple of 64) to LDS, without a stop in registers
  auto stage = [&](elem_t* dst, const elem_t* src, int pieces) {
    for (int i = wave * 64; i < pieces; i += 512)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (i + lane) * 8),
                                       (__attribute__((address_space(3))) void*)(dst + i * 8), 16, 0, 0);
  };
  auto stage_a = [&](int l) { stage(wa, wg + l * a.layer_elems, 4 * D * D / 8); };
  auto stage_m = [&](int l) { stage(wm, wg + l * a.layer_elems + 4 * D * D, 2 * D * M / 8); };
  auto staged = [&] {  // the copies of all waves have arrived
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    barrier_lds();
  };
  const bool reload = L > 1;  // a single layer's weights stay in LDS
  if (WLDS && !reload) {
    stage_a(0);
    stage_m(0);
  }

  const int slot = lr / n, site = lr - slot * n;
  uint32_t okb = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int key = tile_idx(r, h);
    okb |= (!MASKED || (key / n == slot && key / n < cpb)) ? 1u << r : 0u;
  }

  const uint32_t okbits[1][1] = {{okb}};

  for (int64_t grp = blockIdx.x; grp * G < E; grp += gridDim.x) {
    const int64_t g0 = grp * G;
    // thread tid < G keeps configuration (or chain) g0 + tid in the registers
    const int64_t ce = g0 + tid;
    const bool mine = tid < G && ce < E;
    uint64_t sa = 0, sb = 0;
    float2 slr = make_float2(0.f, 0.f);
    if (mine) {
      if constexpr (MODE == 0 || MODE == 3) { sa = a.ecfg[2 * ce]; sb = a.ecfg[2 * ce + 1]; }
      if constexpr (MODE == 1) { sa = a.state[2 * ce]; sb = a.state[2 * ce + 1]; }
      if constexpr (MODE == 2) sa = sb = a.state[ce];
      if constexpr (MODE == 1 || MODE == 2) slr = make_float2(a.state_lr[2 * ce], a.state_lr[2 * ce + 1]);
    }
    const bool rvalid[1] = {busy && slot < cpb && g0 + pair * cpb + slot < E};
    // the (first) block of this wave in the saved activations, and whether it exists
    const int64_t blk = 2 * (grp * a.pairs + pair) + pass0;
    const bool kept = MODE == 3 && busy && g0 + pair * cpb < E;
    auto save = [&](void* dst, int l, const f32x16 (&v)[TW][NB]) {
      constexpr int bytes = 64 * 16 * (int)sizeof(save_t);
      const auto r = rsrc(static_cast<char*>(dst) + l * a.layer_bytes + blk * NB * bytes, kept ? TW * NB * bytes : 0);
#pragma unroll
      for (int i = 0; i < TW * NB; ++i) {
        const f32x16& t = v[i / NB][i % NB];
        if constexpr (WLDS) {
#pragma unroll
          for (int s = 0; s < 2; ++s) rst4(r, lane * 16, __builtin_bit_cast(float4, cvt8(t, s)), i * bytes + 1024 * s);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            rst4(r, lane * 16, make_float4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]), i * bytes + 1024 * q);
        }
      }
    };
    const int steps = MODE == 1 || MODE == 2 ? a.steps : 1;
    for (int s = 0; s < steps; ++s) {
      uint64_t pa = sa, pb = sb;
      double u = 0.0;
      if constexpr (MODE == 1) u = propose_move(pa, pb, n, a.t0 + s, (uint32_t)ce, a.seed, a.pair_thr);
      if constexpr (MODE == 2) {
        u = propose_diag(pa, n, a.t0 + s, (uint32_t)ce, a.seed);
        pb = pa;
      }
      if (tid < G) { cfg_s[tid / cpb][tid % cpb][0] = pa; cfg_s[tid / cpb][tid % cpb][1] = pb; }
      if (WLDS && reload) stage_a(0);
      if (WLDS) staged();
      else barrier_lds();
      f32x16 x[TW][NB];
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        const int pass = pass0 + t;
        int code = 0;
        if (rvalid[0]) {
          const uint64_t al = cfg_s[pair][slot][0], be = cfg_s[pair][slot][1];
          code = EmbedRow<D>::code(pass ? be : al, pass ? al : be, site, n);
        }
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(tabs + code * (D + TABLE_PAD) + 32 * ob + 8 * q + 4 * h);
            x[t][ob][4 * q + 0] = v.x; x[t][ob][4 * q + 1] = v.y; x[t][ob][4 * q + 2] = v.z; x[t][ob][4 * q + 3] = v.w;
          }
      }
#pragma unroll 1
      for (int l = 0; l < L; ++l) {
        const elem_t* W = WLDS ? wa : wg + l * a.layer_elems;
        if (WLDS && reload) stage_m(l);
        if constexpr (MODE == 3) save(a.save_x, l, x);
        if (busy)
#pragma unroll
          for (int t = 0; t < TW; ++t) {
            f32x16 xt[1][NB];
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) xt[0][ob] = x[t][ob];
            tile_attention<P, D, DH, 1, MASKED>(xt, W, W + D * D, W + 2 * D * D, W + 3 * D * D, okbits, a.score_scale, lane,
                                                [&](int hb, const float (&lsev)[1][HPB]) {
              if constexpr (MODE == 3 && WLDS) {  // one store per lane of the first half; the second's is out of range
                const auto r = rsrc(a.save_lse + l * a.lse_layer + (blk + t) * 32 * (NB * HPB), kept ? 32 * NB * HPB * 4 : 0);
                const int off = h == 0 ? (lr * (NB * HPB) + hb * HPB) * 4 : 0x7ffffff0;
                if constexpr (HPB == 4) rst4(r, off, make_float4(lsev[0][0], lsev[0][1], lsev[0][2], lsev[0][3]));
                else rst2(r, off, make_float2(lsev[0][0], lsev[0][1]));
              }
            });
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) x[t][ob] = xt[0][ob];
            __builtin_amdgcn_sched_barrier(0);  // one tile at a time: the registers
          }
        if (WLDS && reload) {
          staged();  // feed-forward weights ready, attention weights free
          if (l + 1 < L) stage_a(l + 1);
        }
        if constexpr (MODE == 3) save(a.save_mid, l, x);  // after the wait, which would be for these stores too
        const elem_t* W1 = WLDS ? wm : W + 4 * D * D;
        if (busy) tile_ffn<P, D, TW>(x, W1, W1 + D * M, bias + l * (M + D), bias + l * (M + D) + M, MB, lane);
        if (WLDS && reload) staged();  // the next layer's attention weights ready, feed-forward weights free
      }
      if constexpr (MODE == 3) save(a.save_last, 0, x);
      if (busy)
#pragma unroll
        for (int t = 0; t < TW; ++t) {
          float v0, v1;
          f32x16 xt[1][NB];
#pragma unroll
          for (int ob = 0; ob < NB; ++ob) xt[0][ob] = x[t][ob];
          tile_head<1, NB>(xt, hws, rvalid, site, h, v0, v1);
          if (h == 0 && site == n - 1 && slot < cpb) {
            const float inv = 1.0f / (float)n;
            const float2 z = make_float2(v0 * inv + a.head_b[0], v1 * inv + a.head_b[1]);
            zsh[pair][slot][pass0 + t] = z;
            if (MODE == 3 && rvalid[0]) {
              const int64_t e = g0 + pair * cpb + slot;
              a.z[(e * 2 + pass0 + t) * 2] = z.x;
              a.z[(e * 2 + pass0 + t) * 2 + 1] = z.y;
            }
          }
        }
      barrier_lds();
      if (mine) {
        const float2 z1 = zsh[tid / cpb][tid % cpb][0], z2 = zsh[tid / cpb][tid % cpb][1];
        const float2 v = symmetrise(z1.x, z1.y, z2.x, z2.y);
        if constexpr (MODE == 0 || MODE == 3) {
          if (MODE == 0 || a.lr) {
            a.lr[2 * ce] = v.x;
            a.lr[2 * ce + 1] = v.y;
          }
        } else if (u < accept_ratio(v.x, slr.x, MODE == 2)) {
          sa = pa;
          sb = pb;
          slr = v;
        }
      }
    }
    if ((MODE == 1 || MODE == 2) && mine) {
      a.state_lr[2 * ce] = slr.x;
      a.state_lr[2 * ce + 1] = slr.y;
      if constexpr (MODE == 1) {
        a.state[2 * ce] = a.record[2 * ce] = sa;
        a.state[2 * ce + 1] = a.record[2 * ce + 1] = sb;
      } else a.state[ce] = a.record[ce] = sa;
    }
    barrier_lds();  // z read before the next group's
  }
}

template <class P, int D>
static size_t stack_lds_t(int M, int layers) {
  return (P::KPL == 8 ? (size_t)(4 * D * D + 2 * D * M) * 2 : 0) + (size_t)layers * (M + D) * 4 + 64 * (D + TABLE_PAD) * 4 + 64 * sizeof(float2);
}

// static LDS of the kernel, at most: z and configurations of 8 pairs of tiles
constexpr size_t STACK_STATIC = 8 * 10 * 2 * (sizeof(float2) + sizeof(uint64_t));

bool stack_supported(bool bf16, int D, int M, int layers, bool span) {
  const size_t lds = D == 32 ? (bf16 ? stack_lds_t<PBF16, 32>(M, layers) : stack_lds_t<PF32, 32>(M, layers))
                             : (bf16 ? stack_lds_t<PBF16, 64>(M, layers) : stack_lds_t<PF32, 64>(M, layers));
  return !span && lds + STACK_STATIC <= 160 * 1024 && (!bf16 || 2 * D * M * 2 <= STACK_FF_BYTES);
}

template <class P, int D, int DH, int MBC, bool MASKED>
static int32_t stack_m(StackArgs a, int mode, int num_cus, hipStream_t st) {
  const int64_t tiles = (a.E + a.cpb - 1) / a.cpb;
  // Two tiles per wave.  A round of the chip (4 pairs per CU with one tile, 8 with two) at n = 32, 4
  // layers, takes 33 and 57 us, so they are taken where 1.8 times their rounds are fewer: 2048 pairs 91
  // and 84 us, 3072 129 and 140, 4096 159 and 143 (per proposal of 2048 chains 70 and 63).  The same choice is the
  // faster one, by 5 to 24%, at widths 16, 32 and 64, n = 4, 8, 16, 24, mlp 64 to 512 (1100 to 20000 pairs: width 32,
  // n = 8, 2500 pairs 48 and 51, 4000 57 and 51; width 32, mlp 512, n = 32, 2500 103 and 105, 20000 534 and 432).  With
  // the activations saved a backward pass follows, and the gain of this kernel is lost in its clock up to 64 pairs per
  // CU (log rho and gradient, BF16, n = 32, 4 layers: 8192 pairs 1603 and 1626 us, 24576 4220 and 4148; with 2 or 3
  // layers, widths 32 and 64, 4000 to 12000 pairs two tiles are 0 to 2% faster).
  const int64_t r1 = (tiles + 4 * num_cus - 1) / (4 * num_cus), r2 = (tiles + 8 * num_cus - 1) / (8 * num_cus);
  const bool two = P::KPL == 8 && (mode == 3 ? tiles > 64LL * num_cus : 18 * r2 < 10 * r1);
  constexpr int T2 = P::KPL == 8 ? 2 : 1;
  auto kern = mode == 0   ? (two ? k_fwd_stack<P, D, DH, MBC, MASKED, 0, T2> : k_fwd_stack<P, D, DH, MBC, MASKED, 0, 1>)
              : mode == 1 ? (two ? k_fwd_stack<P, D, DH, MBC, MASKED, 1, T2> : k_fwd_stack<P, D, DH, MBC, MASKED, 1, 1>)
              : mode == 2 ? (two ? k_fwd_stack<P, D, DH, MBC, MASKED, 2, T2> : k_fwd_stack<P, D, DH, MBC, MASKED, 2, 1>)
                          : (two ? k_fwd_stack<P, D, DH, MBC, MASKED, 3, T2> : k_fwd_stack<P, D, DH, MBC, MASKED, 3, 1>);
  TDO_TRY(allow_full_lds((const void*)kern, STACK_STATIC));
  const size_t lds = stack_lds_t<P, D>(a.M, a.layers);
  a.pairs = two ? (int)std::min<int64_t>(8, (tiles + num_cus - 1) / num_cus) : tiles <= num_cus ? 1 : tiles <= 2 * num_cus ? 2 : 4;
  const int64_t groups = (tiles + a.pairs - 1) / a.pairs;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(groups, num_cus));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * STACK_WAVES), lds, st, a);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

template <class P, int D, int DH>
static int32_t stack_d(const StackArgs& a, bool masked, int mode, int num_cus, hipStream_t st) {
  if constexpr (P::KPL == 8 && D == 64)
    if (a.M == 256) return masked ? stack_m<P, D, DH, 8, true>(a, mode, num_cus, st) : stack_m<P, D, DH, 8, false>(a, mode, num_cus, st);
  return masked ? stack_m<P, D, DH, 0, true>(a, mode, num_cus, st) : stack_m<P, D, DH, 0, false>(a, mode, num_cus, st);
}

template <class P>
static int32_t stack_p(const StackArgs& a, int D, int DH, bool masked, int mode, int num_cus, hipStream_t st) {
  if (D == 32 && DH == 8) return stack_d<P, 32, 8>(a, masked, mode, num_cus, st);
  if (D == 64 && DH == 8) return stack_d<P, 64, 8>(a, masked, mode, num_cus, st);
  if (D == 64 && DH == 16) return stack_d<P, 64, 16>(a, masked, mode, num_cus, st);
  return set_error(TDO_EUNSUPPORTED, "no forward kernel for padded width %d, head width %d", D, DH);
}

int32_t launch_fwd_stack(const StackArgs& a, bool bf16, int D, int DH, bool masked, int mode, int num_cus, hipStream_t st) {
  return bf16 ? stack_p<PBF16>(a, D, DH, masked, mode, num_cus, st) : stack_p<PF32>(a, D, DH, masked, mode, num_cus, st);
}

}  // namespace tdo
