// Forward pass of small batches and Metropolis sweeps in one launch: a workgroup takes its tiles
// through every layer, so that the residual stream never leaves the registers and nothing but the
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
constexpr int STACK_PIECES = 8;  // 16-byte pieces per thread that hold a layer's feed-forward weights (BF16: 64 KB)

// MODE 0: log rho of E configurations; 1, 2: `steps` proposals of every chain (doubled space,
// diagonal); 3: z (and log rho, if lr is given) of E configurations, with the activations that the
// backward pass needs.  Waves 2p and 2p + 1 of a workgroup hold the two passes of cpb = 32 / n configurations,
// p < pairs: 4, or fewer in a batch that leaves CUs idle (a wave alone on its SIMD is faster).
// BF16: a layer's weights are staged in two LDS buffers, attention and feed-forward; each is
// loaded into registers while the other is computed with and stored before the barrier that ends
// that phase (two barriers a layer), so the loads from L2 overlap the products.  FP32: weight
// fragments come through the caches, no staging.
// Bound: latency in a small batch (one tile's chain of products through all layers), the products
// in a large one.  Layer by layer, a proposal of 1024 chains at n = 32 took 77 us, about half of it
// launches, staging and the round trip of the residual stream; here 40 us, and 24 us for 16 chains
// (40 before).
template <class P, int D, int DH, int MBC, bool MASKED, int MODE>
__global__ void __launch_bounds__(512) k_fwd_stack(StackArgs a) {
  constexpr int NB = D / 32, HPB = 32 / DH;
  constexpr bool WLDS = P::KPL == 8;
  using elem_t = typename P::elem_t;
  using save_t = typename P::save_t;
  extern __shared__ __align__(16) char smem[];
  __shared__ float2 zsh[4][10][2];
  __shared__ uint64_t cfg_s[4][10][2];
  const int M = MBC ? 32 * MBC : a.M, MB = M / 32, L = a.layers;
  // LDS: [attention weights][feed-forward weights] (BF16), [b1 M, b2 D] per layer, table [64][D], head weights [64]
  elem_t* wa = reinterpret_cast<elem_t*>(smem);
  elem_t* wm = wa + 4 * D * D;
  float* bias = reinterpret_cast<float*>(smem + (WLDS ? (size_t)(4 * D * D + 2 * D * M) * sizeof(elem_t) : 0));
  float* tabs = bias + L * (M + D);
  float2* hws = reinterpret_cast<float2*>(tabs + 64 * D);
  const elem_t* wg = reinterpret_cast<const elem_t*>(a.wpack);
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), pair = wave >> 1, pass = wave & 1;
  const int64_t E = MODE == 3 && a.n_entries_dev ? *a.n_entries_dev : a.E;
  const int n = a.n, cpb = a.cpb, G = a.pairs * cpb;
  const bool busy = pair < a.pairs;  // the other waves only stage weights

  for (int i = tid; i < L * (M + D); i += 512) {
    const int l = i / (M + D), k = i % (M + D);
    bias[i] = k < M ? a.b1[l * M + k] : a.b2[l * D + k - M];
  }
  for (int i = tid; i < 64 * D; i += 512) tabs[i] = a.table[i];
  if (tid < 64) hws[tid] = tid < a.d_real ? make_float2(a.head_w[2 * tid], a.head_w[2 * tid + 1]) : make_float2(0.f, 0.f);

  // 16-byte pieces of a layer's weights in this thread's registers between load and store (as
  // vectors: arrays indexed in the loops below would live in scratch memory)
  constexpr int NA = WLDS ? (4 * D * D * 2 / 16 + 511) / 512 : 1, NM = WLDS ? STACK_PIECES : 1;
  const int tm = 2 * D * M * 2 / 16;
  int __attribute__((ext_vector_type(4 * NA))) ra;
  int __attribute__((ext_vector_type(4 * NM))) rm;
  auto load_a = [&](int l) {
    const i32x4* s = reinterpret_cast<const i32x4*>(wg + l * a.layer_elems);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const i32x4 v = s[i * 512 + tid];
      ra[4 * i] = v.x; ra[4 * i + 1] = v.y; ra[4 * i + 2] = v.z; ra[4 * i + 3] = v.w;
    }
  };
  auto store_a = [&] {
#pragma unroll
    for (int i = 0; i < NA; ++i)
      reinterpret_cast<i32x4*>(wa)[i * 512 + tid] = i32x4{ra[4 * i], ra[4 * i + 1], ra[4 * i + 2], ra[4 * i + 3]};
  };
  auto load_m = [&](int l) {
    const i32x4* s = reinterpret_cast<const i32x4*>(wg + l * a.layer_elems + 4 * D * D);
#pragma unroll
    for (int i = 0; i < NM; ++i)
      if (i * 512 + tid < tm) {
        const i32x4 v = s[i * 512 + tid];
        rm[4 * i] = v.x; rm[4 * i + 1] = v.y; rm[4 * i + 2] = v.z; rm[4 * i + 3] = v.w;
      }
  };
  auto store_m = [&] {
#pragma unroll
    for (int i = 0; i < NM; ++i)
      if (i * 512 + tid < tm)
        reinterpret_cast<i32x4*>(wm)[i * 512 + tid] = i32x4{rm[4 * i], rm[4 * i + 1], rm[4 * i + 2], rm[4 * i + 3]};
  };
  const bool reload = L > 1;  // a single layer's weights stay in LDS
  if (WLDS && !reload) {
    load_a(0);
    load_m(0);
    store_a();
    store_m();
  }

  const int slot = lr / n, site = lr - slot * n;
  uint32_t okbits[1][1] = {{0}};
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int key = tile_idx(r, h);
    okbits[0][0] |= (!MASKED || (key / n == slot && key / n < cpb)) ? 1u << r : 0u;
  }

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
    // the block of this wave in the saved activations, and whether it exists
    const int64_t blk = 2 * (grp * a.pairs + pair) + pass;
    const bool kept = MODE == 3 && busy && g0 + pair * cpb < E;
    auto save = [&](void* dst, int l, const f32x16 (&v)[1][NB]) {
      constexpr int bytes = 64 * 16 * (int)sizeof(save_t);
      const auto r = rsrc(static_cast<char*>(dst) + l * a.layer_bytes + blk * NB * bytes, kept ? NB * bytes : 0);
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        if constexpr (WLDS) {
#pragma unroll
          for (int s = 0; s < 2; ++s)
            rst4(r, lane * 16, __builtin_bit_cast(float4, cvt8(v[0][ob], s)), ob * bytes + 1024 * s);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            rst4(r, lane * 16, make_float4(v[0][ob][4 * q], v[0][ob][4 * q + 1], v[0][ob][4 * q + 2], v[0][ob][4 * q + 3]), ob * bytes + 1024 * q);
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
      if (WLDS && reload) { load_a(0); store_a(); }
      barrier_lds();
      f32x16 x[1][NB];
      {
        int code = 0;
        if (rvalid[0]) {
          const uint64_t al = cfg_s[pair][slot][0], be = cfg_s[pair][slot][1];
          code = EmbedRow<D>::code(pass ? be : al, pass ? al : be, site, n);
        }
#pragma unroll
        for (int ob = 0; ob < NB; ++ob)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(tabs + code * D + 32 * ob + 8 * q + 4 * h);
            x[0][ob][4 * q + 0] = v.x; x[0][ob][4 * q + 1] = v.y; x[0][ob][4 * q + 2] = v.z; x[0][ob][4 * q + 3] = v.w;
          }
      }
#pragma unroll 1
      for (int l = 0; l < L; ++l) {
        const elem_t* W = WLDS ? wa : wg + l * a.layer_elems;
        if (WLDS && reload) load_m(l);
        if constexpr (MODE == 3) save(a.save_x, l, x);
        if (busy)
          tile_attention<P, D, DH, 1, MASKED>(x, W, W + D * D, W + 2 * D * D, W + 3 * D * D, okbits, a.score_scale, lane,
                                              [&](int hb, const float (&lsev)[1][HPB]) {
            if constexpr (MODE == 3 && WLDS) {  // one store per lane of the first half; the second's is out of range
              const auto r = rsrc(a.save_lse + l * a.lse_layer + blk * 32 * (NB * HPB), kept ? 32 * NB * HPB * 4 : 0);
              const int off = h == 0 ? (lr * (NB * HPB) + hb * HPB) * 4 : 0x7ffffff0;
              if constexpr (HPB == 4) rst4(r, off, make_float4(lsev[0][0], lsev[0][1], lsev[0][2], lsev[0][3]));
              else rst2(r, off, make_float2(lsev[0][0], lsev[0][1]));
            }
          });
        if constexpr (MODE == 3) save(a.save_mid, l, x);
        if (WLDS && reload) {
          store_m();
          barrier_lds();  // feed-forward weights ready, attention weights free
          if (l + 1 < L) load_a(l + 1);
        }
        const elem_t* W1 = WLDS ? wm : W + 4 * D * D;
        if (busy) tile_ffn<P, D, 1>(x, W1, W1 + D * M, bias + l * (M + D), bias + l * (M + D) + M, MB, lane);
        if (WLDS && reload) {
          if (l + 1 < L) store_a();
          barrier_lds();  // the next layer's attention weights ready, feed-forward weights free
        }
      }
      if constexpr (MODE == 3) save(a.save_last, 0, x);
      if (busy) {
        float v0, v1;
        tile_head<1, NB>(x, hws, rvalid, site, h, v0, v1);
        if (h == 0 && site == n - 1 && slot < cpb) {
          const float inv = 1.0f / (float)n;
          const float2 z = make_float2(v0 * inv + a.head_b[0], v1 * inv + a.head_b[1]);
          zsh[pair][slot][pass] = z;
          if (MODE == 3 && rvalid[0]) {
            const int64_t e = g0 + pair * cpb + slot;
            a.z[(e * 2 + pass) * 2] = z.x;
            a.z[(e * 2 + pass) * 2 + 1] = z.y;
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
  return (P::KPL == 8 ? (size_t)(4 * D * D + 2 * D * M) * 2 : 0) + (size_t)layers * (M + D) * 4 + 64 * D * 4 + 64 * sizeof(float2);
}

// static LDS of the kernel: z and configurations of 4 pairs of waves
constexpr size_t STACK_STATIC = 4 * 10 * 2 * (sizeof(float2) + sizeof(uint64_t));

bool stack_supported(bool bf16, int D, int M, int layers, bool span) {
  const size_t lds = D == 32 ? (bf16 ? stack_lds_t<PBF16, 32>(M, layers) : stack_lds_t<PF32, 32>(M, layers))
                             : (bf16 ? stack_lds_t<PBF16, 64>(M, layers) : stack_lds_t<PF32, 64>(M, layers));
  return !span && lds + STACK_STATIC <= 160 * 1024 && (!bf16 || 2 * D * M * 2 <= STACK_PIECES * 512 * 16);
}

template <class P, int D, int DH, int MBC, bool MASKED>
static int32_t stack_m(StackArgs a, int mode, int num_cus, hipStream_t st) {
  auto kern = mode == 0   ? k_fwd_stack<P, D, DH, MBC, MASKED, 0>
              : mode == 1 ? k_fwd_stack<P, D, DH, MBC, MASKED, 1>
              : mode == 2 ? k_fwd_stack<P, D, DH, MBC, MASKED, 2>
                          : k_fwd_stack<P, D, DH, MBC, MASKED, 3>;
  TDO_TRY(allow_full_lds((const void*)kern, STACK_STATIC));
  const size_t lds = stack_lds_t<P, D>(a.M, a.layers);
  const int64_t tiles = (a.E + a.cpb - 1) / a.cpb;
  a.pairs = tiles <= num_cus ? 1 : (tiles <= 2 * num_cus ? 2 : 4);
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
