// Forward pass of the transformer density operator (main text "Transformer
// density operator ansatz"; App. B), one kernel launch per layer.
//
// Work decomposition.  The evaluation list holds E configurations, each
// evaluated in two passes: the direct channel order (alpha, beta) giving
// z(alpha, beta) and the swapped order (beta, alpha) giving z(beta, alpha)
// (Eq. log_sum_exp_conjugate).  For n <= 32 a 32-row block holds
// cpb = 32/n configurations of one pass (block g: pass g&1, configurations
// (g>>1)*cpb ...); attention is masked to rows of the same configuration.  For
// 32 < n <= 64 one configuration-pass spans two blocks (64 rows, rows >= n
// masked).  A wave owns a tile of NBR blocks and keeps its rows in registers
// through the whole layer: QKV projection, per-head softmax(QK^T/sqrt(dh))V,
// W_O and residual, then the ReLU feed-forward sub-layer and residual.
// The layer's packed weights are staged once per workgroup in LDS (BF16) or
// read through the caches (FP32); workgroups are persistent over tiles.
#include <algorithm>

#include "common.h"
#include "fwd_tile.h"
#include "net.h"
#include "netapi.h"

namespace tdo {

// Workgroup size NT: BF16 weights staged in LDS are shared by 8 waves (two per SIMD,
// so that one wave's latencies overlap the other's work) or by 4 waves (one per SIMD,
// with twice the registers); the choice is autotuned per shape.  FP32: by the batch (launch_layer_m).
// A wave of a spanning pass (two row blocks) needs more than half a SIMD's registers:
// with 8 waves it is held to 256 and spills a few values (24 at head width 16 with
// masking), which measured faster than one wave per SIMD.

// MBC: the feed-forward width in 32-column chunks when fixed at compile time (0: a.M / 32), so
// that the chunk loop unrolls and one chunk's LDS reads overlap the previous chunk's products.
// MASKED: some (query, key) pairs of a tile are invalid (several configurations per block, or
// padding rows); a compile-time choice, so that the unmasked kernel holds no mask registers.
template <class P, int D, int DH, bool SPAN, int MBC, bool MASKED, int NT>
__global__ void __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu((SPAN && NT == 512) ? 2 : 1, (SPAN && NT == 512) ? 2 : 8))) k_fwd_layer(FwdArgs a) {
  constexpr int NB = D / 32;            // feature blocks
  constexpr int NBR = SPAN ? 2 : 1;     // row blocks per wave
  constexpr int HPB = 32 / DH;          // heads per 32-feature block
  using elem_t = typename P::elem_t;
  using save_t = typename P::save_t;
  constexpr bool WLDS = (P::KPL == 8);

  extern __shared__ __align__(16) char smem[];
  const int M = MBC ? 32 * MBC : a.M, MB = M / 32;
  const int wtotal = 4 * D * D + 2 * D * M;
  // LDS carve-up: [weights (BF16 only)] [b1 M] [b2 D] [table 64*D] [head weights: 64 float2]
  elem_t* wl = reinterpret_cast<elem_t*>(smem);
  float* b1s = reinterpret_cast<float*>(smem + (WLDS ? (size_t)wtotal * sizeof(elem_t) : 0));
  float* b2s = b1s + M;
  float* tabs = b2s + D;
  float2* hws = reinterpret_cast<float2*>(tabs + (a.first ? 64 * D : 0));  // last layer: (W_h[f][0], W_h[f][1]), 0 past d

  // ---- stage weights, biases and the embedding table
  const elem_t* wg = reinterpret_cast<const elem_t*>(a.wpack);
  if constexpr (WLDS) {
    const int n16 = wtotal * (int)sizeof(elem_t) / 16;
    const int4* src = reinterpret_cast<const int4*>(wg);
    int4* dst = reinterpret_cast<int4*>(wl);
    for (int i = threadIdx.x; i < n16; i += blockDim.x) dst[i] = src[i];
  }
  for (int i = threadIdx.x; i < M; i += blockDim.x) b1s[i] = a.b1[i];
  for (int i = threadIdx.x; i < D; i += blockDim.x) b2s[i] = a.b2[i];
  if (a.first)
    for (int i = threadIdx.x; i < 64 * D; i += blockDim.x) tabs[i] = a.table[i];
  if (a.last)
    for (int i = threadIdx.x; i < 64; i += blockDim.x)
      hws[i] = i < a.d_real ? make_float2(a.head_w[2 * i], a.head_w[2 * i + 1]) : make_float2(0.f, 0.f);
  __syncthreads();
  const elem_t* W = WLDS ? wl : wg;
  const elem_t* Wq = W + 0 * D * D;
  const elem_t* Wk = W + 1 * D * D;
  const elem_t* Wv = W + 2 * D * D;
  const elem_t* Wo = W + 3 * D * D;
  const elem_t* W1 = W + 4 * D * D;
  const elem_t* W2 = W + 4 * D * D + D * M;

  const int lane = threadIdx.x & 63, h = lane >> 5, lr = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int64_t E = a.n_entries_dev ? *a.n_entries_dev : a.n_entries;
  const int n = a.n, cpb = a.cpb;
  const int64_t ntiles = SPAN ? 2 * E : 2 * ((E + cpb - 1) / cpb);
  const float sc = a.score_scale;  // log2(e)/sqrt(dh)

  // valid (query row qb*32+lr, key row kb*32+tile_idx(r, h)) pairs as bit r of okbits[qb][kb]
  uint32_t okbits[NBR][NBR];
#pragma unroll
  for (int qb = 0; qb < NBR; ++qb)
#pragma unroll
    for (int kb = 0; kb < NBR; ++kb) {
      uint32_t bits = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = kb * 32 + tile_idx(r, h);
        bool ok;
        if (SPAN) ok = key < n;
        else ok = a.masked ? ((key / n) == (SPAN ? 0 : lr / n) && (key / n) < cpb) : true;
        bits |= ok ? (1u << r) : 0u;
      }
      okbits[qb][kb] = bits;
    }

  // x of a layer after the first, for the wave's next tile: loaded one tile ahead (one row
  // block per tile; the two of a spanning tile would not fit in the registers), so that the
  // latency of the loads overlaps the current tile's work
  const int64_t tstride = (int64_t)gridDim.x * (blockDim.x >> 6);
  f32x16 xnext[NBR][NB];
  auto fetch_x = [&](int64_t tl) {
    if (a.first || tl >= ntiles) return;
#pragma unroll
    for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
      for (int ob = 0; ob < NB; ++ob) {
        xnext[rb][ob] = load_tile(a.x_in + ((tl * NBR + rb) * NB + ob) * 1024, lane);
      }
  };
  // Neighbouring tiles go to the waves of one workgroup (contiguous activations), but a batch of
  // fewer tiles than the grid has waves goes round the workgroups first, so that all CUs work.
  const int64_t tile0 = ntiles < tstride ? (int64_t)wave * gridDim.x + blockIdx.x
                                         : (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  if (!SPAN) fetch_x(tile0);

  for (int64_t tile = tile0; tile < ntiles; tile += tstride) {
    // keeps the loads of the LDS weights inside the loop: hoisted, they would fill the registers
    asm volatile("" ::: "memory");
    const int pass = (int)(tile & 1);
    // first entry of the tile and the slot/validity of this lane's rows
    const int64_t e0 = SPAN ? (tile >> 1) : (tile >> 1) * cpb;
    int rslot[NBR];
    bool rvalid[NBR];
#pragma unroll
    for (int rb = 0; rb < NBR; ++rb) {
      const int row = rb * 32 + lr;
      if (SPAN) { rslot[rb] = 0; rvalid[rb] = row < n; }
      else { rslot[rb] = lr / n; rvalid[rb] = (lr / n) < cpb && (e0 + lr / n) < E; }
    }

    // ---- residual stream x (feature x row), FP32
    f32x16 x[NBR][NB];
    const int64_t gblk0 = tile * NBR;
    if (a.first) {
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb) {
        const int row = rb * 32 + lr;
        int code = 0;
        if (rvalid[rb]) {
          const int64_t e = e0 + rslot[rb];
          const uint64_t al = a.ecfg[2 * e], be = a.ecfg[2 * e + 1];
          const uint64_t c0 = pass ? be : al, c1 = pass ? al : be;
          code = EmbedRow<D>::code(c0, c1, SPAN ? row : (lr % n), n);
        }
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
          const float* tr = tabs + code * D + 32 * ob;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(tr + 8 * q + 4 * h);
            x[rb][ob][4 * q + 0] = v.x; x[rb][ob][4 * q + 1] = v.y;
            x[rb][ob][4 * q + 2] = v.z; x[rb][ob][4 * q + 3] = v.w;
          }
        }
      }
    } else {
      if (SPAN) fetch_x(tile);
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) x[rb][ob] = xnext[rb][ob];
    }
    if (!SPAN) fetch_x(tile + tstride);
    auto save = [&](void* dst, const f32x16 (&v)[NBR][NB]) {
      save_t* s = reinterpret_cast<save_t*>(dst);
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
          store_tile(s + ((gblk0 + rb) * NB + ob) * 1024, lane, v[rb][ob]);
        }
    };
    if (a.save_x) save(a.save_x, x);

    tile_attention<P, D, DH, NBR, MASKED, NT / 64>(x, Wq, Wk, Wv, Wo, okbits, sc, lane, [&](int hb, const float (&lsev)[NBR][HPB]) {
      if constexpr (P::KPL == 8) {
        // the head block's normalisers are contiguous per row; one store per lane of the first
        // half (the second half's offset is out of range, and the resource is empty when nothing
        // is saved: no branch)
        const auto rl = rsrc(a.save_lse ? a.save_lse + gblk0 * 32 * (NB * HPB) : nullptr,
                             a.save_lse ? NBR * 32 * NB * HPB * 4 : 0);
#pragma unroll
        for (int qb = 0; qb < NBR; ++qb) {
          const int off = h == 0 ? ((qb * 32 + lr) * (NB * HPB) + hb * HPB) * 4 : 0x7ffffff0;
          if constexpr (HPB == 4) rst4(rl, off, make_float4(lsev[qb][0], lsev[qb][1], lsev[qb][2], lsev[qb][3]));
          else rst2(rl, off, make_float2(lsev[qb][0], lsev[qb][1]));
        }
      }
    });
    if (a.save_mid) save(a.save_mid, x);

    tile_ffn<P, D, NBR, NT / 64>(x, W1, W2, b1s, b2s, MB, lane);

    if (!a.last) {
#pragma unroll
      for (int rb = 0; rb < NBR; ++rb)
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
          store_tile(a.x_out + ((gblk0 + rb) * NB + ob) * 1024, lane, x[rb][ob]);
        }
      continue;
    }
    // ---- last layer: save x_L, mean pooling over sites, dense head to z (Eq. global-pool-final)
    if (a.save_last) save(a.save_last, x);
    float v0, v1;
    const int seg = SPAN ? 0 : lr / n, pos = SPAN ? lr : lr - seg * n;
    tile_head<NBR, NB>(x, hws, rvalid, pos, h, v0, v1);
    const int last = SPAN ? 31 : n - 1;  // in a spanning tile every lane's rows are one configuration
    if (h == 0 && pos == last && (SPAN || seg < cpb)) {
      const int64_t e = e0 + seg;
      if (e < E) {
        const float inv = 1.0f / (float)n;
        a.z[(e * 2 + pass) * 2 + 0] = v0 * inv + a.head_b[0];
        a.z[(e * 2 + pass) * 2 + 1] = v1 * inv + a.head_b[1];
      }
    }
  }
}

__global__ void k_symmetrise(const int64_t* __restrict__ E_dev, int64_t E_host, const float* __restrict__ z,
                             float* __restrict__ lr) {
  const int64_t E = E_dev ? *E_dev : E_host;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < E; e += (int64_t)gridDim.x * blockDim.x) {
    const float2 v = symmetrise(z[4 * e], z[4 * e + 1], z[4 * e + 2], z[4 * e + 3]);
    lr[2 * e] = v.x;
    lr[2 * e + 1] = v.y;
  }
}

// ------------------------------------------------------------------ dispatch
template <class P, int D, int DH, bool SPAN, int MBC, bool MASKED, int NT>
static int32_t launch_layer_nt(const FwdArgs& a, int num_cus, hipStream_t st) {
  const size_t wbytes = (P::KPL == 8) ? (size_t)(4 * D * D + 2 * D * a.M) * sizeof(typename P::elem_t) : 0;
  const size_t lds = wbytes + (size_t)(a.M + D) * 4 + (a.first ? 64 * D * 4 : 0) + 64 * sizeof(float2);
  auto kern = k_fwd_layer<P, D, DH, SPAN, MBC, MASKED, NT>;
  TDO_TRY(allow_full_lds((const void*)kern));
  // no more workgroups than tiles (n_entries bounds the entries also where their count is on the device)
  const int64_t tiles = SPAN ? 2 * a.n_entries : 2 * ((a.n_entries + a.cpb - 1) / a.cpb);
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(num_cus * a.blocks_per_cu, tiles));
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(NT), lds, st, a);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

template <class P, int D, int DH, bool SPAN, int MBC, bool MASKED>
static int32_t launch_layer_m(const FwdArgs& a, int num_cus, hipStream_t st) {
  if constexpr (P::KPL == 8) {
    if (a.waves == 4) return launch_layer_nt<P, D, DH, SPAN, MBC, MASKED, 256>(a, num_cus, st);
  } else {
    // FP32: the weights come through the caches.  With 4 waves a wave has the registers to load its fragments
    // ahead (frags_ahead), with 8 a second wave per SIMD covers their latency.  A spanning pass of width 64 spills
    // with 8 (100 registers) and takes 4: microseconds for log rho with 8 and 4 waves, 3 layers, n = 40, 500
    // configurations 252 and 237, 1500 917 and 627, 16000 6790 and 5981.  The others: a round of the chip with 8 waves
    // takes so many hundredths of one with 4 (width 32 spanning 190, one row block of width 64 196, of width 32 180),
    // and 4 are taken where their rounds cost less, which is in batches of few (width 32, n = 50, 1500
    // configurations 346 and 285, 16000 2507 and 2587; one layer of width 64, n = 32, 1100 146 and 118, 6000 387 and 388).
    if constexpr (SPAN && D == 64) return launch_layer_nt<P, D, DH, SPAN, MBC, MASKED, 256>(a, num_cus, st);
    const int64_t tiles = SPAN ? 2 * a.n_entries : 2 * ((a.n_entries + a.cpb - 1) / a.cpb);
    const int64_t r4 = (tiles + 4 * num_cus - 1) / (4 * num_cus), r8 = (tiles + 8 * num_cus - 1) / (8 * num_cus);
    if (a.blocks_per_cu == 1 && 100 * r4 < (SPAN ? 190 : D == 64 ? 196 : 180) * r8)
      return launch_layer_nt<P, D, DH, SPAN, MBC, MASKED, 256>(a, num_cus, st);
  }
  if constexpr (P::KPL == 8 || !SPAN || D == 32)
  return launch_layer_nt<P, D, DH, SPAN, MBC, MASKED, 512>(a, num_cus, st);
}

// the BF16 width-64 kernels with the feed-forward width 4 x 64 fixed at compile time
template <class P, int D, int DH, bool SPAN, bool MASKED>
static int32_t launch_layer_k(const FwdArgs& a, int num_cus, hipStream_t st) {
  if constexpr (P::KPL == 8 && D == 64)
    if (a.M == 256) return launch_layer_m<P, D, DH, SPAN, 8, MASKED>(a, num_cus, st);
  return launch_layer_m<P, D, DH, SPAN, 0, MASKED>(a, num_cus, st);
}

// masking is needed with several configurations per block, or padding rows of a spanning pass
template <class P, int D, int DH, bool SPAN>
static int32_t launch_layer_t(const FwdArgs& a, int num_cus, hipStream_t st) {
  const bool masked = SPAN ? (a.n < 64) : (a.masked != 0);
  return masked ? launch_layer_k<P, D, DH, SPAN, true>(a, num_cus, st) : launch_layer_k<P, D, DH, SPAN, false>(a, num_cus, st);
}

template <class P>
static int32_t launch_layer_p(const FwdArgs& a, int D, int DH, bool span, int num_cus, hipStream_t st) {
  if (D == 32 && DH == 8) return span ? launch_layer_t<P, 32, 8, true>(a, num_cus, st) : launch_layer_t<P, 32, 8, false>(a, num_cus, st);
  if (D == 64 && DH == 8) return span ? launch_layer_t<P, 64, 8, true>(a, num_cus, st) : launch_layer_t<P, 64, 8, false>(a, num_cus, st);
  if (D == 64 && DH == 16) return span ? launch_layer_t<P, 64, 16, true>(a, num_cus, st) : launch_layer_t<P, 64, 16, false>(a, num_cus, st);
  return set_error(TDO_EUNSUPPORTED, "no forward kernel for padded width %d, head width %d", D, DH);
}

int32_t launch_fwd_layer(const FwdArgs& a, bool bf16, int D, int DH, bool span, int num_cus, hipStream_t st) {
  return bf16 ? launch_layer_p<PBF16>(a, D, DH, span, num_cus, st) : launch_layer_p<PF32>(a, D, DH, span, num_cus, st);
}

int32_t launch_symmetrise(const int64_t* E_dev, int64_t E_host, const float* z, float* lr, hipStream_t st) {
  hipLaunchKernelGGL(k_symmetrise, dim3(1024), dim3(256), 0, st, E_dev, E_host, z, lr);
  TDO_HIP(hipGetLastError());
  return TDO_OK;
}

}  // namespace tdo
