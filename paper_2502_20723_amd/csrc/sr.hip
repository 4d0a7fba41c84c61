// Stochastic reconfiguration (App. C, metric tensor and hybrid update):
// solve (S + lambda I) x = g with
//   S_kl = Re sum_b w_b conj(dO_k(x_b)) dO_l(x_b),  dO = O - sum_b w_b O(x_b),
// O_k(x) = d log rho(x) / d theta_k, w normalised to sum 1, for the real
// parameters theta.  With J the 2B x P matrix of rows sqrt(w_b) dRe O(x_b) and
// sqrt(w_b) dIm O(x_b), S = J^T J, so S is never formed: conjugate gradients
// on (J^T J + lambda I) x = g take two passes over J per iteration (rows
// u = J p in segments, then columns J^T u with the segment sums).
//
// The Jacobian comes from tdo_log_rho_jacobian; this call centres and scales
// it in place.  Dot products are two-stage FP64 sums in a fixed order (slices, then the slices, by every
// workgroup that needs the product) and CG's scalars stay on the device, so the iteration count is fixed by
// the caller and the result does not depend on scheduling.  The order of these sums is part of the result: a
// solve stopped on an ill-conditioned system amplifies a change of rounding (256 slices or 128, rows first to
// last or last to first: up to 1e-5 of the update), so the split into slices, segments and accumulators
// is not a tuning choice.  An iteration is five launches (ten with the sums of the slices and the scalars in
// launches of their own: 38 us of 195, now 15 of 162).
#include <algorithm>
#include <cmath>

#include "common.h"
#include "netapi.h"
#include "train.h"

namespace tdo {

namespace {

constexpr int kT = 256;

__device__ double block_reduce(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int h = kT / 2; h > 0; h >>= 1) {
    if (t < h) red[t] += red[t + h];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

}  // namespace

// sc[0] = sum of the weights (B when w is NULL).
__global__ void __launch_bounds__(kT) k_sr_wsum(const double* __restrict__ w, int64_t B, double* __restrict__ sc) {
  __shared__ double red[kT];
  double a = 0.0;
  for (int64_t b = threadIdx.x; b < B; b += kT) a += w ? w[b] : 1.0;
  a = block_reduce(a, red);
  if (threadIdx.x == 0) sc[0] = a;
}

// Columns: subtract the weighted mean of each part (blockIdx.y) and scale row b by sqrt(w_b / sum w).
// Bound: memory, two reads and a write (the second read mostly from the last-level cache).  Eight
// rows' loads are in flight per thread and the parts are two rows of workgroups: B = 256,
// P = 107650 (441 MB): 518 -> 335 us.
__global__ void __launch_bounds__(kT) k_sr_center(double* __restrict__ J, int64_t B, int64_t P, const double* __restrict__ w,
                                                  const double* __restrict__ sc) {
  const double inv = 1.0 / sc[0];
  const int part = blockIdx.y;
  for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < P; k += (int64_t)gridDim.x * kT) {
    double* e = J + part * P + k;
    double mean = 0.0;
#pragma unroll 8
    for (int64_t b = 0; b < B; ++b) mean += (w ? w[b] : 1.0) * inv * e[2 * b * P];
#pragma unroll 8
    for (int64_t b = 0; b < B; ++b) e[2 * b * P] = sqrt((w ? w[b] : 1.0) * inv) * (e[2 * b * P] - mean);
  }
}

// Partial row dots: workgroup (r, s) forms J[r] . p over segment s of kSeg equal
// segments, into up[r][s] (summed in segment order by the column pass).
// Bound: memory, one read of J (441 MB at R = 512, P = 107650: 92 -> 82 us).  Four rows per workgroup,
// which read p once for all, leave too few loads in flight (113 us).  The rows are taken last to first: the
// column pass has just left the last ones in the last-level cache (256 MB), and this pass leaves the first ones
// for the next column pass (with both first to last, 94 and 73 us; so, 81 and 70 us).
constexpr int kSeg = 8;
__global__ void __launch_bounds__(kT) k_sr_rows(const double* __restrict__ J, int64_t R, int64_t P,
                                                const double* __restrict__ p, double* __restrict__ up) {
  __shared__ double red[kT];
  const int64_t seg = (P + kSeg - 1) / kSeg;
  for (int64_t rs = blockIdx.x; rs < R * kSeg; rs += gridDim.x) {
    const int64_t r = R - 1 - rs / kSeg, s = rs % kSeg;
    const double* row = J + r * P;
    const int64_t k1 = std::min<int64_t>(P, (s + 1) * seg);
    double a = 0.0;
#pragma unroll 8
    for (int64_t k = s * seg + threadIdx.x; k < k1; k += kT) a += row[k] * p[k];
    a = block_reduce(a, red);
    if (threadIdx.x == 0) up[r * kSeg + s] = a;
  }
}

// Ap[k] = sum_r J[r][k] u[r] + lambda p[k], one thread per column, with u[r] = sum over s of up[r][s] in
// segment order, formed in LDS for kURows rows at a time; four accumulators over r mod 4 (summed in that
// order; the last R mod 4 rows all in the first), rows first to last.  Bound: memory, one read of J.  R = 512,
// P = 107650: 84 us with four loads in flight, 73 with eight, 70 with the rows in the order that the row pass
// leaves in the cache.
constexpr int kURows = 512;
__global__ void __launch_bounds__(kT) k_sr_cols(const double* __restrict__ J, int64_t R, int64_t P, const double* __restrict__ up,
                                                const double* __restrict__ p, double lambda, double* __restrict__ Ap) {
  __shared__ double u[kURows];
  for (int64_t k0 = (int64_t)blockIdx.x * kT; k0 < P; k0 += (int64_t)gridDim.x * kT) {
    const int64_t k = k0 + threadIdx.x;
    const bool live = k < P;
    const double* col = J + (live ? k : 0);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t r0 = 0; r0 < R; r0 += kURows) {
      const int rows = (int)std::min<int64_t>(kURows, R - r0);
      __syncthreads();  // the previous rows' sums read
      for (int i = threadIdx.x; i < rows; i += kT) {
        double t = 0.0;
#pragma unroll
        for (int s = 0; s < kSeg; ++s) t += up[(r0 + i) * kSeg + s];
        u[i] = t;
      }
      __syncthreads();
      if (!live) continue;
      int i = 0;
#pragma unroll 2
      for (; i + 4 <= rows; i += 4) {
        a[0] += col[(r0 + i) * P] * u[i];
        a[1] += col[(r0 + i + 1) * P] * u[i + 1];
        a[2] += col[(r0 + i + 2) * P] * u[i + 2];
        a[3] += col[(r0 + i + 3) * P] * u[i + 3];
      }
      for (; i < rows; ++i) a[0] += col[(r0 + i) * P] * u[i];
    }
    if (live) Ap[k] = ((a[0] + a[1]) + (a[2] + a[3])) + lambda * p[k];
  }
}

// a . b in a fixed order: kDotParts workgroups sum contiguous slices into part[]; every workgroup of
// the kernel that uses the product sums the parts for itself (dot_parts, a part per thread).
constexpr int kDotParts = 256;
static_assert(kDotParts == kT, "one part per thread");
__device__ __forceinline__ double dot_parts(const double* __restrict__ part, double* red) {
  return block_reduce(part[threadIdx.x], red);
}
// Elements of a slice.
__device__ __forceinline__ int64_t dot_slice(int64_t P) { return (P + kDotParts - 1) / kDotParts; }
__global__ void __launch_bounds__(kT) k_sr_dot(const double* __restrict__ a, const double* __restrict__ b,
                                               int64_t P, double* __restrict__ part) {
  __shared__ double red[kT];
  const int64_t slice = dot_slice(P);
  const int64_t k0 = blockIdx.x * slice, k1 = std::min<int64_t>(P, k0 + slice);
  double s = 0.0;
  for (int64_t k = k0 + threadIdx.x; k < k1; k += kT) s += a[k] * b[k];
  s = block_reduce(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// x <- 0, r <- g, p <- g.
__global__ void k_sr_init(const double* __restrict__ g, int64_t P, double* __restrict__ x, double* __restrict__ r,
                          double* __restrict__ p) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
    x[k] = 0.0;
    r[k] = g[k];
    p[k] = g[k];
  }
}

// out[0] = out[1] = the sum of the parts.
__global__ void __launch_bounds__(kT) k_sr_sum(const double* __restrict__ part, double* __restrict__ out) {
  __shared__ double red[kT];
  const double s = dot_parts(part, red);
  if (threadIdx.x == 0) out[0] = out[1] = s;
}

// alpha = rs / (p . Ap) (0 when p . Ap = 0); x += alpha p; r -= alpha Ap; the parts of the new r . r.  Part i takes
// the place of the first element of slice i of Ap, which nothing reads any more.
__global__ void __launch_bounds__(kT) k_sr_step(int64_t P, const double* __restrict__ rs, const double* __restrict__ pap_part,
                                                const double* __restrict__ p, double* Ap, double* __restrict__ x,
                                                double* __restrict__ r) {
  __shared__ double red[kT];
  const double pAp = dot_parts(pap_part, red);
  const double alpha = pAp != 0.0 ? rs[0] / pAp : 0.0;
  const int64_t slice = dot_slice(P);
  const int64_t k0 = blockIdx.x * slice, k1 = std::min<int64_t>(P, k0 + slice);
  double s = 0.0;
  for (int64_t k = k0 + threadIdx.x; k < k1; k += kT) {
    x[k] += alpha * p[k];
    const double t = r[k] - alpha * Ap[k];
    r[k] = t;
    s += t * t;
  }
  s = block_reduce(s, red);  // every thread has read its elements of Ap
  if (threadIdx.x == 0 && k0 < P) Ap[k0] = s;
}

// beta = rs_new / rs (0 when rs = 0); p = r + beta p; rs_new to its own slot for the next iteration.
__global__ void __launch_bounds__(kT) k_sr_dir(int64_t P, const double* __restrict__ rs, const double* __restrict__ Ap,
                                               const double* __restrict__ r, double* __restrict__ p, double* __restrict__ rs_new) {
  __shared__ double red[kT];
  const int64_t at = threadIdx.x * dot_slice(P);
  const double rn = block_reduce(at < P ? Ap[at] : 0.0, red);
  const double beta = rs[0] != 0.0 ? rn / rs[0] : 0.0;
  for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < P; k += (int64_t)gridDim.x * kT) p[k] = r[k] + beta * p[k];
  if (blockIdx.x == 0 && threadIdx.x == 0) rs_new[0] = rn;
}

// info[0] = |r| / |g| from the recurrence, info[1] = |g|.
__global__ void k_sr_info(const double* __restrict__ rs, const double* __restrict__ gg, double* __restrict__ info) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const double gn = sqrt(gg[0]);
    info[0] = gn > 0.0 ? sqrt(rs[0]) / gn : 0.0;
    info[1] = gn;
  }
}

// Conjugate gradients on (S + lambda) x = g; apply(p, Ap) queues Ap = (S + lambda) p.  part: the parts of
// p . Ap; sc: [0] g . g, [1], [2] r . r, in turn the current and the next one.
template <class Apply>
static int32_t cg(int64_t P, const double* grad, int32_t iters, double* x, double* r, double* p, double* Ap, double* part,
                  double* sc, double* info, hipStream_t stream, Apply&& apply) {
  const unsigned gp = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(P, 256), 4096));
  hipLaunchKernelGGL(k_sr_init, dim3(gp), dim3(256), 0, stream, grad, P, x, r, p);
  hipLaunchKernelGGL(k_sr_dot, dim3(kDotParts), dim3(kT), 0, stream, grad, grad, P, part);
  hipLaunchKernelGGL(k_sr_sum, dim3(1), dim3(kT), 0, stream, part, sc);
  TDO_HIP(hipGetLastError());
  for (int32_t it = 0; it < iters; ++it) {
    TDO_TRY(apply(p, Ap));
    double *rs = sc + 1 + (it & 1), *rs_new = sc + 1 + (~it & 1);
    hipLaunchKernelGGL(k_sr_dot, dim3(kDotParts), dim3(kT), 0, stream, p, Ap, P, part);
    hipLaunchKernelGGL(k_sr_step, dim3(kDotParts), dim3(kT), 0, stream, P, rs, part, p, Ap, x, r);
    hipLaunchKernelGGL(k_sr_dir, dim3(gp), dim3(kT), 0, stream, P, rs, Ap, r, p, rs_new);
    TDO_HIP(hipGetLastError());
  }
  if (info) {
    hipLaunchKernelGGL(k_sr_info, dim3(1), dim3(64), 0, stream, sc + 1 + (iters & 1), sc, info);
    TDO_HIP(hipGetLastError());
  }
  return TDO_OK;
}

// --- the matrix-free form: S p = J^T (J p) from one forward-mode and one reverse-mode pass

// sc[0..2] = sum w, sum w Re t, sum w Im t over the samples (one workgroup, fixed order).
__global__ void __launch_bounds__(kT) k_mf_mean(const float* __restrict__ t, const double* __restrict__ w, int64_t B,
                                                double* __restrict__ sc) {
  __shared__ double red[kT];
  double a = 0.0, re = 0.0, im = 0.0;
  for (int64_t b = threadIdx.x; b < B; b += kT) {
    const double wb = w ? w[b] : 1.0;
    a += wb;
    re += wb * t[2 * b];
    im += wb * t[2 * b + 1];
  }
  a = block_reduce(a, red);
  re = block_reduce(re, red);
  im = block_reduce(im, red);
  if (threadIdx.x == 0) {
    sc[0] = a;
    sc[1] = re;
    sc[2] = im;
  }
}

// seed_b = (w_b / W) (t_b - sum w t / W): the reverse-mode seeds of J^T (J p).
__global__ void k_mf_seeds(const float* __restrict__ t, const double* __restrict__ w, int64_t B,
                           const double* __restrict__ sc, float* __restrict__ seed) {
  const double W = sc[0], mr = sc[1] / W, mi = sc[2] / W;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < B; b += (int64_t)gridDim.x * blockDim.x) {
    const double f = (w ? w[b] : 1.0) / W;
    seed[2 * b] = (float)(f * (t[2 * b] - mr));
    seed[2 * b + 1] = (float)(f * (t[2 * b + 1] - mi));
  }
}

// Ap += lambda p
__global__ void k_mf_shift(int64_t P, double lambda, const double* __restrict__ p, double* __restrict__ Ap) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x)
    Ap[k] += lambda * p[k];
}

}  // namespace tdo

using namespace tdo;

extern "C" int32_t tdo_sr_solve(tdo_ctx_t* ctx, double* jac, int64_t B, int64_t P, const double* weights,
                                const double* grad, double lambda, int32_t iters, double* x, double* info,
                                hipStream_t stream) {
  clear_error();
  TDO_CHECK(ctx != nullptr, TDO_EINVAL, "ctx is NULL");
  TDO_CHECK(B >= 1 && P >= 1, TDO_EINVAL, "B=%lld, P=%lld: both must be >= 1", (long long)B, (long long)P);
  TDO_CHECK(lambda > 0.0 && std::isfinite(lambda), TDO_EINVAL, "diagonal shift lambda=%g must be positive", lambda);
  TDO_CHECK(iters >= 0, TDO_EINVAL, "iters=%d < 0", iters);
  TDO_CHECK(jac && grad && x, TDO_EINVAL, "NULL buffer");
  TDO_HIP(hipSetDevice(ctx->c.device));
  Context& c = ctx->c;
  WsOrder order;
  TDO_TRY(order.begin(&c, stream));
  Arena ar;
  const size_t or_ = ar.take<double>((size_t)P), op = ar.take<double>((size_t)P), oap = ar.take<double>((size_t)P);
  const size_t oup = ar.take<double>(2 * (size_t)B * kSeg), osc = ar.take<double>(8), opart = ar.take<double>(kDotParts);
  TDO_TRY(ensure_workspace(&c, ar.used));
  double* r = at<double>(c.ws, or_);
  double* p = at<double>(c.ws, op);
  double* Ap = at<double>(c.ws, oap);
  double* up = at<double>(c.ws, oup);
  double* sc = at<double>(c.ws, osc);  // [0] sum w, [1..3] the scalars of cg
  double* part = at<double>(c.ws, opart);
  const int64_t R = 2 * B;
  const unsigned gp = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(P, 256), 4096));
  const unsigned gr = (unsigned)std::min<int64_t>(R * kSeg, 16384);
  hipLaunchKernelGGL(k_sr_wsum, dim3(1), dim3(kT), 0, stream, weights, B, sc);
  hipLaunchKernelGGL(k_sr_center, dim3(gp, 2), dim3(kT), 0, stream, jac, B, P, weights, sc);
  TDO_HIP(hipGetLastError());
  return cg(P, grad, iters, x, r, p, Ap, part, sc + 1, info, stream, [&](const double* v, double* Av) -> int32_t {
    hipLaunchKernelGGL(k_sr_rows, dim3(gr), dim3(kT), 0, stream, jac, R, P, v, up);
    hipLaunchKernelGGL(k_sr_cols, dim3(gp), dim3(kT), 0, stream, jac, R, P, up, v, lambda, Av);
    return TDO_OK;
  });
}

// S p = Re sum_b w_b conj(dO_b) (dO_b . p) with t_b = O_b . p from the forward-mode pass:
// sum_b w_b t_b conj... = J^T J p is the reverse-mode product with the seeds w_b (t_b - mean_w t)
// (the mean term vanishes against the centring of O).
extern "C" int32_t tdo_sr_solve_matfree(tdo_ctx_t* ctx, const tdo_arch_t* arch, const float* params, int32_t n,
                                        const uint64_t* cfg, int64_t B, const double* weights, tdo_prec_t prec,
                                        const double* grad, double lambda, int32_t iters, double* x, double* info,
                                        hipStream_t stream) {
  clear_error();
  TDO_CHECK(ctx != nullptr, TDO_EINVAL, "ctx is NULL");
  TDO_CHECK(prec == TDO_FP32 || prec == TDO_BF16, TDO_EINVAL, "unknown precision %d", (int)prec);
  NetPlan npj, npv;
  TDO_TRY(jvp_check(ctx->c, arch, n, B, &npj));
  TDO_TRY(net_plan(&ctx->c, arch, n, prec == TDO_BF16, &npv));
  TDO_CHECK(B >= 1, TDO_EINVAL, "B=%lld < 1", (long long)B);
  TDO_CHECK(lambda > 0.0 && std::isfinite(lambda), TDO_EINVAL, "diagonal shift lambda=%g must be positive", lambda);
  TDO_CHECK(iters >= 0, TDO_EINVAL, "iters=%d < 0", iters);
  TDO_CHECK(params && cfg && grad && x, TDO_EINVAL, "NULL buffer");
  TDO_HIP(hipSetDevice(ctx->c.device));
  Context& c = ctx->c;
  WsOrder order;
  TDO_TRY(order.begin(&c, stream));
  TDO_TRY(check_params_finite(&c, params, npj.pp.nparams, stream));
  const int64_t P = npj.pp.nparams;
  // CG vectors and scalars, the per-sample tangents and seeds, the forward-mode buffers (at most a third
  // of the rest of the budget, less where the reverse mode would not fit), then the reverse-mode plan in
  // what remains
  Arena ar;
  const size_t or_ = ar.take<double>((size_t)P), op = ar.take<double>((size_t)P), oap = ar.take<double>((size_t)P);
  const size_t osc = ar.take<double>(16), opart = ar.take<double>(kDotParts);
  const size_t ot = ar.take<float>(2 * (size_t)B), oseed = ar.take<float>(2 * (size_t)B);
  TDO_CHECK(c.budget > ar.used + 4096, TDO_ENOMEM, "workspace budget %zu too small", c.budget);
  JvpWs j;
  TrainWs t;
  const Arena vectors = ar;
  for (size_t most = (c.budget - ar.used) / 3;; most = std::max(most / 2, jvp_min_bytes(npj))) {
    ar = vectors;
    TDO_TRY(plan_jvp(npj, B, most, ar, &j));
    const int32_t rc = plan_train_at(c, npv, B, 1, ar.used, c.budget, &t);
    if (rc == TDO_OK) break;
    if (rc != TDO_ENOMEM || most <= jvp_min_bytes(npj)) return rc;
  }
  clear_error();
  TDO_TRY(ensure_workspace(&c, t.total));
  void* ws = c.ws;
  double *r = at<double>(ws, or_), *p = at<double>(ws, op), *Ap = at<double>(ws, oap), *sc = at<double>(ws, osc);
  double* part = at<double>(ws, opart);
  float *tv = at<float>(ws, ot), *seed = at<float>(ws, oseed);
  const unsigned gp = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(P, 256), 4096));
  const unsigned gb = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(B, 256), 4096));
  {  // the reverse-mode weight fragments, packed once
    NetWeights w = weights_at(ws, t.woff);
    TDO_TRY(pack_weights(npv, params, &w, stream, at<char>(ws, t.wback)));
  }
  // sc: [0..2] weight sum and weighted tangent sums, [3..5] the scalars of cg
  return cg(P, grad, iters, x, r, p, Ap, part, sc + 3, info, stream, [&](const double* v, double* Av) -> int32_t {
    TDO_TRY(run_jvp(npj, ws, j, params, v, cfg, B, tv, stream));
    hipLaunchKernelGGL(k_mf_mean, dim3(1), dim3(kT), 0, stream, tv, weights, B, sc);
    hipLaunchKernelGGL(k_mf_seeds, dim3(gb), dim3(256), 0, stream, tv, weights, B, sc, seed);
    TDO_HIP(hipGetLastError());
    TDO_TRY(vjp_run(c, npv, t, params, cfg, B, seed, Av, true, stream));
    hipLaunchKernelGGL(k_mf_shift, dim3(gp), dim3(256), 0, stream, P, lambda, v, Av);
    return TDO_OK;
  });
}
