// Robust reweighting between solver epochs (paper Section 4.3, solver
// features: reweighting after Sob et al. 2020, which keeps calibration from
// fitting RFI and unmodelled emission), as the expectation step of a complex
// Student's t noise model: a weight shared by D complex correlations (D = 1
// with a weight per correlation, 4 with one per sample) becomes
//   w = w0 (nu + D) / (nu + w0 sum_k |r_k|^2 / s2),
// s2 the mean of w0 |r|^2 over every complex residual value of the unflagged
// cross-correlation samples with a finite residual.  Other samples keep w0.
//
// Two HBM-bound passes over the residual and the weights: per-workgroup FP64
// partial sums over a fixed grid (rows strided over the wavefronts, lanes
// over channels, fixed-order reductions: the result does not depend on
// scheduling), one workgroup adds the partials in order, then the weights.

#include <cmath>

#include "qc_internal.h"
#include "qc_host.h"

namespace qc {
namespace {

constexpr int RW_BLOCKS = 1024;       // fixed grid of the partial sums
constexpr int RW_THREADS = 256;

// w0 |r|^2 of correlation k of sample s, and whether the sample takes part
template <typename S>
__device__ __forceinline__ void sample_terms(const VisArgs& V, const S* R, const S* W, size_t s, double e[4],
                                             double w0[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double re = (double)R[8 * s + 2 * k], im = (double)R[8 * s + 2 * k + 1];
    w0[k] = (double)W[V.n_wcorr == 4 ? 4 * s + k : s];
    e[k] = w0[k] * (re * re + im * im);
  }
}

template <typename S>
__global__ void __launch_bounds__(RW_THREADS) k_rw_partial(VisArgs V, const S* R, double* part_sum,
                                                            unsigned long long* part_n) {
  __shared__ double s_sum[RW_THREADS / 64];
  __shared__ unsigned long long s_n[RW_THREADS / 64];
  const S* W = reinterpret_cast<const S*>(V.weight);
  const int lane = threadIdx.x & 63;
  const long long wave0 = (long long)blockIdx.x * (RW_THREADS / 64) + (threadIdx.x >> 6);
  const long long n_wave = (long long)gridDim.x * (RW_THREADS / 64);
  double acc = 0.0;
  unsigned long long n = 0;
  for (long long r = wave0; r < V.n_row; r += n_wave) {
    if (V.ant1[r] == V.ant2[r]) continue;            // uniform over the wavefront
    for (int c = lane; c < V.n_chan; c += 64) {
      const size_t s = (size_t)r * V.n_chan + c;
      double e[4], w0[4];
      sample_terms<S>(V, R, W, s, e, w0);
      const double tot = ((e[0] + e[1]) + e[2]) + e[3];
      if (V.flag[s] == 0 && isfinite(tot)) {
        acc += tot;
        n += 4;
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    acc += __shfl_xor(acc, o);
    n += __shfl_xor(n, o);
  }
  if (lane == 0) {
    s_sum[threadIdx.x >> 6] = acc;
    s_n[threadIdx.x >> 6] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    unsigned long long m = 0;
    for (int k = 0; k < RW_THREADS / 64; ++k) {
      t += s_sum[k];
      m += s_n[k];
    }
    part_sum[blockIdx.x] = t;
    part_n[blockIdx.x] = m;
  }
}

// s2 = (sum of the partials, a fixed tree) / (their count); out[1] = count.  One
// workgroup, a thread per partial (one thread adding all 1024 took 77 us).
__global__ void __launch_bounds__(RW_BLOCKS) k_rw_final(const double* part_sum, const unsigned long long* part_n,
                                                        double* out) {
  __shared__ double s_sum[RW_BLOCKS];
  __shared__ unsigned long long s_n[RW_BLOCKS];
  const int i = threadIdx.x;
  s_sum[i] = part_sum[i];
  s_n[i] = part_n[i];
  __syncthreads();
  for (int o = RW_BLOCKS / 2; o > 0; o >>= 1) {
    if (i < o) {
      s_sum[i] += s_sum[i + o];
      s_n[i] += s_n[i + o];
    }
    __syncthreads();
  }
  if (i == 0) {
    out[0] = s_n[0] > 0 ? s_sum[0] / (double)s_n[0] : 0.0;
    out[1] = (double)s_n[0];
  }
}

// w0 (nu + D) / (nu + e / s2) as w0 ((nu + D) s2 / (nu s2 + e)): one FP64 division
// per weight instead of two; with whole-sample reads and writes the pass over
// 1.03e8 samples of four weights (6.7 GB) went from 1.46 to 1.27 ms.  Where s2 or nu is so large or small that
// the products could leave the range, the two divisions (`wide`, the same for
// every sample).
struct RobustRule {
  double nu, s2, nus2, num1, num4;
  bool wide;
  __device__ __forceinline__ RobustRule(double n, double s) : nu(n), s2(s) {
    wide = !(s > 1e-100 && s < 1e100 && n > 1e-100 && n < 1e100);
    nus2 = n * s;
    num1 = (n + 1.0) * s;
    num4 = (n + 4.0) * s;
  }
  template <int D>
  __device__ __forceinline__ double weight(double w0, double e) const {
    if (wide) return w0 * (nu + D) / (nu + e / s2);
    return w0 * ((D == 1 ? num1 : num4) / (nus2 + e));
  }
};

// VEC: residual, weights and output are aligned for four values at a time (the
// host looks); two steps of a row are then read before the first is written.
template <typename S, bool VEC>
__global__ void __launch_bounds__(RW_THREADS) k_rw_apply(VisArgs V, const S* R, double nu, const double* s2n,
                                                          S* out) {
  using V4 = S __attribute__((ext_vector_type(4)));
  constexpr int U = VEC ? 2 : 1;
  const S* W = reinterpret_cast<const S*>(V.weight);
  const bool any = s2n[1] > 0.0;
  const RobustRule rule(nu, s2n[0]);
  const int lane = threadIdx.x & 63;
  const long long wave0 = (long long)blockIdx.x * (RW_THREADS / 64) + (threadIdx.x >> 6);
  const long long n_wave = (long long)gridDim.x * (RW_THREADS / 64);
  for (long long r = wave0; r < V.n_row; r += n_wave) {
    const bool cross = V.ant1[r] != V.ant2[r];
    for (int c0 = lane; c0 < V.n_chan; c0 += 64 * U) {
      V4 x[U][2], w[U];
      uint8_t f[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const size_t s = (size_t)r * V.n_chan + min(c0 + 64 * u, V.n_chan - 1);
        f[u] = V.flag[s];
        if constexpr (VEC) {
          x[u][0] = reinterpret_cast<const V4*>(R)[2 * s];
          x[u][1] = reinterpret_cast<const V4*>(R)[2 * s + 1];
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) x[u][k / 4][k % 4] = R[8 * s + k];
        }
        if (V.n_wcorr == 4) {
          if constexpr (VEC) {
            w[u] = reinterpret_cast<const V4*>(W)[s];
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) w[u][k] = W[4 * s + k];
          }
        } else {
          const S w0 = W[s];
          w[u] = V4{w0, w0, w0, w0};
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + 64 * u;
        if (c >= V.n_chan) break;
        const size_t s = (size_t)r * V.n_chan + c;
        double e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double re = (double)x[u][k / 2][2 * (k % 2)], im = (double)x[u][k / 2][2 * (k % 2) + 1];
          e[k] = (double)w[u][k] * (re * re + im * im);
        }
        const double tot = ((e[0] + e[1]) + e[2]) + e[3];
        const bool use = any && cross && f[u] == 0 && isfinite(tot);
        if (V.n_wcorr == 4) {
          V4 o;
#pragma unroll
          for (int k = 0; k < 4; ++k) o[k] = use ? (S)rule.template weight<1>((double)w[u][k], e[k]) : w[u][k];
          if constexpr (VEC) {
            reinterpret_cast<V4*>(out)[s] = o;
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) out[4 * s + k] = o[k];
          }
        } else {
          out[s] = use ? (S)rule.template weight<4>((double)w[u][0], tot) : w[u][0];
        }
      }
    }
  }
}

template <typename S>
void launch_rw(const VisArgs& V, const void* resid, double nu, double* part_sum, unsigned long long* part_n,
               double* s2n, void* out, hipStream_t s) {
  const S* R = reinterpret_cast<const S*>(resid);
  hipLaunchKernelGGL(k_rw_partial<S>, dim3(RW_BLOCKS), dim3(RW_THREADS), 0, s, V, R, part_sum, part_n);
  hipLaunchKernelGGL(k_rw_final, dim3(1), dim3(RW_BLOCKS), 0, s, (const double*)part_sum,
                     (const unsigned long long*)part_n, s2n);
  long long blocks = (V.n_row + 3) / 4;
  if (blocks > 256 * 64) blocks = 256 * 64;
  if (blocks < 1) blocks = 1;
  const uintptr_t at = reinterpret_cast<uintptr_t>(resid) | reinterpret_cast<uintptr_t>(out) |
                       reinterpret_cast<uintptr_t>(V.weight);
  const dim3 g((unsigned)blocks), b(RW_THREADS);
  if (at % (4 * sizeof(S)) == 0)
    hipLaunchKernelGGL((k_rw_apply<S, true>), g, b, 0, s, V, R, nu, (const double*)s2n, reinterpret_cast<S*>(out));
  else
    hipLaunchKernelGGL((k_rw_apply<S, false>), g, b, 0, s, V, R, nu, (const double*)s2n, reinterpret_cast<S*>(out));
}

}  // namespace
}  // namespace qc

using namespace qc;

extern "C" {

qc_status qc_robust_weights(qc_ctx* ctx, const qc_vis* vis, const void* resid, double nu, void* weight_out,
                            double* s2_out, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!(nu > 0.0) || !std::isfinite(nu)) return fail(ctx, QC_E_ARG, "nu must be finite and > 0");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  qc_status st = validate_rows(ctx, vis, s);
  if (st != QC_OK) return st;
  if (vis->n_row > 0 && (!resid || !weight_out)) return fail(ctx, QC_E_ARG, "resid or weight_out is NULL");
  HIP_TRY(ctx, grow(ctx->d_rw, ctx->rw_cap, (size_t)RW_BLOCKS * 2 + 2));
  double* part_sum = ctx->d_rw;
  unsigned long long* part_n = reinterpret_cast<unsigned long long*>(ctx->d_rw + RW_BLOCKS);
  double* s2n = ctx->d_rw + 2 * RW_BLOCKS;
  VisArgs V;
  ChainArgs ca;
  fill_args(vis, nullptr, 0, -1, V, ca);
  HIP_TRY(ctx, hipEventRecord(ctx->ev0, s));
  if (vis->dtype == QC_C64)
    launch_rw<float>(V, resid, nu, part_sum, part_n, s2n, weight_out, s);
  else
    launch_rw<double>(V, resid, nu, part_sum, part_n, s2n, weight_out, s);
  HIP_TRY(ctx, hipGetLastError());
  HIP_TRY(ctx, call_end(ctx, s));
  if (s2_out) {
    double h[2] = {0.0, 0.0};
    HIP_TRY(ctx, hipMemcpyAsync(h, s2n, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_TRY(ctx, hipStreamSynchronize(s));
    *s2_out = h[1] > 0.0 ? h[0] : NAN;
  }
  return QC_OK;
}

}  // extern "C"
