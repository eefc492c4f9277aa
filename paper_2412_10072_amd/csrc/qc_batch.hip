// Batched solve of many independent calibration problems of uneven size in
// one persistent launch per size bucket, captured in a hipGraph.
//
// Work unit: one solution interval of one problem (intervals are independent,
// paper Section 2.3, so problems and intervals mix freely).  The host sorts
// the intervals into buckets by channel width (which fixes the rows-per-step
// tile) and by size, largest first inside a bucket (longest-processing-time
// order).  For each bucket a persistent kernel with one workgroup per
// resident slot pulls interval indices from a device counter and runs the
// per-interval Gauss-Newton loop (solve_interval) on each until the bucket's
// queue is empty, so every workgroup reaches the exit.  The bucket kernels
// run on parallel branches of one graph.
//
// Schedule: each bucket has (waves per workgroup, rows per step), by default 8
// (4 for a bucket of many intervals) and 4; qc_batch_tune times every candidate
// on the batch itself and keeps the fastest per bucket.  Intervals much larger
// than the rest go to teams of workgroups instead (k_batch_team).

#include <algorithm>
#include <cstring>
#include <vector>

#include "qc_batch.h"
#include "qc_interval.h"

namespace qc {
namespace {

// LM: Levenberg-Marquardt damping for every problem of the batch (kernels of
// their own, as for the single-problem path).  WARM: some problem carries a
// warm-start fallback reference.  Then an interval whose warm start fits
// worse than unit gains returns from its first pass, and this kernel writes
// unit gains and solves it again without the reference.  The item and its
// problem are read as wave-uniform copies: with the problem's pointers and
// sizes in vector registers the MIXED kernel took 160 VGPRs (the warm one
// 168 with spills, LM 239) against 132 (148, 156), and the batch graph at
// six updates 282 against 228 ms.  The MIXED warm kernels stay held to three
// wavefronts per SIMD.
template <typename S, typename T, int RPS, bool LM, bool WARM>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(WARM && !LM && sizeof(T) == 4 ? 3 : 1)))
k_solve_batch(BatchArgs B) {
  __shared__ int s_next;
  __shared__ int s_restart;
  for (;;) {
    if (threadIdx.x == 0) s_next = atomicAdd(B.queue, 1);
    __syncthreads();
    const int k = s_next;
    __syncthreads();
    if (k >= B.n_items) break;
    const BatchItem I = uniform_copy(B.items + B.item_begin + k);
    const BatchProb P = uniform_copy(B.probs + I.prob);
    Job J;
    J.V = &P.vis;
    J.CH = nullptr;
    J.TA = &P.term;
    J.gains = P.gains;
    J.params = nullptr;
    J.gflags = P.gflags;
    J.iters = P.iters;
    J.converged = P.converged;
    J.chisq_first = P.chisq_first;
    J.chisq_last = P.chisq_last;
    J.gt = I.gt;
    J.gf = I.gf;
    J.n_gf = P.term.n_gf;
    J.r_lo = I.r_lo;
    J.r_hi = I.r_hi;
    J.c_lo = I.c_lo;
    J.c_hi = I.c_hi;
    J.tol = B.tol;
    J.max_iter = B.max_iter;
    J.damping = P.damping;
    J.err = B.err;
    J.chisq_ref = WARM ? P.chisq_ref : nullptr;
    J.restarted = P.restarted;
    J.partial = nullptr;
    J.otab = nullptr;
    J.sky = nullptr;
    J.restart_flag = &s_restart;
    J.n_dd = -1;
    constexpr int RST = WARM ? 1 : 0;
    for (int attempt = 0;; ++attempt) {
      if constexpr (WARM) {
        if (threadIdx.x == 0) s_restart = 0;
        __syncthreads();
      }
      // FP64 full-Jones intervals load their next chunk during the current
      // one's work, except in the warm kernel, which would spill with it
      // (FP64 batch graph about 620 -> 540 ms)
      if (P.term.kind == KIND_DIAG) solve_interval<KIND_DIAG, S, T, CHAIN_SINGLE, 1, RPS, false, LM, false, RST, false>(J);
      else solve_interval<KIND_C2X2, S, T, CHAIN_SINGLE, 1, RPS, false, LM, false, RST, !WARM>(J);
      if constexpr (!WARM) break;
      const bool again = s_restart != 0;        // uniform: set before a barrier in the solve
      __syncthreads();                          // read by every thread before it is reset
      if (!again) {
        if (attempt > 0 && threadIdx.x == 0 && P.restarted)
          P.restarted[I.gt * P.term.n_gf + I.gf] = 1;
        break;
      }
      // unit gains for this interval, then the solve again without the reference
      double2* g = P.gains + ((size_t)I.gt * P.term.n_gf + I.gf) * P.vis.n_ant * 4;   // one gain direction
      for (int i = threadIdx.x; i < P.vis.n_ant * 4; i += blockDim.x) {
        const int k = i & 3;
        g[i] = make_double2((k == 0 || k == 3) ? 1.0 : 0.0, 0.0);
      }
      __syncthreads();
      J.chisq_ref = nullptr;
    }
  }
}

// Intervals too large for one workgroup: teams.
//
// A lone workgroup streams an interval at about 10 GB/s, so in a batch of
// uneven problems the largest intervals run long after the rest is done (24
// problems of 5 GB in all: one of 12 wide intervals took 38 of the 50 ms).
// Here an interval's rows are cut into parts that any workgroup may take.  A
// workgroup claims an open part (of the item it worked on last, else of the
// next one that has any), streams it at the current gains and writes its FP64
// block.  The workgroup that completes a group of TEAM_GROUP parts adds the
// group, and the one that completes the item's groups adds those, in index
// order, updates the gains and opens the next pass, so sums do not depend on
// timing, and no pass needs the host or a launch.  A workgroup without a part
// waits only while some item is neither done nor fully claimed by running
// workgroups: every claimed part is being streamed, and an item ends after at
// most max_iter + 1 passes, so every wait ends however many workgroups are
// resident.
template <int KIND, typename S, typename T>
__device__ __forceinline__ bool team_part(const Job& J, const TeamArgs& A, const TeamItem& I, TeamWords* words, int part,
                                          int pass, int* s_last) {
  constexpr int NV = nv_of<KIND, false>();
  const int tid = threadIdx.x;
  const size_t stride = (size_t)J.V->n_ant * NV + 1;
  double* parts = A.parts + I.part_off;
  Job P = J;
  const long long n = I.it.r_hi - I.it.r_lo;
  P.r_lo = I.it.r_lo + (n * part) / I.n_part;
  P.r_hi = I.it.r_lo + (n * (part + 1)) / I.n_part;
  P.partial = parts + (size_t)part * stride;
  solve_interval<KIND, S, T, CHAIN_SINGLE, 1, 4, true, false, false, 2, true>(P);
  team_release();                              // the part, before it is counted
  const int g = part / TEAM_GROUP, g0 = g * TEAM_GROUP;
  const int g_parts = min(TEAM_GROUP, I.n_part - g0);
  if (tid == 0) *s_last = (atomicAdd(&words->parts[g], 1) + 1) % g_parts == 0;
  __syncthreads();
  if (!*s_last) return false;
  const double* src = parts;
  int n_src = I.n_part;
  if (I.n_group > 1) {
    double* sums = parts + (size_t)I.n_part * stride;
    for (size_t i = tid; i < stride; i += blockDim.x) {
      double x = 0.0;
      for (int k = g0; k < g0 + g_parts; ++k) x += ld_shared<true>(parts + (size_t)k * stride + i);
      st_shared<true>(sums + (size_t)g * stride + i, x);
    }
    team_release();
    if (tid == 0) *s_last = (atomicAdd(&words->groups, 1) + 1) % I.n_group == 0;
    __syncthreads();
    if (!*s_last) return false;
    src = sums;
    n_src = I.n_group;
  }
  const bool done = split_update_at<KIND, T, 1, false, true>(J, src, n_src, A.dv + I.dv_off, pass, nullptr);
  team_release();                              // the gains, before the next pass opens
  if (tid == 0 && !done) st_shared<true>(&words->next, (unsigned long long)(pass + 1) << 32);
  return done;
}

// An open part of some item, by one wavefront: 64 items are looked at together,
// from `from` on, and an open one's part is taken by one addition (a
// compare-and-swap had hundreds of waiting workgroups repeat it for each part
// of a pass that opened: 480 us a pass for 6 items of a few parts).  Returns the
// item, pass and part; -1 when every item is done.
__device__ __forceinline__ int team_claim(const TeamArgs& A, int from, int lane, int& pass, int& part) {
  for (;;) {
    for (int base = 0; base < A.n_items; base += 64) {
      const bool in = base + lane < A.n_items;
      int idx = from + base + lane;
      if (idx >= A.n_items) idx -= A.n_items;
      if (!in) idx = 0;
      TeamWords* w = A.words + idx;
      const unsigned n_part = (unsigned)A.items[idx].n_part;
      const unsigned next = (unsigned)ld_shared<true>(&w->next);
      unsigned long long mask = __ballot(in && next < n_part);
      while (mask) {
        const int l = __ffsll(mask) - 1;
        unsigned long long got = 0;
        if (lane == l) got = atomicAdd(&w->next, 1ull);
        const unsigned mine = (unsigned)__shfl((int)(unsigned)got, l);
        if (mine < (unsigned)__shfl((int)n_part, l)) {
          part = (int)mine;
          pass = __shfl((int)(unsigned)(got >> 32), l);
          return __shfl(idx, l);
        }
        mask &= mask - 1;
      }
    }
    if (ld_shared<true>(&A.words[A.n_items].groups) >= A.n_items) return -1;
    __builtin_amdgcn_s_sleep(64);
  }
}

template <typename S, typename T>
__global__ void __launch_bounds__(256) k_batch_team(TeamArgs A) {
  __shared__ int s_item, s_pass, s_part, s_last;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int from = (int)((long long)blockIdx.x * A.n_items / gridDim.x);
  for (;;) {
    if (wave == 0) {
      int pass = 0, part = 0;
      const int k = team_claim(A, from, lane, pass, part);
      if (lane == 0) {
        s_item = k;
        s_pass = pass;
        s_part = part;
      }
    }
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(s_item);
    const int pass = __builtin_amdgcn_readfirstlane(s_pass), part = __builtin_amdgcn_readfirstlane(s_part);
    __syncthreads();
    if (item < 0) break;
    from = item;
    const TeamItem I = uniform_copy(A.items + item);
    const BatchProb P = uniform_copy(A.probs + I.it.prob);
    Job J;
    J.V = &P.vis;
    J.CH = nullptr;
    J.TA = &P.term;
    J.gains = P.gains;
    J.params = nullptr;
    J.gflags = P.gflags;
    J.iters = P.iters;
    J.converged = P.converged;
    J.chisq_first = P.chisq_first;
    J.chisq_last = P.chisq_last;
    J.gt = I.it.gt;
    J.gf = I.it.gf;
    J.n_gf = P.term.n_gf;
    J.c_lo = I.it.c_lo;
    J.c_hi = I.it.c_hi;
    J.r_lo = I.it.r_lo;
    J.r_hi = I.it.r_hi;
    J.tol = A.tol;
    J.max_iter = A.max_iter;
    J.damping = P.damping;
    J.err = A.err;
    J.chisq_ref = nullptr;
    J.restarted = P.restarted;
    J.partial = nullptr;
    J.otab = nullptr;
    J.sky = nullptr;
    J.restart_flag = nullptr;
    J.n_dd = -1;
    TeamWords* words = A.words + item;
    bool done;
    if (P.term.kind == KIND_DIAG) done = team_part<KIND_DIAG, S, T>(J, A, I, words, part, pass, &s_last);
    else done = team_part<KIND_C2X2, S, T>(J, A, I, words, part, pass, &s_last);
    if (done && threadIdx.x == 0) atomicAdd(&A.words[A.n_items].groups, 1);
    __syncthreads();                           // s_last is read by every thread before it is set again
  }
}

__global__ void k_team_reset(int n_items, TeamWords* words) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i <= n_items) words[i] = TeamWords{};
}

__global__ void k_zero_ints(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

template <typename S, typename T, bool LM, bool WARM>
void* batch_kernel(int rps) {
  if (rps == 4) return reinterpret_cast<void*>(k_solve_batch<S, T, 4, LM, WARM>);
  if (rps == 2) return reinterpret_cast<void*>(k_solve_batch<S, T, 2, LM, WARM>);
  return reinterpret_cast<void*>(k_solve_batch<S, T, 1, LM, WARM>);
}

template <bool LM, bool WARM>
void* batch_kernel_prec(int prec_mixed, int vis_c128, int rps) {
  if (prec_mixed) return batch_kernel<float, float, LM, WARM>(rps);
  if (vis_c128) return batch_kernel<double, double, LM, WARM>(rps);
  return batch_kernel<float, double, LM, WARM>(rps);
}

}  // namespace

void* batch_kernel_ptr(int prec_mixed, int vis_c128, int rps, int lm, int warm) {
  if (lm) return warm ? batch_kernel_prec<true, true>(prec_mixed, vis_c128, rps)
                      : batch_kernel_prec<true, false>(prec_mixed, vis_c128, rps);
  return warm ? batch_kernel_prec<false, true>(prec_mixed, vis_c128, rps)
              : batch_kernel_prec<false, false>(prec_mixed, vis_c128, rps);
}

size_t batch_lds_bytes(int prec_mixed, int max_ant, int waves) {
  // the full-Jones term needs the most LDS per antenna
  if (prec_mixed) return interval_lds_bytes<KIND_C2X2, float, 1>(max_ant, waves);
  return interval_lds_bytes<KIND_C2X2, double, 1>(max_ant, waves);
}

hipError_t launch_batch_bucket(const BatchArgs& B, void* kern, int waves, size_t lds, int grid, hipStream_t s) {
  if (B.n_items <= 0) return hipSuccess;
  void* args[] = {const_cast<BatchArgs*>(&B)};
  return hipLaunchKernel(kern, dim3(grid), dim3(64 * waves), args, lds, s);
}

void* team_kernel_ptr(int prec_mixed, int vis_c128) {
  if (prec_mixed) return reinterpret_cast<void*>(k_batch_team<float, float>);
  if (vis_c128) return reinterpret_cast<void*>(k_batch_team<double, double>);
  return reinterpret_cast<void*>(k_batch_team<float, double>);
}

// the larger of a pass of 4 wavefronts and an update with its divergence state
size_t team_lds_bytes(int prec_mixed, int max_ant) {
  const size_t dv = sizeof(double) * 2 * (size_t)max_ant;
  if (prec_mixed)
    return std::max(interval_lds_bytes<KIND_C2X2, float, 1>(max_ant, 4), team_dv_off<KIND_C2X2, float>(max_ant) + dv);
  return std::max(interval_lds_bytes<KIND_C2X2, double, 1>(max_ant, 4), team_dv_off<KIND_C2X2, double>(max_ant) + dv);
}

hipError_t launch_batch_team(const TeamArgs& A, void* kern, size_t lds, int grid, hipStream_t s) {
  if (A.n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_team_reset, dim3(A.n_items / 256 + 1), dim3(256), 0, s, A.n_items, A.words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  void* args[] = {const_cast<TeamArgs*>(&A)};
  return hipLaunchKernel(kern, dim3(grid), dim3(256), args, lds, s);
}

hipError_t launch_zero_ints(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_ints, dim3((n + 63) / 64), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace qc
