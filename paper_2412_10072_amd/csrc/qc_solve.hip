// The solve launch of libqc: the fixed-factor table of diagonal chains and
// the dispatch of a solve to the kernels of its term kind and precision
// (qc_solve_kernels.h, instantiated in the qc_solve_k*.hip units).

#include <algorithm>

#include "qc_interval.h"

namespace qc {

template <int KIND, typename S, typename T>
hipError_t launch_solve_kind(const SolveLaunch& L, const SplitLaunch* P, hipStream_t stream, size_t* lds_out);

namespace {

// Fixed direction-independent factors of a diagonal chain: for every time,
// antenna and channel, the product of the diagonals of the terms with one
// gain direction other than the active one (diagonal matrices commute, so
// the position of the active term does not matter).  One workgroup per
// (time, antenna), lanes over channels.
template <typename T>
__global__ void __launch_bounds__(256) k_chain_table(SolveLaunch L, cx<T>* out) {
  const ChainArgs& CH = L.chain;
  const int n_ant = L.vis.n_ant, n_chan = L.vis.n_chan;
  const int t = blockIdx.x / n_ant;
  const int a = blockIdx.x - t * n_ant;
  for (int c = threadIdx.x; c < n_chan; c += blockDim.x) {
    const double nu = L.vis.freq[c];
    cx<T> h0 = cone<T>(), h1 = cone<T>();
    for (int j = 0; j < CH.n_term; ++j) {
      if (j == CH.active || CH.t[j].n_gdir > 1) continue;
      const m22<T> J = term_jones<T>(CH.t[j], n_ant, t, c, a, 0, nu);
      h0 = h0 * J.a;
      h1 = h1 * J.d;
    }
    const size_t o = (((size_t)t * n_ant + a) * n_chan + c) * 2;
    out[o] = h0;
    out[o + 1] = h1;
  }
}

// Steps of every part: a wavefront per 64-row window of a part (windows start
// at the part's first row, so every window starts a run); within a window a
// run of equal (time, p) is cut into steps of `rows` rows from its first row.
__global__ void __launch_bounds__(64) k_band_steps(VisArgs V, const long long* row_lo, const long long* row_hi,
                                                   int n_part, int windows, int rows, BandStep* steps) {
  const int lane = threadIdx.x;
  const int w = blockIdx.x % windows;
  const int rest = blockIdx.x / windows;
  const int part = rest % n_part;
  const int gt = rest / n_part;
  const long long lo = row_lo[gt], n = row_hi[gt] - lo;
  const long long r_lo = lo + (n * part) / n_part, r_hi = lo + (n * (part + 1)) / n_part;
  const long long r = r_lo + (long long)w * 64 + lane;
  const bool in = r < r_hi;
  const int t = in ? V.row_time[r] : -1;
  const int p = in ? V.ant1[r] : -1;
  const int q = in ? V.ant2[r] : -1;
  const int t_up = __shfl_up(t, 1), p_up = __shfl_up(p, 1);
  int qs[BAND_MAX_ROWS];     // q of the next rows (those past the run are not read: g < k)
  qs[0] = q;
#pragma unroll
  for (int g = 1; g < BAND_MAX_ROWS; ++g) qs[g] = __shfl_down(q, g);
  const bool head = in && (lane == 0 || t_up != t || p_up != p);
  const unsigned long long heads = __ballot(head);
  const unsigned long long ins = __ballot(in);
  if (!in) return;
  // first row of this lane's run, and the row after it
  const unsigned long long upto = (2ull << lane) - 1;     // lanes 0..lane (all 64 for lane 63)
  const int run0 = 63 - __clzll(heads & upto);
  const unsigned long long above = heads & ~upto;
  const int n_in = __popcll(ins);
  const int run1 = above ? __ffsll(above) - 1 : n_in;
  if ((lane - run0) % rows != 0) return;
  BandStep s;
  s.k = min(rows, run1 - lane);
  s.t = t;
  s.p = p;
  int dup = 0;
#pragma unroll
  for (int g = 0; g < BAND_MAX_ROWS; ++g) {
    s.q[g] = (g < s.k && qs[g] != p) ? qs[g] : -1;
#pragma unroll
    for (int h = 0; h < g; ++h)
      if (s.q[g] >= 0 && s.q[g] == s.q[h]) dup = 1;
  }
  s.dup = dup;
  steps[r] = s;
}

// The parts of an interval added per value, the split schedule's step between
// a pass and the update: one workgroup per (interval, 64 values), its 16
// wavefronts each adding every 16th part (a 512-byte read per part), then the 16
// sums in order, so the order of the additions is fixed.  Bound by reading
// the partials once.  Done by the update's single workgroup per interval before,
// which read 472 parts of 1537 values (a direction-dependent term, 64 antennas x
// 4 directions) in 1169 us a pass.
constexpr int SR_WAVES = 16;
__global__ void __launch_bounds__(64 * SR_WAVES) k_split_reduce(const double* partials, int n_part, size_t stride,
                                                                int chunks, const uint8_t* done, double* totals) {
  __shared__ double part_sum[SR_WAVES][64];
  const int interval = blockIdx.x / chunks;
  const int chunk = blockIdx.x - interval * chunks;
  if (done[interval]) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t i = (size_t)chunk * 64 + lane;
  double sum = 0.0;
  if (i < stride) {
    const double* p = partials + (size_t)interval * n_part * stride + i;
#pragma unroll 4
    for (int k = wave; k < n_part; k += SR_WAVES) sum += p[(size_t)k * stride];
  }
  part_sum[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && i < stride) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < SR_WAVES; ++w) t += part_sum[w][lane];
    totals[(size_t)interval * stride + i] = t;
  }
}

// Direction-dependent fixed term j (diagonal gains) by model direction: entry
// ((g * n_ant + a) * n_dir + d) * 2 + hand, g = gain time * n_gf + gain
// frequency.  One workgroup per (gain block, antenna), lanes over directions.
template <typename T>
__global__ void __launch_bounds__(64) k_dd_table(TermArgs tm, int n_ant, int n_dir, cx<T>* out) {
  const int a = blockIdx.x % n_ant;
  const size_t gb = blockIdx.x / n_ant;
  for (int d = threadIdx.x; d < n_dir; d += blockDim.x) {
    const size_t blk = (gb * n_ant + a) * tm.n_gdir + tm.d_map[d];
    const double2 g0 = tm.gains[4 * blk], g3 = tm.gains[4 * blk + 3];
    const size_t o = ((gb * n_ant + a) * n_dir + d) * 2;
    out[o] = cmake<T>((T)g0.x, (T)g0.y);
    out[o + 1] = cmake<T>((T)g3.x, (T)g3.y);
  }
}

// A diagonal chain with one gain direction, folded into one model: while a term
// is solved the others stand still, so
//   E_ij = sum_d o_{p,d,i} M_d,ij conj(o_{q,d,j})
// (o the product of the fixed terms) is the same in every pass, and the solve
// over E, one direction and the active term alone is the single-term solve.  This
// kernel writes E once; a pass then reads 81 bytes per sample instead of 81 +
// 32 (n_dir - 1) and two table entries, in the kernels of the single-term chain.
// Bound by streaming the model once (about one pass of the unfolded solve).
// Measured per solve with this kernel, 64 antennas, 60 times x 256 channels,
// MIXED: 4 directions, delays (13 updates) 18.3 -> 7.9 ms, gains per time (6) 9.0
// -> 4.5, bandpass (10) 15.8 -> 13.6; one direction, delays (14) 12.7 -> 8.0,
// gains 3.9 -> 3.8.
template <typename T, bool FLAT>
__global__ void __launch_bounds__(256) k_chain_fold(SolveLaunch L, T* out) {
  const VisArgs& V = L.vis;
  const ChainArgs& CH = L.chain;
  const T* Mp = reinterpret_cast<const T*>(V.model);
  const cx<T>* otab = reinterpret_cast<const cx<T>*>(L.otab);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n_dir = V.n_dir, n_ant = V.n_ant;
  auto sample = [&](size_t s, long long r, int c) {
    const int p = V.ant1[r], q = V.ant2[r], t = V.row_time[r];
    if ((unsigned)p >= (unsigned)n_ant || (unsigned)q >= (unsigned)n_ant) return;
    const double nu = V.freq[c];
    cx<T> op0 = cone<T>(), op1 = cone<T>(), oq0 = cone<T>(), oq1 = cone<T>();
    if (otab) {
      const cx<T>* tp = otab + (((size_t)t * n_ant + p) * V.n_chan + c) * 2;
      const cx<T>* tq = otab + (((size_t)t * n_ant + q) * V.n_chan + c) * 2;
      op0 = tp[0]; op1 = tp[1];
      oq0 = tq[0]; oq1 = tq[1];
    }
    const cx<T>* ddp[BAND_MAX_DD];
    const cx<T>* ddq[BAND_MAX_DD];
#pragma unroll
    for (int k = 0; k < BAND_MAX_DD; ++k) {
      ddp[k] = ddq[k] = nullptr;
      if (k < L.n_dd) {
        const TermArgs& tj = CH.t[L.dd_term[k]];
        const size_t g = (size_t)tj.t_map[t] * tj.n_gf + tj.f_map[c];
        const cx<T>* base = reinterpret_cast<const cx<T>*>(L.dd_tab[k]) + g * n_ant * n_dir * 2;
        ddp[k] = base + (size_t)p * n_dir * 2;
        ddq[k] = base + (size_t)q * n_dir * 2;
      }
    }
    // the model four directions at a time (one 128-byte line), the index
    // clamped so that the loads go out together
    constexpr int MCH = sizeof(T) == 4 ? 4 : 1;
    m22<T> E = mzero<T>();
    for (int d0 = 0; d0 < n_dir; d0 += MCH) {
      m22<T> Mc[MCH];
#pragma unroll
      for (int k = 0; k < MCH; ++k) Mc[k] = load_m22<T, T>(Mp, s * n_dir + min(d0 + k, n_dir - 1));
#pragma unroll
      for (int k = 0; k < MCH; ++k) {
        const int d = d0 + k;
        if (d >= n_dir) break;
        cx<T> rp0 = op0, rp1 = op1, rq0 = oq0, rq1 = oq1;
        if (L.dd_tabled) {
#pragma unroll
          for (int j = 0; j < BAND_MAX_DD; ++j) {
            if (j < L.n_dd) {
              rp0 = rp0 * ddp[j][2 * d];
              rp1 = rp1 * ddp[j][2 * d + 1];
              rq0 = rq0 * ddq[j][2 * d];
              rq1 = rq1 * ddq[j][2 * d + 1];
            }
          }
        } else {
          for (int j = 0; j < CH.n_term; ++j) {
            if (j == CH.active || CH.t[j].n_gdir <= 1) continue;
            const m22<T> Jp = term_jones<T>(CH.t[j], n_ant, t, c, p, d, nu);
            const m22<T> Jq = term_jones<T>(CH.t[j], n_ant, t, c, q, d, nu);
            rp0 = rp0 * Jp.a;
            rp1 = rp1 * Jp.d;
            rq0 = rq0 * Jq.a;
            rq1 = rq1 * Jq.d;
          }
        }
        E.a = cfma(mulc(rp0, rq0), Mc[k].a, E.a);
        E.b = cfma(mulc(rp0, rq1), Mc[k].b, E.b);
        E.c = cfma(mulc(rp1, rq0), Mc[k].c, E.c);
        E.d = cfma(mulc(rp1, rq1), Mc[k].d, E.d);
      }
    }
    if constexpr (sizeof(T) == 4) {
      float4* o = reinterpret_cast<float4*>(out) + 2 * s;
      o[0] = make_float4(E.a.re, E.a.im, E.b.re, E.b.im);
      o[1] = make_float4(E.c.re, E.c.im, E.d.re, E.d.im);
    } else {
      double2* o = reinterpret_cast<double2*>(out) + 4 * s;
      o[0] = make_double2(E.a.re, E.a.im);
      o[1] = make_double2(E.b.re, E.b.im);
      o[2] = make_double2(E.c.re, E.c.im);
      o[3] = make_double2(E.d.re, E.d.im);
    }
  };
  const long long first = (long long)blockIdx.x * 4 + wave, step = (long long)gridDim.x * 4;
  if constexpr (FLAT) {          // 64 samples as they lie in memory, over rows
    const long long n = V.n_row * V.n_chan;
    for (long long s0 = first * 64; s0 < n; s0 += step * 64) {
      const long long rb = s0 / V.n_chan;
      const unsigned off = (unsigned)(s0 - rb * V.n_chan) + lane;
      const unsigned dr = off / (unsigned)V.n_chan;
      if (s0 + lane < n) sample((size_t)(s0 + lane), rb + dr, (int)(off - dr * (unsigned)V.n_chan));
    }
  } else {
    for (long long r = first; r < V.n_row; r += step)
      for (int c = lane; c < V.n_chan; c += 64) sample((size_t)r * V.n_chan + c, r, c);
  }
}

template <typename T>
hipError_t launch_fold(const SolveLaunch& L, void* out, hipStream_t stream) {
  const long long n_row = L.vis.n_row, n_chan = L.vis.n_chan;
  if (n_row == 0 || n_chan == 0) return hipSuccess;
  const bool flat = flat_samples(n_chan);
  const long long steps = flat ? (n_row * n_chan + 63) / 64 : n_row;
  const dim3 g((unsigned)std::min<long long>((steps + 3) / 4, 256 * 64)), b(256);
  if (flat) hipLaunchKernelGGL((k_chain_fold<T, true>), g, b, 0, stream, L, reinterpret_cast<T*>(out));
  else hipLaunchKernelGGL((k_chain_fold<T, false>), g, b, 0, stream, L, reinterpret_cast<T*>(out));
  return hipGetLastError();
}

}  // namespace

size_t chain_fold_bytes(const SolveLaunch& L) {
  return (size_t)L.vis.n_row * L.vis.n_chan * 4 * (L.prec_mixed ? sizeof(cx<float>) : sizeof(cx<double>));
}

hipError_t launch_chain_fold(const SolveLaunch& L, void* out, hipStream_t stream) {
  if ((L.prec_mixed != 0) == (L.vis_is_c128 != 0)) return hipErrorInvalidValue;   // stored as computed
  return L.prec_mixed ? launch_fold<float>(L, out, stream) : launch_fold<double>(L, out, stream);
}

hipError_t launch_split_reduce(const SplitLaunch& P, int n_int, size_t stride, hipStream_t stream) {
  const int chunks = (int)((stride + 63) / 64);
  const long long grid = (long long)n_int * chunks;
  if (grid == 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_reduce, dim3((unsigned)grid), dim3(64 * SR_WAVES), 0, stream,
                     (const double*)P.partials, P.n_part, stride, chunks, (const uint8_t*)P.state.done, P.totals);
  return hipGetLastError();
}

size_t dd_table_bytes(const SolveLaunch& L, int j) {
  const TermArgs& tm = L.chain.t[j];
  const size_t elt = L.prec_mixed ? sizeof(cx<float>) : sizeof(cx<double>);
  return (size_t)tm.n_gt * tm.n_gf * L.vis.n_ant * L.vis.n_dir * 2 * elt;
}

hipError_t launch_dd_table(const SolveLaunch& L, int j, void* table, hipStream_t stream) {
  const TermArgs& tm = L.chain.t[j];
  const long long grid = (long long)tm.n_gt * tm.n_gf * L.vis.n_ant;
  if (grid == 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  if (L.prec_mixed)
    hipLaunchKernelGGL(k_dd_table<float>, dim3((unsigned)grid), dim3(64), 0, stream, tm, L.vis.n_ant, L.vis.n_dir,
                       reinterpret_cast<cx<float>*>(table));
  else
    hipLaunchKernelGGL(k_dd_table<double>, dim3((unsigned)grid), dim3(64), 0, stream, tm, L.vis.n_ant, L.vis.n_dir,
                       reinterpret_cast<cx<double>*>(table));
  return hipGetLastError();
}

size_t band_lds_bytes_for(int n_ant, int rows) {
  return sizeof(double) * (size_t)n_ant * KindInfo<KIND_DIAG>::NV * (64 / rows);
}

size_t band_gains_bytes(const SolveLaunch& L) {
  const TermArgs& ta = L.chain.t[L.chain.active];
  const size_t cw = 64 / L.band_rows, slices = (L.vis.n_chan + cw - 1) / cw;
  return (size_t)ta.n_gt * slices * cw * L.vis.n_ant * 2 * (L.prec_mixed ? sizeof(cx<float>) : sizeof(cx<double>));
}

hipError_t launch_band_steps(const SolveLaunch& L, int n_part, int rows, BandStep* steps, hipStream_t stream) {
  if (rows != 4 && rows != 8) return hipErrorInvalidValue;
  const TermArgs& ta = L.chain.t[L.chain.active];
  const long long rows_max = (L.vis.n_row + n_part - 1) / n_part + 1;   // rows of the largest part
  const int windows = (int)((rows_max + 63) / 64);
  const long long grid = (long long)ta.n_gt * n_part * windows;
  if (grid == 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_band_steps, dim3((unsigned)grid), dim3(64), 0, stream, L.vis, L.row_lo, L.row_hi, n_part,
                     windows, rows, steps);
  return hipGetLastError();
}

size_t chain_table_bytes(const SolveLaunch& L) {
  const size_t elt = L.prec_mixed ? sizeof(cx<float>) : sizeof(cx<double>);
  return (size_t)L.vis.n_time * L.vis.n_ant * L.vis.n_chan * 2 * elt;
}

hipError_t launch_chain_table(const SolveLaunch& L, void* table, hipStream_t stream) {
  const unsigned grid = (unsigned)((size_t)L.vis.n_time * L.vis.n_ant);
  if (grid == 0) return hipSuccess;
  if (L.prec_mixed)
    hipLaunchKernelGGL(k_chain_table<float>, dim3(grid), dim3(256), 0, stream, L,
                       reinterpret_cast<cx<float>*>(table));
  else
    hipLaunchKernelGGL(k_chain_table<double>, dim3(grid), dim3(256), 0, stream, L,
                       reinterpret_cast<cx<double>*>(table));
  return hipGetLastError();
}

hipError_t launch_solve(const SolveLaunch& L, const SplitLaunch* P, hipStream_t stream, size_t* lds_out) {
  const int kind = L.chain.t[L.chain.active].kind;
  if (L.prec_mixed) {
    if (L.vis_is_c128) return hipErrorInvalidValue;
    switch (kind) {
      case KIND_DIAG: return launch_solve_kind<KIND_DIAG, float, float>(L, P, stream, lds_out);
      case KIND_C2X2: return launch_solve_kind<KIND_C2X2, float, float>(L, P, stream, lds_out);
      case KIND_DELOFF: return launch_solve_kind<KIND_DELOFF, float, float>(L, P, stream, lds_out);
      default: return launch_solve_kind<KIND_DELAY, float, float>(L, P, stream, lds_out);
    }
  }
  if (L.vis_is_c128) {
    switch (kind) {
      case KIND_DIAG: return launch_solve_kind<KIND_DIAG, double, double>(L, P, stream, lds_out);
      case KIND_C2X2: return launch_solve_kind<KIND_C2X2, double, double>(L, P, stream, lds_out);
      case KIND_DELOFF: return launch_solve_kind<KIND_DELOFF, double, double>(L, P, stream, lds_out);
      default: return launch_solve_kind<KIND_DELAY, double, double>(L, P, stream, lds_out);
    }
  }
  switch (kind) {
    case KIND_DIAG: return launch_solve_kind<KIND_DIAG, float, double>(L, P, stream, lds_out);
    case KIND_C2X2: return launch_solve_kind<KIND_C2X2, float, double>(L, P, stream, lds_out);
    case KIND_DELOFF: return launch_solve_kind<KIND_DELOFF, float, double>(L, P, stream, lds_out);
    default: return launch_solve_kind<KIND_DELAY, float, double>(L, P, stream, lds_out);
  }
}

}  // namespace qc
