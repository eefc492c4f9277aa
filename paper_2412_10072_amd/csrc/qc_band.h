// Split pass for terms whose solution intervals are single channels (a
// bandpass solved per channel) on a diagonal chain with one gain direction.
//
// The per-interval accumulation is the one of Algorithm 1 (JHJ and JHr of
// every antenna, Section 2.3, with eq. chain_trick for the chain), but the
// work is laid out for these intervals: one interval is one channel of every
// row, so a wavefront that took one interval would read one sample per row
// at the row stride.  Here a wavefront takes 16 neighbouring channels -- 16
// intervals -- and steps through a part of their rows four rows at a time,
// lane (g, c) = (row g of the step, channel c) (or 8 channels and 8 rows,
// whose LDS slots are half as large: where 16-channel slots do not fit or leave
// too few wavefronts).  Every sample load is then a contiguous segment of channels, and the
// intervals need no reduction across lanes: each lane's channel is its own
// interval.
//
// A step holds up to four (eight) consecutive rows of one time that share
// antenna p and differ in antenna q (a p-run of the row order).  The
// antenna-p sums stay in registers over the run and are summed over the rows
// of the step when p changes; the antenna-q sums go straight to the wavefront's LDS slots
// [antenna][channel][value], which the lanes of one step address without
// collision (distinct q per row, distinct channel per lane), so they are added in
// program order and the result does not depend on timing.  At
// each change of time the LDS slots are added into the part's FP64 partial
// blocks (in the layout the split update sums).
//
// The sums are FP64 in MIXED too (contributions FP32): nothing bounds the rows of
// one time and antenna (a baseline may repeat), and plain FP32 slots over 8000 equal
// rows were off by 1e-4 of the update, where the other MIXED passes compensate
// theirs.
#pragma once

#include "qc_interval.h"

namespace qc {
namespace {

constexpr int BAND_NV = KindInfo<KIND_DIAG>::NV;

// A step read through the scalar cache (its index is the same in every lane);
// R rows.
template <int R>
__device__ __forceinline__ BandStep band_step_at(const BandStep* steps, long long r) {
  using CP = const __attribute__((address_space(4))) int*;
  const CP b = (CP)(steps + r);
  BandStep s;
  s.k = b[0];
  s.t = b[1];
  s.p = b[2];
  s.dup = b[3];
#pragma unroll
  for (int g = 0; g < BAND_MAX_ROWS; ++g) s.q[g] = g < R ? b[4 + g] : -1;
  return s;
}

// LDS slot of (antenna, value, channel) for CW channels per wavefront: the
// values of one (antenna, channel) side by side, so that a lane adds its six with
// three 8-byte (FP64: 16-byte) reads and writes.
template <typename A, int CW>
__device__ __forceinline__ A* band_slot(int ant, int k, int cl) {
  return lds_at<A>(0) + ((size_t)ant * CW + cl) * BAND_NV + k;
}

// Adds a lane's values to the slots of (ant, channel cl).  The lanes of one call
// address distinct slots and only this wavefront does, so plain reads and writes
// do: as LDS atomics (six per step, rows colliding on banks) the additions were
// what bounded the pass, at 2.2 TB/s whatever was loaded ahead (FP32 slots, 256
// channels x 60 times of 64 antennas: 1.24 ms, with these 0.68, and 0.55 in one round
// of workgroups).
template <typename A, int CW>
__device__ __forceinline__ void band_add(int ant, int cl, const A* v) {
  using A2 = A __attribute__((ext_vector_type(2)));
  A2* s = reinterpret_cast<A2*>(band_slot<A, CW>(ant, 0, cl));
  static_assert(BAND_NV == 6, "three pairs");
  A2 x[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) x[j] = s[j];
#pragma unroll
  for (int j = 0; j < 3; ++j) s[j] = x[j] + A2{v[2 * j], v[2 * j + 1]};
}

// Keeps a lane's additions before it apart from those after it, which other
// lanes may have made to the same slots meanwhile (no instruction: a wavefront's
// LDS operations are performed in order).
__device__ __forceinline__ void band_turn() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The same, the rows of a step one after the other (their slots may be the same):
// lane (g, cl) adds where `add` is set.  (To one lane, which has its own turn only,
// the turns would be one addition.)
template <typename A, int CW>
__device__ __forceinline__ void band_add_turns(bool add, int g, int ant, int cl, const A* v) {
#pragma unroll
  for (int h = 0; h < 64 / CW; ++h) {
    if (add && g == h) band_add<A, CW>(ant, cl, v);
    band_turn();
  }
}

// acc += the contribution of one sample, formed in T.
template <typename T>
__device__ __forceinline__ void band_contrib(const m22<T>& B, const m22<T>& WR, T w0, T w1, T w2, T w3, cx<T> g0, cx<T> g1,
                                             double* acc) {
  if constexpr (sizeof(T) == 8) {
    contrib<KIND_DIAG, true, T>(cone<T>(), cone<T>(), B, WR, w0, w1, w2, w3, g0, g1, T(1), acc);
  } else {
    T v[BAND_NV];
#pragma unroll
    for (int k = 0; k < BAND_NV; ++k) v[k] = T(0);
    contrib<KIND_DIAG, true, T>(cone<T>(), cone<T>(), B, WR, w0, w1, w2, w3, g0, g1, T(1), v);
#pragma unroll
    for (int k = 0; k < BAND_NV; ++k) acc[k] += (double)v[k];
  }
}

// x of the lane 8 apart in the same 16-lane row (DPP row rotate by 8)
constexpr int DPP_ROW_ROR8 = 0x128;
__device__ __forceinline__ float ror8(float x) {
  return ffrom((unsigned)__builtin_amdgcn_mov_dpp((int)fbits(x), DPP_ROW_ROR8, 0xF, 0xF, true));
}
__device__ __forceinline__ double ror8(double x) {
  return dfrom((unsigned)__builtin_amdgcn_mov_dpp((int)lo32(x), DPP_ROW_ROR8, 0xF, 0xF, true),
               (unsigned)__builtin_amdgcn_mov_dpp((int)hi32(x), DPP_ROW_ROR8, 0xF, 0xF, true));
}

// Pair sums across the lanes OFF apart, OFF in {32, 16, 8}: lanes with bit
// OFF clear keep x summed over the pair, the others y; the lane's channel
// (its low bits) is kept.
template <int OFF, typename A>
__device__ __forceinline__ A band_pair(A x, A y, bool up) {
  if constexpr (OFF == 8) {
    const A send = up ? x : y;
    const A keep = up ? y : x;
    return keep + ror8(send);
  } else {
    return pair_step<OFF>(x, y, up);
  }
}
template <int OFF, typename A>
__device__ __forceinline__ A band_full(A x) {
  if constexpr (OFF == 8) return x + ror8(x);
  else return full_step<OFF>(x);
}

template <typename A>
__device__ __forceinline__ void lds_add(A* p, A x) {
  __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// An int read through the scalar cache (the index is the same in every lane).
__device__ __forceinline__ int ld_uniform(const int* base, long long i) {
  using CP = const __attribute__((address_space(4))) int*;
  return ((CP)base)[i];
}

// grid: (CW-channel slice, gain time, part), slice fastest; one wavefront
// each, lanes (row g < 64 / CW of the step, channel c < CW).
// ND: direction-dependent fixed terms, read from their tables (L.dd_tab).
template <typename S, typename T, int ND, int CW>
__global__ void __launch_bounds__(64) k_band_pass(SolveLaunch L, int n_part, double* partials, const uint8_t* done) {
  using A = double;                     // the sums
  constexpr int NV = BAND_NV;
  constexpr int NR = 64 / CW;           // rows per step
  const VisArgs& V = L.vis;
  const ChainArgs& CH = L.chain;
  const int act = CH.active;
  const int n_term = CH.n_term;
  const TermArgs& TA = CH.t[act];
  const int n_ant = V.n_ant;
  const int n_chan = V.n_chan;
  const int n_dir = V.n_dir;
  const int n_gf = TA.n_gf;
  const int n_slices = (n_chan + CW - 1) / CW;
  const int slice = blockIdx.x % n_slices;
  const int rest = blockIdx.x / n_slices;
  const int part = rest % n_part;
  const int gt = rest / n_part;
  const int lane = threadIdx.x;
  const int cl = lane & (CW - 1);
  const int g = lane / CW;
  const int c = slice * CW + cl;
  const bool cin = c < n_chan;
  const int cc = cin ? c : n_chan - 1;
  const int interval = gt * n_gf + cc;       // one channel per interval: gain frequency = channel
  const bool live = cin && !done[interval];
  if (!__any(live)) return;

  const int n_vals = n_ant * NV * CW;
  for (int i = lane; i < n_vals; i += 64) lds_at<A>(0)[i] = A(0);
  __syncthreads();

  const long long lo = L.row_lo[gt], n = L.row_hi[gt] - lo;
  const long long r_lo = lo + (n * part) / n_part, r_hi = lo + (n * (part + 1)) / n_part;
  const size_t stride = (size_t)n_ant * NV + 1;
  double* Pc = partials + ((size_t)interval * n_part + part) * stride;
  const S* Dp = reinterpret_cast<const S*>(V.data);
  const S* Mp = reinterpret_cast<const S*>(V.model);
  const S* Wp = reinterpret_cast<const S*>(V.weight);
  const double nu = V.freq[cc];
  const size_t gbase = (size_t)interval * n_ant;       // one gain direction
  const cx<T>* otab = reinterpret_cast<const cx<T>*>(L.otab);
  // direction-dependent fixed terms: table entry (gain time, gain frequency,
  // antenna, model direction); the lane's gain frequency is fixed
  const cx<T>* dtab[ND > 0 ? ND : 1];
  size_t dd_f[ND > 0 ? ND : 1];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    const TermArgs& tj = CH.t[L.dd_term[j]];
    dtab[j] = reinterpret_cast<const cx<T>*>(L.dd_tab[j]);
    dd_f[j] = (size_t)tj.f_map[cc] * n_ant * n_dir * 2;
  }

  bool first = true;          // no FP64 flush yet: the first one stores
  T chi = T(0);
  double chi64 = 0.0;
  A pacc[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) pacc[k] = A(0);
  int p_cur = -1, t_cur = -1;

  // the run's antenna-p sums, summed over the NR rows of the step, into LDS
  auto flush_p = [&]() {
    if (p_cur < 0) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) pacc[j] = band_pair<32>(pacc[j], pacc[j + 4], (lane & 32) != 0);
#pragma unroll
    for (int j = 0; j < 2; ++j) pacc[j] = band_pair<16>(pacc[j], pacc[j + 2], (lane & 16) != 0);
    if constexpr (CW == 8) pacc[0] = band_pair<8>(pacc[0], pacc[1], (lane & 8) != 0);
    // lane (g, c) holds values PER g .. PER g + PER - 1 of its channel
    constexpr int PER = 8 / NR;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int k = PER * g + j;
      if (k < NV && cin) lds_add(band_slot<A, CW>(p_cur, k, cl), pacc[j]);
    }
    band_turn();
#pragma unroll
    for (int k = 0; k < 8; ++k) pacc[k] = A(0);
  };
  // the LDS slots added into the part's FP64 blocks, and cleared
  auto flush_lds = [&]() {
    __syncthreads();
    for (int i = g; i < n_ant * NV; i += NR) {     // (antenna, value)
      A* ps = band_slot<A, CW>(i / NV, i % NV, cl);
      const double x = (double)*ps;
      *ps = A(0);
      if (cin) {
        double* dst = Pc + i;
        *dst = first ? x : *dst + x;
      }
    }
    __syncthreads();
    chi64 += (double)chi;
    chi = T(0);
    first = false;
  };

  long long r = r_lo;
  BandStep st;
  if (r < r_hi) st = band_step_at<NR>(L.band_steps, r);
  while (r < r_hi) {
    const long long r_next = r + max(st.k, 1);
    BandStep nx;
    if (r_next < r_hi) nx = band_step_at<NR>(L.band_steps, r_next);
    const int t = st.t, p = st.p;
    if (t != t_cur) {
      flush_p();
      p_cur = -1;
      if (t_cur >= 0) flush_lds();
      t_cur = t;
    }
    if (p != p_cur) {
      flush_p();
      p_cur = p;
    }
    int q = st.q[0];
#pragma unroll
    for (int h = 1; h < NR; ++h) q = g == h ? st.q[h] : q;
    const bool row_ok = q >= 0;
    const int qq = row_ok ? q : p;
    const size_t s = (size_t)(r + (row_ok ? g : 0)) * n_chan + cc;
    T w0, w1, w2, w3;
    load_w<S, T>(Wp, s, V.n_wcorr, w0, w1, w2, w3);
    const uint8_t fl = V.flag[s];
    const m22<T> Draw = load_m22<S, T>(Dp, s);
    const bool use = row_ok & cin & (fl == 0);
    w0 = use ? w0 : T(0); w1 = use ? w1 : T(0); w2 = use ? w2 : T(0); w3 = use ? w3 : T(0);
    const m22<T> D = select_m(use, Draw);

    // direction-independent fixed factors o (table or per sample), active gains h
    cx<T> op0 = cone<T>(), op1 = cone<T>(), oq0 = cone<T>(), oq1 = cone<T>();
    if (otab) {
      const size_t tp_ = (((size_t)t * n_ant + p) * n_chan + cc) * 2;
      const size_t tq_ = (((size_t)t * n_ant + qq) * n_chan + cc) * 2;
      op0 = otab[tp_]; op1 = otab[tp_ + 1];
      oq0 = otab[tq_]; oq1 = otab[tq_ + 1];
    } else {
      for (int j = 0; j < n_term; ++j) {
        if (j == act || CH.t[j].n_gdir > 1) continue;
        const m22<T> Jp = term_jones<T>(CH.t[j], n_ant, t, cc, p, 0, nu);
        const m22<T> Jq = term_jones<T>(CH.t[j], n_ant, t, cc, qq, 0, nu);
        op0 = op0 * Jp.a; op1 = op1 * Jp.d;
        oq0 = oq0 * Jq.a; oq1 = oq1 * Jq.d;
      }
    }
    const double2 gp0 = L.gains[4 * (gbase + p)], gp3 = L.gains[4 * (gbase + p) + 3];
    const double2 gq0 = L.gains[4 * (gbase + qq)], gq3 = L.gains[4 * (gbase + qq) + 3];
    const cx<T> hp0 = cmake<T>((T)gp0.x, (T)gp0.y), hp1 = cmake<T>((T)gp3.x, (T)gp3.y);
    const cx<T> hq0 = cmake<T>((T)gq0.x, (T)gq0.y), hq1 = cmake<T>((T)gq3.x, (T)gq3.y);
    // table rows of antennas p and q at this time
    const cx<T>* dp_[ND > 0 ? ND : 1];
    const cx<T>* dq_[ND > 0 ? ND : 1];
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      const TermArgs& tj = CH.t[L.dd_term[j]];
      const size_t tb = (size_t)ld_uniform(tj.t_map, t) * tj.n_gf * n_ant * n_dir * 2 + dd_f[j];
      dp_[j] = dtab[j] + tb + (size_t)p * n_dir * 2;
      dq_[j] = dtab[j] + tb + (size_t)qq * n_dir * 2;
    }

    // E_ij = o_{p,i} conj(o_{q,j}) sum_d e_{p,d,i} M_d,ij conj(e_{q,d,j}), with o the
    // direction-independent and e the direction-dependent fixed factors;
    // then V_ij = h_{p,i} E_ij conj(h_{q,j})
    constexpr int MCH = sizeof(T) == 4 ? 4 : 1;
    m22<T> E = mzero<T>();
    for (int d0 = 0; d0 < n_dir; d0 += MCH) {
      m22<T> Mc[MCH];
      cx<T> ep0[MCH], ep1[MCH], eq0[MCH], eq1[MCH];
#pragma unroll
      for (int k = 0; k < MCH; ++k) {
        const int d = min(d0 + k, n_dir - 1);      // clamped: the loads go out together
        Mc[k] = load_m22<S, T>(Mp, s * n_dir + d);
        ep0[k] = ep1[k] = eq0[k] = eq1[k] = cone<T>();
#pragma unroll
        for (int j = 0; j < ND; ++j) {
          ep0[k] = ep0[k] * dp_[j][2 * d];
          ep1[k] = ep1[k] * dp_[j][2 * d + 1];
          eq0[k] = eq0[k] * dq_[j][2 * d];
          eq1[k] = eq1[k] * dq_[j][2 * d + 1];
        }
      }
#pragma unroll
      for (int k = 0; k < MCH; ++k) {
        if (d0 + k < n_dir) {
          E.a = cfma(mulc(ep0[k], eq0[k]), Mc[k].a, E.a);
          E.b = cfma(mulc(ep0[k], eq1[k]), Mc[k].b, E.b);
          E.c = cfma(mulc(ep1[k], eq0[k]), Mc[k].c, E.c);
          E.d = cfma(mulc(ep1[k], eq1[k]), Mc[k].d, E.d);
        }
      }
    }
    E.a = E.a * mulc(op0, oq0);
    E.b = E.b * mulc(op0, oq1);
    E.c = E.c * mulc(op1, oq0);
    E.d = E.d * mulc(op1, oq1);
    E = select_m(use, E);
    m22<T> B, Bc;
    B.a = mulc(E.a, hq0);
    B.b = mulc(E.b, hq1);
    B.c = mulc(E.c, hq0);
    B.d = mulc(E.d, hq1);
    Bc.a = conj(E.a * hp0);
    Bc.b = conj(E.c * hp1);
    Bc.c = conj(E.b * hp0);
    Bc.d = conj(E.d * hp1);
    const m22<T> R = D - rowscale(hp0, hp1, B);
    const m22<T> WR = wmul(R, w0, w1, w2, w3);
    A qv[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) qv[k] = A(0);
    band_contrib<T>(B, WR, w0, w1, w2, w3, hp0, hp1, pacc);
    band_contrib<T>(Bc, herm(WR), w0, w2, w1, w3, hq0, hq1, qv);
    chi = chisq_acc(WR, R, chi);

    const bool add = row_ok && cin;
    if (!st.dup) {
      if (add) band_add<A, CW>(q, cl, qv);
      band_turn();
    } else {
      // two rows of the step share antenna q: one row at a time
      band_add_turns<A, CW>(add, g, q, cl, qv);
    }
    r = r_next;
    st = nx;
  }
  flush_p();
  flush_lds();
  // chi^2 of the channel: the sums of the step's rows
  double cs = chi64;
  cs = band_full<32>(cs);
  cs = band_full<16>(cs);
  if constexpr (CW == 8) cs = band_full<8>(cs);
  if (g == 0 && cin) Pc[stride - 1] = cs;
}

// ---------------------------------------------------------------------------
// The same pass where the model is one direction and the chain the active term
// alone (as it is over a folded chain): no fixed factors.
//
// Bound by latency: six wavefronts per CU (24 KiB of LDS each at 64 antennas, in
// steps of 8 x 8) and 64 samples a step.  So a step is simply the next four (eight) rows, whose
// samples are loaded two steps ahead and whose antennas and gains one step ahead
// (the steps above wait for one another's records), and the gains come from a
// table in the step's own layout [gain time][slice][antenna][hand][channel]
// (k_band_gains, once per pass: 8 cache lines a step instead of one per lane out
// of the solution's FP64 blocks, which lie an interval apart).  The rows of a step
// may differ in antenna p: each lane keeps its own row's p sums and adds them to
// LDS, one row after the other, when its p changes.  Folded bandpass of 256
// channels, 64 antennas, 60 times (2.5 GB a pass): 1.24 -> 0.55 ms with FP32 slots; the
// mean over a solve's passes 0.46 ms with those, 0.52 with the FP64 ones (4.8 TB/s).
// ---------------------------------------------------------------------------
template <typename T, int CW>
__global__ void __launch_bounds__(256) k_band_gains(const double2* gains, int n_gf, int n_ant, int n_slices, size_t n,
                                                    cx<T>* tab) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int cl = (int)(i % CW);
  size_t j = i / CW;
  const int hand = (int)(j & 1);
  j >>= 1;
  const int a = (int)(j % n_ant);
  j /= n_ant;
  const int slice = (int)(j % n_slices);
  const size_t gt = j / n_slices;
  const int c = min(slice * CW + cl, n_gf - 1);        // lanes past the band repeat the last channel
  const double2 g = gains[4 * ((gt * n_gf + c) * n_ant + a) + 3 * hand];
  tab[i] = cmake<T>((T)g.x, (T)g.y);
}

struct BandRow {
  int p, q, t;               // of this lane's row; q = -1: the row adds nothing
};
template <typename T>
struct BandGain {
  cx<T> p0, p1, q0, q1;
};

template <typename S, typename T, int CW>
__global__ void __launch_bounds__(64) k_band_single(SolveLaunch L, int n_part, double* partials, const uint8_t* done) {
  using A = double;                     // the sums
  constexpr int NV = BAND_NV;
  constexpr int NR = 64 / CW;           // rows per step
  const VisArgs& V = L.vis;
  const TermArgs& TA = L.chain.t[L.chain.active];
  const int n_ant = V.n_ant;
  const int n_chan = V.n_chan;
  const int n_gf = TA.n_gf;
  const int n_slices = (n_chan + CW - 1) / CW;
  const int slice = blockIdx.x % n_slices;
  const int rest = blockIdx.x / n_slices;
  const int part = rest % n_part;
  const int gt = rest / n_part;
  const int lane = threadIdx.x;
  const int cl = lane & (CW - 1);
  const int g = lane / CW;
  const int c = slice * CW + cl;
  const bool cin = c < n_chan;
  const int cc = cin ? c : n_chan - 1;
  const int interval = gt * n_gf + cc;       // one channel per interval: gain frequency = channel
  if (!__any(cin && !done[interval])) return;

  const int n_vals = n_ant * NV * CW;
  for (int i = lane; i < n_vals; i += 64) lds_at<A>(0)[i] = A(0);
  __syncthreads();

  const long long lo = L.row_lo[gt], n = L.row_hi[gt] - lo;
  const long long r_lo = lo + (n * part) / n_part, r_hi = lo + (n * (part + 1)) / n_part;
  const size_t stride = (size_t)n_ant * NV + 1;
  double* Pc = partials + ((size_t)interval * n_part + part) * stride;
  const cx<T>* tab = reinterpret_cast<const cx<T>*>(L.band_gains) + ((size_t)gt * n_slices + slice) * n_ant * 2 * CW;
  const S* Dp = reinterpret_cast<const S*>(V.data);
  const S* Mp = reinterpret_cast<const S*>(V.model);
  const S* Wp = reinterpret_cast<const S*>(V.weight);

  bool first = true;          // no FP64 flush yet: the first one stores
  T chi = T(0);
  double chi64 = 0.0;
  A pacc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) pacc[k] = A(0);
  int p_cur = -1, t_cur = -1;

  // the sums of the lanes whose antenna p is over (`over`) into LDS, one row of
  // the step after the other (several rows usually share the antenna)
  auto flush_p = [&](bool over) {
    const bool add = over && p_cur >= 0 && cin;
    band_add_turns<A, CW>(add, g, p_cur, cl, pacc);
#pragma unroll
    for (int k = 0; k < NV; ++k) pacc[k] = over ? A(0) : pacc[k];
  };
  // the LDS slots added into the part's FP64 blocks, and cleared; the blocks of
  // earlier times are read eight at a time
  auto flush_lds = [&]() {
    __syncthreads();
    constexpr int U = 8;
    const int n_av = n_ant * NV;
    for (int i0 = g; i0 < n_av; i0 += NR * U) {      // (antenna, value)
      double x[U], was[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + NR * u;
        x[u] = 0.0;
        was[u] = 0.0;
        if (i < n_av) {
          A* ps = band_slot<A, CW>(i / NV, i % NV, cl);
          x[u] = (double)*ps;
          *ps = A(0);
          if (!first && cin) was[u] = Pc[i];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + NR * u;
        if (i < n_av && cin) Pc[i] = was[u] + x[u];
      }
    }
    __syncthreads();
    chi64 += (double)chi;
    chi = T(0);
    first = false;
  };

  // row of this lane in the step that begins at row r (clamped into the part)
  auto row_at = [&](long long r) -> long long { return min(r + g, r_hi - 1); };
  auto load_row = [&](long long r) -> BandRow {
    const long long rr = row_at(r);
    BandRow a{V.ant1[rr], V.ant2[rr], V.row_time[rr]};
    const bool ok = r + g < r_hi && a.p != a.q && (unsigned)a.p < (unsigned)n_ant && (unsigned)a.q < (unsigned)n_ant;
    a.p = ok ? a.p : 0;
    a.q = ok ? a.q : -1;
    return a;
  };
  auto load_gain = [&](const BandRow& a) -> BandGain<T> {
    const cx<T>* hp = tab + (size_t)a.p * 2 * CW + cl;
    const cx<T>* hq = tab + (size_t)max(a.q, 0) * 2 * CW + cl;
    return {hp[0], hp[CW], hq[0], hq[CW]};
  };
  RawSample<S> x0 = {}, x1 = {}, x2 = {};
  BandRow a0{0, -1, 0}, a1{0, -1, 0}, a2{0, -1, 0};
  BandGain<T> h0 = {}, h1 = {};
  auto load_x = [&](RawSample<S>& x, long long r) {
    raw_load<S>(x, Dp, Mp, Wp, V.flag, (size_t)row_at(r) * n_chan + cc, V.n_wcorr);
  };
  if (r_lo < r_hi) {
    load_x(x0, r_lo);
    a0 = load_row(r_lo);
    load_x(x1, r_lo + NR);
    a1 = load_row(r_lo + NR);
    h0 = load_gain(a0);
  }
  for (long long r = r_lo; r < r_hi; r += NR) {
    load_x(x2, r + 2 * NR);
    a2 = load_row(r + 2 * NR);
    h1 = load_gain(a1);
    // the time of the step's first row
    const int t = __builtin_amdgcn_readfirstlane(a0.t);
    if (t != t_cur) {
      if (t_cur >= 0) {
        flush_p(true);
        p_cur = -1;
        flush_lds();
      }
      t_cur = t;
    }
    const bool row_ok = a0.q >= 0;
    const bool over = row_ok && a0.p != p_cur;
    if (__any(over)) {
      flush_p(over);
      p_cur = over ? a0.p : p_cur;
    }
    T w0, w1, w2, w3;
    raw_weights<S, T>(x0, V.n_wcorr, w0, w1, w2, w3);
    const bool use = row_ok & cin & (x0.f == 0);
    w0 = use ? w0 : T(0); w1 = use ? w1 : T(0); w2 = use ? w2 : T(0); w3 = use ? w3 : T(0);
    const m22<T> D = select_m(use, raw_data<T>(x0));
    const m22<T> E = select_m(use, raw_model<T>(x0));
    m22<T> B, Bc;
    B.a = mulc(E.a, h0.q0);
    B.b = mulc(E.b, h0.q1);
    B.c = mulc(E.c, h0.q0);
    B.d = mulc(E.d, h0.q1);
    Bc.a = conj(E.a * h0.p0);
    Bc.b = conj(E.c * h0.p1);
    Bc.c = conj(E.b * h0.p0);
    Bc.d = conj(E.d * h0.p1);
    const m22<T> R = D - rowscale(h0.p0, h0.p1, B);
    const m22<T> WR = wmul(R, w0, w1, w2, w3);
    A qv[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) qv[k] = A(0);
    band_contrib<T>(B, WR, w0, w1, w2, w3, h0.p0, h0.p1, pacc);
    band_contrib<T>(Bc, herm(WR), w0, w2, w1, w3, h0.q0, h0.q1, qv);
    chi = chisq_acc(WR, R, chi);

    // two rows of the step that share antenna q are added one after the other
    const int q_own = row_ok ? a0.q : -1 - g;
    bool dup = false;
#pragma unroll
    for (int h = 1; h < NR; ++h) dup = dup || __shfl_xor(q_own, h * CW) == q_own;
    const bool add = row_ok && cin;
    if (!__any(dup)) {
      if (add) band_add<A, CW>(a0.q, cl, qv);
      band_turn();
    } else {
      band_add_turns<A, CW>(add, g, a0.q, cl, qv);
    }
    x0 = x1;
    x1 = x2;
    a0 = a1;
    a1 = a2;
    h0 = h1;
  }
  flush_p(true);
  flush_lds();
  // chi^2 of the channel: the sums of the step's rows
  double cs = chi64;
  cs = band_full<32>(cs);
  cs = band_full<16>(cs);
  if constexpr (CW == 8) cs = band_full<8>(cs);
  if (g == 0 && cin) Pc[stride - 1] = cs;
}

// One pass of that kernel, its gain table first.
template <typename S, typename T, int CW>
hipError_t launch_band_single(const SolveLaunch& L, int n_part, double* partials, const uint8_t* done, unsigned grid,
                              size_t lds, hipStream_t stream) {
  const TermArgs& ta = L.chain.t[L.chain.active];
  const int n_slices = (L.vis.n_chan + CW - 1) / CW;
  const size_t n = (size_t)ta.n_gt * n_slices * L.vis.n_ant * 2 * CW;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_band_single<S, T, CW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_band_gains<T, CW>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                     (const double2*)L.gains, ta.n_gf, L.vis.n_ant, n_slices, n, reinterpret_cast<cx<T>*>(L.band_gains));
  hipLaunchKernelGGL((k_band_single<S, T, CW>), dim3(grid), dim3(64), lds, stream, L, n_part, partials, done);
  return hipGetLastError();
}

}  // namespace
}  // namespace qc
