// Host side of the libqc C-ABI: context, argument checks, the device-side
// validation pre-pass (row order, antenna and time ranges, per-interval row
// ranges) and the public entry points declared in include/qc.h.

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "qc_host.h"
#include "qc_hostcheck.h"
#include "qc_schedule.h"

using namespace qc;

namespace qc {

// ---------------------------------------------------------------------------
// validation kernels
// ---------------------------------------------------------------------------

__global__ void k_clear(int* err) {
  if (threadIdx.x == 0 && blockIdx.x == 0) err[0] = 0;
}

// For rows sorted by time, rowpos[t] = first row with row_time >= t
// (t = 0 .. n_time).  Each entry is written by exactly one row when the
// order is valid; bad input raises a flag and every write stays in bounds.
__global__ void k_rows(VisArgs v, long long* rowpos, int* err) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= v.n_row) return;
  const int nt = v.n_time;
  int t = v.row_time[r];
  const int p = v.ant1[r], q = v.ant2[r];
  int bad = 0;
  if ((unsigned)p >= (unsigned)v.n_ant || (unsigned)q >= (unsigned)v.n_ant) bad |= ERR_RANGE;
  if ((unsigned)t >= (unsigned)nt) bad |= ERR_RANGE;
  int tp = (r > 0) ? v.row_time[r - 1] : -1;
  if (r > 0 && tp > t) bad |= ERR_ORDER;
  if (bad) atomicOr(err, bad);
  t = min(max(t, -1), nt - 1);
  tp = min(max(tp, -1), nt - 1);
  for (int tt = tp + 1; tt <= t; ++tt) rowpos[tt] = r;
  if (r == v.n_row - 1)
    for (int tt = max(t, -1) + 1; tt <= nt; ++tt) rowpos[tt] = v.n_row;
}

__global__ void k_rowpos_empty(long long* rowpos, int nt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t <= nt) rowpos[t] = 0;
}

__global__ void k_ranges(const long long* rowpos, const int* tt, int n_gt, long long* lo, long long* hi) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n_gt) return;
  lo[g] = rowpos[tt[g]];
  hi[g] = rowpos[tt[n_gt + g]];
}

// ---------------------------------------------------------------------------
// host checks
// ---------------------------------------------------------------------------

qc_status check_vis(qc_ctx* ctx, const qc_vis* v, bool need_model) {
  const Check c = check_vis_fields(v, need_model);
  return c.st == QC_OK ? QC_OK : fail(ctx, c.st, "%s", c.msg.c_str());
}

qc_status check_term(qc_ctx* ctx, const qc_vis* v, const qc_term* t, int j, HostMaps& hm, hipStream_t s) {
  Check c = check_term_fields(t, j);
  if (c.st != QC_OK) return fail(ctx, c.st, "%s", c.msg.c_str());
  if (t->type == QC_TERM_POINTING) {
    std::vector<double> lm(2 * (size_t)v->n_dir);
    HIP_TRY(ctx, hipMemcpyAsync(lm.data(), t->dir_lm, sizeof(double) * lm.size(), hipMemcpyDeviceToHost, s));
    HIP_TRY(ctx, hipStreamSynchronize(s));
    c = check_dir_lm(lm.data(), v->n_dir, j);
    if (c.st != QC_OK) return fail(ctx, c.st, "%s", c.msg.c_str());
  }
  hm.t_map.resize(v->n_time);
  hm.f_map.resize(v->n_chan);
  hm.d_map.resize(v->n_dir);
  HIP_TRY(ctx, hipMemcpyAsync(hm.t_map.data(), t->t_map, sizeof(int) * v->n_time, hipMemcpyDeviceToHost, s));
  HIP_TRY(ctx, hipMemcpyAsync(hm.f_map.data(), t->f_map, sizeof(int) * v->n_chan, hipMemcpyDeviceToHost, s));
  HIP_TRY(ctx, hipMemcpyAsync(hm.d_map.data(), t->d_map, sizeof(int) * v->n_dir, hipMemcpyDeviceToHost, s));
  HIP_TRY(ctx, hipStreamSynchronize(s));
  c = check_term_maps(t, j, hm.t_map.data(), v->n_time, hm.f_map.data(), v->n_chan, hm.d_map.data(), v->n_dir);
  return c.st == QC_OK ? QC_OK : fail(ctx, c.st, "%s", c.msg.c_str());
}

bool dmap_constant(const HostMaps& hm) {
  for (size_t i = 1; i < hm.d_map.size(); ++i)
    if (hm.d_map[i] != hm.d_map[0]) return false;
  return true;
}

void fill_args(const qc_vis* v, const qc_term* chain, int n_term, int active, VisArgs& va, ChainArgs& ca) {
  va.data = v->data;
  va.model = v->model;
  va.weight = v->weight;
  va.flag = v->flag;
  va.ant1 = v->ant1;
  va.ant2 = v->ant2;
  va.row_time = v->row_time;
  va.freq = v->chan_freq;
  va.n_row = v->n_row;
  va.n_chan = v->n_chan;
  va.n_dir = v->n_dir;
  va.n_ant = v->n_ant;
  va.n_time = v->n_time;
  va.n_wcorr = v->n_wcorr;
  memset(&ca, 0, sizeof ca);
  ca.n_term = n_term;
  ca.active = active;
  for (int j = 0; j < n_term; ++j) {
    const qc_term& t = chain[j];
    TermArgs& ta = ca.t[j];
    ta.kind = (int)t.type;
    ta.n_gt = t.n_gt;
    ta.n_gf = t.n_gf;
    ta.n_gdir = t.n_gdir;
    ta.t_map = t.t_map;
    ta.f_map = t.f_map;
    ta.d_map = t.d_map;
    ta.gains = reinterpret_cast<const double2*>(t.gains);
    ta.params = t.params;
    if (t.type == QC_TERM_POINTING) {
      // one parameter pair per antenna, a gain per model direction: every chain
      // path treats the term as direction dependent
      ta.n_gdir = v->n_dir;
      ta.dir_lm = t.dir_lm;
      ta.beta = 4.0 * std::log(2.0) / ((t.beam_fwhm * t.beam_freq) * (t.beam_fwhm * t.beam_freq));
    }
  }
}

qc_status read_err(qc_ctx* ctx, hipStream_t s) {
  int h = 0;
  HIP_TRY(ctx, hipMemcpyAsync(&h, ctx->d_err, sizeof(int), hipMemcpyDeviceToHost, s));
  HIP_TRY(ctx, hipStreamSynchronize(s));
  if (h & ERR_ORDER) return fail(ctx, QC_E_ARG, "row_time is not non-decreasing");
  if (h & ERR_RANGE) return fail(ctx, QC_E_RANGE, "antenna or time index out of range");
  if (h & ERR_NONFINITE) return fail(ctx, QC_E_NONFINITE, "non-finite value in an unflagged sample");
  return QC_OK;
}

// Validates the rows on the device and (when active >= 0) computes the row
// and channel ranges of every solution interval of the active term.
qc_status validate_rows(qc_ctx* ctx, const qc_vis* v, hipStream_t s) {
  qc_status st = check_vis(ctx, v, true);
  if (st != QC_OK) return st;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  VisArgs va;
  ChainArgs ca;
  fill_args(v, nullptr, 0, -1, va, ca);
  HIP_TRY(ctx, grow(ctx->d_rowpos, ctx->rowpos_cap, (size_t)v->n_time + 1));
  HIP_TRY(ctx, solve_take(ctx, s, false));
  hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, s, ctx->d_err);
  if (v->n_row > 0) {
    const long long nb = (v->n_row + 255) / 256;
    hipLaunchKernelGGL(k_rows, dim3((unsigned)nb), dim3(256), 0, s, va, ctx->d_rowpos, ctx->d_err);
  }
  HIP_TRY(ctx, hipGetLastError());
  return read_err(ctx, s);
}

qc_status prepare(qc_ctx* ctx, const qc_vis* v, const qc_term* chain, int n_term, int active,
                  std::vector<HostMaps>& maps, hipStream_t s, const PrepScratch* fixed, bool need_model) {
  qc_status st = check_vis(ctx, v, need_model);
  if (st != QC_OK) return st;
  if (!chain || n_term <= 0) return fail(ctx, QC_E_ARG, "empty chain");
  if (n_term > QC_MAX_TERMS) return fail(ctx, QC_E_UNSUPPORTED, "n_term=%d exceeds %d", n_term, QC_MAX_TERMS);
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  maps.assign(n_term, HostMaps());
  for (int j = 0; j < n_term; ++j) {
    st = check_term(ctx, v, &chain[j], j, maps[j], s);
    if (st != QC_OK) return st;
  }
  VisArgs va;
  ChainArgs ca;
  fill_args(v, chain, n_term, active, va, ca);
  // device scratch: the context's (grown as needed) or the caller's fixed block
  PrepScratch sc;
  if (fixed) {
    sc = *fixed;
  } else {
    HIP_TRY(ctx, grow(ctx->d_rowpos, ctx->rowpos_cap, (size_t)v->n_time + 1));
    sc.rowpos = ctx->d_rowpos;
  }
  HIP_TRY(ctx, solve_take(ctx, s, active >= 0 && !fixed));
  hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, s, ctx->d_err);
  if (v->n_row > 0) {
    const long long nb = (v->n_row + 255) / 256;
    hipLaunchKernelGGL(k_rows, dim3((unsigned)nb), dim3(256), 0, s, va, sc.rowpos, ctx->d_err);
  } else {
    hipLaunchKernelGGL(k_rowpos_empty, dim3((v->n_time + 256) / 256), dim3(256), 0, s, sc.rowpos, v->n_time);
  }
  HIP_TRY(ctx, hipGetLastError());
  if (active >= 0) {
    const qc_term& ta = chain[active];
    const HostMaps& hm = maps[active];
    std::vector<int> tt, clo, chi;
    ctx->max_int_chan = interval_extents(hm.t_map, hm.f_map, ta.n_gt, ta.n_gf, tt, clo, chi);
    if (!fixed) {
      HIP_TRY(ctx, grow(ctx->d_rowlo, ctx->rowlo_cap, (size_t)ta.n_gt));
      HIP_TRY(ctx, grow(ctx->d_rowhi, ctx->rowhi_cap, (size_t)ta.n_gt));
      HIP_TRY(ctx, grow(ctx->d_tt, ctx->tt_cap, 2 * (size_t)ta.n_gt));
      HIP_TRY(ctx, grow(ctx->d_chlo, ctx->chlo_cap, (size_t)ta.n_gf));
      HIP_TRY(ctx, grow(ctx->d_chhi, ctx->chhi_cap, (size_t)ta.n_gf));
      sc.rowlo = ctx->d_rowlo;
      sc.rowhi = ctx->d_rowhi;
      sc.tt = ctx->d_tt;
      sc.chlo = ctx->d_chlo;
      sc.chhi = ctx->d_chhi;
    }
    ctx->h_clo = clo;
    ctx->h_chi = chi;
    HIP_TRY(ctx, hipMemcpyAsync(sc.tt, tt.data(), sizeof(int) * tt.size(), hipMemcpyHostToDevice, s));
    HIP_TRY(ctx, hipMemcpyAsync(sc.chlo, clo.data(), sizeof(int) * clo.size(), hipMemcpyHostToDevice, s));
    HIP_TRY(ctx, hipMemcpyAsync(sc.chhi, chi.data(), sizeof(int) * chi.size(), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_ranges, dim3((ta.n_gt + 255) / 256), dim3(256), 0, s, sc.rowpos, sc.tt, ta.n_gt,
                       sc.rowlo, sc.rowhi);
    HIP_TRY(ctx, hipGetLastError());
  }
  return read_err(ctx, s);
}

int resolve_damping(qc_damping d, const qc_term& t) {
  if (d == QC_DAMP_AUTO) {
    // full steps for delay and phase-only terms: a common phase or delay
    // leaves the model unchanged, so there is no scale mode to overshoot
    if (t.type == QC_TERM_DELAY || t.type == QC_TERM_PHASE || t.type == QC_TERM_DELAY_OFFSET) return 0;
    // pointing: the beams enter the model as the product b_p b_q (as amplitudes do)
    if (t.type == QC_TERM_POINTING) return 2;
    return t.direction_dependent ? 1 : 2;
  }
  return (int)d;
}

}  // namespace qc

// ---------------------------------------------------------------------------
// allocation-free scratch (qc_solve_interval_static)
// ---------------------------------------------------------------------------

// A fixed device array for the scratch of qc_solve_interval_static: each
// device that loads the library holds its own copy until the process ends.
// Host code never passes the array's name to a kernel or a copy (on the host
// it is a stand-in, not a device address): it uses the address that
// hipGetSymbolAddress returns for the current device, kept per device.
static __device__ __align__(256) unsigned char scratch[QC_STATIC_SCRATCH_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[MAX_DEVICES] = {};

// The address of this device's scratch array, looked up once per device
// with the device current.
qc_status static_scratch_ptr(int device, unsigned char** out) {
  if (device < 0 || device >= MAX_DEVICES) return QC_E_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return QC_E_DEVICE;
    g_scratch_ptr[device] = reinterpret_cast<unsigned char*>(p);
  }
  *out = g_scratch_ptr[device];
  return QC_OK;
}

// Carves the prepare scratch of a solve out of the static array; returns the
// bytes it needs (those beyond QC_STATIC_SCRATCH_BYTES are not carved).
size_t carve_static(unsigned char* base, const qc_vis* v, const qc_term& ta, PrepScratch& sc) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    unsigned char* p = base + off;
    off += (bytes + 255) & ~size_t(255);
    return p;
  };
  const size_t n_time = v ? (size_t)std::max(v->n_time, 0) : 0;
  const size_t n_gt = (size_t)std::max(ta.n_gt, 0), n_gf = (size_t)std::max(ta.n_gf, 0);
  sc.rowpos = reinterpret_cast<long long*>(take(sizeof(long long) * (n_time + 1)));
  sc.rowlo = reinterpret_cast<long long*>(take(sizeof(long long) * n_gt));
  sc.rowhi = reinterpret_cast<long long*>(take(sizeof(long long) * n_gt));
  sc.tt = reinterpret_cast<int*>(take(sizeof(int) * 2 * n_gt));
  sc.chlo = reinterpret_cast<int*>(take(sizeof(int) * n_gf));
  sc.chhi = reinterpret_cast<int*>(take(sizeof(int) * n_gf));
  return off;
}

}  // namespace

// ---------------------------------------------------------------------------
// public API
// ---------------------------------------------------------------------------

extern "C" {

qc_status qc_ctx_create(int32_t device, qc_ctx** out) {
  if (!out) return QC_E_ARG;
  *out = nullptr;
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return QC_E_DEVICE;
  if (hipSetDevice(device) != hipSuccess) return QC_E_DEVICE;
  qc_ctx* c = new qc_ctx();
  c->device = device;
  if (hipMalloc(reinterpret_cast<void**>(&c->d_err), sizeof(int) * 4) != hipSuccess) {
    delete c;
    return QC_E_NOMEM;
  }
  hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, device);
  if (c->n_cu <= 0) c->n_cu = 256;
  if (static_scratch_ptr(device, &c->static_scratch) != QC_OK) {
    hipFree(c->d_err);
    delete c;
    return QC_E_DEVICE;
  }
  if (hipEventCreate(&c->ev0) != hipSuccess || hipEventCreate(&c->ev1) != hipSuccess ||
      hipEventCreate(&c->solve_use.ev) != hipSuccess || hipEventCreate(&c->outtab_use.ev) != hipSuccess) {
    hipFree(c->d_err);
    delete c;
    return QC_E_DEVICE;
  }
  *out = c;
  return QC_OK;
}

qc_status qc_ctx_destroy(qc_ctx* ctx) {
  if (!ctx) return QC_E_ARG;
  hipSetDevice(ctx->device);
  hipDeviceSynchronize();
  hipFree(ctx->d_err);
  hipFree(ctx->d_rowpos);
  hipFree(ctx->d_rowlo);
  hipFree(ctx->d_rowhi);
  hipFree(ctx->d_tt);
  hipFree(ctx->d_chlo);
  hipFree(ctx->d_chhi);
  hipFree(ctx->d_dh);
  hipFree(ctx->d_partials);
  hipFree(ctx->d_otab);
  hipFree(ctx->d_outtab);
  hipFree(ctx->d_fold);
  hipFree(ctx->d_fl_stat);
  hipFree(ctx->d_fl_groups);
  hipFree(ctx->d_fl_hist);
  hipFree(ctx->d_fl_count);
  hipFree(ctx->d_fl_rows);
  hipFree(ctx->d_fl_new);
  hipFree(ctx->d_rw);
  hipFree(ctx->d_pc);
  hipFree(ctx->d_pc_off);
  hipFree(ctx->d_dv);
  hipFree(ctx->d_passes);
  hipFree(ctx->d_totals);
  if (ctx->h_done) hipHostFree(ctx->h_done);
  hipFree(ctx->d_done);
  hipFree(ctx->d_active);
  hipFree(ctx->d_pt_int);
  hipFree(ctx->d_pt_dbl);
  hipFree(ctx->d_lm);
  hipFree(ctx->d_acc);
  hipFree(ctx->d_band);
  hipFree(ctx->d_bandg);
  hipFree(ctx->d_ptab);
  hipFree(ctx->d_ddtab);
  hipEventDestroy(ctx->ev0);
  hipEventDestroy(ctx->ev1);
  hipEventDestroy(ctx->solve_use.ev);
  hipEventDestroy(ctx->outtab_use.ev);
  for (hipEvent_t ev : ctx->ev_pass)
    if (ev) hipEventDestroy(ev);
  delete ctx;
  return QC_OK;
}

qc_status qc_ctx_sync(qc_ctx* ctx) {
  if (!ctx) return QC_E_ARG;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  HIP_TRY(ctx, hipStreamSynchronize(ctx->last_stream));
  qc_status st = read_err(ctx, ctx->last_stream);
  hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, ctx->last_stream, ctx->d_err);
  HIP_TRY(ctx, hipStreamSynchronize(ctx->last_stream));
  return st;
}

const char* qc_last_error(const qc_ctx* ctx) { return ctx ? ctx->msg.c_str() : "null context"; }

double qc_last_kernel_ms(qc_ctx* ctx) {
  if (!ctx || !ctx->timed) return -1.0;
  if (hipEventSynchronize(ctx->ev_end) != hipSuccess) return -1.0;
  float ms = 0.f;
  if (hipEventElapsedTime(&ms, ctx->ev0, ctx->ev_end) != hipSuccess) return -1.0;
  return (double)ms;
}

}  // extern "C"

// The work of one pass over the intervals of a solve, as the choices below see it.
struct PassShape {
  int n_int;
  double n_samples, avg, rows;   // samples in all and per interval, rows per interval
  int rps;                       // rows per wavefront step
  double chunks;                 // steps per row
  double step_us;                // one step of a lone workgroup of four wavefronts
  int fit;                       // workgroups of four wavefronts that the chip holds
  bool fp64, wide;               // wide: kernels held to four wavefronts
  double stream_us;              // one read of the inputs

  double steps(int waves) const { return std::ceil(rows / (waves * (double)rps)) * chunks; }
  // Estimate of one fused pass in microseconds: the workgroups of a round take their
  // steps one after the other or wait for the memory; the last round may leave
  // the chip half empty.  Eight wavefronts on a compute unit take a fifth (FP64:
  // two fifths) longer per step than four: full-Jones, 80 intervals of 1.3e5
  // samples, MIXED 1.44 / 1.21 us, FP64 1.46 / 0.92 us.
  double fused_us(int waves) const {
    const int fit_w = std::max(1, fit * 4 / waves);
    const double us = steps(waves) * step_us * (waves <= 4 ? 1.0 : fp64 ? 1.4 : 1.2);
    const int full = n_int / fit_w, rest = n_int - full * fit_w;
    return 12.0 + full * std::max(stream_us * fit_w / n_int, us) +
           (rest ? std::max(stream_us * rest / n_int, us) : 0.0);
  }
};

static PassShape pass_shape(const qc_ctx* ctx, const qc_vis* vis, const qc_term& ta, bool single, const SolveLaunch& L) {
  PassShape S;
  S.n_int = ta.n_gt * ta.n_gf;
  S.n_samples = (double)vis->n_row * vis->n_chan;
  S.rows = (double)vis->n_row / std::max(ta.n_gt, 1);
  S.avg = S.n_samples / std::max(S.n_int, 1);
  const int n_dir = single ? 1 : vis->n_dir;
  const bool lane_rows = !single && L.max_int_chan <= 4 && ta.n_gdir == 1 && !L.left_general;
  S.fp64 = !L.prec_mixed;
  S.wide = !single && (L.left_general || (!L.diag_chain && S.fp64));
  S.rps = single ? (L.rows_per_step > 0 ? L.rows_per_step : 4) : lane_rows ? 64 : 1;
  S.chunks = lane_rows ? L.max_int_chan : std::ceil(L.max_int_chan / (64.0 / S.rps));
  S.step_us = single ? 1.25 : lane_rows ? 10.0 : 1.25 * (1.0 + 0.75 * n_dir);
  S.fit = ctx->n_cu * (S.fp64 ? 2 : single ? 4 : 3);
  const double real = L.vis_is_c128 ? 8.0 : 4.0;
  const double bytes = S.n_samples * (real * (8.0 + 8.0 * n_dir + vis->n_wcorr) + 1.0);
  S.stream_us = bytes / (S.fp64 ? 4.2e6 : 6e6);                  // 6 TB/s, FP64 4.2 TB/s
  return S;
}

// Wavefronts per workgroup of the fused schedule, where the caller has not chosen.
//
// Where the intervals leave the chip room, eight: an interval's pass is a chain of
// steps, and twice the wavefronts halve it.  Measured (whole solves, four / eight):
// 24 diagonal FP64 intervals of 840 samples 0.49 / 0.40 ms, 400 MIXED ones of 3040
// 0.37 / 0.31 ms; 190 full-Jones FP64 ones of 1.2e5 5.2 / 3.9 ms; chains over four
// directions, 64 intervals of 9920 samples 13.5 / 7.7 ms.  Room is one workgroup per
// compute unit, two for the MIXED single-term kernels (400 FP64 ones of 3840
// samples 0.48 / 0.52 ms; 640 MIXED ones of 1.3e5 8.6 / 9.5 ms).
// Where many small intervals wait in line, fewer: each is mostly sums and block
// solves, which a workgroup does at the pace of its barriers, so more intervals at once
// are worth more than a shorter one.  25600 full-Jones MIXED intervals of 112
// samples 5.5 ms with four, 3.7 with two, 3.0 with one; of 480 samples 9.1 / 7.4 / 6.9;
// of 960 8.9 / 7.3 / 7.6 (diagonal FP64 10.5 / 9.3 / 9.1); 12800 of 3968 12.6 /
// 12.5 / 13.4; 1600 of 960 0.58 / 0.55 / 0.80.  A wavefront alone takes up to 16
// steps, two together up to 16 each.
// Levenberg-Marquardt stays at four: its accepted steps hang on the last bits of
// chi^2, which differ with the number of partial sums.
static int fused_waves(const qc_ctx* ctx, const PassShape& S, bool single, bool lm) {
  if (lm) return 4;
  if (S.n_int <= ctx->n_cu * (single && !S.fp64 ? 2 : 1)) return S.wide ? 4 : 8;
  if (single && S.n_int >= 8 * ctx->n_cu) {
    if (S.steps(1) <= 16.0) return 1;
    if (S.steps(2) <= 16.0) return 2;
  }
  return 4;
}

// Values of one part's sums: every block's (qc_interval.h: KindInfo NV, or NV_FB for full
// blocks) and chi^2.
static size_t split_values(const qc_vis* vis, const qc_term& ta, bool left_general) {
  const int nv = left_general ? (ta.type == QC_TERM_DIAGONAL ? 8
                                 : ta.type == QC_TERM_COMPLEX2X2 ? 24 : (ta.type == QC_TERM_DELAY_OFFSET ? 14 : 5))
                              : (ta.type == QC_TERM_DIAGONAL ? 6
                                 : ta.type == QC_TERM_COMPLEX2X2 ? 16 : (ta.type == QC_TERM_DELAY_OFFSET ? 10 : 4));
  return (size_t)vis->n_ant * (ta.n_gdir == 1 ? 1 : 4) * nv + 1;
}

// Parts per interval of a solve (1: the fused schedule), by an estimate of
// one pass of each schedule in microseconds.
//
// Fused: a workgroup takes an interval of its own (PassShape::fused_us).  Split: the
// same work spread over the chip, plus the launches, the sums of the
// parts and an update kernel.  Measured (MI355X, whole solves, fused with four
// wavefronts against split): 35 diagonal intervals of 1.6e5 samples 9.1 / 1.1 ms (eight:
// 5.1); 80 full-Jones ones of 1.3e5 5.5 / 1.5 ms (3.3); 190 FP64 ones of 1.2e5 5.2 /
// 4.1 (3.9); 1100 of them 19.2 / 16.2 ms, 1600 22.0 / 22.0; 640
// diagonal ones 8.6 / 8.9 ms; 400 of 3040 samples 0.37 / 0.49 ms; 4 of 19200
// samples 1.13 / 0.35 ms (0.70); one delay interval of 5.7e5 samples x 3 directions
// 201 / 1.1 ms.  Constants: a step of a lone workgroup takes 1.2-1.4 us in
// the single-term kernels, 3.6-5.1 us in the chain kernels over 3-4
// directions and 9-11 us with one row per lane; a pass with its update costs about
// 12 us beyond its steps fused and 25 us split; FP64 passes read 4.2 TB/s.
// Levenberg-Marquardt keeps to large intervals (2^18 samples on average): its
// accepted steps hang on the last bits of chi^2, which differ between the schedules.
//
// The parts of all intervals together fill whole rounds of the chip: a few
// workgroups over a round run on an empty one.  80 full-Jones intervals take 1.82 ms in
// 13 parts each (1040 workgroups of 1024 at once), 1.50 in 8; 190 FP64 ones 4.47 ms in
// 6 (1140 of 512), 4.07 in 8 (1520).
static int split_parts(const qc_ctx* ctx, const qc_vis* vis, const qc_term& ta, const PassShape& S, int waves, bool lm) {
  const int n_int = S.n_int;
  const bool large = n_int < 4 * ctx->n_cu && S.avg >= (double)(1 << 18);   // split whatever the estimate
  if (lm && !large) return 1;
  if (!large) {
    const double split_us = 25.0 + std::max(S.stream_us, n_int * S.steps(4) * S.step_us / S.fit);
    if (S.fused_us(S.wide ? std::min(waves, 4) : waves) <= 1.1 * split_us + 10.0) return 1;
  }
  const double wg = std::min((double)SPLIT_WG_PER_CU, std::max((double)SPLIT_WG_PER_CU_MIN,
                                                               S.n_samples / SPLIT_PART_SAMPLES / ctx->n_cu));
  const double most = std::max(2.0, std::min(S.rows / SPLIT_MIN_ROWS, S.avg / SPLIT_MIN_SAMPLES));
  // the fewest parts from this number on that leave at most a sixteenth of their
  // last round empty; else the fullest up to twice as many
  const int least = (int)std::max(2.0, std::min(std::floor(wg * ctx->n_cu / n_int), std::floor(most)));
  int parts = least;
  double best = 0.0;
  for (int p = least; p <= std::min(2 * least, (int)most) && best < 0.9375; ++p) {
    const double rounds = (double)n_int * p / S.fit;
    const double full = rounds / std::ceil(rounds);
    if (full > best) {
      best = full;
      parts = p;
    }
  }
  return parts;
}

// Wavefronts' parts of the band pass per gain time: BAND_WAVES_PER_CU of them per compute
// unit, or as many as its LDS holds.
static int band_parts(const qc_ctx* ctx, const qc_vis* vis, const qc_term& ta, int rows) {
  const long long units = (long long)((vis->n_chan + 64 / rows - 1) / (64 / rows)) * ta.n_gt;
  const double rows_per_int = (double)vis->n_row / std::max(ta.n_gt, 1);
  const int fit = (int)(160 * 1024 / band_lds_bytes_for(vis->n_ant, rows));
  const int parts = (int)((long long)std::max(1, std::min(BAND_WAVES_PER_CU, fit)) * ctx->n_cu / units);
  return std::max(2, std::min(parts, (int)std::max(1.0, rows_per_int / 32.0)));
}

// The parts that the memory for their sums allows (split_parts_within).
static int parts_in_memory(const qc_ctx* ctx, int parts, int n_int, size_t values) {
  const size_t held = ctx->d_partials ? ctx->partials_cap * sizeof(double) : 0;
  size_t free_b = 0, total_b = 0;
  if ((double)parts * n_int * (double)values * sizeof(double) > (double)held &&
      hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    free_b = 0;
  }
  return split_parts_within(parts, n_int, values, held, free_b);
}

// Memory of the context that a call can do without (spare_fits); false: the call goes
// without.
static bool spare_memory(qc_ctx* ctx, unsigned char*& ptr, size_t& cap, size_t bytes) {
  if (bytes == 0) return false;
  if (ptr && bytes <= cap) return true;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (!spare_fits(bytes, free_b, total_b)) return false;
  if (grow(ptr, cap, bytes) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// qc_solve_interval; fixed != NULL: the allocation-free form (prepare scratch
// in `fixed`, always the fused schedule, no fixed-factor table, no pointing);
// sky != NULL: the model predicted from point components in the passes
static qc_status solve_interval_impl(qc_ctx* ctx, const qc_vis* vis, qc_term* chain, int32_t n_term,
                                     int32_t active, const qc_solve_opts* opts, qc_solve_stats* stats,
                                     const PrepScratch* fixed, const qc_sky* sky = nullptr,
                                     const double* uvw = nullptr) {
  if (!ctx) return QC_E_ARG;
  if (!opts) return fail(ctx, QC_E_ARG, "opts is NULL");
  if (!chain || n_term <= 0 || active < 0 || active >= n_term)
    return fail(ctx, QC_E_ARG, "active=%d outside the chain of %d terms", active, n_term);
  const int prec_v = enum_value(opts->prec), damp_v = enum_value(opts->damping);
  if (prec_v != QC_PREC_FP64 && prec_v != QC_PREC_MIXED) return fail(ctx, QC_E_ARG, "bad precision %d", prec_v);
  if (damp_v < QC_DAMP_FULL || damp_v > QC_DAMP_LM) return fail(ctx, QC_E_ARG, "bad damping %d", damp_v);
  if (opts->max_iter < 0) return fail(ctx, QC_E_ARG, "max_iter < 0");
  if (vis && prec_v == QC_PREC_MIXED && enum_value(vis->dtype) != QC_C64)
    return fail(ctx, QC_E_ARG, "MIXED precision needs complex64 data");
  hipStream_t s = reinterpret_cast<hipStream_t>(opts->stream);
  ctx->last_stream = s;
  if (fixed && enum_value(chain[active].type) == QC_TERM_POINTING)
    return fail(ctx, QC_E_UNSUPPORTED, "the allocation-free solve takes no active POINTING term");
  if (sky) {
    if (!uvw && vis && vis->n_row > 0) return fail(ctx, QC_E_ARG, "uvw is NULL");
    bool diag = true;
    for (int j = 0; j < n_term; ++j)
      if (enum_value(chain[j].type) == QC_TERM_COMPLEX2X2) diag = false;
    const bool single = vis && n_term == 1 && vis->n_dir == 1 && chain[active].n_gdir == 1;
    if (!single && !diag)
      return fail(ctx, QC_E_UNSUPPORTED, "the predicted model takes a single term or a chain of diagonal terms");
    if (enum_value(chain[active].type) == QC_TERM_POINTING)
      return fail(ctx, QC_E_UNSUPPORTED, "the predicted model takes no active POINTING term");
    if (damp_v == QC_DAMP_LM)
      return fail(ctx, QC_E_UNSUPPORTED, "the predicted model takes no Levenberg-Marquardt damping");
  }
  std::vector<HostMaps> maps;
  qc_status st = prepare(ctx, vis, chain, n_term, active, maps, s, fixed, sky == nullptr);
  if (st != QC_OK) return st;
  SkyArgs sk;
  memset(&sk, 0, sizeof sk);
  if (sky) {
    st = prepare_sky(ctx, sky, vis->n_dir, uvw, s, sk);
    if (st != QC_OK) return st;
  }
  if (chain[active].type == QC_TERM_POINTING) {
    ctx->solve_passes = false;
    return solve_pointing(ctx, vis, chain, n_term, active, opts, stats, s);
  }
  SolveLaunch L;
  memset(&L, 0, sizeof L);
  fill_args(vis, chain, n_term, active, L.vis, L.chain);
  L.vis_is_c128 = vis->dtype == QC_C128;
  L.prec_mixed = opts->prec == QC_PREC_MIXED;
  L.diag_chain = 1;
  for (int j = 0; j < n_term; ++j)
    if (chain[j].type == QC_TERM_COMPLEX2X2) L.diag_chain = 0;
  // A chain of diagonal terms commutes, so its diagonal-chain evaluation takes
  // any left factor (direction-dependent ones and pointing beams included).
  // Otherwise a left factor that is not diagonal, or differs by direction,
  // needs the full per-antenna blocks (eq. jonesfactor, eq. g_derivative_dd).
  L.left_general = 0;
  if (!L.diag_chain)
    for (int j = 0; j < active; ++j)
      if (chain[j].type == QC_TERM_COMPLEX2X2 || chain[j].type == QC_TERM_POINTING || !dmap_constant(maps[j]))
        L.left_general = 1;
  qc_term& ta = chain[active];
  L.gains = reinterpret_cast<double2*>(ta.gains);
  L.params = ta.params;
  L.gflags = ta.gain_flags;
  L.row_lo = fixed ? fixed->rowlo : ctx->d_rowlo;
  L.row_hi = fixed ? fixed->rowhi : ctx->d_rowhi;
  L.chan_lo = fixed ? fixed->chlo : ctx->d_chlo;
  L.chan_hi = fixed ? fixed->chhi : ctx->d_chhi;
  if (stats) {
    L.iters = stats->iters;
    L.converged = stats->converged;
    L.chisq_first = stats->chisq_first;
    L.chisq_last = stats->chisq_last;
    L.restarted = stats->restarted;
  }
  L.chisq_ref = opts->chisq_ref;
  L.sky = sk;
  L.tol = opts->tol;
  L.max_iter = opts->max_iter;
  L.damping = resolve_damping(opts->damping, ta);
  L.err = ctx->d_err;
  L.waves = ctx->waves ? ctx->waves : 4;
  L.waves_auto = 0;
  L.max_int_chan = ctx->max_int_chan;
  L.dir_ident = ta.n_gdir > 1 && ta.n_gdir == vis->n_dir && ta.n_gdir <= 4;
  for (int d = 0; L.dir_ident && d < vis->n_dir; ++d)
    if (maps[active].d_map[d] != d) L.dir_ident = 0;
  L.rows_per_step = ctx->rows_per_step == 8 ? 0 : ctx->rows_per_step;   // 8: the one-channel split only
  // schedule: fused (one workgroup per interval) or split (each interval's rows
  // streamed by several workgroups), by split_parts
  const int n_int = ta.n_gt * ta.n_gf;
  int parts = 1;
  const bool lm = opts->damping == QC_DAMP_LM;
  const bool single_chain = (n_term == 1 && vis->n_dir == 1 && ta.n_gdir == 1);
  // intervals of one channel each, in channel order, for the band pass below
  bool one_chan = ta.type == QC_TERM_DIAGONAL && ctx->max_int_chan == 1 && ta.n_gf == vis->n_chan;
  for (int g = 0; one_chan && g < ta.n_gf; ++g)
    if (ctx->h_clo[g] != g) one_chan = false;
  // diagonal chains: the direction-dependent fixed terms, when all are
  // diagonal gains and at most BAND_MAX_DD, tabulated once per solve for every
  // pass (the band pass takes no other kind).  A pointing term differs by
  // direction through its beam although it has one gain direction.
  L.n_dd = 0;
  L.dd_tabled = !fixed && L.diag_chain && !L.left_general;
  for (int j = 0; L.dd_tabled && j < n_term; ++j) {
    const bool dd = chain[j].n_gdir > 1 || enum_value(chain[j].type) == QC_TERM_POINTING;
    if (j == active || !dd) continue;
    if (chain[j].type != QC_TERM_DIAGONAL || L.n_dd == BAND_MAX_DD) L.dd_tabled = 0;
    else L.dd_term[L.n_dd++] = j;
  }
  if (!L.dd_tabled) L.n_dd = 0;
  // A diagonal chain whose active term has one gain direction: folded into one
  // model where several passes will read it, the model is stored as it is
  // computed (MIXED of complex64, FP64 of complex128) and the memory is there.
  // (Levenberg-Marquardt keeps its arithmetic.  Intervals of up to 4 channels keep
  // the one-row-per-lane kernel of chains unless the band pass takes them: the
  // single-term kernels read a row's channels on 16 lanes.)
  bool fold = !fixed && !sky && !lm && L.diag_chain && !single_chain && ta.n_gdir == 1 && opts->max_iter >= 3 &&
              L.prec_mixed != L.vis_is_c128;
  // intervals of one channel each, in channel order, on a diagonal chain with
  // one gain direction: the split pass over 16 channels per wavefront
  const bool band_fits = !sky && L.diag_chain && !L.left_general && one_chan && ta.n_gdir == 1 && vis->n_row < (1LL << 31) &&
                         band_lds_bytes_for(vis->n_ant, 8) <= (L.prec_mixed ? 160 : 64) * 1024;
  bool band = band_fits && (L.dd_tabled || fold);
  fold = fold && (band || ctx->max_int_chan > 4);
  // 4 rows x 16 channels per step, or as asked; 8 x 8, whose LDS slots are half as
  // large, where those do not fit and, in MIXED, where they leave a compute unit
  // fewer than six wavefronts (solves of 10 updates, 4 x 16 / 8 x 8: 28 antennas, 100
  // times x 256 channels 2.40 / 2.57 ms; 64, 100 x 512 26.0 / 19.2; four directions
  // folded, 60 x 256 9.6 / 7.3; FP32 slots took 17.1 and 6.8 in 4 x 16)
  const size_t rows4 = band_lds_bytes_for(vis->n_ant, 4);
  L.band_rows = (ctx->rows_per_step == 8 || rows4 > 64 * 1024 ||
                 (L.prec_mixed && ctx->rows_per_step != 4 && rows4 > 160 * 1024 / 6)) ? 8 : 4;
  if (lm && ta.type == QC_TERM_DELAY_OFFSET)
    return fail(ctx, QC_E_UNSUPPORTED, "Levenberg-Marquardt takes no delay-and-offset term");
  int waves = 4;
  auto choose = [&]() {
    const bool single = single_chain || (fold && !band);
    const PassShape shape = pass_shape(ctx, vis, ta, single, L);
    waves = ctx->waves ? ctx->waves : fused_waves(ctx, shape, single, lm);
    parts = 1;
    if (fixed) return;                         // the split schedule's state is context memory
    if (ctx->split_parts > 1) {
      parts = ctx->split_parts;
    } else if (ctx->split_parts == 0 && !opts->chisq_ref && n_int > 0) {
      parts = split_parts(ctx, vis, ta, shape, waves, lm);
      if (parts > 1 && band) parts = band_parts(ctx, vis, ta, L.band_rows);
      if (parts > 1) parts = parts_in_memory(ctx, parts, n_int, split_values(vis, ta, L.left_general != 0));
    }
  };
  choose();
  if (fold && ((band && parts == 1) || !spare_memory(ctx, ctx->d_fold, ctx->fold_cap, chain_fold_bytes(L)))) {
    fold = false;
    band = band_fits && L.dd_tabled;
    choose();
  }
  if (parts > 1 && opts->chisq_ref)
    return fail(ctx, QC_E_UNSUPPORTED, "the split schedule does not take chisq_ref");
  band = band && parts > 1;
  ctx->last_split_parts = parts;
  ctx->last_route = (parts > 1 ? QC_ROUTE_SPLIT : 0) | (fold ? QC_ROUTE_FOLD : 0) | (band ? QC_ROUTE_BAND : 0);
  // diagonal chains: the direction-independent terms other than the active
  // one are fixed during the solve; tabulate their product once
  bool other_di = false;
  for (int j = 0; j < n_term; ++j)
    if (j != active && chain[j].n_gdir == 1) other_di = true;
  const bool want_tab = !fixed && L.diag_chain && !single_chain && other_di;
  L.otab = nullptr;
  if (want_tab) HIP_TRY(ctx, grow(ctx->d_otab, ctx->otab_cap, chain_table_bytes(L)));
  SplitLaunch P;
  if (parts > 1) {
    const int ng = ta.n_gdir == 1 ? 1 : 4;
    const size_t stride = split_values(vis, ta, L.left_general != 0);
    HIP_TRY(ctx, grow(ctx->d_partials, ctx->partials_cap, stride * (size_t)n_int * parts));
    HIP_TRY(ctx, grow(ctx->d_passes, ctx->passes_cap, (size_t)n_int));
    HIP_TRY(ctx, grow(ctx->d_done, ctx->done_cap, (size_t)n_int));
    HIP_TRY(ctx, grow(ctx->d_active, ctx->active_cap, 1));
    HIP_TRY(ctx, grow(ctx->d_dv, ctx->dv_cap, (size_t)n_int * vis->n_ant * ng * 2));
    P.state.dv = ctx->d_dv;
    P.n_part = parts;
    P.partials = ctx->d_partials;
    P.totals = nullptr;
    if (parts > SPLIT_DIRECT_PARTS) {
      HIP_TRY(ctx, grow(ctx->d_totals, ctx->totals_cap, stride * (size_t)n_int));
      P.totals = ctx->d_totals;
    }
    for (hipEvent_t& ev : ctx->ev_pass)
      if (!ev) HIP_TRY(ctx, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    if (!ctx->h_done) {
      HIP_TRY(ctx, hipHostMalloc(reinterpret_cast<void**>(&ctx->h_done), sizeof(int), hipHostMallocCoherent));
      *ctx->h_done = 0;
    }
    P.state.all_done = ctx->h_done;
    P.state.run = ++ctx->split_run;
    P.state.passes = ctx->d_passes;
    P.state.done = ctx->d_done;
    P.state.n_active = ctx->d_active;
    P.state.lm = nullptr;
    P.state.acc = nullptr;
    if (lm) {
      HIP_TRY(ctx, grow(ctx->d_lm, ctx->lm_cap, (size_t)n_int * LM_STATE));
      HIP_TRY(ctx, grow(ctx->d_acc, ctx->acc_cap, (size_t)n_int * vis->n_ant * ng * 4));
      P.state.lm = ctx->d_lm;
      P.state.acc = ctx->d_acc;
    }
  }
  size_t dd_off[BAND_MAX_DD] = {0, 0};
  L.ptab = nullptr;
  if (parts > 1 && (single_chain || fold) && !sky && !L.prec_mixed &&
      (ta.type == QC_TERM_DELAY || ta.type == QC_TERM_DELAY_OFFSET)) {
    const size_t bytes = sizeof(double) * 4 * (size_t)n_int * vis->n_ant * ctx->max_int_chan;
    if (spare_memory(ctx, ctx->d_ptab, ctx->ptab_cap, bytes)) L.ptab = ctx->d_ptab;
  }
  L.band_gains = nullptr;
  if (band && (fold || single_chain)) {
    HIP_TRY(ctx, grow(ctx->d_bandg, ctx->bandg_cap, band_gains_bytes(L)));
    L.band_gains = ctx->d_bandg;
  } else if (band) {
    HIP_TRY(ctx, grow(ctx->d_band, ctx->band_cap, (size_t)std::max<long long>(vis->n_row, 1)));
  }
  if (L.n_dd > 0) {
    size_t dd_bytes = 0;
    for (int j = 0; j < L.n_dd; ++j) {
      dd_off[j] = dd_bytes;
      dd_bytes += (dd_table_bytes(L, L.dd_term[j]) + 255) / 256 * 256;
    }
    HIP_TRY(ctx, grow(ctx->d_ddtab, ctx->ddtab_cap, dd_bytes));
  }
  size_t lds = 0;
  hipError_t e = hipSuccess;
  HIP_TRY(ctx, hipEventRecord(ctx->ev0, s));
  if (want_tab) {
    e = launch_chain_table(L, ctx->d_otab, s);
    L.otab = ctx->d_otab;
  }
  if (band && !L.band_gains && e == hipSuccess) {
    e = launch_band_steps(L, parts, L.band_rows, ctx->d_band, s);
    L.band_steps = ctx->d_band;
  }
  for (int j = 0; j < L.n_dd && e == hipSuccess; ++j) {
    L.dd_tab[j] = ctx->d_ddtab + dd_off[j];
    e = launch_dd_table(L, L.dd_term[j], ctx->d_ddtab + dd_off[j], s);
  }
  if (fold && e == hipSuccess) {
    e = launch_chain_fold(L, ctx->d_fold, s);
    // from here the solve is that of the active term alone over the folded model
    L.vis.model = ctx->d_fold;
    L.vis.n_dir = 1;
    L.chain.t[0] = L.chain.t[active];
    L.chain.active = 0;
    L.chain.n_term = 1;
    L.otab = nullptr;
    L.n_dd = 0;
    L.dd_tabled = 1;
    L.dir_ident = 0;
  }
  if (e != hipSuccess) {
    // reported below
  } else if (parts <= 1) {
    L.waves = waves;
    L.waves_auto = ctx->waves == 0;
    e = launch_solve(L, nullptr, s, &lds);
  } else {
    P.phase = 0;
    e = launch_solve(L, &P, s, &lds);
    P.phase = 1;
    // a pass per update; with LM a rejected attempt takes one more pass
    const int max_rounds = lm ? 2 * opts->max_iter + 2 : opts->max_iter + 1;
    for (int k = 0; k < max_rounds && e == hipSuccess; ++k) {
      e = launch_solve(L, &P, s, &lds);
      if (e != hipSuccess) break;
      // the next pass is launched while this one runs: the host waits for the
      // pass before it (a pass over intervals that are all done returns at once)
      HIP_TRY(ctx, hipEventRecord(ctx->ev_pass[k & 1], s));
      if (k > 0) HIP_TRY(ctx, hipEventSynchronize(ctx->ev_pass[(k - 1) & 1]));
      if (__atomic_load_n(ctx->h_done, __ATOMIC_ACQUIRE) == P.state.run) break;
    }
  }
  if (e != hipSuccess) {
    ctx->timed = false;
    if (lds > 160 * 1024)
      return fail(ctx, QC_E_UNSUPPORTED, "per-interval state needs %zu B of LDS (n_ant=%d)", lds, vis->n_ant);
    return fail(ctx, QC_E_DEVICE, "solve launch: %s", hipGetErrorString(e));
  }
  if (!fixed) ctx->solve_passes = parts > 1;
  HIP_TRY(ctx, call_end(ctx, s, fixed ? nullptr : &ctx->solve_use));
  return QC_OK;
}

extern "C" {

qc_status qc_solve_interval(qc_ctx* ctx, const qc_vis* vis, qc_term* chain, int32_t n_term, int32_t active,
                            const qc_solve_opts* opts, qc_solve_stats* stats) {
  return solve_interval_impl(ctx, vis, chain, n_term, active, opts, stats, nullptr);
}

qc_status qc_solve_interval_sky(qc_ctx* ctx, const qc_vis* vis, const qc_sky* sky, const double* uvw,
                                qc_term* chain, int32_t n_term, int32_t active, const qc_solve_opts* opts,
                                qc_solve_stats* stats) {
  if (!ctx) return QC_E_ARG;
  if (!sky) return fail(ctx, QC_E_ARG, "sky is NULL");
  return solve_interval_impl(ctx, vis, chain, n_term, active, opts, stats, nullptr, sky, uvw);
}

qc_status qc_solve_interval_static(qc_ctx* ctx, const qc_vis* vis, qc_term* chain, int32_t n_term,
                                   int32_t active, const qc_solve_opts* opts, qc_solve_stats* stats) {
  if (!ctx) return QC_E_ARG;
  if (!chain || n_term <= 0 || active < 0 || active >= n_term)
    return fail(ctx, QC_E_ARG, "active=%d outside the chain of %d terms", active, n_term);
  if (!ctx->static_scratch) return fail(ctx, QC_E_DEVICE, "no scratch array on device %d", ctx->device);
  PrepScratch sc;
  const size_t need = carve_static(ctx->static_scratch, vis, chain[active], sc);
  if (need > QC_STATIC_SCRATCH_BYTES)
    return fail(ctx, QC_E_UNSUPPORTED, "the allocation-free solve needs %zu B of scratch, more than its %d B",
                need, (int)QC_STATIC_SCRATCH_BYTES);
  return solve_interval_impl(ctx, vis, chain, n_term, active, opts, stats, &sc);
}

int32_t qc_ctx_last_split(const qc_ctx* ctx) { return ctx ? ctx->last_split_parts : -1; }

int32_t qc_ctx_last_route(const qc_ctx* ctx) { return ctx ? ctx->last_route : -1; }

qc_status qc_ctx_set_split(qc_ctx* ctx, int32_t parts) {
  if (!ctx) return QC_E_ARG;
  if (parts < 0) return fail(ctx, QC_E_ARG, "parts must be >= 0");
  ctx->split_parts = parts;
  return QC_OK;
}

qc_status qc_ctx_set_tile(qc_ctx* ctx, int32_t waves, int32_t rows_per_step) {
  if (!ctx) return QC_E_ARG;
  if (waves != 0 && waves != 1 && waves != 2 && waves != 4 && waves != 8)
    return fail(ctx, QC_E_ARG, "waves must be 1, 2, 4 or 8 (0 = default)");
  if (rows_per_step != 0 && rows_per_step != 1 && rows_per_step != 2 && rows_per_step != 4 && rows_per_step != 8)
    return fail(ctx, QC_E_ARG, "rows_per_step must be 1, 2, 4 or 8 (0 = from the interval width)");
  ctx->waves = waves;
  ctx->rows_per_step = rows_per_step;
  return QC_OK;
}

qc_status qc_solve_chain(qc_ctx* ctx, const qc_vis* vis, qc_term* chain, int32_t n_term, int32_t n_epoch,
                         const qc_solve_opts* opts, qc_solve_stats* stats) {
  if (!ctx) return QC_E_ARG;
  if (n_epoch < 0) return fail(ctx, QC_E_ARG, "n_epoch < 0");
  for (int e = 0; e < n_epoch; ++e) {
    for (int n = 0; n < n_term; ++n) {
      qc_solve_stats* st = stats ? &stats[(size_t)e * n_term + n] : nullptr;
      qc_status s = qc_solve_interval(ctx, vis, chain, n_term, n, opts, st);
      if (s != QC_OK) return s;
    }
  }
  return QC_OK;
}

qc_status qc_solve_chain_robust(qc_ctx* ctx, const qc_vis* vis, qc_term* chain, int32_t n_term, int32_t n_epoch,
                                const qc_solve_opts* opts, double nu, void* resid_work, void* weight_work,
                                qc_solve_stats* stats) {
  if (!ctx) return QC_E_ARG;
  if (!vis || !opts) return fail(ctx, QC_E_ARG, "vis or opts is NULL");
  if (n_epoch < 0) return fail(ctx, QC_E_ARG, "n_epoch < 0");
  if (!(nu > 0.0) || !std::isfinite(nu)) return fail(ctx, QC_E_ARG, "nu must be finite and > 0");
  if (n_epoch > 1 && vis->n_row > 0 && (!resid_work || !weight_work))
    return fail(ctx, QC_E_ARG, "resid_work or weight_work is NULL");
  qc_vis wv = *vis;                            // the weights of the current epoch
  for (int e = 0; e < n_epoch; ++e) {
    for (int n = 0; n < n_term; ++n) {
      qc_solve_stats* st = stats ? &stats[(size_t)e * n_term + n] : nullptr;
      qc_status s = qc_solve_interval(ctx, &wv, chain, n_term, n, opts, st);
      if (s != QC_OK) return s;
    }
    if (e + 1 < n_epoch) {
      // the residual of the whole chain, then weights from the prior ones
      qc_status s = qc_residual(ctx, vis, chain, n_term, nullptr, resid_work, opts->stream);
      if (s != QC_OK) return s;
      s = qc_robust_weights(ctx, vis, resid_work, nu, weight_work, nullptr, opts->stream);
      if (s != QC_OK) return s;
      wv.weight = weight_work;
    }
  }
  return QC_OK;
}

qc_status qc_delay_init(qc_ctx* ctx, const qc_vis* vis, qc_term* k_term, int32_t ref_ant, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!k_term) return fail(ctx, QC_E_ARG, "term is NULL");
  if (k_term->type != QC_TERM_DELAY && k_term->type != QC_TERM_DELAY_OFFSET)
    return fail(ctx, QC_E_ARG, "qc_delay_init needs a DELAY or DELAY_OFFSET term");
  if (!vis) return fail(ctx, QC_E_ARG, "vis is NULL");
  if (ref_ant < 0 || ref_ant >= vis->n_ant) return fail(ctx, QC_E_ARG, "ref_ant=%d outside [0,%d)", ref_ant, vis->n_ant);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  std::vector<HostMaps> maps;
  qc_status st = prepare(ctx, vis, k_term, 1, 0, maps, s);
  if (st != QC_OK) return st;
  DelayInitLaunch L;
  memset(&L, 0, sizeof L);
  ChainArgs ca;
  fill_args(vis, k_term, 1, 0, L.vis, ca);
  L.vis_is_c128 = vis->dtype == QC_C128;
  L.offset = k_term->type == QC_TERM_DELAY_OFFSET ? 1 : 0;
  L.n_gt = k_term->n_gt;
  L.n_gf = k_term->n_gf;
  L.n_gdir = k_term->n_gdir;
  L.ref_ant = ref_ant;
  L.row_lo = ctx->d_rowlo;
  L.row_hi = ctx->d_rowhi;
  L.chan_lo = ctx->d_chlo;
  L.chan_hi = ctx->d_chhi;
  L.params = k_term->params;
  L.max_chan = ctx->max_int_chan;
  L.fft = delay_init_lds(L.max_chan, true) <= 64 * 1024;     // up to 1024 channels per interval
  if (delay_init_lds(L.max_chan, L.fft != 0) > 64 * 1024)
    return fail(ctx, QC_E_UNSUPPORTED, "delay interval of %d channels exceeds the LDS budget", ctx->max_int_chan);
  HIP_TRY(ctx, launch_delay_init(L, s));
  return QC_OK;
}

qc_status qc_ws_features(qc_ctx* ctx, const qc_vis* vis, const qc_term* layout, float* feat, double* chisq_unit,
                         int32_t ref_ant, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!layout || !feat) return fail(ctx, QC_E_ARG, "layout or feat is NULL");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  std::vector<HostMaps> maps;
  qc_status st = prepare(ctx, vis, layout, 1, 0, maps, s);
  if (st != QC_OK) return st;
  FeatLaunch L;
  memset(&L, 0, sizeof L);
  ChainArgs ca;
  fill_args(vis, layout, 1, 0, L.vis, ca);
  L.vis_is_c128 = vis->dtype == QC_C128;
  L.n_gt = layout->n_gt;
  L.n_gf = layout->n_gf;
  L.row_lo = ctx->d_rowlo;
  L.row_hi = ctx->d_rowhi;
  L.chan_lo = ctx->d_chlo;
  L.chan_hi = ctx->d_chhi;
  L.feat = feat;
  L.feat_stride = vis->n_ant * 8;
  L.chisq_unit = chisq_unit;
  if (ref_ant >= vis->n_ant) return fail(ctx, QC_E_ARG, "ref_ant=%d outside [0,%d)", ref_ant, vis->n_ant);
  L.ref_ant = ref_ant;
  hipError_t e = launch_ws_features(L, 4, s);
  if (e == hipErrorInvalidValue) return fail(ctx, QC_E_UNSUPPORTED, "too many antennas for the feature pass");
  HIP_TRY(ctx, e);
  return QC_OK;
}

static qc_status check_mlp(qc_ctx* ctx, int batch, int n_in, int n_hid, int n_out) {
  if (batch <= 0 || n_in <= 0 || n_hid <= 0 || n_out <= 0)
    return fail(ctx, QC_E_ARG, "bad MLP shape batch=%d in=%d hid=%d out=%d", batch, n_in, n_hid, n_out);
  return QC_OK;
}

qc_status qc_mlp_forward(qc_ctx* ctx, const float* params, const float* x, int32_t batch, int32_t n_in,
                         int32_t n_hid, int32_t n_out, float* y, float* pre, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!params || !x || !y || !pre) return fail(ctx, QC_E_ARG, "a pointer is NULL");
  qc_status st = check_mlp(ctx, batch, n_in, n_hid, n_out);
  if (st != QC_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  const float* W1 = params;
  const float* b1 = W1 + (size_t)n_hid * n_in;
  const float* W2 = b1 + n_hid;
  const float* b2 = W2 + (size_t)n_out * n_hid;
  HIP_TRY(ctx, launch_linear_fwd(x, W1, b1, pre, batch, n_in, n_hid, 0, s));
  HIP_TRY(ctx, launch_linear_fwd(pre, W2, b2, y, batch, n_hid, n_out, 1, s));
  return QC_OK;
}

qc_status qc_mlp_backward(qc_ctx* ctx, const float* params, const float* x, const float* pre, const float* dy,
                          int32_t batch, int32_t n_in, int32_t n_hid, int32_t n_out, float* grad, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!params || !x || !pre || !dy || !grad) return fail(ctx, QC_E_ARG, "a pointer is NULL");
  qc_status st = check_mlp(ctx, batch, n_in, n_hid, n_out);
  if (st != QC_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  HIP_TRY(ctx, grow(ctx->d_dh, ctx->dh_cap, (size_t)batch * n_hid));
  const float* W2 = params + (size_t)n_hid * n_in + n_hid;
  float* gW1 = grad;
  float* gb1 = gW1 + (size_t)n_hid * n_in;
  float* gW2 = gb1 + n_hid;
  float* gb2 = gW2 + (size_t)n_out * n_hid;
  HIP_TRY(ctx, launch_linear_bwd_out(pre, dy, W2, gW2, gb2, ctx->d_dh, batch, n_hid, n_out, s));
  HIP_TRY(ctx, launch_linear_bwd_w(x, ctx->d_dh, gW1, gb1, batch, n_in, n_hid, 0, s));
  return QC_OK;
}

qc_status qc_adam_step(qc_ctx* ctx, float* params, const float* grad, float* m, float* v, int32_t n, float lr,
                       float b1, float b2, float eps, int32_t step, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!params || !grad || !m || !v || n <= 0 || step <= 0) return fail(ctx, QC_E_ARG, "bad Adam arguments");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  HIP_TRY(ctx, launch_adam(params, grad, m, v, n, lr, b1, b2, eps, step, s));
  return QC_OK;
}

qc_status qc_mse_grad(qc_ctx* ctx, const float* y, const float* t, int32_t n, float* dy, float* loss, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!y || !t || !dy || n <= 0) return fail(ctx, QC_E_ARG, "bad MSE arguments");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  HIP_TRY(ctx, launch_mse(y, t, dy, loss, n, s));
  return QC_OK;
}

qc_status qc_ws_gains(qc_ctx* ctx, const float* y, int32_t n_int, int32_t n_ant, void* gains, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!y || !gains || n_int < 0 || n_ant <= 0) return fail(ctx, QC_E_ARG, "bad warm-start gain arguments");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  HIP_TRY(ctx, launch_ws_gains(y, n_ant * 4, n_int, n_ant, reinterpret_cast<double2*>(gains), s));
  return QC_OK;
}

qc_status qc_ws_labels(qc_ctx* ctx, const void* gains, int32_t n_int, int32_t n_ant, int32_t ref_ant, float* y,
                       void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!gains || !y || n_int < 0 || n_ant <= 0 || ref_ant < 0 || ref_ant >= n_ant)
    return fail(ctx, QC_E_ARG, "bad warm-start label arguments");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  HIP_TRY(ctx, launch_ws_labels(reinterpret_cast<const double2*>(gains), n_int, n_ant, ref_ant, y, s));
  return QC_OK;
}

// Whether the outputs read the direction-independent chain from a table.  It
// pays where a sample's chain takes more than one gain block that the wavefront's
// lanes share: several such terms (residual of a K.B.G.dE chain over 4
// directions, 64 antennas, 60 times x 256 channels: 1969 -> 1582 us), complex64
// outputs through solutions narrower than 16 channels (one per channel, 40 x
// 512: residual 1425 -> 826 us, CORRECT 1222 -> 623, weights 938 -> 387; their
// FP64 blocks of 64 bytes lie one per lane), complex128 ones through phasors.  It
// does not for one delay term in complex64 (CORRECT 1298 against 1398 us with a
// table) nor for 32-channel solutions in complex128 (251 against 329 us), whose
// entries are as long as the gain blocks.  The baselines must outnumber the
// antennas enough to pay for it (four rows per time and antenna), and it stays
// below OUT_TABLE_BYTES.  A full product is tabulated only where every term is
// direction independent.
constexpr size_t OUT_TABLE_BYTES = (size_t)1 << 30;
static bool out_table_pays(const OutputLaunch& L, const qc_vis* vis, const qc_term* chain, int n_term,
                           const std::vector<HostMaps>& maps) {
  constexpr int NARROW = 16;
  int di = 0;
  bool costly = false;
  for (int j = 0; j < n_term; ++j) {
    if (L.chain.t[j].n_gdir > 1) {
      if (!L.diag_chain) return false;
      continue;
    }
    ++di;
    if (L.vis_is_c128) {
      if (chain[j].type != QC_TERM_DIAGONAL && chain[j].type != QC_TERM_COMPLEX2X2 &&
          chain[j].type != QC_TERM_AMPLITUDE)
        costly = true;
    } else {
      // (f_map does not decrease) a gain frequency of fewer than NARROW channels, but the last
      int first = 0;
      for (int c = 1; c < vis->n_chan && !costly; ++c) {
        if (maps[j].f_map[c] == maps[j].f_map[c - 1]) continue;
        costly = c - first < NARROW;
        first = c;
      }
    }
  }
  if (di == 0 || !(costly || di > 1)) return false;
  return vis->n_row >= 4LL * vis->n_time * vis->n_ant && out_table_bytes(L) <= OUT_TABLE_BYTES;
}

static qc_status outputs_common(qc_ctx* ctx, const qc_vis* vis, const qc_term* chain, int32_t n_term, int mode,
                                const uint8_t* dir_mask, void* out, void* stream, const qc_sky* sky = nullptr,
                                const double* uvw = nullptr) {
  if (!ctx) return QC_E_ARG;
  if (!out) return fail(ctx, QC_E_ARG, "out is NULL");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ctx->last_stream = s;
  if (sky && !uvw && vis && vis->n_row > 0) return fail(ctx, QC_E_ARG, "uvw is NULL");
  std::vector<HostMaps> maps;
  qc_status st = prepare(ctx, vis, chain, n_term, -1, maps, s, nullptr, sky == nullptr);
  if (st != QC_OK) return st;
  SkyArgs sk;
  memset(&sk, 0, sizeof sk);
  if (sky) {
    st = prepare_sky(ctx, sky, vis->n_dir, uvw, s, sk);
    if (st != QC_OK) return st;
  }
  if (mode == 1 || mode == 3) {
    for (int j = 0; j < n_term; ++j)
      if (!dmap_constant(maps[j]) || chain[j].type == QC_TERM_POINTING)
        return fail(ctx, QC_E_ARG, "%s needs a direction-independent chain (term %d)",
                    mode == 1 ? "CORRECT" : "corrected weights", j);
  }
  OutputLaunch L;
  memset(&L, 0, sizeof L);
  fill_args(vis, chain, n_term, 0, L.vis, L.chain);
  L.vis_is_c128 = vis->dtype == QC_C128;
  L.mode = mode;
  L.diag_chain = 1;
  for (int j = 0; j < n_term; ++j)
    if (chain[j].type == QC_TERM_COMPLEX2X2) L.diag_chain = 0;
  unsigned mask = 0;
  for (int d = 0; d < vis->n_dir; ++d)
    if (!dir_mask || dir_mask[d]) mask |= 1u << d;
  L.dir_mask = mask;
  L.out = out;
  L.w_vec = mode == 3 && vis->n_wcorr == 4 && reinterpret_cast<uintptr_t>(vis->weight) % 16 == 0 &&
            reinterpret_cast<uintptr_t>(out) % 16 == 0;
  L.sky = sk;
  L.tab = nullptr;
  void* table = nullptr;
  if (!sky && out_table_pays(L, vis, chain, n_term, maps)) {
    // (without memory for it the chain is formed per sample)
    if (spare_memory(ctx, ctx->d_outtab, ctx->outtab_cap, out_table_bytes(L))) table = ctx->d_outtab;
  }
  HIP_TRY(ctx, hipEventRecord(ctx->ev0, s));
  if (table) {
    HIP_TRY(ctx, scratch_take(ctx->outtab_use, s));
    HIP_TRY(ctx, launch_out_table(L, table, s));
    L.tab = table;
  }
  HIP_TRY(ctx, launch_outputs(L, s));
  HIP_TRY(ctx, call_end(ctx, s, table ? &ctx->outtab_use : nullptr));
  return QC_OK;
}

qc_status qc_apply_gains(qc_ctx* ctx, const qc_vis* vis, const qc_term* chain, int32_t n_term,
                         qc_apply_mode mode, const uint8_t* dir_mask, void* out, void* stream) {
  const int mode_v = enum_value(mode);
  if (mode_v != QC_CORRUPT && mode_v != QC_CORRECT) return fail(ctx, QC_E_ARG, "bad apply mode %d", mode_v);
  return outputs_common(ctx, vis, chain, n_term, mode == QC_CORRECT ? 1 : 0, dir_mask, out, stream);
}

qc_status qc_residual(qc_ctx* ctx, const qc_vis* vis, const qc_term* chain, int32_t n_term,
                      const uint8_t* dir_mask, void* out, void* stream) {
  return outputs_common(ctx, vis, chain, n_term, 2, dir_mask, out, stream);
}

qc_status qc_corrected_weights(qc_ctx* ctx, const qc_vis* vis, const qc_term* chain, int32_t n_term,
                               void* weight_out, void* stream) {
  return outputs_common(ctx, vis, chain, n_term, 3, nullptr, weight_out, stream);
}

qc_status qc_residual_sky(qc_ctx* ctx, const qc_vis* vis, const qc_sky* sky, const double* uvw,
                          const qc_term* chain, int32_t n_term, const uint8_t* dir_mask, void* out, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!sky) return fail(ctx, QC_E_ARG, "sky is NULL");
  return outputs_common(ctx, vis, chain, n_term, 2, dir_mask, out, stream, sky, uvw);
}

qc_status qc_corrupt_sky(qc_ctx* ctx, const qc_vis* vis, const qc_sky* sky, const double* uvw,
                         const qc_term* chain, int32_t n_term, const uint8_t* dir_mask, void* out, void* stream) {
  if (!ctx) return QC_E_ARG;
  if (!sky) return fail(ctx, QC_E_ARG, "sky is NULL");
  return outputs_common(ctx, vis, chain, n_term, 0, dir_mask, out, stream, sky, uvw);
}

}  // extern "C"
