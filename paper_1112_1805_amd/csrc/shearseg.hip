// Host side of the shearlet-segmentation library: plan (filter bank, its pruned layout
// and the column work lists on the device), workspace layout, launch orchestration of the
// ADMM of Section 3, and the C ABI declared in include/shearseg.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "host.hpp"
#include "misc.hpp"
#include "tv_launch.hpp"
#include "nl.hpp"
#include "nl_launch.hpp"

thread_local shs::Recorder* shs::g_rec = nullptr;

namespace {

thread_local std::string g_err;

shs_status fail(shs_status s, const std::string& msg) {
  g_err = msg;
  return s;
}

#define HIPCHK(expr)                                                                      \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess) return fail(SHS_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

#define LAUNCHCHK(what)                                                                   \
  do {                                                                                    \
    hipError_t e_ = hipGetLastError();                                                    \
    if (e_ != hipSuccess) return fail(SHS_E_DEVICE, std::string("launch ") + what + ": " + hipGetErrorString(e_)); \
  } while (0)

// Makes the plan's device current for the duration of a call and restores the caller's.
struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// ---------------------------------------------------------------- kernel timing
enum KClass {
  KC_ROW_SOLVE, KC_COL_SYN, KC_COL_ANA, KC_COL_FINAL, KC_COL_FWD, KC_ROW_C2R, KC_ROW_R2C, KC_ROW_PRIME,
  KC_ROW_ENERGY, KC_MID, KC_REDUCE, KC_OTHER, KC_BATCH, KC_ROW_SHRINK, KC_ROW_PD, KC_TV_RHS, KC_TV_UPDATE,
  KC_COL_SOLVE, KC_NL_DUAL, KC_NL_PRIMAL, KC_COUNT
};
const char* const kKClassName[KC_COUNT] = {"row_solve", "col_syn", "col_ana", "col_final", "col_fwd", "row_c2r",
                                           "row_r2c", "row_prime", "row_energy", "pixel", "reduce", "other",
                                           "batch_solve", "row_shrink", "row_pd", "tv_rhs", "tv_update",
                                           "col_solve", "nl_dual", "nl_primal"};

struct Prof {
  std::mutex mu;
  bool on = false;
  uint32_t mask = ~0u;                 // kernel classes that are timed (bit per class)
  std::vector<hipEvent_t> pool;        // reused across sessions
  size_t used = 0;
  std::vector<int> cls;                // class of event pair i (events 2i, 2i+1)
};
Prof& prof() {
  static Prof p;
  return p;
}
bool profiling_on() {
  Prof& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  return P.on;
}
// Set while a batch graph is being captured: no timing events inside graphs.
thread_local int g_capturing = 0;
struct CaptureScope {
  CaptureScope() { ++g_capturing; }
  ~CaptureScope() { --g_capturing; }
};

// Brackets the launches made during its lifetime with HIP events on stream s (when on).
struct Timed {
  hipStream_t s;
  hipEvent_t stop = nullptr;
  Timed(hipStream_t s_, int cls) : s(s_) {
    Prof& P = prof();
    if (!P.on || g_capturing || !((P.mask >> cls) & 1u)) return;
    std::lock_guard<std::mutex> g(P.mu);
    while (P.pool.size() < P.used + 2) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return;
      P.pool.push_back(e);
    }
    hipEvent_t start = P.pool[P.used];
    stop = P.pool[P.used + 1];
    P.used += 2;
    P.cls.push_back(cls);
    (void)hipEventRecord(start, s);
  }
  ~Timed() {
    if (stop) (void)hipEventRecord(stop, s);
  }
};

size_t store_bytes(int store) { return store == SHS_STORE_F32 ? 4 : 2; }

template <template <int> class F>
int by_size(int n) {
  switch (n) {
    case 64: return F<64>::value;
    case 128: return F<128>::value;
    case 256: return F<256>::value;
    case 512: return F<512>::value;
    case 1024: return F<1024>::value;
    case 2048: return F<2048>::value;
  }
  return 0;
}
template <int N> struct RpbOf { static constexpr int value = RowGeom<N>::RPB; };

// Stage twiddle table of fft_run<L, R, RM> (thread read order), copied from the base table
// exp(-2 pi i m / NT) so both hold identical values.
template <int L, int R, int RM>
void fill_stage_tw(const std::vector<float2>& tw, int NT, float2* out) {
  constexpr int T = L / R;
  const int step = NT / L;
  for (int r = 1; r < R; ++r)
    for (int t = 0; t < T; ++t) out[(r - 1) * T + t] = tw[(r * t * step) % NT];
  for (int r = 1; r < RM; ++r)
    for (int tr = 0; tr < R; ++tr) out[(R - 1) * T + (r - 1) * R + tr] = tw[(r * tr * (L / (R * RM)) * step) % NT];
}
template <int N>
void fill_plan_tw(std::vector<float2>& tw) {
  tw.resize(tw_table_size<N>());
  fill_stage_tw<N / 2, RowGeom<N>::R, RowGeom<N>::RM>(tw, N, tw.data() + row_sw_off<N>());
  fill_stage_tw<N, ColGeom<N>::R, ColGeom<N>::RM>(tw, N, tw.data() + col_sw_off<N>());
}
// Stage table of a mixed-radix transform of length L (gstage): W_{Ns R}^{i k} at
// i Ns + k - 1, copied from the base table of NT = L * step entries.
void fill_stage_tw_g(const FftPlan& pl, const std::vector<float2>& tw, int NT, float2* out) {
  const int L = pl.L, step = NT / L;
  for (int e = 0; e < L; ++e) out[e] = tw[0];
  int Ns = 1;
  for (int s = 0; s < pl.ns; ++s) {
    const int R = pl.radix[s];
    for (int i = 1; i < R; ++i)
      for (int k = 0; k < Ns; ++k)
        if (Ns > 1) out[i * Ns + k - 1] = tw[(long long)i * k * (L / (Ns * R)) * step % NT];
    Ns *= R;
  }
}
// exp(-2 pi i m / n), m < n, from double precision.
std::vector<float2> base_twiddles(int n) {
  std::vector<float2> tw(n);
  for (int m = 0; m < n; ++m) {
    const double a = -2.0 * M_PI * double(m) / double(n);
    tw[m] = make_float2(float(std::cos(a)), float(std::sin(a)));
  }
  return tw;
}
// float2 entries of the stage lists, and of all that follows a mixed-radix plan's base table.
constexpr size_t kPlansLen = (3 * sizeof(FftPlan) + sizeof(float2) - 1) / sizeof(float2);
size_t tables_g_len(int n) { return size_t(n) / 2 * 3 + n + kPlansLen; }
// The tables of a mixed-radix plan behind its base table: what a row pass copies
// (exp(-2 pi i k / N) for k <= M = N/2, the inverse and the forward transform's stage tables
// of M - 1 entries each, one unused entry), then the columns' stage table (N), then the three
// stage lists themselves.
void fill_stage_tables_g(const FftPlan& inv, const FftPlan& fwd, const FftPlan& col, const std::vector<float2>& tw,
                         float2* out) {
  const int n = col.L;
  const int M = n / 2;
  std::vector<float2> tab(n);
  std::copy(tw.begin(), tw.begin() + M + 1, out);
  fill_stage_tw_g(inv, tw, n, tab.data());
  std::copy(tab.begin(), tab.begin() + M - 1, out + M + 1);
  fill_stage_tw_g(fwd, tw, n, tab.data());
  std::copy(tab.begin(), tab.begin() + M - 1, out + 2 * M);
  out[3 * M - 1] = tw[0];
  fill_stage_tw_g(col, tw, n, out + 3 * M);
  const FftPlan plans[3] = {inv, fwd, col};
  std::memcpy(out + 3 * M + n, plans, sizeof(plans));
}
void fill_stage_tables(int n, std::vector<float2>& tw) {
  switch (n) {
    case 64: fill_plan_tw<64>(tw); break;
    case 128: fill_plan_tw<128>(tw); break;
    case 256: fill_plan_tw<256>(tw); break;
    case 512: fill_plan_tw<512>(tw); break;
    case 1024: fill_plan_tw<1024>(tw); break;
    case 2048: fill_plan_tw<2048>(tw); break;
  }
}
template <int N> struct WOf { static constexpr int value = ColGeom<N>::W; };

constexpr int kRed1Blocks = 256;
constexpr int kDoneSlot = 7;   // entry of sdev that holds a reduction's count of blocks done
constexpr int kDotBlocks = 1024;

struct Layout {
  size_t g, w, bw, state_end;
  size_t t1, t2, v, z, zs, us, part, parts, red1, sdev, hctr, total;
  long long nrow_parts, nparts;
};

Layout make_layout(const shs_plan* p) {
  Layout L{};
  const size_t n = p->n, nn = n * n, q = p->q, eta = p->eta, P = p->P;
  const size_t plane = n * P;  // float2 per dense spectrum
  size_t off = 0;
  L.g = off;   off = align256(off + q * eta * nn * store_bytes(p->store));
  L.w = off;   off = align256(off + q * nn * 4);
  L.bw = off;  off = align256(off + q * nn * 4);
  L.state_end = off;
  L.t1 = off;  off = align256(off + q * size_t(p->t_ls) * 8);
  L.t2 = off;  off = align256(off + q * size_t(p->t_ls) * 8);
  L.v = off;   off = align256(off + q * plane * 8);
  L.z = off;   off = align256(off + q * plane * 8);
  L.zs = off;  off = align256(off + q * nn * 4);
  L.us = off;  off = align256(off + q * nn * 4);
  L.part = off; off = align256(off + size_t(std::max(p->n_part, 1)) * q * n * p->W * 8);
  L.nrow_parts = (long long)(q * eta) * (n / p->rpb);
  const long long npix = (long long)((nn + 255) / 256);
  L.nparts = L.nrow_parts + std::max<long long>(2 * npix, kDotBlocks);
  L.parts = off; off = align256(off + size_t(L.nparts) * 4 * 8);
  L.red1 = off;  off = align256(off + kRed1Blocks * 4 * 8);
  L.sdev = off;  off = align256(off + 8 * 8);   // totals [0, 5), counters: history row [6], blocks done [7]
  L.hctr = L.sdev + 6 * 8;
  L.total = off;
  return L;
}

bool get_ops_pow2(int n, Ops& o);

bool get_ops(const shs_plan* p, Ops& o) {
  if (p->generic) { o = mixed_ops(); return true; }
  return get_ops_pow2(p->n, o);
}

bool get_ops_pow2(int n, Ops& o) {
  switch (n) {
    case 64: o = pow2_ops<64>(); return true;
    case 128: o = pow2_ops<128>(); return true;
    case 256: o = pow2_ops<256>(); return true;
    case 512: o = pow2_ops<512>(); return true;
    case 1024: o = pow2_ops<1024>(); return true;
    case 2048: o = pow2_ops<2048>(); return true;
  }
  return false;
}

int row_class(int mode) {
  switch (mode) {
    case ROW_SOLVE: return KC_ROW_SOLVE;
    case ROW_C2R: return KC_ROW_C2R;
    case ROW_R2C: return KC_ROW_R2C;
    case ROW_PRIME: return KC_ROW_PRIME;
    case ROW_ENERGY: return KC_ROW_ENERGY;
    case ROW_SHRINK: return KC_ROW_SHRINK;
    case ROW_PD: return KC_ROW_PD;
  }
  return KC_OTHER;
}

// Everything a compute call needs, resolved from plan + workspace.
struct Ctx {
  const shs_plan* p;
  Layout L;
  Ops ops;
  char* ws;
  hipStream_t s;
  FilterWeights fw;
  template <class T> T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

shs_status make_ctx(const shs_plan* p, void* ws, size_t ws_bytes, void* stream, Ctx& c) {
  if (!p) return fail(SHS_E_INVALID, "null plan");
  c.p = p;
  c.L = make_layout(p);
  if (!get_ops(p, c.ops)) return fail(SHS_E_UNSUPPORTED, "unsupported size");
  if (!ws) return fail(SHS_E_WORKSPACE, "null workspace");
  if (ws_bytes < c.L.total)
    return fail(SHS_E_WORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes < required " +
                                     std::to_string(c.L.total));
  if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return fail(SHS_E_WORKSPACE, "workspace must be 256-byte aligned");
  c.ws = static_cast<char*>(ws);
  c.s = static_cast<hipStream_t>(stream);
  std::memset(&c.fw, 0, sizeof(c.fw));
  return SHS_OK;
}

SpecLayout dense_layout(const shs_plan* p) { return SpecLayout{nullptr, (long long)p->n * p->P, 1, p->P}; }
SpecLayout pruned_layout(const shs_plan* p) { return SpecLayout{p->tcol, p->t_ls, p->eta, p->P}; }

void run_row(const Ctx& c, int mode, int store, bool stats, RowParams rp, int channels) {
  rp.tw = c.p->tw;
  rp.eta = c.p->eta;
  rp.real_cs = (long long)c.p->n * c.p->n;
  rp.fw = c.fw;
  rp.partials = c.at<double>(c.L.parts);
  Timed tm(c.s, row_class(mode));
  c.ops.row(c.p, mode, store, stats, rp, channels, c.s);
}

ColParams col_params(const Ctx& c, int labels) {
  const shs_plan* p = c.p;
  ColParams cp{};
  cp.psiw = p->psiw;
  cp.fwin = p->fwin;
  cp.fgeo = p->fgeo;
  cp.tl = pruned_layout(p);
  cp.strips = p->strips_ana;
  cp.part = c.at<float2>(c.L.part);
  cp.tw = p->tw;
  cp.P = p->P;
  cp.eta = p->eta;
  cp.labels = labels;
  cp.nnz = int(p->nnz);
  cp.inv_n2 = 1.0f / (float(p->n) * float(p->n));
  return cp;
}

void run_col(const Ctx& c, int kind, const ColParams& cp, int nblocks, int labels) {
  static const int cls[4] = {KC_COL_FWD, KC_COL_SYN, KC_COL_ANA, KC_COL_FINAL};
  Timed tm(c.s, cls[kind]);
  c.ops.col(c.p, kind, cp, nblocks, labels, c.s);
}

// u-step of the TV model on per-label spectra: Z = V / (1 + eigenvalues) column-wise.
void run_col_solve(const Ctx& c, const ColParams& cp, int labels) {
  Timed tm(c.s, KC_COL_SOLVE);
  c.ops.col_solve(c.p, cp, labels, c.s);
}

// Row spectra V (count dense planes) -> pruned coefficient spectra T1 (count * eta planes).
void enqueue_synthesis_cols(const Ctx& c, int count) {
  const shs_plan* p = c.p;
  ColParams cp = col_params(c, count);
  cp.in = c.at<float2>(c.L.v);
  cp.out = c.at<float2>(c.L.v);          // column FFT in place: V -> U
  // Small plans: the synthesis transforms its columns itself, which saves a launch where launches
  // are what is waited for: 128^2, q = 3 (132 blocks) 4.2 + 4.5 -> 5.7 us, one image of 512^2, q = 1
  // 28.3 -> 25.5 us for the whole forward transform.  The two forms round differently in the last
  // bit, so the choice is the plan's, not the launch's: an image's coefficients do not depend on how
  // many images share its launch.  Up to 256^2 this form is never the slower one (q = 8 at 256^2 40.8
  // against 41.8 us, a batch of 32 images 1,233 against 1,232 us per iteration); larger plans whose
  // launches fill the GPU (four blocks of four waves per CU) keep the separate launch: at 512^2, q = 4
  // (2,024 blocks) both forms take 27 us, at 1024^2, q = 5 (2,795) the separate launch 128 and this
  // 129.  Mixed-radix sides keep it as well: 30 iterations at 360^2, q = 2 took 3.07 ms with it and
  // 3.18 with the transform inside (a longer chain per block, a strip more of LDS).
  cp.fwd = !p->generic && (p->n <= 256 || (long long)p->n_syn * p->q <= 1024) ? 1 : 0;
  if (!cp.fwd) {
    rec_step(BS_FWD);
    run_col(c, COL_FWD, cp, p->NS, count);
  }
  cp.in = c.at<float2>(c.L.v);
  cp.out = c.at<float2>(c.L.t1);
  cp.items = p->items_syn;
  rec_step(BS_SYN);
  run_col(c, COL_SYN, cp, p->n_syn, count);
}

// S: real images [count][N][N] -> pruned coefficient spectra T1.
void enqueue_synthesis(const Ctx& c, const float* real_in, int count) {
  RowParams rp{};
  rp.real_in = real_in;
  rp.spec_out = c.at<float2>(c.L.v);
  rp.lout = dense_layout(c.p);
  run_row(c, ROW_R2C, ST_F32, false, rp, count);
  enqueue_synthesis_cols(c, count);
}

// The middle step of a solver iteration (MID_*): Z -> pixels -> V.
void run_mid(const Ctx& c, int mode, const float* d_s, float gamma, bool have_z, bool stats, bool emit) {
  const shs_plan* p = c.p;
  MidParams mp{};
  mp.z = have_z ? c.at<float2>(c.L.z) : nullptr;
  mp.v = c.at<float2>(c.L.v);
  mp.w = c.at<float>(c.L.w);
  mp.bw = c.at<float>(c.L.bw);
  mp.s = d_s;
  mp.partials = c.at<double>(c.L.parts) + c.L.nrow_parts * 4;
  mp.tw = p->tw;
  mp.n2 = (long long)p->n * p->n;
  mp.P = p->P;
  mp.q = p->q;
  mp.gamma = gamma;
  mp.emit = emit ? 1 : 0;
  mp.stats = stats ? 1 : 0;
  rec_step(BS_MID);
  Timed tm(c.s, KC_MID);
  c.ops.mid(p, mode, mp, c.s);
}

// Adjoint column side: pruned spectra T2 (count * eta planes) -> Z (count dense planes).
void enqueue_analysis(const Ctx& c, int count) {
  const shs_plan* p = c.p;
  ColParams cp = col_params(c, count);
  cp.in = c.at<float2>(c.L.t2);
  cp.out = c.at<float2>(c.L.z);
  cp.items = p->items_ana;
  rec_step(BS_ANA);
  run_col(c, COL_ANA, cp, p->n_ana, count);
  rec_step(BS_FINAL);
  if (p->n_part > 0) run_col(c, COL_FINAL, cp, p->NS, count);
}

// Sums nparts partial rows: one block up to eight rows per thread (no second step), else a block per
// 256 rows, at most kRed1Blocks of them.
void launch_reduce(hipStream_t s, const double* parts, long long nparts, double* red, double* sdev, double* hist_row,
                   double gamma, int* hist_ctr) {
  const int blocks = nparts <= 2048 ? 1 : int(std::min<long long>(kRed1Blocks, (nparts + 255) / 256));
  hipLaunchKernelGGL(k_reduce, dim3(blocks), dim3(256), 0, s, parts, nparts, (nparts + blocks - 1) / blocks, red,
                     reinterpret_cast<unsigned*>(sdev + kDoneSlot), sdev, hist_row, gamma, hist_ctr);
}
// Zeroes the workspace's two counters (history row, blocks done of a reduction): before the
// first launch of a call that reduces.
void enqueue_zero_counters(const Ctx& c) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, c.s, reinterpret_cast<uint32_t*>(c.at<double>(c.L.hctr)), 4LL, 0u);
}

// hist_ctr: NULL (hist_row is the row itself) or the device row counter (hist_row is the
// history's first row).
void enqueue_reduce(const Ctx& c, long long nparts, double* hist_row, double gamma, int* hist_ctr = nullptr) {
  if (g_rec) {
    rec_step(BS_REDUCE);
    LaunchRec& r = rec_add(RK_REDUCE, &k_reduce, 256, 1, 1, 0);
    r.parts = c.at<double>(c.L.parts);
    r.nparts = nparts;
    r.red1 = c.at<double>(c.L.red1);
    r.sdev = c.at<double>(c.L.sdev);
    r.gamma = gamma;
    return;
  }
  Timed tm(c.s, KC_REDUCE);
  launch_reduce(c.s, c.at<double>(c.L.parts), nparts, c.at<double>(c.L.red1), c.at<double>(c.L.sdev), hist_row, gamma,
                hist_ctr);
}

// Per-filter weights and thresholds from a host Lambda (J+1 per-scale or eta per-filter).
shs_status set_lambda(Ctx& c, const shs_params* prm) {
  const int eta = c.p->eta, J = c.p->J;
  if (!prm->lambda) return fail(SHS_E_INVALID, "null lambda");
  float lam_f[kMaxFilters] = {};   // eta <= kMaxFilters (J <= 6); no heap allocation
  if (prm->lambda_len == eta) {
    for (int f = 0; f < eta; ++f) lam_f[f] = prm->lambda[f];
  } else if (prm->lambda_len == J + 1) {
    int f = 0;
    lam_f[f++] = prm->lambda[0];
    for (int j = 0; j < J; ++j)
      for (int i = 0; i < (4 << j); ++i) lam_f[f++] = prm->lambda[j + 1];
  } else {
    return fail(SHS_E_INVALID, "lambda_len must be J+1 or eta");
  }
  for (int f = 0; f < eta; ++f)
    if (!(lam_f[f] >= 0.f) || !std::isfinite(lam_f[f]))
      return fail(SHS_E_INVALID, "lambda entries must be finite and >= 0");
  std::memset(&c.fw, 0, sizeof(c.fw));
  for (int f = 0; f < eta; ++f) {
    c.fw.lam[f] = lam_f[f];
    c.fw.thr[f] = prm->gamma * lam_f[f];
  }
  return SHS_OK;
}

// Exact energy <u, s> + sum_l sum_j lambda_j ||S_j u_l||_1 of u [q][N][N] (device), FP64.
shs_status energy_of(const Ctx& c, const float* d_u, const float* d_s, double* out) {
  const shs_plan* p = c.p;
  enqueue_synthesis(c, d_u, p->q);
  RowParams rp{};
  rp.spec_in = c.at<float2>(c.L.t1);
  rp.lin = pruned_layout(p);
  run_row(c, ROW_ENERGY, ST_F32, true, rp, p->q * p->eta);
  LAUNCHCHK("energy rows");
  const long long nn = (long long)p->n * p->n * p->q;
  {
    Timed tm(c.s, KC_OTHER);
    hipLaunchKernelGGL(k_dot, dim3(kDotBlocks), dim3(256), 0, c.s, d_u, d_s, nn,
                       c.at<double>(c.L.parts) + c.L.nrow_parts * 4);
  }
  enqueue_reduce(c, c.L.nrow_parts + kDotBlocks, nullptr, 1.0);
  LAUNCHCHK("energy reduce");
  double tot[8];
  HIPCHK(hipMemcpyAsync(tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
  HIPCHK(hipStreamSynchronize(c.s));
  if (tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite energy");
  *out = tot[SLOT_WS] + tot[SLOT_L1];
  return SHS_OK;
}

// ---------------------------------------------------------------- plan construction
void free_plan(shs_plan* p) {
  if (!p) return;
  delete p->graphs;
  void* bufs[] = {p->psi, p->tw, p->eig, p->psiw, p->pwin, p->tcol, p->items_syn, p->items_ana, p->fwin,
                  p->strips_ana};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  delete p;
}

template <class T>
shs_status upload(T** dst, const std::vector<T>& v) {
  const size_t bytes = std::max<size_t>(v.size(), 1) * sizeof(T);
  if (hipMalloc(dst, bytes) != hipSuccess) return fail(SHS_E_NOMEM, "plan table allocation");
  if (!v.empty()) HIPCHK(hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return SHS_OK;
}

// Column work list: per strip, the filters whose column range meets it, cut into runs of
// at most `fc` filters.  Analysis lists also assign partial-accumulator slots.
void build_items(const std::vector<std::vector<int>>& per_strip, const std::vector<int>& strip_flist_off, int fc,
                 bool with_parts, std::vector<int4>& items, std::vector<int2>* strips, int* nparts) {
  items.clear();
  int slot = 0;
  for (size_t s = 0; s < per_strip.size(); ++s) {
    const int nf = int(per_strip[s].size());
    const int nit = (nf + fc - 1) / fc;
    if (strips) strips->push_back(make_int2(int(items.size()), nit));
    for (int i = 0; i < nit; ++i) {
      const int cnt = std::min(fc, nf - i * fc);
      int part = -1;
      if (with_parts && nit > 1) part = slot++;
      items.push_back(make_int4(int(s), strip_flist_off[s] + i * fc, cnt, part));
    }
  }
  if (nparts) *nparts = slot;
}

// Filters meeting each strip (grouped by strip in flist), kept for re-cutting the synthesis
// work items while the plan is tuned.
struct StripLists {
  std::vector<std::vector<int>> per_strip;
  std::vector<int> strip_off;
};

shs_status build_pruned_layout(shs_plan* p, StripLists* keep) {
  const int n = p->n, half = p->M + 1, eta = p->eta, W = p->W;
  // 1. column windows of every filter
  int2* dwin = nullptr;
  if (hipMalloc(&dwin, size_t(eta) * half * sizeof(int2)) != hipSuccess) return fail(SHS_E_NOMEM, "window scratch");
  hipLaunchKernelGGL(k_filter_windows, dim3((eta * half + 255) / 256), dim3(256), 0, 0, p->psi, n, p->PP, eta, dwin);
  std::vector<int2> win(size_t(eta) * half);
  const hipError_t e1 = hipGetLastError();
  const hipError_t e2 = hipMemcpy(win.data(), dwin, win.size() * sizeof(int2), hipMemcpyDeviceToHost);
  (void)hipFree(dwin);
  if (e1 != hipSuccess || e2 != hipSuccess) return fail(SHS_E_DEVICE, "filter window scan");
  // 2. compact value offsets and per-filter column ranges (whole strips)
  std::vector<int4> pwin(win.size());
  std::vector<int4> tcol(eta);
  std::vector<int> s0(eta), s1(eta);
  long long off = 0, toff = 0;
  for (int j = 0; j < eta; ++j) {
    int c0 = -1, c1 = -1;
    for (int k1 = 0; k1 < half; ++k1) {
      const int2 w = win[size_t(j) * half + k1];
      pwin[size_t(j) * half + k1] = make_int4(w.x, w.y, int(off), 0);
      off += w.y;
      if (w.y > 0) { if (c0 < 0) c0 = k1; c1 = k1; }
    }
    if (c0 < 0) c0 = c1 = 0;
    s0[j] = c0 / W;
    s1[j] = c1 / W;
    const int cb = s0[j] * W, pitch = (s1[j] - s0[j] + 1) * W;
    tcol[j] = make_int4(cb, pitch, int(toff & 0xffffffffLL), int(toff >> 32));
    toff += (long long)n * pitch;
  }
  if (off >= (1LL << 29)) return fail(SHS_E_UNSUPPORTED, "filter bank too large");
  p->nnz = off;
  p->t_ls = toff;
  // 3. work lists
  std::vector<std::vector<int>> per_strip(p->NS);
  std::vector<int> flist, strip_off(p->NS);
  for (int s = 0; s < p->NS; ++s) {
    for (int j = 0; j < eta; ++j)
      if (s >= s0[j] && s <= s1[j]) per_strip[s].push_back(j);
    strip_off[s] = int(flist.size());
    flist.insert(flist.end(), per_strip[s].begin(), per_strip[s].end());
  }
  const long long pairs = (long long)flist.size();
  const int fc_syn = int(std::min<long long>(kItemMax, std::max<long long>(1, (pairs * p->q + 1249) / 2500)));
  const int fc_ana = int(std::min<long long>(kItemMax, std::max<long long>(2, (pairs * p->q + 749) / 1500)));
  std::vector<int4> isyn, iana;
  std::vector<int2> strips;
  build_items(per_strip, strip_off, fc_syn, false, isyn, nullptr, nullptr);
  build_items(per_strip, strip_off, fc_ana, true, iana, &strips, &p->n_part);
  p->n_syn = int(isyn.size());
  p->n_ana = int(iana.size());
  p->fc_syn = fc_syn;
  if (keep) {
    keep->per_strip = per_strip;
    keep->strip_off = strip_off;
  }
  shs_status st;
  if ((st = upload(&p->pwin, pwin)) != SHS_OK) return st;
  if ((st = upload(&p->tcol, tcol)) != SHS_OK) return st;
  if ((st = upload(&p->items_syn, isyn)) != SHS_OK) return st;
  if ((st = upload(&p->items_ana, iana)) != SHS_OK) return st;
  // the work list: every entry's column windows and plane geometry
  const size_t entries = flist.size();
  std::vector<int4> list(entries * (W + 1), make_int4(0, 0, 0, 0));   // windows, then geometry
  for (int s = 0; s < p->NS; ++s)
    for (size_t k = 0; k < per_strip[s].size(); ++k) {
      const size_t e = size_t(strip_off[s]) + k;
      const int j = per_strip[s][k];
      list[entries * W + e] = tcol[j];
      for (int c = 0; c < W && s * W + c < half; ++c) list[e * W + c] = pwin[size_t(j) * half + s * W + c];
    }
  if ((st = upload(&p->fwin, list)) != SHS_OK) return st;
  p->fgeo = p->fwin + entries * W;
  if ((st = upload(&p->strips_ana, strips)) != SHS_OK) return st;
  // 4. compact filter values
  if (hipMalloc(&p->psiw, size_t(std::max<long long>(off, 1)) * 4) != hipSuccess) return fail(SHS_E_NOMEM, "psiw");
  hipLaunchKernelGGL(k_filter_compact, dim3(4, std::min(eta * half, 65535)), dim3(256), 0, 0, p->psi, n, p->PP, eta,
                     p->pwin, p->psiw);
  LAUNCHCHK("filter compaction");
  HIPCHK(hipDeviceSynchronize());
  return SHS_OK;
}


shs_status check_params(const shs_params* prm) {
  if (!(prm->gamma > 0.f) || !std::isfinite(prm->gamma)) return fail(SHS_E_INVALID, "gamma must be > 0");
  if (prm->iters < 0) return fail(SHS_E_INVALID, "iters must be >= 0");
  if (prm->tol < 0.0 || (prm->tol > 0.0 && prm->check_every < 1)) return fail(SHS_E_INVALID, "bad tol/check_every");
  return SHS_OK;
}

// Zeroes `bytes` (a multiple of 4) of the workspace from `off` with a fill kernel, so that it
// can be captured in a graph.
void enqueue_zero(const Ctx& c, size_t off, size_t bytes) {
  const long long words = (long long)(bytes / 4);
  hipLaunchKernelGGL(k_fill_u32, dim3(unsigned((words + 255) / 256)), dim3(256), 0, c.s,
                     reinterpret_cast<uint32_t*>(c.ws + off), words, 0u);
}
// Zero solver state (v = w = b = 0).
void enqueue_zero_state(const Ctx& c) { enqueue_zero(c, c.L.g, c.L.state_end - c.L.g); }

void enqueue_epilogue(const Ctx& c, float* d_u, int32_t* d_labels) {
  if (!d_u && !d_labels) return;
  const long long n2 = (long long)c.p->n * c.p->n;
  Timed tm(c.s, KC_OTHER);
  hipLaunchKernelGGL(k_epilogue, dim3(unsigned((n2 + 255) / 256)), dim3(256), 0, c.s, c.at<float>(c.L.w), c.p->q, n2,
                     d_u, d_labels);
}

// One ADMM iteration of one image (Section 3): u-update from the adjoint of the previous
// iteration's (v - b_v) (absent on the first iteration), w/b_w update, forward transform,
// v/b_v update fused with the next adjoint's row FFT (when `emit`), optional FP64 residual
// reduction into `hist_row`.  Enqueues only; no host synchronisation.
void enqueue_iteration(const Ctx& c, const float* d_s, float gamma, bool have_adjoint_input, bool stats, bool emit,
                       double* hist_row, int* hist_ctr = nullptr) {
  const shs_plan* p = c.p;
  const Layout& L = c.L;
  const int q = p->q;
  if (have_adjoint_input) enqueue_analysis(c, q);
  run_mid(c, MID_ADMM, d_s, gamma, have_adjoint_input, stats, true);
  enqueue_synthesis_cols(c, q);
  RowParams rp{};
  rp.spec_in = c.at<float2>(L.t1);
  rp.lin = pruned_layout(p);
  rp.spec_out = c.at<float2>(L.t2);
  rp.lout = pruned_layout(p);
  rp.g = c.ws + L.g;
  rp.emit = emit ? 1 : 0;
  rp.fresh = have_adjoint_input ? 0 : 1;
  rec_step(BS_ROW);
  run_row(c, ROW_SOLVE, p->store, stats, rp, q * p->eta);
  if (stats) enqueue_reduce(c, L.nrow_parts + c.ops.mid_blocks(p), hist_row, gamma, hist_ctr);
}

TvParams tv_params(const Ctx& c, const float* d_s, float lambda, float gamma) {
  const shs_plan* p = c.p;
  TvParams tp{};
  tp.g = c.ws + c.L.g;
  tp.t = c.at<float>(c.L.t1);            // the filtered spectra's place, unused here
  tp.b = c.at<float>(c.L.t2);
  tp.w = c.at<float>(c.L.w);
  tp.bw = c.at<float>(c.L.bw);
  tp.s = d_s;
  tp.u = c.at<float>(c.L.zs);
  tp.rhs = c.at<float>(c.L.us);
  tp.partials = c.at<double>(c.L.parts);
  tp.n = p->n;
  tp.q = p->q;
  tp.gamma = gamma;
  tp.lambda = lambda;
  tp.radius = gamma * lambda;
  return tp;
}

// One ADMM iteration of the TV model: right-hand side (grad^T of v - b_v, w - b_w, data
// term), the u-solve on the DFT (row R2C, column FFT / divide / inverse, row C2R), then
// the pixel update of g, w, b_w with residual partials.
void enqueue_tv_iteration(const Ctx& c, const float* d_s, float lambda, float gamma, bool first, bool write_w,
                          bool stats, double* hist_row) {
  const shs_plan* p = c.p;
  const Layout& L = c.L;
  const int q = p->q;
  const long long n2 = (long long)p->n * p->n;
  TvParams tp = tv_params(c, d_s, lambda, gamma);
  tp.fresh = first ? 1 : 0;
  tp.write_w = write_w ? 1 : 0;
  {
    Timed tm(c.s, KC_TV_RHS);
    tv_launch(p->store, TV_RHS, false, tp, c.s);
  }
  RowParams rp{};
  rp.real_in = c.at<float>(L.us);
  rp.spec_out = c.at<float2>(L.v);
  rp.lout = dense_layout(p);
  run_row(c, ROW_R2C, ST_F32, false, rp, q);
  ColParams cp = col_params(c, q);
  cp.in = c.at<float2>(L.v);
  cp.out = c.at<float2>(L.z);
  run_col_solve(c, cp, q);
  RowParams rz{};
  rz.spec_in = c.at<float2>(L.z);
  rz.lin = dense_layout(p);
  rz.real_out = c.at<float>(L.zs);
  run_row(c, ROW_C2R, ST_F32, false, rz, q);
  {
    Timed tm(c.s, KC_TV_UPDATE);
    tv_launch(p->store, TV_UPDATE, stats, tp, c.s);
  }
  if (stats) enqueue_reduce(c, tv_blocks(n2), hist_row, gamma);
}

// <w, s> + lambda TV(w) (FP64), synchronising.
shs_status tv_energy_of(const Ctx& c, const float* d_s, float lambda, double* out) {
  const long long n2 = (long long)c.p->n * c.p->n;
  TvParams tp = tv_params(c, d_s, lambda, 1.f);
  {
    Timed tm(c.s, KC_OTHER);
    hipLaunchKernelGGL(k_tv_energy, dim3(unsigned((n2 + 255) / 256)), dim3(256), 0, c.s, tp);
  }
  enqueue_reduce(c, (n2 + 255) / 256, nullptr, 1.0);
  LAUNCHCHK("tv energy");
  double tot[8];
  HIPCHK(hipMemcpyAsync(tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
  HIPCHK(hipStreamSynchronize(c.s));
  if (tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite energy");
  *out = tot[SLOT_WS] + tot[SLOT_L1];
  return SHS_OK;
}

// One primal-dual iteration (Chambolle-Pock for the functional of Section 3), from the row
// spectra of ubar: K ubar (synthesis), the dual step fused into the row pass (y <- clip(y +
// sigma K ubar), then the row FFT of y), K^T y (analysis), the primal step and extrapolation
// with their row transforms (the next ubar's spectra unless this is the last iteration).
void enqueue_pd_iteration(const Ctx& c, const float* d_s, float tau, float sigma, bool first, bool last, bool stats,
                          double* hist_row) {
  const shs_plan* p = c.p;
  const Layout& L = c.L;
  const int q = p->q;
  enqueue_synthesis_cols(c, q);
  RowParams rp{};
  rp.spec_in = c.at<float2>(L.t1);
  rp.lin = pruned_layout(p);
  rp.spec_out = c.at<float2>(L.t2);
  rp.lout = pruned_layout(p);
  rp.g = c.ws + L.g;
  rp.emit = 1;
  rp.fresh = first ? 1 : 0;
  rp.sigma = sigma;
  run_row(c, ROW_PD, p->store, stats, rp, q * p->eta);
  enqueue_analysis(c, q);
  run_mid(c, MID_PD, d_s, tau, true, stats, !last);
  if (stats) enqueue_reduce(c, L.nrow_parts + c.ops.mid_blocks(p), hist_row, 1.0);
}

}  // namespace

// A batch of images of different sizes and label counts (one plan per distinct shape).
// A solve of the whole batch is one captured graph, replayed on the caller's stream with a
// single launch.  Images are split into lanes by kernel class (the same kernels and the same
// occupancy); in a lane every step of an iteration is one grouped launch covering all its
// images (grouped.hpp), and the lanes are independent branches of the graph that run side by
// side.
struct shs_batch {
  int count = 0, device = 0;
  std::vector<shs_plan*> plans;
  std::vector<int> plan_of;
  std::vector<size_t> ws_off;
  size_t ws_total = 0;
  std::vector<std::vector<int>> lanes; // images by kernel class (see batch_class)
  hipStream_t main = nullptr;          // capture stream (default priority)
  std::vector<hipStream_t> lane_s;     // one capture branch per lane (default priority)
  std::vector<hipEvent_t> lane_e;
  hipEvent_t fork = nullptr;
  std::vector<double> key;             // pointers and parameters baked into the graph
  hipGraphExec_t graph = nullptr;      // the whole solve
  void* arena = nullptr;               // device task tables of the grouped launches

  void drop_graph() {
    if (graph) (void)hipGraphExecDestroy(graph);
    graph = nullptr;
    if (arena) (void)hipFree(arena);
    arena = nullptr;
    key.clear();
  }
};

namespace {
// One iteration of a batch as launches: grouped launches (tables at arena offsets) and the
// per-image FP64 reductions, in the order of the iteration's steps.
struct BatchItem {
  bool group = true;
  const void* fn = nullptr;
  int threads = 0;
  size_t lds = 0;
  unsigned blocks = 0;
  size_t tasks_off = 0, bt_off = 0;
  LaunchRec red;       // !group: one image's reduction
};
using BatchIter = std::vector<BatchItem>;

size_t arena_put(std::vector<char>& a, const void* data, size_t bytes) {
  const size_t off = align256(a.size());
  a.resize(off + bytes);
  std::memcpy(a.data() + off, data, bytes);
  return off;
}

template <class P>
void put_group(const std::vector<const LaunchRec*>& recs, P LaunchRec::*field, std::vector<char>& arena,
               BatchItem& it) {
  std::vector<GroupTask<P>> tasks(recs.size());
  std::vector<uint16_t> bt;
  unsigned start = 0;
  for (size_t k = 0; k < recs.size(); ++k) {
    const LaunchRec& r = *recs[k];
    GroupTask<P>& T = tasks[k];
    std::memset(static_cast<void*>(&T), 0, sizeof(T));
    T.p = r.*field;
    T.gp = r.gp;
    T.gx = r.gx;
    T.gy = r.gy;
    T.start = int(start);
    const unsigned nb = unsigned(r.gx) * unsigned(r.gy);
    bt.insert(bt.end(), nb, uint16_t(k));
    start += nb;
    it.lds = std::max(it.lds, r.lds);
  }
  it.blocks = start;
  it.tasks_off = arena_put(arena, tasks.data(), tasks.size() * sizeof(GroupTask<P>));
  it.bt_off = arena_put(arena, bt.data(), bt.size() * sizeof(uint16_t));
}

// Groups one iteration's records of all images (image order) by step, then by kernel.
void build_batch_iter(const std::vector<LaunchRec>& recs, std::vector<char>& arena, BatchIter& out) {
  for (int step = 0; step < BS_COUNT; ++step) {
    std::vector<std::pair<const void*, int>> keys;
    std::vector<std::vector<const LaunchRec*>> groups;
    for (const LaunchRec& r : recs) {
      if (r.step != step) continue;
      if (r.kind == RK_REDUCE) {
        BatchItem it;
        it.group = false;
        it.red = r;
        out.push_back(it);
        continue;
      }
      size_t g = 0;
      while (g < keys.size() && !(keys[g].first == r.fn && keys[g].second == r.threads)) ++g;
      if (g == keys.size()) {
        keys.emplace_back(r.fn, r.threads);
        groups.emplace_back();
      }
      groups[g].push_back(&r);
    }
    for (size_t g = 0; g < groups.size(); ++g) {
      BatchItem it;
      it.fn = keys[g].first;
      it.threads = keys[g].second;
      const int kind = groups[g][0]->kind;
      if (kind == RK_ROW) put_group(groups[g], &LaunchRec::rp, arena, it);
      else if (kind == RK_COL) put_group(groups[g], &LaunchRec::cp, arena, it);
      else put_group(groups[g], &LaunchRec::mp, arena, it);
      out.push_back(it);
    }
  }
}

// Kernel class of an image: the power-of-two side, or for the mixed-radix path the rows per wave and
// waves per block of its row pass, its column blocks' width, and the blocks per CU its column
// passes' LDS allows (a grouped launch takes its largest image's LDS, so only images of one
// occupancy share a launch).  The middle step of a class is one launch per block size.  Coarser
// classes (any column width in one launch, four LDS classes: 68 instead of 108 launches per iteration
// of 64 images) gain nothing on balance, per iteration: 64 images of 96..768 12.0 -> 12.4 ms and 13.5 ->
// 13.5, 32 of them in FP16 6.99 -> 6.95, 32 of 96..256 1.04 -> 1.02.
int batch_class(const shs_plan* p) {
  if (!p->generic) return p->n;
  const int bpc = std::min(6, int(160 * 1024 / col_g_lds_bytes(p, 1)));
  return 100000 + (col_g_threads(p->pcol) / 64) * 1000 + p->wpb * 100 + p->rw * 10 + bpc;
}

void launch_batch_iter(const BatchIter& iter, char* dbase, hipStream_t s) {
  for (const BatchItem& it : iter) {
    if (it.group) {
      void* tasks = dbase + it.tasks_off;
      void* bt = dbase + it.bt_off;
      void* args[] = {&tasks, &bt};
      (void)hipLaunchKernel(it.fn, dim3(it.blocks), dim3(it.threads), args, it.lds, s);
    } else {
      const LaunchRec& r = it.red;
      launch_reduce(s, r.parts, r.nparts, r.red1, r.sdev, nullptr, r.gamma, nullptr);
    }
  }
}
}  // namespace

// ---------------------------------------------------------------- schedule tuning
// Mixed-radix plans pick their launch schedule by timing candidates on their own kernels
// at plan creation: rows per wave and waves per block of the row pass, the stage order of
// the row FFT, the stage order of the column FFT, and the filters per synthesis work item.
// The row-pass geometry and the synthesis item size leave the solution bit-identical (the
// residual partial sums are grouped by block, so the histories can differ in the last
// bits); the stage order changes the FFT's rounding (results stay within the parity
// bounds, and are fixed for a given schedule).  The choice is cached per (arch, N, J, q, store) for
// the process, and in the file named by SHEARSEG_TUNE_CACHE when set (one line per key, see
// schedule.hpp); SHEARSEG_TUNE=0 keeps the default schedule.
std::mutex g_tune_mu;
std::vector<std::pair<std::string, TuneCfg>> g_tune;   // process cache
bool g_tune_loaded = false;

void tune_cache_load() {
  if (g_tune_loaded) return;
  g_tune_loaded = true;
  const char* path = std::getenv("SHEARSEG_TUNE_CACHE");
  if (!path || !*path) return;
  FILE* f = std::fopen(path, "r");
  if (!f) return;
  char line[512];
  while (std::fgets(line, sizeof(line), f)) {
    std::string key;
    TuneCfg c;
    if (parse_schedule_line(line, key, c)) g_tune.emplace_back(key, c);
  }
  std::fclose(f);
}
void tune_cache_store(const std::string& key, const TuneCfg& c) {
  g_tune.emplace_back(key, c);
  const char* path = std::getenv("SHEARSEG_TUNE_CACHE");
  if (!path || !*path) return;
  if (FILE* f = std::fopen(path, "a")) {
    std::fprintf(f, "%s\n", schedule_line(key, c).c_str());
    std::fclose(f);
  }
}

// Installs a schedule in the plan: FFT plans and their twiddle tables, rows per wave, and
// the synthesis work items.
shs_status apply_schedule(shs_plan* p, const TuneCfg& c, const StripLists& sl) {
  FftPlan pr, pf, pc;
  if (!row_plans_from(p->M, c.prow, pr, pf) || !fft_plan_from(p->n, c.pcol, pc, true))
    return fail(SHS_E_DEVICE, "bad schedule");
  const int n = p->n;
  const std::vector<float2> tw = base_twiddles(n);
  std::vector<float2> tabs(tables_g_len(n));
  fill_stage_tables_g(pr, pf, pc, tw, tabs.data());
  HIPCHK(hipMemcpy(p->tw + n, tabs.data(), tabs.size() * sizeof(float2), hipMemcpyHostToDevice));
  p->prow = pr;
  p->pfwd = pf;
  p->pcol = pc;
  p->rw = c.rw;
  p->wpb = c.wpb;
  p->rpb = c.wpb * c.rw;
  p->nbuf = row_g_bufs(pr, c.rw);
  if (c.fc_syn != p->fc_syn) {
    std::vector<int4> isyn;
    build_items(sl.per_strip, sl.strip_off, c.fc_syn, false, isyn, nullptr, nullptr);
    int4* d = nullptr;
    const shs_status st = upload(&d, isyn);
    if (st != SHS_OK) return st;
    (void)hipFree(p->items_syn);
    p->items_syn = d;
    p->n_syn = int(isyn.size());
    p->fc_syn = c.fc_syn;
  }
  return SHS_OK;
}

shs_status tune_schedule(shs_plan* p, const StripLists& sl) {
  hipDeviceProp_t prop{};
  HIPCHK(hipGetDeviceProperties(&prop, p->device));
  const std::string key = std::string(prop.gcnArchName).substr(0, std::string(prop.gcnArchName).find(':')) +
                          "/n" + std::to_string(p->n) + "/J" + std::to_string(p->J) + "/q" + std::to_string(p->q) +
                          "/s" + std::to_string(p->store);
  std::lock_guard<std::mutex> lock(g_tune_mu);
  tune_cache_load();
  TuneCfg base;
  base.rw = p->rw;
  base.wpb = p->wpb;
  base.fc_syn = p->fc_syn;
  const std::vector<std::vector<int>> row_lists = stage_lists(p->M, false), col_lists = stage_lists(p->n, true);
  base.prow = row_lists[0];
  base.pcol = col_lists[0];
  for (auto& e : g_tune)   // an entry that the tuner could not have chosen is passed over
    if (e.first == key && schedule_ok(p->n, e.second, kItemMax)) {
      const shs_status st = apply_schedule(p, e.second, sl);
      if (st == SHS_OK)
        std::snprintf(p->schedule, sizeof(p->schedule), "%s: rows/wave %d, waves/block %d, row radices %s, "
                      "column radices %s, synthesis run %d (cached)", key.c_str(), p->rw, p->wpb,
                      join_radices(e.second.prow, 'x').c_str(),
                      join_radices(e.second.pcol, 'x').c_str(), p->fc_syn);
      return st;
    }
  const char* off = std::getenv("SHEARSEG_TUNE");
  if (off && std::string(off) == "0") {
    std::snprintf(p->schedule, sizeof(p->schedule), "%s: rows/wave %d, waves/block %d, row radices %s, "
                  "column radices %s, synthesis run %d (default)", key.c_str(), p->rw, p->wpb,
                  join_radices(base.prow, 'x').c_str(),
                  join_radices(base.pcol, 'x').c_str(), p->fc_syn);
    return SHS_OK;
  }
  const auto t0 = std::chrono::steady_clock::now();
  // a workspace for one label's channels, sized for the smallest rows per block
  const int rw0 = p->rw, rpb0 = p->rpb;
  p->rw = 1;
  p->rpb = 1;
  const Layout L = make_layout(p);
  p->rw = rw0;
  p->rpb = rpb0;
  void* ws = nullptr;
  if (hipMalloc(&ws, L.total) != hipSuccess) return fail(SHS_E_NOMEM, "tuning workspace");
  struct Free {
    void* w;
    ~Free() { (void)hipFree(w); }
  } fr{ws};
  HIPCHK(hipMemset(ws, 0, L.total));
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  struct FreeEv {
    hipEvent_t a, b;
    ~FreeEv() { (void)hipEventDestroy(a); (void)hipEventDestroy(b); }
  } fe{e0, e1};
  CaptureScope cs;   // no profiling events while tuning
  auto time_ms = [&](auto&& launch) -> float {
    launch();
    (void)hipEventRecord(e0, 0);
    for (int r = 0; r < 3; ++r) launch();
    (void)hipEventRecord(e1, 0);
    float ms = 1e30f;
    if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return 1e30f;
    return ms;
  };
  TuneCfg best = base;
  int tried = 0;
  // row pass: rows per wave x row stage order (one label's channels, state update on)
  float best_row = 1e30f;
  for (int rw : {1, 2, 4})
   for (int wpb : {4, 2, 1}) {
    for (const auto& ord : row_lists) {
      if (!row_shape_ok(p->n, rw, wpb, ord)) continue;
      TuneCfg c = best;
      c.rw = rw;
      c.wpb = wpb;
      c.prow = ord;
      shs_status st = apply_schedule(p, c, sl);
      if (st != SHS_OK) return st;
      Ctx cx;
      if ((st = make_ctx(p, ws, L.total, nullptr, cx)) != SHS_OK) return st;
      RowParams rp{};
      rp.spec_in = cx.at<float2>(cx.L.t1);
      rp.lin = pruned_layout(p);
      rp.spec_out = cx.at<float2>(cx.L.t2);
      rp.lout = pruned_layout(p);
      rp.g = cx.ws + cx.L.g;
      rp.emit = 1;
      const float ms = time_ms([&] { run_row(cx, ROW_SOLVE, p->store, false, rp, p->eta); });
      ++tried;
      if (ms < best_row) { best_row = ms; best.rw = rw; best.wpb = wpb; best.prow = ord; }
    }
   }
  // column passes: column stage order x synthesis run length (one label)
  float best_col = 1e30f;
  std::vector<int> fcs;
  for (int fc : {1, 2, 4, 8, 16}) if (fc <= kItemMax) fcs.push_back(fc);
  for (const auto& ord : col_lists) {
    for (int fc : fcs) {
      TuneCfg c = best;
      c.pcol = ord;
      c.fc_syn = fc;
      shs_status st = apply_schedule(p, c, sl);
      if (st != SHS_OK) return st;
      Ctx cx;
      if ((st = make_ctx(p, ws, L.total, nullptr, cx)) != SHS_OK) return st;
      ColParams cp = col_params(cx, 1);
      const float ms = time_ms([&] {
        ColParams a = cp;
        a.in = cx.at<float2>(cx.L.v);
        a.out = cx.at<float2>(cx.L.t1);
        a.items = p->items_syn;
        run_col(cx, COL_SYN, a, p->n_syn, 1);
        ColParams b = cp;
        b.in = cx.at<float2>(cx.L.t2);
        b.out = cx.at<float2>(cx.L.z);
        b.items = p->items_ana;
        run_col(cx, COL_ANA, b, p->n_ana, 1);
      });
      ++tried;
      if (ms < best_col) { best_col = ms; best.pcol = ord; best.fc_syn = fc; }
    }
  }
  LAUNCHCHK("schedule tuning");
  shs_status st = apply_schedule(p, best, sl);
  if (st != SHS_OK) return st;
  tune_cache_store(key, best);
  const double tms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  std::snprintf(p->schedule, sizeof(p->schedule), "%s: rows/wave %d, waves/block %d, row radices %s, column "
                "radices %s, synthesis run %d (tuned: %d candidates, %.0f ms)", key.c_str(), p->rw, p->wpb,
                join_radices(best.prow, 'x').c_str(),
                join_radices(best.pcol, 'x').c_str(), p->fc_syn, tried, tms);
  return SHS_OK;
}

// ---------------------------------------------------------------- graph replay
constexpr int kGraphIters = 8;   // ADMM iterations per captured graph

namespace {
// Enqueues `reps` x `k` steady-state ADMM iterations (adjoint input present, next adjoint
// input emitted, statistics only when a history is kept) on c.s by replaying a captured
// graph of k iterations.  The graph is captured on first use for this key.
shs_status replay_iterations(const Ctx& c, const float* d_s, float gamma, double* d_hist, int* hctr, int k, int reps) {
  const shs_plan* p = c.p;
  GraphCache& G = *p->graphs;
  std::vector<uint64_t> key;
  key.reserve(8 + 2 * kMaxFilters);
  auto put = [&](const void* ptr) { key.push_back(uint64_t(reinterpret_cast<uintptr_t>(ptr))); };
  put(c.ws); put(d_s); put(d_hist); put(hctr);
  key.push_back(uint64_t(k));
  uint32_t gb;
  std::memcpy(&gb, &gamma, 4);
  key.push_back(gb);
  for (int f = 0; f < p->eta; ++f) {
    uint32_t a, b;
    std::memcpy(&a, &c.fw.thr[f], 4);
    std::memcpy(&b, &c.fw.lam[f], 4);
    key.push_back((uint64_t(a) << 32) | b);
  }
  std::lock_guard<std::mutex> lock(G.mu);
  hipGraphExec_t exec = nullptr;
  for (size_t i = 0; i < G.entries.size(); ++i) {
    if (G.entries[i].key == key) {
      GraphCache::Entry e = G.entries[i];
      G.entries.erase(G.entries.begin() + long(i));
      G.entries.push_back(e);
      exec = e.exec;
      break;
    }
  }
  if (!exec) {
    if (!G.cap) HIPCHK(hipStreamCreateWithFlags(&G.cap, hipStreamNonBlocking));
    Ctx cc = c;
    cc.s = G.cap;
    {
      CaptureScope cs;
      HIPCHK(hipStreamBeginCapture(G.cap, hipStreamCaptureModeThreadLocal));
      for (int i = 0; i < k; ++i) enqueue_iteration(cc, d_s, gamma, true, d_hist != nullptr, true, d_hist, hctr);
      const hipError_t el = hipGetLastError();
      hipGraph_t g = nullptr;
      const hipError_t ee = hipStreamEndCapture(G.cap, &g);
      if (el != hipSuccess || ee != hipSuccess || !g) {
        if (g) (void)hipGraphDestroy(g);
        return fail(SHS_E_DEVICE, "capture of the iteration graph failed");
      }
      const hipError_t ei = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
      (void)hipGraphDestroy(g);
      if (ei != hipSuccess) return fail(SHS_E_DEVICE, std::string("graph instantiate: ") + hipGetErrorString(ei));
    }
    if (G.entries.size() >= GraphCache::kMax) {
      (void)hipGraphExecDestroy(G.entries.front().exec);
      G.entries.erase(G.entries.begin());
    }
    G.entries.push_back(GraphCache::Entry{key, exec});
  }
  for (int r = 0; r < reps; ++r) HIPCHK(hipGraphLaunch(exec, c.s));
  return SHS_OK;
}
}  // namespace

// ---------------------------------------------------------------- allocation-free solve
// Workspace of shs_solve_noalloc: one file-scope device array per GPU, held until the
// process ends.  Host code never passes `scratch` itself (on the host it is only a stand-in
// for the symbol); it uses the device address that hipGetSymbolAddress returns for the
// current device, looked up once per device on the first call there.
static __device__ __align__(256) unsigned char scratch[SHS_NOALLOC_MAX_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};

// Device address of `scratch` on `device` (which must be current).
shs_status scratch_address(int device, void** out) {
  if (device < 0 || device >= kScratchDevices) return fail(SHS_E_UNSUPPORTED, "device ordinal too large");
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(SHS_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return SHS_OK;
}
}  // namespace

// ===================================================================== C ABI
extern "C" {

const char* shs_status_str(shs_status s) {
  switch (s) {
    case SHS_OK: return "ok";
    case SHS_E_INVALID: return "invalid argument";
    case SHS_E_UNSUPPORTED: return "unsupported";
    case SHS_E_NOMEM: return "out of device memory";
    case SHS_E_DEVICE: return "device error";
    case SHS_E_NUMERIC: return "non-finite value";
    case SHS_E_WORKSPACE: return "workspace too small or missing";
  }
  return "unknown status";
}

const char* shs_last_error(void) { return g_err.c_str(); }

shs_status shs_profile_begin(void) { return shs_profile_begin_classes(nullptr); }

shs_status shs_profile_begin_classes(const char* classes) {
  uint32_t mask = 0;
  if (!classes || !*classes) {
    mask = ~0u;
  } else {
    // comma-separated names, matched in place (no allocation)
    const char* p = classes;
    for (;;) {
      const char* e = p;
      while (*e && *e != ',') ++e;
      const size_t len = size_t(e - p);
      int c = 0;
      while (c < KC_COUNT && !(std::strlen(kKClassName[c]) == len && std::strncmp(kKClassName[c], p, len) == 0)) ++c;
      if (c == KC_COUNT) {
        g_err.assign("unknown kernel class '").append(p, len).append("'");
        return SHS_E_INVALID;
      }
      mask |= 1u << c;
      if (!*e) break;
      p = e + 1;
    }
  }
  Prof& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  P.on = true;
  P.mask = mask;
  P.used = 0;
  P.cls.clear();
  return SHS_OK;
}

int32_t shs_profile_end(shs_kernel_time* out, int32_t max_entries) {
  Prof& P = prof();
  std::lock_guard<std::mutex> g(P.mu);
  P.on = false;
  double ms[KC_COUNT] = {0};
  int64_t cnt[KC_COUNT] = {0};
  for (size_t i = 0; i < P.cls.size(); ++i) {
    if (hipEventSynchronize(P.pool[2 * i + 1]) != hipSuccess) { g_err = "event synchronize"; return -1; }
    float t = 0.f;
    if (hipEventElapsedTime(&t, P.pool[2 * i], P.pool[2 * i + 1]) != hipSuccess) { g_err = "event elapsed"; return -1; }
    ms[P.cls[i]] += t;
    cnt[P.cls[i]] += 1;
  }
  int32_t k = 0;
  for (int c = 0; c < KC_COUNT && k < max_entries; ++c) {
    if (!cnt[c]) continue;
    if (out) {
      std::memset(out[k].name, 0, sizeof(out[k].name));
      std::strncpy(out[k].name, kKClassName[c], sizeof(out[k].name) - 1);
      out[k].launches = cnt[c];
      out[k].total_ms = ms[c];
    }
    ++k;
  }
  P.used = 0;
  P.cls.clear();
  return k;
}

int32_t shs_num_filters(int32_t J) { return J < 1 || J > 12 ? -1 : 1 + 4 * ((1 << J) - 1); }

shs_status shs_plan_create(const shs_shape* shape, int device, shs_plan** out) {
  if (!shape || !out) return fail(SHS_E_INVALID, "null argument");
  *out = nullptr;
  const int n = shape->n;
  if (n < 2) return fail(SHS_E_INVALID, "n must be >= 2");
  if (shape->q < 1 || shape->q > SHS_MAX_LABELS) return fail(SHS_E_INVALID, "q must be in 1..8");
  if (shape->channels < 1 || shape->channels > SHS_MAX_CHANNELS) return fail(SHS_E_INVALID, "channels must be in 1..4");
  if (shape->J < 1 || shape->J > 6 || (1LL << (2 * shape->J)) > 2LL * n)
    return fail(SHS_E_INVALID, "J must satisfy J >= 1 and 4^J <= 2N");
  if (shape->store < SHS_STORE_F32 || shape->store > SHS_STORE_F16) return fail(SHS_E_INVALID, "bad store type");
  Ops o;
  FftPlan prow{}, pfwd{}, pcol{};
  const bool pow2 = get_ops_pow2(n, o);
  if (!pow2) {
    // mixed-radix path: N a multiple of 8 in [64, 1024] whose prime factors are <= 23
    const auto rows = stage_lists(n / 2, false), cols = stage_lists(n, true);
    if (n % 8 != 0 || n < 64 || n > kGenericMaxN || rows.empty() || cols.empty() ||
        !row_plans_from(n / 2, rows[0], prow, pfwd) || !fft_plan_from(n, cols[0], pcol, true))
      return fail(SHS_E_UNSUPPORTED,
                  "n must be a power of two in 64..2048 or a multiple of 8 in 64..1024 with prime factors <= 23");
  }
  if (device < 0) return fail(SHS_E_INVALID, "bad device");
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return fail(SHS_E_DEVICE, "no such HIP device");
  DeviceGuard dg(device);
  if (!dg.ok) return fail(SHS_E_DEVICE, "hipSetDevice failed");

  shs_plan* p = new (std::nothrow) shs_plan{};
  if (!p) return fail(SHS_E_NOMEM, "host allocation");
  p->graphs = new (std::nothrow) GraphCache();
  if (!p->graphs) { delete p; return fail(SHS_E_NOMEM, "host allocation"); }
  p->n = n; p->C = shape->channels; p->q = shape->q; p->J = shape->J; p->store = shape->store;
  p->eta = shs_num_filters(shape->J);
  p->M = n / 2;
  p->generic = pow2 ? 0 : 1;
  p->prow = prow;
  p->pfwd = pfwd;
  p->pcol = pcol;
  p->W = pow2 ? by_size<WOf>(n) : kGW;
  // generic rows: as many rows per wave (up to 4, in blocks that divide N) as keep every
  // stage one pass over the wave's lanes
  p->rw = 1;
  if (!pow2)
    while (p->rw < 4 && n % (8 * p->rw) == 0 && row_g_bufs(prow, 2 * p->rw) == 1) p->rw *= 2;
  p->nbuf = pow2 ? 0 : row_g_bufs(prow, p->rw);
  p->wpb = 4;
  p->rpb = pow2 ? by_size<RpbOf>(n) : p->wpb * p->rw;
  p->NS = p->M / p->W + 1;
  p->P = p->NS * p->W;  // columns of a dense spectrum plane (strip tiled); columns M+1.. unused
  p->PP = p->M + 16;    // row pitch of the dense filter bank
  p->device = device;
  const size_t psi_bytes = size_t(p->eta) * n * p->PP * 4;
  if (hipMalloc(&p->psi, psi_bytes) != hipSuccess) { free_plan(p); return fail(SHS_E_NOMEM, "filter bank allocation"); }
  std::vector<float2> tw = base_twiddles(n);
  // append the row and column stage tables
  if (pow2) {
    fill_stage_tables(n, tw);
  } else {
    const std::vector<float2> base = tw;
    tw.resize(size_t(n) + tables_g_len(n));
    fill_stage_tables_g(p->prow, p->pfwd, p->pcol, base, tw.data() + n);
  }
  if (hipMalloc(&p->tw, tw.size() * 8) != hipSuccess) { free_plan(p); return fail(SHS_E_NOMEM, "twiddle allocation"); }
  std::vector<float> eig(n);
  for (int k = 0; k < n; ++k) {
    const double sn = std::sin(M_PI * double(k) / double(n));
    eig[k] = float(4.0 * sn * sn);
  }
  if (!pow2) p->fft = reinterpret_cast<FftPlan*>(p->tw + n + tables_g_len(n) - kPlansLen);
  if (hipMalloc(&p->eig, size_t(n) * 4) != hipSuccess) { free_plan(p); return fail(SHS_E_NOMEM, "eigenvalue table"); }
  if (hipMemcpy(p->eig, eig.data(), size_t(n) * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(p->tw, tw.data(), tw.size() * 8, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(p->psi, 0, psi_bytes) != hipSuccess) {
    free_plan(p);
    return fail(SHS_E_DEVICE, "plan initialisation copy");
  }
  const long long total = (long long)p->eta * n * (p->M + 1);
  hipLaunchKernelGGL(k_filter_gen, dim3(unsigned((total + 255) / 256)), dim3(256), 0, 0, p->psi, n, p->J, p->PP,
                     p->eta);
  if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
    free_plan(p);
    return fail(SHS_E_DEVICE, "filter generation failed");
  }
  // dynamic LDS beyond the runtime's default limit
  {
    Ops ops;
    if (!get_ops(p, ops) || !ops.reserve(p)) {
      free_plan(p);
      return fail(SHS_E_DEVICE, "cannot reserve LDS for the plan's kernels");
    }
  }
  StripLists sl;
  shs_status st = build_pruned_layout(p, &sl);
  if (st == SHS_OK && p->generic) st = tune_schedule(p, sl);
  if (st != SHS_OK) {
    free_plan(p);
    return st;
  }
  if (!p->generic)
    std::snprintf(p->schedule, sizeof(p->schedule), "n%d: power-of-two path, row FFT %d-point (compile-time "
                  "radices), column strips of %d, synthesis run %d", n, p->M, p->W, p->fc_syn);
  *out = p;
  return SHS_OK;
}

shs_status shs_plan_destroy(shs_plan* p) {
  if (!p) return SHS_OK;
  DeviceGuard dg(p->device);
  free_plan(p);
  return SHS_OK;
}

size_t shs_workspace_bytes(const shs_plan* p) { return p ? make_layout(p).total : 0; }
size_t shs_state_bytes(const shs_plan* p) { return p ? make_layout(p).state_end : 0; }

const char* shs_plan_describe(const shs_plan* p) { return p ? p->schedule : ""; }

shs_status shs_filters(const shs_plan* p, float* d_psi, void* stream) {
  if (!p || !d_psi) return fail(SHS_E_INVALID, "null argument");
  DeviceGuard dg(p->device);
  const size_t w = size_t(p->M + 1) * 4;
  HIPCHK(hipMemcpy2DAsync(d_psi, w, p->psi, size_t(p->PP) * 4, w, size_t(p->eta) * p->n, hipMemcpyDeviceToDevice,
                          static_cast<hipStream_t>(stream)));
  return SHS_OK;
}

shs_status shs_datacost(const shs_plan* p, const float* d_img, const float* h_codebook, float pw, float* d_s,
                        void* stream) {
  if (!p || !d_img || !h_codebook || !d_s) return fail(SHS_E_INVALID, "null argument");
  if (!(pw > 0.f) || !std::isfinite(pw)) return fail(SHS_E_INVALID, "p must be > 0");
  DeviceGuard dg(p->device);
  Codebook cb{};
  for (int k = 0; k < p->q; ++k)
    for (int c = 0; c < p->C; ++c) cb.c[k * 4 + c] = h_codebook[k * p->C + c];
  const long long n2 = (long long)p->n * p->n;
  hipLaunchKernelGGL(k_datacost, dim3(unsigned((n2 + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     d_img, p->C, cb, p->q, pw, d_s, n2);
  LAUNCHCHK("datacost");
  return SHS_OK;
}

shs_status shs_solve_pd(const shs_plan* p, const shs_pd_params* prm, const float* d_s, void* d_ws, size_t ws_bytes,
                        float* d_u, int32_t* d_labels, double* d_hist, shs_stats* h_stats, void* stream) {
  if (!p || !prm || !d_s) return fail(SHS_E_INVALID, "null argument");
  if (!(prm->tau > 0.f) || !(prm->sigma > 0.f) || !std::isfinite(prm->tau) || !std::isfinite(prm->sigma))
    return fail(SHS_E_INVALID, "tau and sigma must be finite and > 0");
  if (double(prm->tau) * double(prm->sigma) > 1.0 + 1e-6)
    return fail(SHS_E_INVALID, "tau * sigma must be <= 1 (||K|| = 1)");
  if (prm->iters < 0) return fail(SHS_E_INVALID, "iters must be >= 0");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  shs_params lp{};
  lp.lambda = prm->lambda;
  lp.lambda_len = prm->lambda_len;
  lp.gamma = 1.f;                        // thresholds = lambda_j (the dual box)
  if ((st = set_lambda(c, &lp)) != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  // zero start: u (in w) and the spectra of ubar; y (in the g array) is written, not read, by
  // the first iteration
  enqueue_zero(c, c.L.w, size_t(p->q) * n2 * 4);
  enqueue_zero(c, c.L.v, size_t(p->q) * p->n * p->P * 8);
  enqueue_zero_counters(c);
  LAUNCHCHK("initial state");
  double tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool have = false;
  for (int it = 0; it < prm->iters; ++it) {
    const bool last = it == prm->iters - 1;
    const bool stats = d_hist != nullptr || (last && h_stats != nullptr);
    enqueue_pd_iteration(c, d_s, prm->tau, prm->sigma, it == 0, last, stats, d_hist ? d_hist + 4LL * it : nullptr);
    LAUNCHCHK("primal-dual iteration");
    if (last && h_stats) {
      HIPCHK(hipMemcpyAsync(tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
      HIPCHK(hipStreamSynchronize(c.s));
      have = true;
      if (tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite value in the primal-dual iteration");
    }
  }
  enqueue_epilogue(c, d_u, d_labels);
  LAUNCHCHK("epilogue");
  if (h_stats) {
    shs_stats out{};
    out.iters_done = prm->iters;
    if (have) {
      out.r_primal = std::sqrt(tot[SLOT_DB2]);
      out.r_dual = std::sqrt(tot[SLOT_DY2]);
      out.r_combined = tot[SLOT_DY2] + tot[SLOT_DB2];
      out.energy_surrogate = tot[SLOT_WS] + tot[SLOT_L1];
    }
    double e = 0.0;
    st = energy_of(c, c.at<float>(c.L.w), d_s, &e);
    if (st != SHS_OK) return st;
    out.energy = e;
    *h_stats = out;
  }
  return SHS_OK;
}

shs_status shs_solve_tv(const shs_plan* p, const shs_params* prm, const float* d_s, void* d_ws, size_t ws_bytes,
                        float* d_u, int32_t* d_labels, double* d_hist, shs_stats* h_stats, void* stream) {
  if (!p || !prm || !d_s || !prm->lambda) return fail(SHS_E_INVALID, "null argument");
  shs_status st = check_params(prm);
  if (st != SHS_OK) return st;
  if (prm->lambda_len != 1) return fail(SHS_E_INVALID, "the TV model takes one weight (lambda_len = 1)");
  const float lam = prm->lambda[0];
  if (!(lam >= 0.f) || !std::isfinite(lam)) return fail(SHS_E_INVALID, "lambda must be finite and >= 0");
  if (prm->resume) return fail(SHS_E_INVALID, "the TV solver starts from the zero state only");
  if (p->q > kTvMaxLabels) return fail(SHS_E_UNSUPPORTED, "too many labels for the TV solver");
  DeviceGuard dg(p->device);
  Ctx c;
  st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  // the first iteration reads no state
  if (prm->iters == 0) enqueue_zero_state(c);
  enqueue_zero_counters(c);
  LAUNCHCHK("initial state");
  const double rnorm = std::sqrt(double(p->q) * double(n2));
  double tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool have = false;
  int done = 0;
  for (int it = 0; it < prm->iters; ++it) {
    const bool last = it == prm->iters - 1;
    const bool check = prm->tol > 0.0 && ((it + 1) % prm->check_every == 0 || last);
    const bool stats = d_hist != nullptr || check || (last && h_stats != nullptr);
    // w is read by statistics and by the result only: written where the next iteration or the
    // end of the solve needs it
    const bool next_stats = d_hist != nullptr || (it + 2 == prm->iters && h_stats != nullptr) ||
                            (prm->tol > 0.0 && ((it + 2) % prm->check_every == 0 || it + 2 == prm->iters));
    enqueue_tv_iteration(c, d_s, lam, prm->gamma, it == 0, last || check || next_stats, stats,
                         d_hist ? d_hist + 4LL * it : nullptr);
    LAUNCHCHK("TV iteration");
    done = it + 1;
    if (check || (last && h_stats)) {
      HIPCHK(hipMemcpyAsync(tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
      HIPCHK(hipStreamSynchronize(c.s));
      have = true;
      if (tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite residual at iteration " + std::to_string(it + 1));
      if (check && std::sqrt(tot[SLOT_DY2] + tot[SLOT_DB2]) <= prm->tol * rnorm) break;
    }
  }
  enqueue_epilogue(c, d_u, d_labels);
  LAUNCHCHK("epilogue");
  if (h_stats) {
    shs_stats out{};
    out.iters_done = done;
    if (have) {
      out.r_primal = std::sqrt(tot[SLOT_DB2]);
      out.r_dual = std::sqrt(tot[SLOT_DY2]) / prm->gamma;
      out.r_combined = tot[SLOT_DY2] + tot[SLOT_DB2];
      out.energy_surrogate = tot[SLOT_WS] + tot[SLOT_L1];
    }
    double e = 0.0;
    if ((st = tv_energy_of(c, d_s, lam, &e)) != SHS_OK) return st;
    out.energy = e;
    *h_stats = out;
  }
  return SHS_OK;
}

shs_status shs_nl_graph(int32_t n, int32_t channels, const float* h_img, const shs_nl_graph_params* prm,
                        int32_t* h_nbr, int32_t* h_rev, int32_t* h_max_degree) {
  if (!h_img || !prm || !h_nbr || !h_rev) return fail(SHS_E_INVALID, "null argument");
  if (channels < 1 || channels > SHS_MAX_CHANNELS) return fail(SHS_E_INVALID, "channels must be 1..4");
  if (prm->patch < 1 || prm->patch % 2 == 0) return fail(SHS_E_INVALID, "patch must be odd and >= 1");
  if (prm->window < 3 || prm->window % 2 == 0) return fail(SHS_E_INVALID, "window must be odd and >= 3");
  if (n < prm->window || n > 4096) return fail(SHS_E_INVALID, "n must be in window..4096");
  if (prm->m < 1 || 2 * prm->m > kNlMaxBlocks) return fail(SHS_E_INVALID, "m must be 1..8");
  if (!(prm->a > 0.f) || !std::isfinite(prm->a)) return fail(SHS_E_INVALID, "a must be finite and > 0");
  NlGraphCfg g{n, channels, prm->patch, prm->window, prm->m, double(prm->a)};
  const int md = nl_build_graph(g, h_img, h_nbr, h_rev);
  if (h_max_degree) *h_max_degree = md;
  return SHS_OK;
}

shs_status shs_solve_nl(const shs_plan* p, const shs_nl_params* prm, const float* d_s, const int32_t* d_nbr,
                        const int32_t* d_rev, void* d_ws, size_t ws_bytes, float* d_u, int32_t* d_labels,
                        double* d_hist, shs_stats* h_stats, void* stream) {
  if (!p || !prm || !d_s || !d_nbr || !d_rev) return fail(SHS_E_INVALID, "null argument");
  if (prm->blocks < 1 || prm->blocks > kNlMaxBlocks) return fail(SHS_E_INVALID, "blocks must be 1..16");
  if (prm->blocks > p->eta) return fail(SHS_E_UNSUPPORTED, "the plan's state holds q * eta images: need eta >= blocks");
  if (prm->max_degree < 0 || prm->max_degree > prm->blocks) return fail(SHS_E_INVALID, "bad max_degree");
  if (!(prm->tau > 0.f) || !(prm->sigma > 0.f) || !std::isfinite(prm->tau) || !std::isfinite(prm->sigma))
    return fail(SHS_E_INVALID, "tau and sigma must be finite and > 0");
  if (double(prm->tau) * double(prm->sigma) * 4.0 * std::max(prm->max_degree, 1) > 1.0 + 1e-6)
    return fail(SHS_E_INVALID, "tau * sigma * 4 * max_degree must be <= 1 (||D||^2 <= 4 max_degree)");
  if (!(prm->lambda >= 0.f) || !std::isfinite(prm->lambda)) return fail(SHS_E_INVALID, "lambda must be >= 0");
  if (prm->iters < 0) return fail(SHS_E_INVALID, "iters must be >= 0");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  const long long npix = (n2 + 255) / 256;
  // Zero start: u; y and ubar are written, not read, by the first iteration.  The records of y
  // (16-bit types: padded to whole words) take the state's place, or where they do not fit
  // there the spectra's, which this solver does not use; the neighbour records' indexes follow.
  enqueue_zero(c, c.L.w, size_t(p->q) * n2 * 4);
  const size_t ybytes = align256(size_t(prm->blocks) * n2 * nl_record_bytes(p->store, p->q));
  const size_t ibytes = align256(size_t(prm->blocks) * n2 * 4);
  const bool in_state = ybytes <= c.L.w - c.L.g, idx_in_state = in_state && ybytes + ibytes <= c.L.w - c.L.g;
  const size_t yoff = in_state ? c.L.g : c.L.t1;
  const size_t ioff = idx_in_state ? c.L.g + ybytes : in_state ? c.L.t1 : c.L.t1 + ybytes;
  if ((in_state ? (idx_in_state ? 0 : ibytes) : ybytes + ibytes) > c.L.zs - c.L.t1)
    return fail(SHS_E_UNSUPPORTED, "the graph's blocks do not fit the plan's workspace");
  NlParams np{};
  np.y = c.ws + yoff;
  np.u = c.at<float>(c.L.w);
  np.ubar = c.at<float>(c.L.us);
  np.ysum = c.at<float>(c.L.zs);
  np.s = d_s;
  np.nbr = d_nbr;
  np.rev = d_rev;
  np.src = c.at<int32_t>(ioff);
  np.n2 = n2;
  np.q = p->q;
  np.M2 = prm->blocks;
  np.lambda = prm->lambda;
  np.tau = prm->tau;
  np.sigma = prm->sigma;
  if (prm->iters > 0) nl_launch(p->store, NL_INDEX, np, c.s);
  enqueue_zero_counters(c);
  LAUNCHCHK("initial state");
  double tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool have = false;
  for (int it = 0; it < prm->iters; ++it) {
    const bool last = it == prm->iters - 1;
    const bool stats = d_hist != nullptr || (last && h_stats != nullptr);
    NlParams pd = np, pp = np;
    pd.partials = c.at<double>(c.L.parts);
    pp.partials = c.at<double>(c.L.parts) + npix * 4;
    pd.stats = pp.stats = stats ? 1 : 0;
    pd.fresh = it == 0 ? 1 : 0;
    {
      Timed tm(c.s, KC_NL_DUAL);
      nl_launch(p->store, NL_DUAL, pd, c.s);
    }
    {
      Timed tm(c.s, KC_NL_PRIMAL);
      nl_launch(p->store, NL_PRIMAL, pp, c.s);
    }
    if (stats) enqueue_reduce(c, 2 * npix, d_hist ? d_hist + 4LL * it : nullptr, 1.0);
    LAUNCHCHK("NL primal-dual iteration");
    if (last && h_stats) {
      HIPCHK(hipMemcpyAsync(tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
      HIPCHK(hipStreamSynchronize(c.s));
      have = true;
      if (tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite value in the NL iteration");
    }
  }
  enqueue_epilogue(c, d_u, d_labels);
  LAUNCHCHK("epilogue");
  if (h_stats) {
    shs_stats out{};
    out.iters_done = prm->iters;
    if (have) {
      out.r_primal = std::sqrt(tot[SLOT_DB2]);
      out.r_dual = std::sqrt(tot[SLOT_DY2]);
      out.r_combined = tot[SLOT_DY2] + tot[SLOT_DB2];
      out.energy_surrogate = tot[SLOT_WS] + tot[SLOT_L1];
    }
    NlParams pe = np;
    pe.partials = c.at<double>(c.L.parts);
    {
      Timed tm(c.s, KC_OTHER);
      nl_launch(p->store, NL_ENERGY, pe, c.s);
    }
    enqueue_reduce(c, npix, nullptr, 1.0);
    LAUNCHCHK("NL energy");
    double e[8];
    HIPCHK(hipMemcpyAsync(e, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
    HIPCHK(hipStreamSynchronize(c.s));
    if (e[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite energy");
    out.energy = e[SLOT_WS] + e[SLOT_L1];
    *h_stats = out;
  }
  return SHS_OK;
}

// The transform entry points take any number of images and run them in groups of at
// most q (the plan's label count sizes the workspace's spectra).
shs_status shs_shearlet_forward(const shs_plan* p, int32_t count, const float* d_f, float* d_c, void* d_ws,
                                size_t ws_bytes, void* stream) {
  if (!p || !d_f || !d_c) return fail(SHS_E_INVALID, "null argument");
  if (count < 1) return fail(SHS_E_INVALID, "count must be >= 1");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  for (int i0 = 0; i0 < count; i0 += p->q) {
    const int k = std::min(p->q, count - i0);
    enqueue_synthesis(c, d_f + i0 * n2, k);
    RowParams rp{};
    rp.spec_in = c.at<float2>(c.L.t1);
    rp.lin = pruned_layout(p);
    rp.real_out = d_c + (long long)i0 * p->eta * n2;
    run_row(c, ROW_C2R, ST_F32, false, rp, k * p->eta);
    LAUNCHCHK("forward");
  }
  return SHS_OK;
}

shs_status shs_shearlet_adjoint(const shs_plan* p, int32_t count, const float* d_c, float* d_f, void* d_ws,
                                size_t ws_bytes, void* stream) {
  if (!p || !d_f || !d_c) return fail(SHS_E_INVALID, "null argument");
  if (count < 1) return fail(SHS_E_INVALID, "count must be >= 1");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  for (int i0 = 0; i0 < count; i0 += p->q) {
    const int k = std::min(p->q, count - i0);
    RowParams rp{};
    rp.real_in = d_c + (long long)i0 * p->eta * n2;
    rp.spec_out = c.at<float2>(c.L.t2);
    rp.lout = pruned_layout(p);
    run_row(c, ROW_R2C, ST_F32, false, rp, k * p->eta);
    enqueue_analysis(c, k);
    RowParams rz{};
    rz.spec_in = c.at<float2>(c.L.z);
    rz.lin = dense_layout(p);
    rz.real_out = d_f + i0 * n2;
    run_row(c, ROW_C2R, ST_F32, false, rz, k);
    LAUNCHCHK("adjoint");
  }
  return SHS_OK;
}

// S^T S_lambda S: forward transform, soft shrinkage of every coefficient and the adjoint,
// with the shrinkage inside the row pass between the two column passes (the coefficient
// images are never stored).
shs_status shs_shearlet_denoise(const shs_plan* p, int32_t count, const float* h_lambda, int32_t lambda_len,
                                const float* d_f, float* d_out, void* d_ws, size_t ws_bytes, void* stream) {
  if (!p || !d_f || !d_out || !h_lambda) return fail(SHS_E_INVALID, "null argument");
  if (count < 1) return fail(SHS_E_INVALID, "count must be >= 1");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  shs_params prm{};
  prm.lambda = h_lambda;
  prm.lambda_len = lambda_len;
  prm.gamma = 1.f;
  if ((st = set_lambda(c, &prm)) != SHS_OK) return st;
  const long long n2 = (long long)p->n * p->n;
  for (int i0 = 0; i0 < count; i0 += p->q) {
    const int k = std::min(p->q, count - i0);
    enqueue_synthesis(c, d_f + i0 * n2, k);
    RowParams rp{};
    rp.spec_in = c.at<float2>(c.L.t1);
    rp.lin = pruned_layout(p);
    rp.spec_out = c.at<float2>(c.L.t2);
    rp.lout = pruned_layout(p);
    run_row(c, ROW_SHRINK, ST_F32, false, rp, k * p->eta);
    enqueue_analysis(c, k);
    RowParams rz{};
    rz.spec_in = c.at<float2>(c.L.z);
    rz.lin = dense_layout(p);
    rz.real_out = d_out + i0 * n2;
    run_row(c, ROW_C2R, ST_F32, false, rz, k);
    LAUNCHCHK("denoise");
  }
  return SHS_OK;
}

shs_status shs_energy(const shs_plan* p, const shs_params* prm, const float* d_s, const float* d_u, void* d_ws,
                      size_t ws_bytes, double* h_energy, void* stream) {
  if (!p || !prm || !d_s || !d_u || !h_energy) return fail(SHS_E_INVALID, "null argument");
  DeviceGuard dg(p->device);
  Ctx c;
  shs_status st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  shs_params tmp = *prm;
  if (!(tmp.gamma > 0.f)) tmp.gamma = 1.f;
  st = set_lambda(c, &tmp);
  if (st != SHS_OK) return st;
  enqueue_zero_counters(c);
  return energy_of(c, d_u, d_s, h_energy);
}

}  // extern "C"

namespace {
// shs_solve; allow_graphs = false keeps every launch eager (no graph capture or
// instantiation, which may allocate).
shs_status solve_impl(const shs_plan* p, const shs_params* prm, const float* d_s, void* d_ws, size_t ws_bytes,
                      float* d_u, int32_t* d_labels, double* d_hist, shs_stats* h_stats, void* stream,
                      bool allow_graphs) {
  if (!p || !prm || !d_s) return fail(SHS_E_INVALID, "null argument");
  shs_status st = check_params(prm);
  if (st != SHS_OK) return st;
  DeviceGuard dg(p->device);
  Ctx c;
  st = make_ctx(p, d_ws, ws_bytes, stream, c);
  if (st != SHS_OK) return st;
  st = set_lambda(c, prm);
  if (st != SHS_OK) return st;

  const int q = p->q;
  const long long n2 = (long long)p->n * p->n;
  if (!prm->resume) {
    // the first iteration writes the whole state without reading it
    if (prm->iters == 0) enqueue_zero_state(c);
  } else {
    RowParams rp{};
    rp.g = c.ws + c.L.g;
    rp.spec_out = c.at<float2>(c.L.t2);
    rp.lout = pruned_layout(p);
    run_row(c, ROW_PRIME, p->store, false, rp, q * p->eta);
  }
  LAUNCHCHK("initial state");

  const double rnorm = std::sqrt(double(q) * double(n2));
  int done = 0;
  bool have_adjoint_input = prm->resume != 0;
  double last_tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool have_last = false;
  // History rows are addressed through a device counter (reset here), so the launches of
  // every steady-state iteration are identical.
  int* hctr = d_hist ? c.at<int>(c.L.hctr) : nullptr;
  enqueue_zero_counters(c);
  // FP16 state overflows to inf beyond 65504: the last iteration's non-finite flag is
  // always reduced and checked for it (one synchronisation), also without h_stats.
  const bool f16_guard = p->store == SHS_STORE_F16;
  // Steady-state iterations (not the first, not the last; no host check in between) are
  // replayed from captured graphs of kGraphIters iterations unless kernel timing is on.
  const bool graphs = allow_graphs && prm->tol == 0.0 && prm->iters >= 4 && !profiling_on();
  for (int it = 0; it < prm->iters; ++it) {
    const bool last = it == prm->iters - 1;
    if (graphs && it >= 1 && it + kGraphIters < prm->iters) {
      const int reps = (prm->iters - 1 - it) / kGraphIters;
      st = replay_iterations(c, d_s, prm->gamma, d_hist, hctr, kGraphIters, reps);
      if (st != SHS_OK) return st;
      it += reps * kGraphIters - 1;
      have_adjoint_input = true;
      done = it + 1;
      continue;
    }
    const bool check = prm->tol > 0.0 && ((it + 1) % prm->check_every == 0 || last);
    const bool want_last = last && (h_stats != nullptr || f16_guard);
    const bool stats = d_hist != nullptr || check || want_last;
    enqueue_iteration(c, d_s, prm->gamma, have_adjoint_input, stats, !last, d_hist, hctr);
    LAUNCHCHK("iteration");
    have_adjoint_input = true;
    done = it + 1;
    if (check || want_last) {
      HIPCHK(hipMemcpyAsync(last_tot, c.at<double>(c.L.sdev), 5 * 8, hipMemcpyDeviceToHost, c.s));
      HIPCHK(hipStreamSynchronize(c.s));
      have_last = true;
      if (last_tot[4] != 0.0) return fail(SHS_E_NUMERIC, "non-finite residual at iteration " + std::to_string(it + 1));
      if (check && std::sqrt(last_tot[SLOT_DY2] + last_tot[SLOT_DB2]) <= prm->tol * rnorm) break;
    }
  }
  enqueue_epilogue(c, d_u, d_labels);
  LAUNCHCHK("epilogue");
  if (h_stats) {
    shs_stats out{};
    out.iters_done = done;
    if (have_last) {
      out.r_primal = std::sqrt(last_tot[SLOT_DB2]);
      out.r_dual = std::sqrt(last_tot[SLOT_DY2]) / prm->gamma;
      out.r_combined = last_tot[SLOT_DY2] + last_tot[SLOT_DB2];
      out.energy_surrogate = last_tot[SLOT_WS] + last_tot[SLOT_L1];
    }
    double e = 0.0;
    st = energy_of(c, c.at<float>(c.L.w), d_s, &e);
    if (st != SHS_OK) return st;
    out.energy = e;
    *h_stats = out;
  }
  return SHS_OK;
}

}  // namespace

extern "C" {

shs_status shs_solve(const shs_plan* p, const shs_params* prm, const float* d_s, void* d_ws, size_t ws_bytes,
                     float* d_u, int32_t* d_labels, double* d_hist, shs_stats* h_stats, void* stream) {
  return solve_impl(p, prm, d_s, d_ws, ws_bytes, d_u, d_labels, d_hist, h_stats, stream, true);
}

shs_status shs_solve_noalloc(const shs_plan* p, const shs_params* prm, const float* d_s, float* d_u,
                             int32_t* d_labels, double* d_hist, shs_stats* h_stats, void* stream) {
  if (!p || !prm || !d_s) return fail(SHS_E_INVALID, "null argument");
  const size_t need = shs_workspace_bytes(p);
  if (need > SHS_NOALLOC_MAX_BYTES)
    return fail(SHS_E_WORKSPACE, "this plan needs " + std::to_string(need) + " bytes of workspace; the "
                "allocation-free solve holds at most " + std::to_string((unsigned long long)SHS_NOALLOC_MAX_BYTES));
  DeviceGuard dg(p->device);
  if (!dg.ok) return fail(SHS_E_DEVICE, "hipSetDevice failed");
  void* ws = nullptr;
  const shs_status st = scratch_address(p->device, &ws);
  if (st != SHS_OK) return st;
  return solve_impl(p, prm, d_s, ws, need, d_u, d_labels, d_hist, h_stats, stream, false);
}

shs_status shs_batch_create(int32_t count, const shs_shape* shapes, int device, shs_batch** out) {
  if (!out || !shapes || count < 1) return fail(SHS_E_INVALID, "null argument or count < 1");
  if (count > 65535) return fail(SHS_E_UNSUPPORTED, "at most 65535 images per batch");
  *out = nullptr;
  shs_batch* b = new (std::nothrow) shs_batch{};
  if (!b) return fail(SHS_E_NOMEM, "host allocation");
  b->count = count;
  b->device = device;
  for (int i = 0; i < count; ++i) {
    const shs_shape& s = shapes[i];
    int found = -1;
    for (size_t k = 0; k < b->plans.size(); ++k) {
      const shs_plan* p = b->plans[k];
      if (p->n == s.n && p->C == s.channels && p->q == s.q && p->J == s.J && p->store == s.store) found = int(k);
    }
    if (found < 0) {
      shs_plan* p = nullptr;
      const shs_status st = shs_plan_create(&s, device, &p);
      if (st != SHS_OK) {
        const std::string msg = g_err;
        shs_batch_destroy(b);
        return fail(st, "image " + std::to_string(i) + ": " + msg);
      }
      b->plans.push_back(p);
      found = int(b->plans.size()) - 1;
    }
    b->plan_of.push_back(found);
    b->ws_off.push_back(b->ws_total);
    b->ws_total += align256(shs_workspace_bytes(b->plans[found]));
  }
  {
    std::vector<int> keys;
    for (int i = 0; i < count; ++i) {
      const int k = batch_class(b->plans[b->plan_of[i]]);
      size_t l = 0;
      while (l < keys.size() && keys[l] != k) ++l;
      if (l == keys.size()) {
        keys.push_back(k);
        b->lanes.emplace_back();
      }
      b->lanes[l].push_back(i);
    }
  }
  DeviceGuard dg(device);
  bool ok = hipStreamCreateWithFlags(&b->main, hipStreamNonBlocking) == hipSuccess &&
            hipEventCreateWithFlags(&b->fork, hipEventDisableTiming) == hipSuccess;
  for (size_t l = 0; ok && l < b->lanes.size(); ++l) {
    hipStream_t st = nullptr;
    hipEvent_t ev = nullptr;
    ok = hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess &&
         hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess;
    if (st) b->lane_s.push_back(st);
    if (ev) b->lane_e.push_back(ev);
  }
  if (!ok) {
    shs_batch_destroy(b);
    return fail(SHS_E_DEVICE, "batch stream creation");
  }
  *out = b;
  return SHS_OK;
}

shs_status shs_batch_destroy(shs_batch* b) {
  if (!b) return SHS_OK;
  DeviceGuard dg(b->device);
  b->drop_graph();
  if (b->main) (void)hipStreamDestroy(b->main);
  if (b->fork) (void)hipEventDestroy(b->fork);
  for (hipStream_t st : b->lane_s) (void)hipStreamDestroy(st);
  for (hipEvent_t ev : b->lane_e) (void)hipEventDestroy(ev);
  for (shs_plan* p : b->plans) shs_plan_destroy(p);
  delete b;
  return SHS_OK;
}

size_t shs_batch_workspace_bytes(const shs_batch* b) { return b ? b->ws_total : 0; }

shs_status shs_solve_batch(shs_batch* b, const shs_params* params, const float* const* d_s, void* d_ws,
                           size_t ws_bytes, float* const* d_u, int32_t* const* d_labels, double* d_stats,
                           void* stream) {
  if (!b || !params || !d_s) return fail(SHS_E_INVALID, "null argument");
  if (!d_ws || ws_bytes < b->ws_total) return fail(SHS_E_WORKSPACE, "batch workspace too small");
  if (reinterpret_cast<uintptr_t>(d_ws) % 256 != 0) return fail(SHS_E_WORKSPACE, "workspace must be 256-byte aligned");
  const int iters = params[0].iters;
  for (int i = 0; i < b->count; ++i) {
    const shs_status st = check_params(&params[i]);
    if (st != SHS_OK) return fail(st, "image " + std::to_string(i) + ": " + g_err);
    if (!d_s[i]) return fail(SHS_E_INVALID, "null data term of image " + std::to_string(i));
    if (params[i].iters != iters) return fail(SHS_E_UNSUPPORTED, "all images of a batch run the same iteration count");
    if (params[i].tol != 0.0 || params[i].resume) return fail(SHS_E_UNSUPPORTED, "batch solves take no tol / resume");
  }
  DeviceGuard dg(b->device);
  // per-image contexts, all on the capture stream
  std::vector<Ctx> ctx(b->count);
  for (int i = 0; i < b->count; ++i) {
    const shs_plan* p = b->plans[b->plan_of[i]];
    shs_status st = make_ctx(p, static_cast<char*>(d_ws) + b->ws_off[i], shs_workspace_bytes(p), nullptr, ctx[i]);
    if (st == SHS_OK) st = set_lambda(ctx[i], &params[i]);
    if (st != SHS_OK) return fail(st, "image " + std::to_string(i) + ": " + g_err);
    ctx[i].s = b->main;
  }
  // graph cache key: every pointer and parameter baked into the graph
  std::vector<double> key;
  key.push_back(double(reinterpret_cast<uintptr_t>(d_ws)));
  key.push_back(double(reinterpret_cast<uintptr_t>(d_stats)));
  key.push_back(iters);
  for (int i = 0; i < b->count; ++i) {
    key.push_back(double(reinterpret_cast<uintptr_t>(d_s[i])));
    key.push_back(double(reinterpret_cast<uintptr_t>(d_u ? d_u[i] : nullptr)));
    key.push_back(double(reinterpret_cast<uintptr_t>(d_labels ? d_labels[i] : nullptr)));
    key.push_back(params[i].gamma);
    for (int f = 0; f < ctx[i].p->eta; ++f) key.push_back(ctx[i].fw.lam[f]);
  }
  if (key != b->key || !b->graph) {
    b->drop_graph();
    // the iteration variants, recorded for all images and grouped
    struct Variant {
      bool adj, stats, emit;
    };
    std::vector<Variant> vars;
    if (iters == 1) vars = {{false, true, false}};
    else if (iters == 2) vars = {{false, false, true}, {true, true, false}};
    else if (iters >= 3) vars = {{false, false, true}, {true, false, true}, {true, true, false}};
    std::vector<char> arena;
    const size_t nl = b->lanes.size();
    std::vector<std::vector<BatchIter>> its(nl, std::vector<BatchIter>(vars.size()));
    for (size_t l = 0; l < nl; ++l) {
      for (size_t v = 0; v < vars.size(); ++v) {
        Recorder rec;
        CaptureScope cs;        // no timing events while recording
        g_rec = &rec;
        for (int i : b->lanes[l])
          enqueue_iteration(ctx[i], d_s[i], params[i].gamma, vars[v].adj, vars[v].stats, vars[v].emit, nullptr);
        g_rec = nullptr;
        build_batch_iter(rec.recs, arena, its[l][v]);
      }
    }
    if (!arena.empty()) {
      if (hipMalloc(&b->arena, arena.size()) != hipSuccess) return fail(SHS_E_NOMEM, "batch task tables");
      HIPCHK(hipMemcpy(b->arena, arena.data(), arena.size(), hipMemcpyHostToDevice));
    }
    char* dbase = static_cast<char*>(b->arena);
    auto tail = [&](int i) {   // epilogue + statistics of image i (zeros when no iteration ran)
      const Ctx& c = ctx[i];
      enqueue_epilogue(c, d_u ? d_u[i] : nullptr, d_labels ? d_labels[i] : nullptr);
      if (d_stats && iters > 0)
        hipLaunchKernelGGL(k_copy_f64, dim3(1), dim3(64), 0, c.s, c.at<double>(c.L.sdev), 5, d_stats + 5LL * i);
      else if (d_stats)
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, c.s, reinterpret_cast<uint32_t*>(d_stats + 5LL * i),
                           10LL, 0u);
    };
    {
      CaptureScope cs;
      HIPCHK(hipStreamBeginCapture(b->main, hipStreamCaptureModeThreadLocal));
      bool ok = hipEventRecord(b->fork, b->main) == hipSuccess;
      for (size_t l = 0; ok && l < nl; ++l) {
        hipStream_t ls = b->lane_s[l];
        ok = hipStreamWaitEvent(ls, b->fork, 0) == hipSuccess;
        for (int i : b->lanes[l]) {
          ctx[i].s = ls;
          if (iters == 0) enqueue_zero_state(ctx[i]);
          enqueue_zero_counters(ctx[i]);
        }
        if (iters >= 1) launch_batch_iter(its[l][0], dbase, ls);
        for (int it = 1; it + 1 < iters; ++it) launch_batch_iter(its[l][1], dbase, ls);
        if (iters >= 2) launch_batch_iter(its[l].back(), dbase, ls);
        for (int i : b->lanes[l]) tail(i);
        ok = ok && hipEventRecord(b->lane_e[l], ls) == hipSuccess &&
             hipStreamWaitEvent(b->main, b->lane_e[l], 0) == hipSuccess;
      }
      const hipError_t el = ok ? hipGetLastError() : hipErrorUnknown;
      hipGraph_t g = nullptr;
      const hipError_t ee = hipStreamEndCapture(b->main, &g);
      if (el != hipSuccess || ee != hipSuccess || !g) {
        if (g) (void)hipGraphDestroy(g);
        b->drop_graph();
        return fail(SHS_E_DEVICE, "capture of the batch graph failed");
      }
      const hipError_t ei = hipGraphInstantiate(&b->graph, g, nullptr, nullptr, 0);
      (void)hipGraphDestroy(g);
      if (ei != hipSuccess) {
        b->graph = nullptr;
        b->drop_graph();
        return fail(SHS_E_DEVICE, std::string("graph instantiate: ") + hipGetErrorString(ei));
      }
    }
    b->key = key;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  Timed tm(s, KC_BATCH);
  HIPCHK(hipGraphLaunch(b->graph, s));
  return SHS_OK;
}

}  // extern "C"
