// Declarations shared by the library's host code and the translation units that instantiate
// and launch its kernels (one unit per group of sizes, so that they compile in parallel).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "shearseg.h"
#include "kernels.hpp"
#include "generic.hpp"
#include "grouped.hpp"

using namespace shs;

struct shs_plan {
  int n, C, q, J, store, eta, M, P, PP, W, NS, device;
  int generic;         // 1: mixed-radix path (N not a power of two)
  int rpb;             // rows per row-pass block
  int rw;              // generic path: rows per wave of the row pass (1, 2 or 4)
  int wpb;             // generic path: waves per row-pass block (1, 2 or 4)
  int nbuf;            // generic path: LDS buffers per row-pass wave (row_g_bufs)
  FftPlan prow, pfwd, pcol;  // mixed-radix transforms: inverse rows, forward rows, columns
  FftPlan* fft;        // the same three in device memory (FFT_* order)
  float* psi;          // [eta][N][PP] dense filter bank (half spectrum)
  float2* tw;          // [N] exp(-2 pi i m / N), then (power-of-two N) the FFT stage tables
  float* eig;          // [N] 4 sin^2(pi k / N): DFT eigenvalues of one forward-difference pair (TV)
  // pruned layout
  float* psiw;         // filter values inside each column window
  int4* pwin;          // [eta][M+1] {a, L, value offset, 0}
  int4* tcol;          // [eta] {cb, pitch, off_lo, off_hi} of the filtered spectra
  long long t_ls;      // label stride of the filtered spectra (float2)
  // column work lists
  int4* items_syn;     // {strip, first work-list entry, count, -1}
  int4* items_ana;     // {strip, first work-list entry, count, partial slot or -1}
  int4* fwin;          // work list, entries grouped by strip: column windows [entry][W]
  int4* fgeo;          // and plane geometry [entry]
  int2* strips_ana;    // per strip {first analysis item, items}
  int n_syn, n_ana, n_part;
  int fc_syn;          // filters per synthesis work item
  long long nnz;       // stored filter values
  struct GraphCache* graphs;  // captured steady-state iterations of shs_solve
  char schedule[256];  // chosen launch schedule (shs_plan_describe)
};

// Executable graphs of steady-state ADMM iterations, keyed by everything the captured
// launches bake in (workspace, data term, history, thresholds, iteration count).  Captured
// on a stream of the plan's own and launched on the caller's stream; a few entries, least
// recently used dropped first.  The mutex makes lookups, captures and launches of one plan
// safe from several host threads.
struct GraphCache {
  struct Entry {
    std::vector<uint64_t> key;
    hipGraphExec_t exec;
  };
  std::mutex mu;
  hipStream_t cap = nullptr;
  std::vector<Entry> entries;   // most recently used last
  static constexpr size_t kMax = 6;
  ~GraphCache() {
    for (Entry& e : entries) (void)hipGraphExecDestroy(e.exec);
    if (cap) (void)hipStreamDestroy(cap);
  }
};

namespace shs {

// ---------------------------------------------------------------- launch recording (batches)
// While a Recorder is installed (this thread), the launchers below append a description of
// each launch, with the grouped kernel of its configuration, instead of launching; the
// batch solve turns one iteration's records of all images into grouped launches.  Each
// record carries the step of the iteration it belongs to.
enum BatchStep { BS_ANA, BS_FINAL, BS_MID, BS_FWD, BS_SYN, BS_ROW, BS_REDUCE, BS_COUNT };
enum RecKind { RK_ROW, RK_COL, RK_MID, RK_REDUCE };
struct LaunchRec {
  int step = 0, kind = 0;
  const void* fn = nullptr;    // grouped kernel of the launch's configuration
  int threads = 0, gx = 0, gy = 0;
  size_t lds = 0;              // dynamic LDS bytes
  RowParams rp{};
  ColParams cp{};
  MidParams mp{};
  GenParams gp{};
  // RK_REDUCE (one image's FP64 reduction)
  double* parts = nullptr;
  long long nparts = 0;
  double* red1 = nullptr;
  double* sdev = nullptr;
  double gamma = 1.0;
};
struct Recorder {
  std::vector<LaunchRec> recs;
  int step = 0;
};
extern thread_local Recorder* g_rec;
inline void rec_step(int s) {
  if (g_rec) g_rec->step = s;
}
// Row-pass modes of a batch's iterations (the others have no grouped kernel).
constexpr bool batch_row_mode(int mode) { return mode == ROW_SOLVE; }
template <class F>
LaunchRec& rec_add(int kind, F fn, int threads, int gx, int gy, size_t lds) {
  LaunchRec r;
  r.step = g_rec->step;
  r.kind = kind;
  r.fn = reinterpret_cast<const void*>(fn);
  r.threads = threads;
  r.gx = gx;
  r.gy = gy;
  r.lds = lds;
  g_rec->recs.push_back(r);
  return g_rec->recs.back();
}

// Launchers of one size: row passes by mode, column passes by kind (COL_*), and the TV
// model's column solve.
struct Ops {
  void (*row)(const shs_plan*, int, int, bool, const RowParams&, int, hipStream_t);
  void (*col)(const shs_plan*, int, const ColParams&, int, int, hipStream_t);
  void (*col_solve)(const shs_plan*, const ColParams&, int, hipStream_t);
  // middle step (MID_*) and its blocks
  void (*mid)(const shs_plan*, int, const MidParams&, hipStream_t);
  int (*mid_blocks)(const shs_plan*);
  // Lets the path's kernels take LDS (static and dynamic together) beyond the runtime's default
  // limit, where the plan can need it (as much as the largest plan of the path needs: plans are
  // created in any order); false if the runtime refuses.
  bool (*reserve)(const shs_plan*);
};
enum { COL_FWD = 0, COL_SYN = 1, COL_ANA = 2, COL_FINAL = 3 };

// Power-of-two sizes (pow2_*.hip) and the mixed-radix path (mixed_*.hip).
template <int N> Ops pow2_ops();
extern template Ops pow2_ops<64>();
extern template Ops pow2_ops<128>();
extern template Ops pow2_ops<256>();
extern template Ops pow2_ops<512>();
extern template Ops pow2_ops<1024>();
extern template Ops pow2_ops<2048>();
Ops mixed_ops();

constexpr size_t kDefaultLds = 64 * 1024;   // a block's static and dynamic LDS without a raised limit
// Threads of a column-pass block: one per butterfly of the stage with the most of them, in
// whole waves, up to 256.
inline int col_g_threads(const FftPlan& pl) {
  int rmin = pl.radix[0];
  for (int i = 1; i < pl.ns; ++i) rmin = pl.radix[i] < rmin ? pl.radix[i] : rmin;
  const int waves = (pl.L / rmin * kGW + 63) / 64;
  return 64 * (waves < 4 ? waves : 4);
}
// Dynamic LDS of a column-pass block: the twiddle table, `extra` strips (the spectrum or the
// accumulator) and the transform's buffers.
inline size_t col_g_lds_bytes(const shs_plan* p, int extra) {
  return (size_t(extra + col_bufs(p->pcol)) * p->n * kGW + col_tab_len(p->n)) * sizeof(float2);
}
}  // namespace shs
