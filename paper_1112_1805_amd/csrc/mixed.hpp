// Launcher of one mixed-radix row pass; the mixed_*.hip units instantiate it for their modes
// and storage types.
#pragma once
#include "host.hpp"

namespace shs {

inline GenParams mixed_params(const shs_plan* p) { return GenParams{p->prow, p->pcol, p->n, p->wpb}; }

template <int MODE, int ST, bool STATS>
void mixed_row(const shs_plan* p, const RowParams& rp, int channels, hipStream_t s) {
  // p->wpb waves per block, p->rw rows per wave
  const dim3 grid(p->n / p->rpb, channels);
  const int threads = 64 * p->wpb;
  const size_t lds = row_g_lds_bytes(p->M, p->rw, p->wpb, p->n);
  if constexpr (batch_row_mode(MODE)) {
    if (g_rec) {
      LaunchRec* r = nullptr;
      switch (p->rw) {
        case 4: r = &rec_add(RK_ROW, &kg_row_g<MODE, ST, STATS, 4>, threads, p->n / p->rpb, channels, lds); break;
        case 2: r = &rec_add(RK_ROW, &kg_row_g<MODE, ST, STATS, 2>, threads, p->n / p->rpb, channels, lds); break;
        default: r = &rec_add(RK_ROW, &kg_row_g<MODE, ST, STATS, 1>, threads, p->n / p->rpb, channels, lds); break;
      }
      r->rp = rp;
      r->gp = mixed_params(p);
      return;
    }
  }
  const GenParams gp = mixed_params(p);
  switch (p->rw) {
    case 4: hipLaunchKernelGGL((k_row_g<MODE, ST, STATS, 4>), grid, dim3(threads), lds, s, rp, gp); break;
    case 2: hipLaunchKernelGGL((k_row_g<MODE, ST, STATS, 2>), grid, dim3(threads), lds, s, rp, gp); break;
    default: hipLaunchKernelGGL((k_row_g<MODE, ST, STATS, 1>), grid, dim3(threads), lds, s, rp, gp); break;
  }
}

#define SHS_MIXED_ROWS(X)                                                                    \
  X(ROW_SOLVE, ST_F32, true) X(ROW_SOLVE, ST_F32, false) X(ROW_SOLVE, ST_BF16, true)         \
  X(ROW_SOLVE, ST_BF16, false) X(ROW_SOLVE, ST_F16, true) X(ROW_SOLVE, ST_F16, false)        \
  X(ROW_PD, ST_F32, true) X(ROW_PD, ST_F32, false) X(ROW_PD, ST_BF16, true)                  \
  X(ROW_PD, ST_BF16, false) X(ROW_PD, ST_F16, true) X(ROW_PD, ST_F16, false)                 \
  X(ROW_PRIME, ST_F32, false) X(ROW_PRIME, ST_BF16, false) X(ROW_PRIME, ST_F16, false)       \
  X(ROW_C2R, ST_F32, false) X(ROW_R2C, ST_F32, false) X(ROW_ENERGY, ST_F32, true)            \
  X(ROW_SHRINK, ST_F32, false)
#define SHS_MIXED_ROW_EXTERN(MODE, ST, STATS) \
  extern template void mixed_row<MODE, ST, STATS>(const shs_plan*, const RowParams&, int, hipStream_t);
SHS_MIXED_ROWS(SHS_MIXED_ROW_EXTERN)
#define SHS_MIXED_ROW_HERE(MODE, ST, STATS) \
  template void shs::mixed_row<MODE, ST, STATS>(const shs_plan*, const RowParams&, int, hipStream_t);

}  // namespace shs
