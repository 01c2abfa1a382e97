// Launcher of one mixed-radix row pass; the mixed_*.hip units instantiate it for their modes
// and storage types.
#pragma once
#include "host.hpp"

namespace shs {

inline GenParams mixed_params(const shs_plan* p) {
  return GenParams{p->fft, p->n, p->wpb, p->rw == 4 ? 2 : p->rw == 2 ? 1 : 0, p->nbuf, 0};
}

template <int MODE, int ST, bool STATS>
void mixed_row(const shs_plan* p, const RowParams& rp, int channels, hipStream_t s) {
  // p->wpb waves per block, p->rw rows per wave
  const dim3 grid(p->n / p->rpb, channels);
  const int threads = 64 * p->wpb;
  const size_t lds = row_g_lds_bytes(p->M, p->rw, p->wpb, p->nbuf);
  if constexpr (batch_row_mode(MODE)) {
    if (g_rec) {
      LaunchRec& r = rec_add(RK_ROW, &kg_row_g<MODE, ST, STATS>, threads, p->n / p->rpb, channels, lds);
      r.rp = rp;
      r.gp = mixed_params(p);
      return;
    }
  }
  hipLaunchKernelGGL((k_row_g<MODE, ST, STATS>), grid, dim3(threads), lds, s, rp, mixed_params(p));
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
