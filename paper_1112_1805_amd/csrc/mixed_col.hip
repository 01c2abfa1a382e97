// Mixed-radix column passes, the plain row transforms, and the launch table of the path.
#include "mixed.hpp"
#include "generic_col.hpp"

SHS_MIXED_ROW_HERE(ROW_C2R, ST_F32, false)
SHS_MIXED_ROW_HERE(ROW_R2C, ST_F32, false)

namespace shs {

static void mixed_row_any(const shs_plan* p, int mode, int store, bool stats, const RowParams& rp, int channels,
                          hipStream_t s) {
#define SHS_CASE(MODE, ST, STATS) \
  if (mode == MODE && store == ST && stats == STATS) return mixed_row<MODE, ST, STATS>(p, rp, channels, s);
  SHS_MIXED_ROWS(SHS_CASE)
#undef SHS_CASE
}

static void mixed_col(const shs_plan* p, int kind, const ColParams& cp, int nblocks, int labels, hipStream_t s) {
  const dim3 grid(nblocks, labels), block(256);
  const size_t e = size_t(p->n) * kGW * sizeof(float2);
  const size_t t = size_t(col_tab_len(p->n)) * sizeof(float2);
  if (g_rec) {
    LaunchRec* r = nullptr;
    switch (kind) {
      case 0: r = &rec_add(RK_COL, &kg_colg_fwd, 256, nblocks, labels, t + 2 * e); break;
      case 1: r = &rec_add(RK_COL, &kg_colg_syn, 256, nblocks, labels, t + 3 * e); break;
      case 2: r = &rec_add(RK_COL, &kg_colg_ana, 256, nblocks, labels, t + 3 * e); break;
      case 3: r = &rec_add(RK_COL, &kg_colg_final, 256, nblocks, labels, t + 2 * e); break;
    }
    if (r) {
      r->cp = cp;
      r->gp = mixed_params(p);
    }
    return;
  }
  switch (kind) {
    case 0: hipLaunchKernelGGL(k_colg_fwd, grid, block, t + 2 * e, s, cp, mixed_params(p)); break;
    case 1: hipLaunchKernelGGL(k_colg_syn, grid, block, t + 3 * e, s, cp, mixed_params(p)); break;
    case 2: hipLaunchKernelGGL(k_colg_ana, grid, block, t + 3 * e, s, cp, mixed_params(p)); break;
    case 3: hipLaunchKernelGGL(k_colg_final, grid, block, t + 2 * e, s, cp, mixed_params(p)); break;
  }
}

static void mixed_col_solve(const shs_plan* p, const ColParams& cp, int labels, hipStream_t s) {
  const size_t e = size_t(p->n) * kGW * sizeof(float2);
  hipLaunchKernelGGL(k_colg_solve, dim3(p->NS, labels), dim3(256), 2 * e, s, cp, mixed_params(p), p->eig);
}

Ops mixed_ops() { return Ops{&mixed_row_any, &mixed_col, &mixed_col_solve}; }

bool mixed_reserve_lds() {
  const int lds3 = (3 * kGenericMaxN * kGW + col_tab_len(kGenericMaxN)) * int(sizeof(float2));
  const int lds2 = (2 * kGenericMaxN * kGW + col_tab_len(kGenericMaxN)) * int(sizeof(float2));
  const auto reserve = [](auto fn, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) ==
           hipSuccess;
  };
  return reserve(&k_colg_syn, lds3) && reserve(&k_colg_ana, lds3) && reserve(&k_colg_fwd, lds2) &&
         reserve(&k_colg_final, lds2) && reserve(&k_colg_solve, lds2) && reserve(&kg_colg_syn, lds3) &&
         reserve(&kg_colg_ana, lds3) && reserve(&kg_colg_fwd, lds2) && reserve(&kg_colg_final, lds2);
}

}  // namespace shs
