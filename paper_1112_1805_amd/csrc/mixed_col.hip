// Mixed-radix forward and finishing column passes, the TV column solve, the plain row
// transforms, and the launch table of the path.
#include "generic_col.hpp"

SHS_MIXED_ROW_HERE(ROW_C2R, ST_F32, false)
SHS_MIXED_ROW_HERE(ROW_R2C, ST_F32, false)
SHS_MIXED_COL_HERE(COL_FWD)
SHS_MIXED_COL_HERE(COL_FINAL)

namespace shs {

SHS_MIXED_COL_EXTERN(COL_SYN)
SHS_MIXED_COL_EXTERN(COL_ANA)

static __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_colg_solve(ColParams p, GenParams gp, const float* __restrict__ eig) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* lsw = gsm;
  float2* bz = gsm + col_tab_len(n);
  float2* b0 = bz + E;
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  const int cols = strip_cols(blockIdx.x, M);
  const long long strip = blockIdx.y * (long long)n * p.P + (long long)blockIdx.x * E;
  __syncthreads();
  col_transform_g<false>(gp, lsw, b0, b0 + E, NoEarlyCol{}, StripRead{PlaneBuf(p.in + strip, E), cols >= kGW, cols},
    [&](auto& a, int bf, int nb, int c, const auto&) {
      constexpr int R = sizeof(a) / sizeof(cpx);
      const float e1 = c < cols ? eig[blockIdx.x * kGW + c] : 0.f;
      const float scale = c < cols ? p.inv_n2 : 0.f;
      static_for<R>([&](auto k) {
        const int pos = bf + k * nb;
        st(bz + pos * kGW + c, a[k] * (scale / (1.f + eig[pos] + e1)));
      });
    });
  __syncthreads();
  col_transform_g<true>(gp, lsw, b0, b0 + E, NoEarlyCol{},
    [&](auto& a, int bf, int nb, int c) {
      constexpr int R = sizeof(a) / sizeof(cpx);
      static_for<R>([&](auto k) { a[k] = ld(bz + (bf + k * nb) * kGW + c); });
    },
    StripWrite{PlaneBuf(p.out + strip, E), cols >= kGW, cols});
}

static void mixed_row_any(const shs_plan* p, int mode, int store, bool stats, const RowParams& rp, int channels,
                          hipStream_t s) {
#define SHS_CASE(MODE, ST, STATS) \
  if (mode == MODE && store == ST && stats == STATS) return mixed_row<MODE, ST, STATS>(p, rp, channels, s);
  SHS_MIXED_ROWS(SHS_CASE)
#undef SHS_CASE
}

static void mixed_col_any(const shs_plan* p, int kind, const ColParams& cp, int nblocks, int labels, hipStream_t s) {
  switch (kind) {
    case COL_FWD: mixed_col<COL_FWD>(p, cp, nblocks, labels, s); break;
    case COL_SYN: mixed_col<COL_SYN>(p, cp, nblocks, labels, s); break;
    case COL_ANA: mixed_col<COL_ANA>(p, cp, nblocks, labels, s); break;
    case COL_FINAL: mixed_col<COL_FINAL>(p, cp, nblocks, labels, s); break;
  }
}

static void mixed_col_solve(const shs_plan* p, const ColParams& cp, int labels, hipStream_t s) {
  hipLaunchKernelGGL(k_colg_solve, dim3(p->NS, labels), dim3(col_g_threads(p->pcol)), col_g_lds_bytes(p, 1), s, cp,
                     mixed_params(p), p->eig);
}

void mixed_mid(const shs_plan* p, int mode, const MidParams& mp, hipStream_t s);
int mixed_mid_blocks(const shs_plan* p);
bool mixed_mid_reserve();

static bool mixed_reserve(const shs_plan* p) {
  // three strips, the table and a work item's windows; every label's row slots, second buffers
  // and the waves' sums (mixed_mid.hip)
  const size_t col = (3 * size_t(p->n) * kGW + col_tab_len(p->n)) * sizeof(float2) + sizeof(ItemStage<kGW>);
  const size_t mid = (size_t(3) + 4 * p->q + 32) * p->M * sizeof(float2) + 16 * 4 * sizeof(double);
  if (col <= kDefaultLds && mid <= kDefaultLds) return true;
  const int bytes = (3 * kGenericMaxN * kGW + col_tab_len(kGenericMaxN)) * int(sizeof(float2));
  return mixed_col_reserve<COL_FWD>() && mixed_col_reserve<COL_SYN>() && mixed_col_reserve<COL_ANA>() &&
         mixed_col_reserve<COL_FINAL>() &&
         hipFuncSetAttribute(reinterpret_cast<const void*>(&k_colg_solve), hipFuncAttributeMaxDynamicSharedMemorySize,
                             bytes) == hipSuccess &&
         mixed_mid_reserve();
}

Ops mixed_ops() {
  return Ops{&mixed_row_any, &mixed_col_any, &mixed_col_solve, &mixed_mid, &mixed_mid_blocks, &mixed_reserve};
}

}  // namespace shs
