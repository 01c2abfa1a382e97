// Mixed-radix middle step: adjoint rows back, pixel step, row transform.
#include "mixed.hpp"

namespace shs {

// Launch shape of the middle step.  A wave transforms rw of the block's slots (row, label) at
// a time: as many as the row pass takes rows, but fewer where that leaves SIMDs without a wave
// (the launch then takes as long as one wave's instructions); no more rows per block than the
// waves' slots need; waves for the transforms and for one or two pixel pairs per thread.
struct MidShape {
  GenParams gp;
  int threads;
  size_t lds;
};
constexpr size_t kMidLdsMax = 152 * 1024;
static MidShape mid_shape(const shs_plan* p) {
  MidShape m{mixed_params(p), 0, 0};
  int rw = p->rw;                    // 1, 2 or 4
  while (rw > 1 && p->n * p->q / rw < 1024) rw /= 2;
  for (;; rw /= 2) {                 // one row per wave always fits
    int lrb = 0, waves = 1;
    while ((p->q << lrb) % rw != 0) ++lrb;
    const int slots = p->q << lrb, groups = slots / rw;
    while (waves < 8 && (waves < groups || waves * 128 < p->M)) waves *= 2;
    m.gp.lrb = lrb;
    m.gp.lrw = rw == 4 ? 2 : rw == 2 ? 1 : 0;
    m.gp.nbuf = row_g_bufs(p->prow, rw);
    m.threads = 64 * waves;
    m.lds = (size_t(row_tab_len(p->n)) + (size_t(slots) + (m.gp.nbuf == 2 ? size_t(waves) * rw : 0)) * p->M) *
            sizeof(float2);
    if (m.lds <= kMidLdsMax || rw == 1) return m;
  }
}
int mixed_mid_blocks(const shs_plan* p) { return p->n >> mid_shape(p).gp.lrb; }

template <int MODE, bool STATS>
static void launch_mid(const shs_plan* p, const MidParams& mp, hipStream_t s) {
  const MidShape m = mid_shape(p);
  if constexpr (MODE == MID_ADMM) {
    if (g_rec) {
      LaunchRec& r = rec_add(RK_MID, &kg_mid_g<MODE, STATS>, m.threads, p->n >> m.gp.lrb, 1, m.lds);
      r.mp = mp;
      r.gp = m.gp;
      return;
    }
  }
  hipLaunchKernelGGL((k_mid_g<MODE, STATS>), dim3(p->n >> m.gp.lrb), dim3(m.threads), m.lds, s, mp, m.gp);
}

void mixed_mid(const shs_plan* p, int mode, const MidParams& mp, hipStream_t s) {
  if (mode == MID_PD) mp.stats ? launch_mid<MID_PD, true>(p, mp, s) : launch_mid<MID_PD, false>(p, mp, s);
  else mp.stats ? launch_mid<MID_ADMM, true>(p, mp, s) : launch_mid<MID_ADMM, false>(p, mp, s);
}

bool mixed_mid_reserve() {
  const auto one = [](auto fn) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                               int(kMidLdsMax)) == hipSuccess;
  };
  return one(&k_mid_g<MID_ADMM, true>) && one(&k_mid_g<MID_ADMM, false>) && one(&k_mid_g<MID_PD, true>) &&
         one(&k_mid_g<MID_PD, false>) && one(&kg_mid_g<MID_ADMM, true>) && one(&kg_mid_g<MID_ADMM, false>);
}

}  // namespace shs
