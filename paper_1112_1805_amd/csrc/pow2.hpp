// Launchers of the power-of-two sizes; each pow2_*.hip instantiates pow2_ops for its sizes.
#pragma once
#include "host.hpp"

namespace shs {

// ---------------------------------------------------------------- per-size launchers
template <int N>
struct Pipe {
  using RG = RowGeom<N>;
  using CG = ColCfg<N>;

  template <int MODE, int ST, bool STATS>
  static void row_t(const RowParams& rp, int channels, hipStream_t s) {
    dim3 grid(N / RG::RPB, channels);
    if constexpr (batch_row_mode(MODE)) {
      if (g_rec) {
        rec_add(RK_ROW, &kg_row<N, MODE, ST, STATS>, RG::THREADS, N / RG::RPB, channels, 0).rp = rp;
        return;
      }
    }
    hipLaunchKernelGGL((k_row<N, MODE, ST, STATS>), grid, dim3(RG::THREADS), 0, s, rp);
  }
  static void row(const shs_plan*, int mode, int store, bool stats, const RowParams& rp, int channels, hipStream_t s) {
    switch (mode) {
      case ROW_SOLVE:
        if (store == ST_F32) { stats ? row_t<ROW_SOLVE, ST_F32, true>(rp, channels, s) : row_t<ROW_SOLVE, ST_F32, false>(rp, channels, s); }
        else if (store == ST_BF16) { stats ? row_t<ROW_SOLVE, ST_BF16, true>(rp, channels, s) : row_t<ROW_SOLVE, ST_BF16, false>(rp, channels, s); }
        else { stats ? row_t<ROW_SOLVE, ST_F16, true>(rp, channels, s) : row_t<ROW_SOLVE, ST_F16, false>(rp, channels, s); }
        break;
      case ROW_PRIME:
        if (store == ST_F32) row_t<ROW_PRIME, ST_F32, false>(rp, channels, s);
        else if (store == ST_BF16) row_t<ROW_PRIME, ST_BF16, false>(rp, channels, s);
        else row_t<ROW_PRIME, ST_F16, false>(rp, channels, s);
        break;
      case ROW_C2R: row_t<ROW_C2R, ST_F32, false>(rp, channels, s); break;
      case ROW_R2C: row_t<ROW_R2C, ST_F32, false>(rp, channels, s); break;
      case ROW_ENERGY: row_t<ROW_ENERGY, ST_F32, true>(rp, channels, s); break;
      case ROW_SHRINK: row_t<ROW_SHRINK, ST_F32, false>(rp, channels, s); break;
      case ROW_PD:
        if (store == ST_F32) { stats ? row_t<ROW_PD, ST_F32, true>(rp, channels, s) : row_t<ROW_PD, ST_F32, false>(rp, channels, s); }
        else if (store == ST_BF16) { stats ? row_t<ROW_PD, ST_BF16, true>(rp, channels, s) : row_t<ROW_PD, ST_BF16, false>(rp, channels, s); }
        else { stats ? row_t<ROW_PD, ST_F16, true>(rp, channels, s) : row_t<ROW_PD, ST_F16, false>(rp, channels, s); }
        break;
    }
  }
  static void col(const shs_plan*, int kind, const ColParams& cp, int nblocks, int labels, hipStream_t s) {
    const dim3 grid(nblocks, labels), block(CG::THREADS);
    if (g_rec) {
      LaunchRec* r = nullptr;
      switch (kind) {
        case 0: r = &rec_add(RK_COL, &kg_col_fwd<N>, CG::THREADS, nblocks, labels, 0); break;
        case 1: r = &rec_add(RK_COL, &kg_col_syn<N>, CG::THREADS, nblocks, labels, 0); break;
        case 2: r = &rec_add(RK_COL, &kg_col_ana<N>, CG::THREADS, nblocks, labels, 0); break;
        case 3: r = &rec_add(RK_COL, &kg_col_final<N>, CG::THREADS, nblocks, labels, 0); break;
      }
      if (r) r->cp = cp;
      return;
    }
    switch (kind) {
      case 0: hipLaunchKernelGGL((k_col_fwd<N>), grid, block, 0, s, cp); break;
      case 1: hipLaunchKernelGGL((k_col_syn<N>), grid, block, 0, s, cp); break;
      case 2: hipLaunchKernelGGL((k_col_ana<N>), grid, block, 0, s, cp); break;
      case 3: hipLaunchKernelGGL((k_col_final<N>), grid, block, 0, s, cp); break;
    }
  }
};

template <int N>
void launch_col_solve(const shs_plan* p, const ColParams& cp, int labels, hipStream_t s) {
  hipLaunchKernelGGL(k_col_solve<N>, dim3(p->NS, labels), dim3(ColCfg<N>::THREADS), 0, s, cp, p->eig);
}

template <int N>
struct MidPipe {
  template <int MODE, bool STATS>
  static void launch(const shs_plan* p, const MidParams& mp, hipStream_t s) {
    const int threads = 64 * MidGeom<N>::waves(p->q);
    const size_t lds = MidGeom<N>::lds(p->q);
    if constexpr (MODE == MID_ADMM) {
      if (g_rec) {
        rec_add(RK_MID, &kg_mid<N, STATS>, threads, blocks(p), 1, lds).mp = mp;
        return;
      }
    }
    hipLaunchKernelGGL((k_mid<N, MODE, STATS>), dim3(blocks(p)), dim3(threads), lds, s, mp);
  }
  static int blocks(const shs_plan*) { return N / MidGeom<N>::RB; }
  static void mid(const shs_plan* p, int mode, const MidParams& mp, hipStream_t s) {
    if (mode == MID_PD) mp.stats ? launch<MID_PD, true>(p, mp, s) : launch<MID_PD, false>(p, mp, s);
    else mp.stats ? launch<MID_ADMM, true>(p, mp, s) : launch<MID_ADMM, false>(p, mp, s);
  }
  static bool reserve(const shs_plan* p) {
    if (MidGeom<N>::lds(p->q) + MidGeom<N>::lds_static <= kDefaultLds) return true;
    const auto one = [](auto fn) {
      return hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 int(MidGeom<N>::lds(SHS_MAX_LABELS))) == hipSuccess;
    };
    return one(&k_mid<N, MID_ADMM, true>) && one(&k_mid<N, MID_ADMM, false>) && one(&k_mid<N, MID_PD, true>) &&
           one(&k_mid<N, MID_PD, false>) && one(&kg_mid<N, true>) && one(&kg_mid<N, false>);
  }
};

template <int N>
Ops pow2_ops() {
  return Ops{&Pipe<N>::row, &Pipe<N>::col, &launch_col_solve<N>, &MidPipe<N>::mid, &MidPipe<N>::blocks,
             &MidPipe<N>::reserve};
}

}  // namespace shs
