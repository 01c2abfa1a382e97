// Pixel kernels of the TV model, by storage type and label count.
#include "tv_launch.hpp"

namespace shs {

template <int ST, int Q>
static void launch(int kind, bool stats, const TvParams& p, hipStream_t s) {
  const dim3 g{unsigned(tv_blocks((long long)p.n * p.n))}, b{256};
  if (kind == TV_RHS) hipLaunchKernelGGL((k_tv_rhs<ST, Q>), g, b, 0, s, p);
  else if (stats) hipLaunchKernelGGL((k_tv_update<ST, Q, true>), g, b, 0, s, p);
  else hipLaunchKernelGGL((k_tv_update<ST, Q, false>), g, b, 0, s, p);
}
template <int ST>
static void launch_q(int kind, bool stats, const TvParams& p, hipStream_t s) {
  switch (p.q) {
    case 1: launch<ST, 1>(kind, stats, p, s); break;
    case 2: launch<ST, 2>(kind, stats, p, s); break;
    case 3: launch<ST, 3>(kind, stats, p, s); break;
    case 4: launch<ST, 4>(kind, stats, p, s); break;
    case 5: launch<ST, 5>(kind, stats, p, s); break;
    case 6: launch<ST, 6>(kind, stats, p, s); break;
    case 7: launch<ST, 7>(kind, stats, p, s); break;
    case 8: launch<ST, 8>(kind, stats, p, s); break;
    default: break;
  }
}
void tv_launch(int store, int kind, bool stats, const TvParams& p, hipStream_t s) {
  switch (store) {
    case ST_F32: launch_q<ST_F32>(kind, stats, p, s); break;
    case ST_BF16: launch_q<ST_BF16>(kind, stats, p, s); break;
    default: launch_q<ST_F16>(kind, stats, p, s); break;
  }
}

}  // namespace shs
