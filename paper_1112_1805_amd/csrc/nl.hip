// Kernels of the nonlocal model's iteration, by storage type, label count and block count.
#include "nl_launch.hpp"

namespace shs {

template <int ST, int Q>
static void launch(int kind, long long blocks, hipStream_t s, const NlParams& p) {
  const dim3 g{unsigned(blocks)}, b{256};
  // ten blocks (five neighbours picked per pixel) is the paper's graph
  if (p.M2 <= 10) {
    if (kind == NL_DUAL) hipLaunchKernelGGL((k_nl_dual<ST, Q, 10>), g, b, 0, s, p);
    else hipLaunchKernelGGL((k_nl_primal<ST, Q, 10>), g, b, 0, s, p);
  } else {
    if (kind == NL_DUAL) hipLaunchKernelGGL((k_nl_dual<ST, Q, kNlMaxBlocks>), g, b, 0, s, p);
    else hipLaunchKernelGGL((k_nl_primal<ST, Q, kNlMaxBlocks>), g, b, 0, s, p);
  }
}
template <int ST>
static void launch_q(int kind, long long blocks, hipStream_t s, const NlParams& p) {
  switch (p.q) {
    case 1: launch<ST, 1>(kind, blocks, s, p); break;
    case 2: launch<ST, 2>(kind, blocks, s, p); break;
    case 3: launch<ST, 3>(kind, blocks, s, p); break;
    case 4: launch<ST, 4>(kind, blocks, s, p); break;
    case 5: launch<ST, 5>(kind, blocks, s, p); break;
    case 6: launch<ST, 6>(kind, blocks, s, p); break;
    case 7: launch<ST, 7>(kind, blocks, s, p); break;
    case 8: launch<ST, 8>(kind, blocks, s, p); break;
    default: break;
  }
}
void nl_launch(int store, int kind, const NlParams& p, hipStream_t s) {
  const long long blocks = (p.n2 + 255) / 256;
  if (kind == NL_INDEX) {
    hipLaunchKernelGGL(k_nl_index, dim3(unsigned(blocks)), dim3(256), 0, s, p);
  } else if (kind == NL_ENERGY) {
    hipLaunchKernelGGL(k_nl_energy, dim3(unsigned(blocks)), dim3(256), 0, s, p);
  } else {
    switch (store) {
      case ST_F32: launch_q<ST_F32>(kind, blocks, s, p); break;
      case ST_BF16: launch_q<ST_BF16>(kind, blocks, s, p); break;
      default: launch_q<ST_F16>(kind, blocks, s, p); break;
    }
  }
}
size_t nl_record_bytes(int store, int q) {
  return store == ST_F32 ? size_t(q) * 4 : q == 1 ? 2 : size_t(q + 1) / 2 * 4;
}

}  // namespace shs
