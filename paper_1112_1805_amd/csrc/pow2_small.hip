// Kernels of the image sides 64, 128, 256.
#include "pow2.hpp"

template Ops shs::pow2_ops<64>();
template Ops shs::pow2_ops<128>();
template Ops shs::pow2_ops<256>();
