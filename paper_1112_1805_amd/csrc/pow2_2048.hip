// Kernels of the image side 2048.
#include "pow2.hpp"

template Ops shs::pow2_ops<2048>();
