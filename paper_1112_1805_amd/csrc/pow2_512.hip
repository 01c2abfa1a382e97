// Kernels of the image side 512.
#include "pow2.hpp"

template Ops shs::pow2_ops<512>();
