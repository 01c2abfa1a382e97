// Kernels of the image side 1024.
#include "pow2.hpp"

template Ops shs::pow2_ops<1024>();
