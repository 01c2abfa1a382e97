// Launches of the nonlocal model's kernels (instantiated in nl.hip).
#pragma once
#include "nl_iter.hpp"

namespace shs {

enum { NL_INDEX = 0, NL_DUAL = 1, NL_PRIMAL = 2, NL_ENERGY = 3 };
void nl_launch(int store, int kind, const NlParams& p, hipStream_t s);
// Bytes of one record of the dual variable (all labels of a pixel, one block).
size_t nl_record_bytes(int store, int q);

}  // namespace shs
