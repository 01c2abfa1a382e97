// Launches of the TV model's pixel kernels (instantiated in tv.hip).
#pragma once
#include "tv.hpp"

namespace shs {

enum { TV_RHS = 0, TV_UPDATE = 1 };
inline long long tv_blocks(long long n2) { return (n2 + kTvPerBlock - 1) / kTvPerBlock; }
void tv_launch(int store, int kind, bool stats, const TvParams& p, hipStream_t s);

}  // namespace shs
