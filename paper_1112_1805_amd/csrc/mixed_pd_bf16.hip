// Mixed-radix row pass of the primal-dual solver, BF16 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_PD, ST_BF16, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_BF16, false)
