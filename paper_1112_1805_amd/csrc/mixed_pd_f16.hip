// Mixed-radix row pass of the primal-dual solver, F16 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_PD, ST_F16, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_F16, false)
