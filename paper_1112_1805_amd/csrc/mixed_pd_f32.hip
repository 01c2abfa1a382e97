// Mixed-radix row pass of the primal-dual solver, F32 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_PD, ST_F32, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_F32, false)
