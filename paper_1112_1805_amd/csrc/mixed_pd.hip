// Mixed-radix row pass of the primal-dual solver.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_PD, ST_F32, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_F32, false)
SHS_MIXED_ROW_HERE(ROW_PD, ST_BF16, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_BF16, false)
SHS_MIXED_ROW_HERE(ROW_PD, ST_F16, true)
SHS_MIXED_ROW_HERE(ROW_PD, ST_F16, false)
