// Mixed-radix row pass of the ADMM solver, F16 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_F16, true)
SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_F16, false)
