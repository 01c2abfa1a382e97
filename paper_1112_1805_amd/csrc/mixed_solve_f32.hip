// Mixed-radix row pass of the ADMM solver, F32 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_F32, true)
SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_F32, false)
