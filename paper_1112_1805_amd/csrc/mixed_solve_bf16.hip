// Mixed-radix row pass of the ADMM solver, BF16 state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_BF16, true)
SHS_MIXED_ROW_HERE(ROW_SOLVE, ST_BF16, false)
