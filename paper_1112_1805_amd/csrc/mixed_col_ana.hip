// Mixed-radix analysis column pass.
#include "generic_col.hpp"

SHS_MIXED_COL_HERE(COL_ANA)
