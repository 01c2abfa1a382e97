// Mixed-radix synthesis column pass.
#include "generic_col.hpp"

SHS_MIXED_COL_HERE(COL_SYN)
