// Mixed-radix row passes of the transforms, the energy and the resumed state.
#include "mixed.hpp"

SHS_MIXED_ROW_HERE(ROW_PRIME, ST_F32, false)
SHS_MIXED_ROW_HERE(ROW_PRIME, ST_BF16, false)
SHS_MIXED_ROW_HERE(ROW_PRIME, ST_F16, false)
SHS_MIXED_ROW_HERE(ROW_ENERGY, ST_F32, true)
SHS_MIXED_ROW_HERE(ROW_SHRINK, ST_F32, false)
