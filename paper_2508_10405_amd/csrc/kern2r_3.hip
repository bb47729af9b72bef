// Resident 2D kernels with 3 rows per lane (padded z extents up to 192).
#define RES_BZ 3
#include "resident_inst.h"
