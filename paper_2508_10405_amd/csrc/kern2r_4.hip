// Resident 2D kernels with 4 rows per lane (padded z extents up to 256).
#define RES_BZ 4
#include "resident_inst.h"
