// Resident 2D kernels with 2 rows per lane (padded z extents up to 128).
#define RES_BZ 2
#include "resident_inst.h"
