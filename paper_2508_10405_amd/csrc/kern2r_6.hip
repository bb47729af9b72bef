// Resident 2D kernels with 6 rows per lane (padded z extents up to 384).
#define RES_BZ 6
#include "resident_inst.h"
