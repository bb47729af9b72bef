// Resident 2D kernels with 5 rows per lane (padded z extents up to 320).
#define RES_BZ 5
#include "resident_inst.h"
