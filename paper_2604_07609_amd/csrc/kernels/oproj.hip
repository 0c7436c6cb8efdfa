// attention output projection
#include "../phase_kernels.h"

PHASE_KERNEL8(k_oproj, PH_OPROJ)
