// down projection
#include "../phase_kernels.h"

PHASE_KERNEL8(k_down, PH_DOWN)
