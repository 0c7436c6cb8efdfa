// gate and up projections
#include "../phase_kernels.h"

PHASE_KERNEL8(k_gateup, PH_GATEUP)
