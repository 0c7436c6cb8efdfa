// gate and up projections of the experts
#include "../phase_kernels.h"

PHASE_KERNEL8(k_moe_gateup, PH_MOE_GATEUP)
