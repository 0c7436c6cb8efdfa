// down projection of the experts
#include "../phase_kernels.h"

PHASE_KERNEL8(k_moe_down, PH_MOE_DOWN)
