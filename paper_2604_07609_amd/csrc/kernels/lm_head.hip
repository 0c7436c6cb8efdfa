// LM head
#include "../phase_kernels.h"

PHASE_KERNEL8(k_lm_head, PH_LM_HEAD)
