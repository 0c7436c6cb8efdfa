// QKV projection
#include "../phase_kernels.h"

PHASE_KERNEL8(k_qkv, PH_QKV)
