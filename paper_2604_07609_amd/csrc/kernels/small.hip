// embedding, sampler and the small steps of a mixture-of-experts layer
#include "../phase_kernels.h"

PHASE_KERNEL(k_embed, PH_EMBED)
PHASE_KERNEL(k_sample_publish, PH_SAMPLE)
PHASE_KERNEL(k_moe_router, PH_ROUTER)
PHASE_KERNEL(k_moe_route, PH_ROUTE)
PHASE_KERNEL(k_moe_combine, PH_MOE_COMBINE)
PHASE_KERNEL(k_moe_permute, PH_MOE_PERMUTE)
