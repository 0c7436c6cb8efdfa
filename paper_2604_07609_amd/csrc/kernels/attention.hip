// attention and the merge of its partial results
#include "../phase_kernels.h"

PHASE_KERNEL8(k_attention, PH_ATTN)
PHASE_KERNEL(k_attention_combine, PH_ATTN_COMBINE)
