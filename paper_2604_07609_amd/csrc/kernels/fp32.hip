// the phases of an fp32 model
#include "../phase_kernels.h"

PHASE_KERNEL_F32(k_embed_f32, PH_EMBED)
PHASE_KERNEL_F32(k_qkv_f32, PH_QKV)
PHASE_KERNEL_F32(k_attention_f32, PH_ATTN)
PHASE_KERNEL_F32(k_oproj_f32, PH_OPROJ)
PHASE_KERNEL_F32(k_gateup_f32, PH_GATEUP)
PHASE_KERNEL_F32_DOWN(k_down_f32, PH_DOWN)
PHASE_KERNEL_F32(k_lm_head_f32, PH_LM_HEAD)
PHASE_KERNEL_F32(k_sample_publish_f32, PH_SAMPLE)
