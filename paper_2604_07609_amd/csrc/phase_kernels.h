// One named kernel per phase, so that profiles attribute time to the step of the forward pass. They are defined in kernels/*.hip,
// a few per file (compiled in parallel).
#pragma once
#include "phases.h"

#define PHASE_KERNEL_DECL(name) __global__ void name(DevCtx c, u32 layer);
#define PHASE_KERNEL_BODY(PH, F32)                               \
  {                                                              \
    __shared__ PhaseSharedOf<PH, F32>::type sh;                  \
    run_phase<PH, F32>(c, layer, sh, blockIdx.x, gridDim.x);     \
  }
// small phases and the phases of an fp32 model: four waves, two workgroups per compute unit
#define PHASE_KERNEL(name, PH) __global__ void __launch_bounds__(BLK_THREADS, 2) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, false)
#define PHASE_KERNEL_F32(name, PH) __global__ void __launch_bounds__(BLK_THREADS, 2) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, true)
// the GEMMs and the attention of a bf16 model: eight waves, at most 256 registers per lane
#define PHASE_KERNEL8(name, PH) __global__ void __launch_bounds__(512) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, false)

PHASE_KERNEL_DECL(k_embed)
PHASE_KERNEL_DECL(k_qkv)
PHASE_KERNEL_DECL(k_attention)
PHASE_KERNEL_DECL(k_oproj)
PHASE_KERNEL_DECL(k_gateup)
PHASE_KERNEL_DECL(k_down)
PHASE_KERNEL_DECL(k_lm_head)
PHASE_KERNEL_DECL(k_sample_publish)
PHASE_KERNEL_DECL(k_attention_combine)
PHASE_KERNEL_DECL(k_moe_router)
PHASE_KERNEL_DECL(k_moe_route)
PHASE_KERNEL_DECL(k_moe_gateup)
PHASE_KERNEL_DECL(k_moe_down)
PHASE_KERNEL_DECL(k_moe_combine)
PHASE_KERNEL_DECL(k_moe_permute)
// fp32 models
PHASE_KERNEL_DECL(k_embed_f32)
PHASE_KERNEL_DECL(k_qkv_f32)
PHASE_KERNEL_DECL(k_attention_f32)
PHASE_KERNEL_DECL(k_oproj_f32)
PHASE_KERNEL_DECL(k_gateup_f32)
PHASE_KERNEL_DECL(k_down_f32)
PHASE_KERNEL_DECL(k_lm_head_f32)
PHASE_KERNEL_DECL(k_sample_publish_f32)
