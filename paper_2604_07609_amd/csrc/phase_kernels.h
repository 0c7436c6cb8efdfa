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
// small phases and the other phases of an fp32 model: four waves, two workgroups per compute unit
#define PHASE_KERNEL(name, PH) __global__ void __launch_bounds__(BLK_THREADS, 2) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, false)
#define PHASE_KERNEL_F32(name, PH) __global__ void __launch_bounds__(BLK_THREADS, 2) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, true)
// the down projection of an fp32 model: eight waves (gemm_f32.h)
#define PHASE_KERNEL_F32_DOWN(name, PH) __global__ void __launch_bounds__(64 * F32_DOWN_WAVES) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, true)
// The GEMMs and the attention of a bf16 model: eight waves, two per SIMD, which stay on their compute unit for the whole launch (up to
// 1.5 ms). With all 512 registers of a SIMD's lanes between the two, nothing else fits on the chip meanwhile, and the small
// kernels and copies of blink_submit and blink_poll_outputs wait for the end of the launch. So 240 registers per wave at
// most (the attribute counts half of gfx950's unified file): 32 are left, what those need. Beside prefill iterations of
// 8000 tokens (32 q / 8 kv heads of 128, d 4096, FFN 14336) a submit takes 30 us instead of 536 and a poll 25 instead of 549, on
// average; prefill and decode iterations take what they took with 256.
#define PHASE_KERNEL8(name, PH) \
  __global__ void __launch_bounds__(512) __attribute__((amdgpu_num_vgpr(120))) name(DevCtx c, u32 layer) PHASE_KERNEL_BODY(PH, false)

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
