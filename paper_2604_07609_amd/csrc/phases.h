// The ordered list of phases of one loop iteration and their dispatch. A phase is a grid-wide step that
// must be complete before the next begins (a kernel boundary in host-enqueued mode, a grid barrier in
// the resident loop). Shapes are read from the device metadata written by the scheduler step.
#pragma once
#include "blink_device.h"
#include "sched.h"
#include "forward.h"
#include "gemm_dma.h"
#include "gemm_f32.h"
#include "attention_mfma.h"
#include "sampler.h"
#include "moe.h"

enum {
  PH_EMBED = 0,
  PH_NORM1, PH_QKV, PH_ROPE, PH_ATTN, PH_OPROJ, PH_NORM2, PH_GATEUP, PH_DOWN,   // per layer
  PH_FINAL_NORM, PH_LM_HEAD, PH_SAMPLE,
  PH_ATTN_COMBINE,  // bf16 path only, directly after PH_ATTN of the same layer
  PH_UNUSED13, PH_UNUSED14, PH_UNUSED15,   // (no kernels)
  PH_ROUTER, PH_ROUTE, PH_MOE_GATEUP, PH_MOE_DOWN, PH_MOE_COMBINE,  // mixture of experts: in place of PH_GATEUP and PH_DOWN
  PH_MOE_PERMUTE                                                    // (runs between PH_ROUTE and PH_MOE_GATEUP)
};
#define PH_LAYER_FIRST PH_NORM1
#define PH_LAYER_LAST PH_DOWN

// LDS of a phase kernel of a bf16 model, and of an fp32 model (the GEMMs and the attention have kernels of their own per kind of
// model, so that neither is charged the other's LDS and registers)
struct NoShared {};
template <int PH, bool F32> struct PhaseSharedOf { typedef NoShared type; };
template <> struct PhaseSharedOf<PH_QKV, false> { typedef GemmShared8 type; };
template <> struct PhaseSharedOf<PH_OPROJ, false> { typedef GemmShared8 type; };
template <> struct PhaseSharedOf<PH_GATEUP, false> { typedef GemmShared8 type; };
template <> struct PhaseSharedOf<PH_DOWN, false> { typedef GemmShared8 type; };
template <> struct PhaseSharedOf<PH_LM_HEAD, false> { typedef GemmShared8 type; };
template <> struct PhaseSharedOf<PH_ROUTER, false> { typedef MfmaShared type; };
template <> struct PhaseSharedOf<PH_ATTN, false> { typedef AttnShared8 type; };
template <> struct PhaseSharedOf<PH_SAMPLE, false> { typedef SamplerShared type; };
template <> struct PhaseSharedOf<PH_MOE_GATEUP, false> { typedef MoeShared type; };
template <> struct PhaseSharedOf<PH_MOE_DOWN, false> { typedef MoeShared type; };
template <> struct PhaseSharedOf<PH_MOE_COMBINE, false> { typedef MoeLists type; };
template <> struct PhaseSharedOf<PH_MOE_PERMUTE, false> { typedef MoeLists type; };
template <> struct PhaseSharedOf<PH_QKV, true> { typedef F32GemmShared<F32_WAVES> type; };
template <> struct PhaseSharedOf<PH_OPROJ, true> { typedef F32GemmShared<F32_WAVES> type; };
template <> struct PhaseSharedOf<PH_GATEUP, true> { typedef F32GemmShared<F32_WAVES> type; };
template <> struct PhaseSharedOf<PH_DOWN, true> { typedef F32GemmShared<F32_DOWN_WAVES> type; };
template <> struct PhaseSharedOf<PH_LM_HEAD, true> { typedef F32GemmShared<F32_WAVES> type; };
template <> struct PhaseSharedOf<PH_ATTN, true> { typedef AttnShared type; };
template <> struct PhaseSharedOf<PH_SAMPLE, true> { typedef SamplerShared type; };

// fp32 path: the norms, the SiLU gate, the residual adds and the rotary embedding + KV write are fused into the GEMMs here too
template <int PH>
__device__ __forceinline__ void run_phase_f32(const DevCtx& c, u32 layer, typename PhaseSharedOf<PH, true>::type& sh, u32 wg, u32 nwg) {
  const IterMeta* m = c.meta;
  const LayerW* L = c.layers + layer;
  F32GemmArgs a{};
  a.T = m->n_tokens;
  a.eps = c.eps;
  switch (PH) {
    case PH_EMBED: phase_embed<float>(c, wg, nwg); break;
    case PH_QKV:
      a.A = c.x; a.lda = c.d; a.gain = L->g1; a.W = (const float*)L->wqkv; a.out = c.qkv; a.ldo = c.qkv_n; a.N = c.qkv_n; a.K = c.d;
      a.positions = c.positions; a.slot_mapping = c.slot_mapping; a.rope_tab = c.rope_tab;
      a.Kc = (float*)c.kv + (u64)layer * c.kv_layer_stride; a.Vc = a.Kc + c.kv_kv_stride;
      a.nq = c.nq; a.nkv = c.nkv; a.hd = c.hd; a.bs = c.bs;
      gemm_f32<FA_NORM, FE_ROPE, F32_WAVES>(a, *(F32GemmShared<F32_WAVES>*)&sh, wg, nwg);
      break;
    case PH_ATTN: phase_attention_f32(c, layer, *(AttnShared*)&sh, wg, nwg); break;
    case PH_OPROJ:
      a.A = c.attn; a.lda = c.nq * c.hd; a.W = (const float*)L->wo; a.out = c.x; a.ldo = c.d; a.N = c.d; a.K = c.nq * c.hd;
      gemm_f32<FA_PLAIN, FE_ADD, F32_WAVES>(a, *(F32GemmShared<F32_WAVES>*)&sh, wg, nwg);
      break;
    case PH_GATEUP:
      a.A = c.x; a.lda = c.d; a.gain = L->g2; a.W = (const float*)L->wgu; a.out = c.gu; a.ldo = c.F; a.N = 2 * c.F; a.K = c.d;
      gemm_f32<FA_NORM, FE_GATE, F32_WAVES>(a, *(F32GemmShared<F32_WAVES>*)&sh, wg, nwg);
      break;
    case PH_DOWN:
      a.A = c.gu; a.lda = c.F; a.W = (const float*)L->wd; a.out = c.x; a.ldo = c.d; a.N = c.d; a.K = c.F;
      gemm_f32<FA_PLAIN, FE_ADD, F32_DOWN_WAVES>(a, *(F32GemmShared<F32_DOWN_WAVES>*)&sh, wg, nwg);
      break;
    case PH_LM_HEAD:      // one row per sampling sequence (its last token)
      a.T = m->n_samples; a.rows = c.last_idx; a.A = c.x; a.lda = c.d; a.gain = c.gf; a.W = (const float*)c.lm; a.out = c.logits; a.ldo = c.V;
      a.N = c.V; a.K = c.d;
      gemm_f32<FA_NORM, FE_STORE, F32_WAVES>(a, *(F32GemmShared<F32_WAVES>*)&sh, wg, nwg);
      break;
    case PH_SAMPLE:
      if (c.spec_k) phase_sample_publish_spec(c, *(SamplerShared*)&sh, wg, nwg);
      else phase_sample_publish(c, *(SamplerShared*)&sh, wg, nwg);
      break;
  }
}

// bf16 path: MFMA GEMMs on packed operands with the norms, the residual adds and the SiLU gate fused into their
// epilogues; the separate norm phases do not exist here.
template <int PH>
__device__ __forceinline__ void run_phase_bf16(const DevCtx& c, u32 layer, typename PhaseSharedOf<PH, false>::type& sh, u32 wg, u32 nwg) {
  const IterMeta* m = c.meta;
  const LayerWP* P = c.players + layer;
  MfmaGemmArgs a{};
  a.T = m->n_tokens;
  a.TBS = c.TBS;
  a.eps = c.eps;
  a.tune_nw = c.tune_nw;
  a.part = c.gemm_part;
  a.part_count = c.gemm_part_count;
  switch (PH) {
    case PH_EMBED: phase_embed_packed(c, wg, nwg); break;
    case PH_QKV:
      a.Wp = P->wqkv; a.Xp = c.xq; a.N = c.qkv_n; a.K = c.d; a.ssq_in = c.ssq;
      a.positions = c.positions; a.slot_mapping = c.slot_mapping; a.rope_tab = c.rope_tab; a.qbuf = c.qbuf;
      a.Kc = (f16_t*)c.kv + (u64)layer * c.kv_layer_stride; a.Vc = a.Kc + c.kv_kv_stride;
      a.nq = c.nq; a.nkv = c.nkv; a.hd = c.hd; a.bs = c.bs;
      gemm_bf16<EPI_QKV_ROPE>(a, m->plan & 0xffu, *(GemmShared8*)&sh, wg, nwg);
      break;
    case PH_ATTN: phase_attention_mfma(c, layer, *(AttnShared8*)&sh, wg, nwg); break;
    case PH_ATTN_COMBINE: attn_decode_combine(c, wg, nwg); break;
    case PH_ROUTER:     // router logits of every token; its first workgroup also clears the experts' counters for this layer
      if (wg == 0)
        for (u32 e = threadIdx.x; e < c.n_experts; e += blockDim.x) c.moe_count[e * MOE_COUNT_STRIDE] = 0;
      a.Wp = P->wr; a.Xp = c.xq; a.N = c.n_experts; a.K = c.d; a.ssq_in = c.ssq; a.out = c.moe_logits; a.ldo = c.n_experts;
      gemm_router<EPI_SCALED_STORE>(a, *(MfmaShared*)&sh, wg, nwg);
      break;
    case PH_ROUTE: moe_route(c, layer, wg, nwg); break;
    case PH_MOE_PERMUTE: moe_permute(c, layer, *(MoeLists*)&sh, wg, nwg); break;
    case PH_MOE_GATEUP: moe_gateup(c, layer, *(MoeShared*)&sh, wg, nwg); break;
    case PH_MOE_DOWN: moe_down(c, layer, *(MoeShared*)&sh, wg, nwg); break;
    case PH_MOE_COMBINE: moe_combine(c, layer, *(MoeLists*)&sh, wg, nwg); break;
    case PH_OPROJ:
      a.Wp = P->wo; a.Xp = c.aq; a.N = c.d; a.K = c.nq * c.hd; a.x = c.x; a.ldx = c.d; a.g_next = c.layers[layer].g2;
      a.Xp_next = c.xq; a.ssq_out = c.ssq;
      gemm_bf16<EPI_RESIDUAL>(a, (m->plan >> 8) & 0xffu, *(GemmShared8*)&sh, wg, nwg);
      break;
    case PH_GATEUP:
      a.Wp = P->wgu; a.Xp = c.xq; a.N = 2 * c.F; a.K = c.d; a.ssq_in = c.ssq; a.Hp = c.hq;
      gemm_bf16<EPI_SILU_GATE>(a, (m->plan >> 16) & 0xffu, *(GemmShared8*)&sh, wg, nwg);
      break;
    case PH_DOWN:
      a.Wp = P->wd; a.Xp = c.hq; a.N = c.d; a.K = c.F; a.x = c.x; a.ldx = c.d;
      a.g_next = layer + 1 < c.n_layers ? c.layers[layer + 1].g1 : c.gf;
      a.Xp_next = c.xq; a.ssq_out = c.ssq;
      gemm_bf16<EPI_RESIDUAL>(a, m->plan >> 24, *(GemmShared8*)&sh, wg, nwg);
      break;
    case PH_LM_HEAD:
      a.Wp = c.lm_p; a.Xp = c.xq; a.N = c.V; a.K = c.d; a.T = m->n_samples; a.tok_index = c.last_idx; a.ssq_in = c.ssq;
      a.out = c.logits; a.ldo = c.V;
      gemm_bf16<EPI_SCALED_STORE>(a, m->plan_lm, *(GemmShared8*)&sh, wg, nwg);
      break;
    case PH_SAMPLE:
      if (c.spec_k) phase_sample_publish_spec(c, *(SamplerShared*)&sh, wg, nwg);
      else phase_sample_publish(c, *(SamplerShared*)&sh, wg, nwg);
      break;
    default: break;   // the norms and the rotary / KV-write step are fused into the GEMMs
  }
}

template <int PH, bool F32>
__device__ __forceinline__ void run_phase(const DevCtx& c, u32 layer, typename PhaseSharedOf<PH, F32>::type& sh, u32 wg, u32 nwg) {
  if (c.meta->skip || c.meta->kind == KIND_IDLE) return;
  if constexpr (F32) run_phase_f32<PH>(c, layer, sh, wg, nwg);
  else run_phase_bf16<PH>(c, layer, sh, wg, nwg);
}
