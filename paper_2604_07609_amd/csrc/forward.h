// Forward pass of the Llama-style decoder over paged KV: the embedding and, for fp32 models, the attention. Each phase is a device function that loops over its work
// items with a workgroup stride, reading the batch shape from the device-resident metadata, so the
// same code runs from a host-enqueued kernel sequence and from the resident loop kernel. The model is
// the decoder that the paper's engine treats as opaque (section 4.3); shapes come from the workloads.
#pragma once
#include "blink_device.h"

template <typename WT> struct WLoad;
template <> struct WLoad<float> {
  static __device__ __forceinline__ float get(const float* p, u64 i) { return p[i]; }
  static __device__ __forceinline__ void load8(const float* p, float* o) {
    const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
};
template <> struct WLoad<bf16_t> {
  static __device__ __forceinline__ void load8(const bf16_t* p, float* o) {
    const uint4 a = *(const uint4*)p;
    const u32 w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
};

__device__ __forceinline__ u64 packed_act_off(u32 t, u32 k, u32 TBS) {   // same layout as mfma_gemm.h
  return ((u64)((k >> 5) * TBS + (t >> 4)) * 64 + (t & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

// ---- embedding gather: x[t] = E[input_ids[t]] ---------------------------------------------------------------
template <typename WT>
__device__ __forceinline__ void phase_embed(const DevCtx& c, u32 wg, u32 nwg) {
  const u32 T = c.meta->n_tokens, d = c.d;
  const WT* E = (const WT*)c.embed;
  const u32 per_row = d / 8;
  for (u64 i = (u64)wg * BLK_THREADS + threadIdx.x; i < (u64)T * per_row; i += (u64)nwg * BLK_THREADS) {
    const u32 t = (u32)(i / per_row), j = (u32)(i % per_row) * 8;
    float v[8];
    WLoad<WT>::load8(E + (u64)c.input_ids[t] * d + j, v);
    float* o = c.x + (u64)t * d + j;
    *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(o + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
}

// ---- embedding gather of the bf16 path: residual stream, packed operand of the first GEMM (x * g1 of layer 0)
// and the partial sums of squares its RMSNorm needs; one thread per (token, 16 columns) --------------------------
__device__ __forceinline__ void phase_embed_packed(const DevCtx& c, u32 wg, u32 nwg) {
  const u32 T = c.meta->n_tokens, d = c.d, per_row = d / 16;
  const bf16_t* E = (const bf16_t*)c.embed;
  const float* g = c.layers[0].g1;
  for (u64 i = (u64)wg * BLK_THREADS + threadIdx.x; i < (u64)T * per_row; i += (u64)nwg * BLK_THREADS) {
    const u32 t = (u32)(i / per_row), nt = (u32)(i % per_row), k0 = nt * 16;
    float v[16];
    WLoad<bf16_t>::load8(E + (u64)c.input_ids[t] * d + k0, v);
    WLoad<bf16_t>::load8(E + (u64)c.input_ids[t] * d + k0 + 8, v + 8);
    float* o = c.x + (u64)t * d + k0;
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) *(float4*)(o + 4 * j) = make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32 w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float a = v[8 * h + 2 * j], b = v[8 * h + 2 * j + 1];
        ss += a * a + b * b;
        w[j] = pack_f16x2(a * g[k0 + 8 * h + 2 * j], b * g[k0 + 8 * h + 2 * j + 1]);
      }
      *(uint4*)(c.xq + packed_act_off(t, k0 + 8 * h, c.TBS)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    c.ssq[(u64)t * per_row + nt] = ss;
  }
}

// ---- paged attention of an fp32 model: one workgroup (four waves) per (token, kv head, up to GT of its q heads) ----------------
// Bound by the bytes of the context's keys and values: a wave takes every fourth KV block, NB of them a step, with the next step's keys
// and values on their way while it works on this one's. Keys: four lanes a token, so that a load instruction covers whole 64-byte
// pieces of sixteen tokens; values: whole rows of the tokens. Scores meet in the four lanes by DPP, the running maximum over
// the wave by DPP and lane swaps, and a token's probability goes to the lanes of its values by a shuffle; the output stays in
// registers until the waves' results are merged, in their order, at the end. (As one thread per key, a row of keys is a 32-byte
// piece per lane and load and the values wait for a block id each: 512 sequences x 2 kv heads of 64 at 25 / 324 / 1024 / 2024 keys
// 20 / 120 / 505 / 987 us, now 13 / 38 / 130 / 245 = 4.1 TB/s.)
#define ATT_MAX_G 8
struct AttnShared {
  float m[4][ATT_MAX_G], l[4][ATT_MAX_G];
  float o[4][ATT_MAX_G][128];
};
template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __uint_as_float((u32)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xF, 0xF, true)); }
// over the lanes l, l ^ 16, l ^ 32, l ^ 48 (ALL) or l, l ^ 32
template <bool ALL, typename F>
__device__ __forceinline__ float across_rows(float v, F f) {
  if (ALL) { const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false); v = f(__uint_as_float(a[0]), __uint_as_float(a[1])); }
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int HD, int GT>
__device__ __forceinline__ void attn_f32(const DevCtx& c, u32 layer, AttnShared& sh, u32 wg, u32 nwg) {
  constexpr int KD = HD / 16, NB = (HD == 64 ? 4 : 2) / (GT > 128 / HD ? 2 : 1);   // float4 of a key (or value) block per lane; blocks of a step
  constexpr u32 LD = HD / 4, VT = 64 / LD;                  // lanes of a row of values, rows per load
  const u32 T = c.meta->n_tokens, G = c.nq / c.nkv, parts = (G + GT - 1) / GT;
  const u32 lane = threadIdx.x & 63, w = (u32)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const u32 kt = lane >> 2, kp = lane & 3, vt = lane / LD, vd = lane % LD;
  const float* const Kc = (const float*)c.kv + (u64)layer * c.kv_layer_stride;
  const float* const Vc = Kc + c.kv_kv_stride;
  const float scale = 1.0f / sqrtf((float)HD);
  auto fmax2 = [](float x, float y) { return fmaxf(x, y); };
  auto add2 = [](float x, float y) { return x + y; };
  typedef const __attribute__((address_space(4))) u32 const_u32;
  for (u32 item = wg; item < T * c.nkv * parts; item += nwg) {
    const u32 t = item / (c.nkv * parts), g = item / parts % c.nkv, h0 = item % parts * GT, heads = min((u32)GT, G - h0);
    const u32 n = (u32)__builtin_amdgcn_readfirstlane((u32)c.positions[t] + 1), nblk = (n + 15) / 16;
    const u64 bta = (u64)(c.block_tables + (u64)c.tok_bslot[t] * c.max_blocks_per_seq);
    const u32 bt_hi = (u32)__builtin_amdgcn_readfirstlane((u32)(bta >> 32)), bt_lo = (u32)__builtin_amdgcn_readfirstlane((u32)bta);
    const_u32* const bt = (const_u32*)(((u64)bt_hi << 32) | (u64)bt_lo);
    float4 q[GT][KD], acc[GT];
    float m[GT], l[GT];                                     // running maximum, this lane's share of the sum
#pragma unroll
    for (int h = 0; h < GT; ++h) {
      const float* qp = c.qkv + (u64)t * c.qkv_n + (u64)(g * G + min(h0 + h, G - 1)) * HD + kp * 4;
#pragma unroll
      for (int i = 0; i < KD; ++i) {
        const float4 v = *(const float4*)(qp + 16 * i);
        q[h][i] = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
      }
      m[h] = -INFINITY; l[h] = 0.f; acc[h] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // this wave's blocks: w, w + 4, ...; past the last one that again (loaded, not used)
    float4 k[NB][KD], v[NB][KD];
    auto block = [&](u32 s, int j) -> u64 { return ((u64)bt[min((s * NB + j) * 4 + w, nblk - 1)] * c.nkv + g) * (16 * HD); };
    auto load_k = [&](u32 s) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const float* kb = Kc + block(s, j) + kt * HD + kp * 4;
#pragma unroll
        for (int i = 0; i < KD; ++i) k[j][i] = *(const float4*)(kb + 16 * i);
      }
    };
    auto load_v = [&](u32 s) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const float* vb = Vc + block(s, j) + vt * HD + vd * 4;
#pragma unroll
        for (int i = 0; i < KD; ++i) v[j][i] = *(const float4*)(vb + i * (int)VT * HD);
      }
    };
    const u32 steps = nblk > w ? ((nblk - w + 3) / 4 + NB - 1) / NB : 0u;
    if (steps) { load_k(0); load_v(0); }
    for (u32 s = 0; s < steps; ++s) {
      float p[GT][NB];
#pragma unroll
      for (int h = 0; h < GT; ++h) {
        float cm = -INFINITY;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          float d = 0.f;
#pragma unroll
          for (int i = 0; i < KD; ++i) d += q[h][i].x * k[j][i].x + q[h][i].y * k[j][i].y + q[h][i].z * k[j][i].z + q[h][i].w * k[j][i].w;
          d += dpp<0xB1>(d);                                // the four lanes of the token
          d += dpp<0x4E>(d);
          p[h][j] = ((s * NB + j) * 4 + w) * 16 + kt < n ? d : -INFINITY;
          cm = fmaxf(cm, p[h][j]);
        }
        cm = fmaxf(cm, dpp<0x124>(cm));                     // the four tokens of a row of sixteen lanes (rotations by 4 and 8), then the rows
        cm = fmaxf(cm, dpp<0x128>(cm));
        cm = across_rows<true>(cm, fmax2);
        const float mn = fmaxf(m[h], cm), corr = __expf(m[h] - mn);       // (finite: a wave's first block has a visible key; exp(-inf) = 0)
        float ps = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) { p[h][j] = __expf(p[h][j] - mn); ps += p[h][j]; }
        l[h] = l[h] * corr + ps;
        m[h] = mn;
        acc[h].x *= corr; acc[h].y *= corr; acc[h].z *= corr; acc[h].w *= corr;
      }
      load_k(s + 1);
      if (((s * NB + NB - 1) * 4 + w) * 16 + 16 > n) {       // rows behind the context hold what an earlier request left there: not even times 0
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int i = 0; i < KD; ++i)
            if (((s * NB + j) * 4 + w) * 16 + vt + VT * i >= n) v[j][i] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < KD; ++i)
#pragma unroll
          for (int h = 0; h < GT; ++h) {
            const float pj = __shfl(p[h][j], (int)(4 * (vt + VT * i)));   // the probability of this lane's token
            acc[h].x += pj * v[j][i].x; acc[h].y += pj * v[j][i].y; acc[h].z += pj * v[j][i].z; acc[h].w += pj * v[j][i].w;
          }
      load_v(s + 1);
    }
    __syncthreads();                                        // the previous item's results have been read
#pragma unroll
    for (int h = 0; h < GT; ++h) {
      l[h] += dpp<0x124>(l[h]);
      l[h] += dpp<0x128>(l[h]);
      l[h] = across_rows<true>(l[h], add2);
      acc[h].x = across_rows<HD == 64>(acc[h].x, add2); acc[h].y = across_rows<HD == 64>(acc[h].y, add2);
      acc[h].z = across_rows<HD == 64>(acc[h].z, add2); acc[h].w = across_rows<HD == 64>(acc[h].w, add2);
      if (lane < LD) *(float4*)&sh.o[w][h][vd * 4] = acc[h];
      if (lane == 0) { sh.m[w][h] = m[h]; sh.l[w][h] = l[h]; }
    }
    __syncthreads();
    for (u32 i = threadIdx.x; i < heads * HD; i += BLK_THREADS) {
      const u32 h = i / HD, d = i % HD;
      float M = sh.m[0][h], L = 0.f, O = 0.f;               // (wave 0 has the first block)
#pragma unroll
      for (int ww = 1; ww < 4; ++ww) M = fmaxf(M, sh.m[ww][h]);
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {                      // a wave without blocks has m = -inf and contributes 0
        const float f = __expf(sh.m[ww][h] - M);
        L += sh.l[ww][h] * f;
        O += sh.o[ww][h][d] * f;
      }
      c.attn[(u64)t * (c.nq * HD) + (u64)(g * G + h0 + h) * HD + d] = O / L;
    }
  }
}

__device__ __forceinline__ void phase_attention_f32(const DevCtx& c, u32 layer, AttnShared& sh, u32 wg, u32 nwg) {
  const u32 G = c.nq / c.nkv;      // (q heads of one kv head that share its loads: up to four of 64, two of 128, what the registers hold)
  if (c.hd == 64) {
    if (G == 1) attn_f32<64, 1>(c, layer, sh, wg, nwg);
    else if (G == 2) attn_f32<64, 2>(c, layer, sh, wg, nwg);
    else attn_f32<64, 4>(c, layer, sh, wg, nwg);
  } else if (G == 1) attn_f32<128, 1>(c, layer, sh, wg, nwg);
  else attn_f32<128, 2>(c, layer, sh, wg, nwg);
}
