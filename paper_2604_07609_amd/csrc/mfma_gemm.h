// GEMMs of the forward pass of a bf16 model on the CDNA4 matrix cores, the only dense contractions of the serving
// step. The weights are stored in bf16 (8 significant bits); for the matrix cores they are re-encoded once, at init,
// as IEEE half precision scaled by 2^8 (exact for every bf16 value of magnitude 2^-25 .. 255: a half holds 11
// significant bits), and the activation operands between the GEMMs are carried in half precision too
// (v_mfma_f32_16x16x32_f16, fp32 accumulation; same rate and the same bytes as the bf16 instruction). With bf16
// activation operands the roundings between the GEMMs (unit roundoff 2^-8, about eight per layer) add up to 3e-2 of
// the largest logit over 32 layers; half precision cuts each of them by eight. Activations saturate at the largest
// finite half instead of overflowing. Both operands live in HBM already in MFMA operand order, so that every
// wave-wide load is one contiguous kilobyte:
//
//   weights      Wp[n/16][k/32][lane][8]      lane = n%16 + 16*((k%32)/8), element = k%8   (packed once at init)
//   activations  Xp[k/32][t/16][lane][8]      lane = t%16 + 16*((k%32)/8), element = k%8   (written packed by the
//                                                                                  producing kernel's epilogue)
//
// The k dimension of both is padded with zeros to a multiple of 64 (an even number of k-steps).
//
// out[t][n] = sum_k X[t][k] * W[n][k]. Every GEMM kernel runs eight waves per workgroup and one workgroup per compute unit. The
// schedule is chosen per launch from the token count T of the iteration and the shape of the matrix (gemm_plan.h):
//   tiles whose operands go from memory straight to LDS (gemm_dma.h): T > 64, and tall matrices at any T.
//   stream (T <= 64 otherwise, decode at small batch): a workgroup owns 1 or 2 16-row weight tiles and all token blocks; its
//     eight waves split K and keep two batches of 1 KB operand loads in flight each; weight loads are non-temporal;
//     partial sums are reduced through LDS in a fixed order. HBM bound: the weight matrix once.
// Epilogues fuse what follows the GEMM in the model: RMSNorm scale of the *input* (a per-token scalar,
// applied to the accumulator), residual add, SiLU-gating, rotary embedding and the KV-cache write, and re-packing of
// the result as the next GEMM's activation operand together with the partial sums of squares the next RMSNorm needs.
#pragma once
#include "blink_device.h"
#include "gemm_plan.h"

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

#define W_SCALE 256.0f            // packed weights hold W * 2^8 (keeps small weights in the normal range of a half)
#define W_SCALE_INV (1.0f / 256.0f)

struct MfmaGemmArgs {
  const f16_t* Wp;         // packed weights (half precision, scaled by W_SCALE)
  const f16_t* Xp;         // packed activations (half precision; K = inner dimension)
  u32 N, K;                // logical output rows and inner dimension (K % 32 == 0; the packed operands hold gemm_k_tiles(K) k-steps)
  u32 T;                   // tokens (columns)
  u32 TBS;                 // token-block stride of the packed activation buffers (the operand Xp and, unless TBS_out is set, the outputs)
  u32 TBS_out;             // 0, or the token-block stride of the packed output Hp when it differs from the operand's
  u32 col0;                // output column of token 0 (EPI_SCALED_STORE row of `out`, EPI_SILU_GATE column of Hp): a grouped
                           // GEMM writes each group's columns behind the previous group's
  const u32* tok_index;    // optional indirection: column t reads token tok_index[t] of Xp / ssq_in (LM head)
  const float* ssq_in;     // [token][K/16] partial sums of squares of the un-normalised input (null: no scaling)
  float eps;
  // EPI_SCALED_STORE
  float* out; u32 ldo;
  // EPI_RESIDUAL
  float* x; u32 ldx;       // residual stream, updated in place
  const float* g_next;     // gain of the RMSNorm that consumes x next
  f16_t* Xp_next;          // packed half(x * g_next), inner dimension N
  float* ssq_out;          // [token][N/16]
  // EPI_SILU_GATE
  f16_t* Hp;               // packed activations with inner dimension N/2
  // EPI_QKV_ROPE
  const i32* positions;
  const i32* slot_mapping;
  const float2* rope_tab;
  f16_t* qbuf;
  f16_t* Kc;               // this layer's K cache and V cache (half precision)
  f16_t* Vc;
  u32 nq, nkv, hd, bs;
  u64* part;               // split K: the slices' sums, at most one 256 x 128 tile of floats per compute unit, and a count per tile (zeros between launches)
  u32* part_count;
  u32 tune_nw;             // tests and tuning. Low three bits: 0 automatic choice of weight tiles per workgroup of the streaming schedule, 1/2 forced.
                           // Bit 5 (launcher): never a kernel chain without the decode attention's merge kernels, bit 7: always the one for whole contexts, bit 3: always
                           // the one whose attention merges chunks itself. Bit 4 (set in that chain): it does.
                           // Bit 6: epilogues load their operands tile by tile (not in waves with four row tiles, epilogue_cols). Bit 11: tall matrices stream too at T <= 64.
                           // Bits 12-14: force the tile shape at T > 64, with them bits 24-27 the slices of K (gemm_plan).
                           // Bit 15 (scheduler): the decode attention's work items are always chunks, bit 22: always whole
                           // contexts; bit 23: the decode attention kernel with static items. Bits 16-19: 15 prompt attention with shared KV tiles, 1, 2, 4 or 8 the
                           // other kernel with that many waves per item, other values that kernel. Bit 30: mixed launches run their decode part first in every workgroup.
};

#define GEMM_MAX_WAVES 8
struct MfmaShared {
  float red[GEMM_MAX_WAVES][4][64][4];       // [wave][token block][lane][4]
  float rstd[256];                           // norm scales of the tokens
};

__device__ __forceinline__ u64 packed_off(u32 t, u32 k, u32 TBS) {
  return ((u64)((k >> 5) * TBS + (t >> 4)) * 64 + (t & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

__device__ __forceinline__ f16x8_t as_f16x8(uint4 v) { return *(const f16x8_t*)&v; }
__device__ __forceinline__ f16x8_t ld_op(const f16_t* p) {   // one lane's 16 bytes of a packed tile
  return as_f16x8(*(const uint4*)p);
}

// rstd (times the inverse of the weight scale) of COUNT (<= 256) tokens starting at column t0 into
// rstd[0 .. COUNT) (LDS), by a workgroup of THREADS. Sixteen lanes share a token: each reads every sixteenth 16-byte piece of the
// token's partial sums (256 contiguous bytes per token and load), and a butterfly over the sixteen lanes finishes the sum.
// A chain of memory latencies in front of a launch's first product (or, beside its first operands, of its first epilogue), so
// every load is unconditional (clamped) and a batch of them is written out: with the loads behind a run-time count of tokens
// they came one at a time, 16 to 64 latencies, wherever the compiler was short of registers (QKV 6144 x 4096 of one
// token 15 us, 509 tokens 58 us).
template <int COUNT, int THREADS>
__device__ __forceinline__ void compute_rstd(const MfmaGemmArgs& a, u32 t0, float* rstd) {
  constexpr int G = THREADS / 16, P = (COUNT + G - 1) / G, U = P > 8 ? 1 : P == 8 ? 2 : 4;   // tokens at a time, passes, pieces per batch
  const u32 tid = threadIdx.x;
  __syncthreads();   // the previous readers of rstd are done
  if (a.ssq_in == nullptr) {
    if (tid < COUNT) rstd[tid] = W_SCALE_INV;
  } else {
    const u32 np = a.K / 16, l16 = tid & 15, grp = tid >> 4;
    const float* pp[P];
    float s[P];
#pragma unroll
    for (int it = 0; it < P; ++it) {
      const u32 t = min(t0 + min(grp + G * it, (u32)COUNT - 1), a.T - 1);   // clamped: results of padding tokens are dropped
      pp[it] = a.ssq_in + (u64)(a.tok_index ? a.tok_index[t] : t) * np;
      s[it] = 0.f;
    }
    if ((np & 3u) == 0) {
      for (u32 q0 = 0; q0 < np; q0 += 64 * U) {
        float4 v[U][P];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int it = 0; it < P; ++it) v[u][it] = *(const float4*)(pp[it] + min(q0 + 64 * u + l16 * 4, np - 4));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int it = 0; it < P; ++it) s[it] += q0 + 64 * u + l16 * 4 < np ? (v[u][it].x + v[u][it].y) + (v[u][it].z + v[u][it].w) : 0.f;
      }
    } else {
      for (u32 q0 = 0; q0 < np; q0 += 16) {
        float v[P];
#pragma unroll
        for (int it = 0; it < P; ++it) v[it] = pp[it][min(q0 + l16, np - 1)];
#pragma unroll
        for (int it = 0; it < P; ++it) s[it] += q0 + l16 < np ? v[it] : 0.f;
      }
    }
#pragma unroll
    for (int it = 0; it < P; ++it) {
      float v = s[it];
      v += __shfl_xor(v, 1); v += __shfl_xor(v, 2); v += __shfl_xor(v, 4); v += __shfl_xor(v, 8);
      const u32 tl = grp + G * it;
      if (l16 == 0 && tl < COUNT) rstd[tl] = W_SCALE_INV / sqrtf(v / (float)a.K + a.eps);
    }
  }
  __syncthreads();
}

// What several epilogues compute is written out once: left to the compiler, which product is rounded and which goes into a fused
// multiply-add depends on what it is inlined into, and a last bit here moves near ties of a router.
// Sum of the squares of a lane's four values of the residual stream.
__device__ __forceinline__ float sum_squares(float v0, float v1, float v2, float v3) { return fmaf(v3, v3, fmaf(v2, v2, fmaf(v1, v1, v0 * v0))); }

// A pair of the rotary embedding, (c, s) the cosine and sine of its angle.
__device__ __forceinline__ void rotate(float& lo, float& hi, float c, float s) {
  const float a = fmaf(lo, c, -(hi * s));
  hi = fmaf(hi, c, lo * s);
  lo = a;
}

// Epilogue of one 16(n) x 16(t) accumulator tile held by one wave. rl: index of the tile's first token in sh.rstd.
template <int EPI>
__device__ __forceinline__ void epilogue_tile(const MfmaGemmArgs& a, floatx4_t acc, u32 nt, u32 t_base, const float* rstd16) {
  const u32 lane = threadIdx.x & 63;
  const u32 t = t_base + (lane & 15);
  const u32 n0 = nt * 16 + (lane >> 4) * 4;
  const bool tv = t < a.T;
  if (EPI == EPI_SCALED_STORE) {
    if (!tv) return;
    const float r = rstd16[lane & 15];
    float* o = a.out + (u64)(t + a.col0) * a.ldo + n0;
    if (n0 + 3 < a.N && (a.ldo & 3) == 0) {
      *(float4*)o = make_float4(acc[0] * r, acc[1] * r, acc[2] * r, acc[3] * r);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (n0 + i < a.N) o[i] = acc[i] * r;
    }
  } else if (EPI == EPI_RESIDUAL) {
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (tv) {
      float* xp = a.x + (u64)t * a.ldx + n0;
      const float4 old = *(const float4*)xp;
      v[0] = old.x + acc[0] * W_SCALE_INV; v[1] = old.y + acc[1] * W_SCALE_INV;
      v[2] = old.z + acc[2] * W_SCALE_INV; v[3] = old.w + acc[3] * W_SCALE_INV;
      *(float4*)xp = make_float4(v[0], v[1], v[2], v[3]);
      const float4 g = *(const float4*)(a.g_next + n0);
      *(uint2*)(a.Xp_next + packed_off(t, n0, a.TBS)) = make_uint2(pack_f16x2(v[0] * g.x, v[1] * g.y), pack_f16x2(v[2] * g.z, v[3] * g.w));
    }
    float s = sum_squares(v[0], v[1], v[2], v[3]);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lane < 16 && tv) a.ssq_out[(u64)t * (a.N / 16) + nt] = s;
  } else if (EPI == EPI_QKV_ROPE) {
    if (!tv) return;
    const float r = rstd16[lane & 15];
    const u32 hd = a.hd, half = hd / 2, head = n0 / hd, p = (n0 % hd) >> 1;   // rows: (p, p+half, p+1, p+1+half)
    float lo0 = acc[0] * r, hi0 = acc[1] * r, lo1 = acc[2] * r, hi1 = acc[3] * r;
    if (head < a.nq + a.nkv) {
      const float4 cs = *(const float4*)(a.rope_tab + (u64)a.positions[t] * half + p);   // (cos,sin) of pairs p, p+1
      rotate(lo0, hi0, cs.x, cs.y);
      rotate(lo1, hi1, cs.z, cs.w);
    }
    if (head < a.nq) {
      const float sc = 1.0f / sqrtf((float)hd);
      f16_t* q = a.qbuf + ((u64)t * a.nq + head) * hd;
      *(u32*)(q + p) = pack_f16x2(lo0 * sc, lo1 * sc);
      *(u32*)(q + half + p) = pack_f16x2(hi0 * sc, hi1 * sc);
    } else {
      const u32 slot = (u32)a.slot_mapping[t];
      if (head < a.nq + a.nkv) {
        f16_t* k = a.Kc + (((u64)(slot / a.bs) * a.nkv + (head - a.nq)) * a.bs + slot % a.bs) * hd;
        *(u32*)(k + p) = pack_f16x2(lo0, lo1);
        *(u32*)(k + half + p) = pack_f16x2(hi0, hi1);
      } else {   // V is kept dimension-major inside a block: [hd][16 tokens]
        f16_t* v = a.Vc + ((u64)(slot / a.bs) * a.nkv + (head - a.nq - a.nkv)) * a.bs * hd + slot % a.bs;
        v[(u64)p * a.bs] = f32_to_f16(lo0);
        v[(u64)(p + 1) * a.bs] = f32_to_f16(lo1);
        v[(u64)(half + p) * a.bs] = f32_to_f16(hi0);
        v[(u64)(half + p + 1) * a.bs] = f32_to_f16(hi1);
      }
    }
  } else {  // EPI_SILU_GATE
    if (!tv) return;
    const float r = rstd16[lane & 15];
    const float g0 = acc[0] * r, u0 = acc[1] * r, g1 = acc[2] * r, u1 = acc[3] * r;
    const float h0 = g0 / (1.f + __expf(-g0)) * u0, h1 = g1 / (1.f + __expf(-g1)) * u1;
    const u32 j = n0 >> 1;   // pair index = inner index of the next GEMM
    *(u32*)(a.Hp + packed_off(t + a.col0, j, a.TBS_out ? a.TBS_out : a.TBS)) = pack_f16x2(h0, h1);
  }
}

// EPI_QKV_ROPE of one tile with its operands already loaded: `r` = the token's norm scale, `slot` = its place in the paged
// cache, `cs` = (cos, sin) of the two rotary pairs of this lane's rows at the token's position (unused for V rows).
__device__ __forceinline__ void rope_finish(const MfmaGemmArgs& a, floatx4_t acc, u32 nt, u32 t, float r, u32 slot, float4 cs) {
  if (t >= a.T) return;
  const u32 lane = threadIdx.x & 63, n0 = nt * 16 + (lane >> 4) * 4;
  const u32 hd = a.hd, half = hd / 2, head = n0 / hd, p = (n0 % hd) >> 1;   // rows: (p, p+half, p+1, p+1+half)
  float lo0 = acc[0] * r, hi0 = acc[1] * r, lo1 = acc[2] * r, hi1 = acc[3] * r;
  if (head < a.nq + a.nkv) {
    rotate(lo0, hi0, cs.x, cs.y);
    rotate(lo1, hi1, cs.z, cs.w);
  }
  if (head < a.nq) {
    const float sc = 1.0f / sqrtf((float)hd);
    f16_t* q = a.qbuf + ((u64)t * a.nq + head) * hd;
    *(u32*)(q + p) = pack_f16x2(lo0 * sc, lo1 * sc);
    *(u32*)(q + half + p) = pack_f16x2(hi0 * sc, hi1 * sc);
  } else if (head < a.nq + a.nkv) {
    f16_t* k = a.Kc + (((u64)(slot / a.bs) * a.nkv + (head - a.nq)) * a.bs + slot % a.bs) * hd;
    *(u32*)(k + p) = pack_f16x2(lo0, lo1);
    *(u32*)(k + half + p) = pack_f16x2(hi0, hi1);
  } else {   // V is kept dimension-major inside a block: [hd][16 tokens]
    f16_t* v = a.Vc + ((u64)(slot / a.bs) * a.nkv + (head - a.nq - a.nkv)) * a.bs * hd + slot % a.bs;
    v[(u64)p * a.bs] = f32_to_f16(lo0);
    v[(u64)(p + 1) * a.bs] = f32_to_f16(lo1);
    v[(u64)(half + p) * a.bs] = f32_to_f16(hi0);
    v[(u64)(half + p + 1) * a.bs] = f32_to_f16(hi1);
  }
}

// EPI_RESIDUAL of one tile with its operands already loaded: `old` = this lane's four residual values of token
// min(t, T - 1) (the caller's unconditional load), `g` = the next norm's gains of its four rows.
__device__ __forceinline__ void residual_finish(const MfmaGemmArgs& a, floatx4_t acc, u32 nt, u32 t, float4 old, float4 g) {
  const u32 lane = threadIdx.x & 63, n0 = nt * 16 + (lane >> 4) * 4;
  const bool tv = t < a.T;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (tv) {
    v[0] = old.x + acc[0] * W_SCALE_INV; v[1] = old.y + acc[1] * W_SCALE_INV;
    v[2] = old.z + acc[2] * W_SCALE_INV; v[3] = old.w + acc[3] * W_SCALE_INV;
    *(float4*)(a.x + (u64)t * a.ldx + n0) = make_float4(v[0], v[1], v[2], v[3]);
    *(uint2*)(a.Xp_next + packed_off(t, n0, a.TBS)) = make_uint2(pack_f16x2(v[0] * g.x, v[1] * g.y), pack_f16x2(v[2] * g.z, v[3] * g.w));
  }
  float s = sum_squares(v[0], v[1], v[2], v[3]);
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  if (lane < 16 && tv) a.ssq_out[(u64)t * (a.N / 16) + nt] = s;
}

// All loads of this wave have come. Said to the compiler where it may go on without using what they brought: it keeps their registers
// apart from then on by waiting before it writes to them again, and where that is inside a loop it waits there in every
// round, for the tiles on their way to LDS as well, which it knows nothing of.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0), the other counters at their most
// The same for one load whose result not every path uses.
template <typename T>
__device__ __forceinline__ void loaded(const T& v) { asm volatile("" : : "v"(v)); }

// Epilogue of the TJ accumulator tiles a wave holds for one row tile (tokens t_base + 16 j + lane % 16); a residual add or rotary embedding comes
// here from waves with one or two row tiles (with four: epilogue_cols). Those read memory (the residual stream, the
// positions and the rotary table), and request the operands of all tiles first: written one tile after the other, every tile's loads would wait
// behind the previous tile's stores (the compiler has to assume that they may alias), a chain of TJ memory latencies.
// Tokens behind the last one read the last token's operands (an unconditional load) and store nothing.
// (Bit 6 of the tuning word: tile by tile, for comparison.)
template <int EPI, int TJ>
__device__ __forceinline__ void epilogue_row(const MfmaGemmArgs& a, const floatx4_t (&acc)[TJ], u32 nt, u32 t_base, const float* rstd) {
  if ((EPI != EPI_RESIDUAL && EPI != EPI_QKV_ROPE) || (a.tune_nw & 0x40u)) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) epilogue_tile<EPI>(a, acc[j], nt, t_base + j * 16, rstd + j * 16);
    return;
  }
  // (The lane comes anew, by an empty asm: without it the streaming schedule of the same kernel comes out slower, QKV 5120 x 2048 at 96
  // tokens 20.6 us instead of 19.8.)
  u32 lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const u32 n0 = nt * 16 + (lane >> 4) * 4;
  const u32 hd = a.hd, half = hd / 2, head = EPI == EPI_QKV_ROPE ? n0 / hd : 0u, p = EPI == EPI_QKV_ROPE ? (n0 % hd) >> 1 : 0u;   // rows: (p, p+half, p+1, p+1+half)
  const bool rot = head < a.nq + a.nkv;
  float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
  if (EPI == EPI_RESIDUAL) g = *(const float4*)(a.g_next + n0);
  u32 t[TJ], tc[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) { t[j] = t_base + j * 16 + (lane & 15); tc[j] = min(t[j], a.T - 1); }
  if (EPI == EPI_RESIDUAL) {
    float4 old[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) old[j] = *(const float4*)(a.x + (u64)tc[j] * a.ldx + n0);
#pragma unroll
    for (int j = 0; j < TJ; ++j) residual_finish(a, acc[j], nt, t[j], old[j], g);
  } else {   // EPI_QKV_ROPE
    i32 pos[TJ];
    u32 slot[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) { pos[j] = a.positions[tc[j]]; slot[j] = (u32)a.slot_mapping[tc[j]]; }
    float4 cs[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) cs[j] = *(const float4*)(a.rope_tab + (u64)(rot ? pos[j] : 0) * half + (rot ? p : 0u));   // (cos,sin) of pairs p, p+1
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      loaded(cs[j].x); loaded(cs[j].y); loaded(cs[j].z); loaded(cs[j].w);
      loaded(slot[j]);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) rope_finish(a, acc[j], nt, t[j], rstd[j * 16 + (lane & 15)], slot[j], cs[j]);
  }
}

// Transposes the 4 x 4 matrix M[i][lane / 16] that lanes l, l + 16, l + 32, l + 48 hold as r[i]: afterwards lane group g holds row g,
// r[c] = M[g][c]. (v_permlane16_swap exchanges the odd groups of its first operand with the even ones of its second,
// v_permlane32_swap the upper half of the first with the lower half of the second.)
__device__ __forceinline__ void swap16(u32& a, u32& b) { const auto v = __builtin_amdgcn_permlane16_swap(a, b, false, false); a = v[0]; b = v[1]; }
__device__ __forceinline__ void swap32(u32& a, u32& b) { const auto v = __builtin_amdgcn_permlane32_swap(a, b, false, false); a = v[0]; b = v[1]; }
__device__ __forceinline__ void transpose4(u32 (&r)[4]) {
  swap16(r[0], r[1]); swap16(r[2], r[3]);
  swap32(r[0], r[2]); swap32(r[1], r[3]);
}

// Epilogue of the 4 x TJ accumulator tiles (64 rows from row tile nt0, a multiple of four; tokens t_base + 16 j + lane % 16) of a wave
// of the wide tiles. A column of tiles (16 tokens) at a time, with the operands of the next columns on their way: one row tile
// after the other, two tiles' loads at a time, an epilogue is a chain of eight to sixteen memory latencies with little in flight
// (256 x 256 tiles, every compute unit at it: 76 us with the residual add). And the four row tiles of a column are exchanged
// between the lanes first, so that a lane stores 16 bytes of one row's neighbours instead of four pieces of 4 bytes: the gate's
// result is a whole packed tile (1 KB) per column, queries and keys are runs of 64 bytes per token.
// Tokens behind the last one are computed and stored like the others, into rows that the buffers have for it (16 behind the
// last token's; for keys and values the query buffer's), so that no store stands in a branch, where the loads behind it would
// have to wait for it. QKV 6144 x 4096 at 509 / 1700 / 8000 tokens 58 / 120 / 466 us before and 45 / 92 / 346 now (with compute_rstd and
// without waits in the main loop), gate/up 28672 x 4096 at 1700 / 8000 tokens 351 / 1506 and 341 / 1452 (means of a pass).
template <int EPI, int TJ>
__device__ __forceinline__ void epilogue_cols(const MfmaGemmArgs& a, const floatx4_t (&acc)[4][TJ], u32 nt0, u32 t_base, const float* rstd) {
  u32 lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));               // (nothing of this is kept in registers from one item to the next)
  const u32 lc = lane & 15, lg = lane >> 4;
  constexpr int DMAX = EPI == EPI_QKV_ROPE ? 2 : 3, D = TJ < DMAX ? TJ : DMAX;   // columns whose operands are on their way
  if (t_base >= a.T) return;
  if constexpr (EPI == EPI_SILU_GATE) {
    const u32 tbs = a.TBS_out ? a.TBS_out : a.TBS;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      if (t_base + j * 16 >= a.T) return;
      const u32 t = t_base + j * 16 + lc + a.col0;
      const float r = rstd[j * 16 + lc];
      u32 h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float g0 = acc[i][j][0] * r, u0 = acc[i][j][1] * r, g1 = acc[i][j][2] * r, u1 = acc[i][j][3] * r;
        const float h0 = g0 / (1.f + __expf(-g0)) * u0, h1 = g1 / (1.f + __expf(-g1)) * u1;
        h[i] = pack_f16x2(h0, h1);
      }
      transpose4(h);                           // this lane: outputs nt0 * 8 + lg * 8 .. + 7 of its token
      *(uint4*)(a.Hp + ((u64)((nt0 >> 2) * tbs + (t >> 4)) * 64 + (t & 15) + 16 * lg) * 8) = make_uint4(h[0], h[1], h[2], h[3]);
    }
  } else if constexpr (EPI == EPI_RESIDUAL) {
    const u32 NT = a.N / 16;
    const bool two = nt0 + 2 < NT;             // (rows come in pairs of tiles: the second pair may be behind the last row)
    float4 g[4], old[D][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = *(const float4*)(a.g_next + (i < 2 || two ? nt0 + i : nt0) * 16 + lg * 4);
    auto request = [&](int j, float4 (&o)[4]) {
      const float* xp = a.x + (u64)min(t_base + j * 16 + lc, a.T - 1) * a.ldx + nt0 * 16 + lg * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = *(const float4*)(xp + (i < 2 || two ? i * 16 : 0));
    };
#pragma unroll
    for (int j = 0; j < D; ++j) request(j, old[j]);
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      if (t_base + j * 16 >= a.T) { wait_loads(); return; }
      const u32 t = t_base + j * 16 + lc;
      float ss[4];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if (p == 1 && !two) break;
        u32 k[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int i = 2 * p + q;
          const float4 o = old[j % D][i];
          const float v0 = o.x + acc[i][j][0] * W_SCALE_INV, v1 = o.y + acc[i][j][1] * W_SCALE_INV;
          const float v2 = o.z + acc[i][j][2] * W_SCALE_INV, v3 = o.w + acc[i][j][3] * W_SCALE_INV;
          *(float4*)(a.x + (u64)t * a.ldx + (nt0 + i) * 16 + lg * 4) = make_float4(v0, v1, v2, v3);
          k[q][0] = pack_f16x2(v0 * g[i].x, v1 * g[i].y);
          k[q][1] = pack_f16x2(v2 * g[i].z, v3 * g[i].w);
          float s = sum_squares(v0, v1, v2, v3);
          s += __shfl_xor(s, 16);
          ss[i] = s + __shfl_xor(s, 32);
        }
        // even lane groups take eight values of the pair's first row tile, odd ones of its second
        swap16(k[0][0], k[1][0]); swap16(k[0][1], k[1][1]);
        *(uint4*)(a.Xp_next + ((u64)(((nt0 + 2 * p) >> 1) * a.TBS + (t >> 4)) * 64 + lc + 16 * ((lg & 1) * 2 + (lg >> 1))) * 8) =
            make_uint4(k[0][0], k[0][1], k[1][0], k[1][1]);
      }
      // the sums of squares of the four row tiles, a tile per lane group
      const float s01 = lg & 1 ? ss[1] : ss[0], s23 = lg & 1 ? ss[3] : ss[2];
      if (two) a.ssq_out[(u64)t * NT + nt0 + lg] = lg & 2 ? s23 : s01;
      else if (lg < 2) a.ssq_out[(u64)t * NT + nt0 + lg] = s01;
      if (j + D < TJ) request(j + D, old[j % D]);
    }
  } else {                                     // EPI_QKV_ROPE: 64 rows are the pairs p0 .. p0 + 31 of one head
    const u32 hd = a.hd, half = hd / 2, head = nt0 * 16 / hd, p0 = (nt0 * 16 % hd) >> 1;
    u32 at[TJ], pos[TJ];                       // cache slots (keys and values) and positions (queries and keys)
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const u32 t = min(t_base + j * 16 + lc, a.T - 1);
      at[j] = (u32)a.slot_mapping[t]; pos[j] = (u32)a.positions[t];
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) { loaded(at[j]); loaded(pos[j]); }
    auto cache_row = [&](f16_t* cache, u32 h, int j) -> f16_t* {       // the 16-token block's part of kv head h
      return cache + ((u64)(at[j] / a.bs) * a.nkv + h) * (a.bs * hd);
    };
    f16_t* const spare = a.qbuf + ((u64)a.T * a.nq) * hd;              // (rows behind the last token's)
    if (head < a.nq + a.nkv) {
      float4 cs[D][4];
      auto request = [&](int j, float4 (&o)[4]) {
        const float2* tab = a.rope_tab + (u64)pos[j] * half + p0 + lg * 2;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = *(const float4*)(tab + i * 8);    // (cos, sin) of pairs p, p + 1
      };
#pragma unroll
      for (int j = 0; j < D; ++j) request(j, cs[j]);
      const float sc = 1.0f / sqrtf((float)hd);
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        if (t_base + j * 16 >= a.T) { wait_loads(); return; }
        const u32 t = t_base + j * 16 + lc;
        const float r = rstd[j * 16 + lc];
        u32 lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float lo0 = acc[i][j][0] * r, hi0 = acc[i][j][1] * r, lo1 = acc[i][j][2] * r, hi1 = acc[i][j][3] * r;
          const float4 w = cs[j % D][i];
          rotate(lo0, hi0, w.x, w.y);
          rotate(lo1, hi1, w.z, w.w);
          lo[i] = head < a.nq ? pack_f16x2(lo0 * sc, lo1 * sc) : pack_f16x2(lo0, lo1);
          hi[i] = head < a.nq ? pack_f16x2(hi0 * sc, hi1 * sc) : pack_f16x2(hi0, hi1);
        }
        if (j + D < TJ) request(j + D, cs[j % D]);
        transpose4(lo);                        // this lane: pairs p0 + lg * 8 .. + 7 of its token
        transpose4(hi);
        f16_t* out = a.qbuf + ((u64)t * a.nq + head) * hd;
        if (head >= a.nq) out = t < a.T ? cache_row(a.Kc, head - a.nq, j) + at[j] % a.bs * hd : spare;
        out += p0 + lg * 8;
        *(uint4*)out = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        *(uint4*)(out + half) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      }
    } else {                                   // V: dimension-major inside a block, [hd][16 tokens]
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        if (t_base + j * 16 >= a.T) return;
        const bool tv = t_base + j * 16 + lc < a.T;
        const float r = rstd[j * 16 + lc];
        f16_t* v = tv ? cache_row(a.Vc, head - a.nq - a.nkv, j) + at[j] % a.bs : spare;
        const u32 step = tv ? a.bs : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const u32 p = p0 + i * 8 + lg * 2;
          v[p * step] = f32_to_f16(acc[i][j][0] * r);
          v[(p + 1) * step] = f32_to_f16(acc[i][j][2] * r);
          v[(half + p) * step] = f32_to_f16(acc[i][j][1] * r);
          v[(half + p + 1) * step] = f32_to_f16(acc[i][j][3] * r);
        }
      }
    }
  }
}

// ---- stream schedule: T <= 64 ------------------------------------------------------------------------------------
// Weight loads bypass temporal caching: every weight byte is used once per launch, while the activation operand
// is re-read by every workgroup and should stay in L2.
__device__ __forceinline__ f16x8_t ld_op_stream(const f16_t* p) {
  typedef u32 u32x4_t __attribute__((ext_vector_type(4)));
  const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)p);
  return *(const f16x8_t*)&v;
}

// Work item of a workgroup in the round that starts at item `base`. Workgroups are dealt to the eight XCDs round-robin
// (workgroup id modulo 8), and each XCD has its own L2: the workgroups of one XCD take consecutive items, so that the
// operand blocks those items share are fetched into that L2 once. Returns ~0u when the round has no item for `wg`.
__device__ __forceinline__ u32 xcd_item(u32 base, u32 total, u32 wg, u32 nwg) {
  const u32 cnt = min(nwg, total - base);
  if (nwg & 7u) return wg < cnt ? base + wg : ~0u;
  const u32 q = (cnt + 7) / 8, x = wg & 7u, l = wg >> 3, off = x * q + l;
  return (l < q && off < cnt) ? base + off : ~0u;
}

template <int U, int NW, int TW>
struct StreamBuf {
  f16x8_t w[U][NW];
  f16x8_t x[U][TW];
};

// NW consecutive 16-row weight tiles per workgroup: every activation tile a wave loads is used for NW MFMAs, which
// divides the L2 traffic of the activation operand by NW (it is TW/NW times the weight bytes).
// k-tiles per batch of loads (two batches are in flight per wave). Measured on MI355X under the budget of 256 registers
// per lane (an eight-wave workgroup per compute unit): the widest variants keep fewer k-tiles per batch.
// GRID2D (64 < T <= 256, four token blocks per item): the work items are (tile group, group of 64 tokens) pairs, the
// token group varying fastest and the items of one round dealt to the XCDs in runs, so that the workgroups running
// together share weight rows in L2; the weight loads are ordinary (cached) ones then.
constexpr int stream_batch(int NW, int TW) {
  return NW == 1 ? (TW == 1 ? 8 : (TW == 2 ? 6 : 4))
       : ((NW * TW >= 8) ? 2 : (NW + TW >= 5 ? 3 : 4));
}
template <int EPI, int NW, int TW, int U = stream_batch(NW, TW), bool GRID2D = false, int THREADS = 512>
__device__ __forceinline__ void gemm_stream(const MfmaGemmArgs& a, MfmaShared& sh, u32 wg, u32 nwg) {
  const u32 lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const u32 NT = (a.N + 15) / 16, KT = gemm_k_tiles(a.K);
  const u32 TG = GRID2D ? (a.T + 63) / 64 : 1u;            // groups of 64 tokens
  const u32 NG = ((NT + NW - 1) / NW) * TG;                // work items: groups of NW tiles x token groups
  constexpr u32 KS = THREADS / 64;                         // waves of the workgroup: each takes a slice of K
  const u32 kb = (u32)((u64)KT * w / KS), ke = (u32)((u64)KT * (w + 1) / KS);
  const u32 nbatch = (KT / KS + (KT % KS ? 1 : 0) + U - 1) / U;   // same count in every wave (loads past `ke` are zeros)
  u32 round = 0;
  auto item_of = [&](u32 r) -> u32 {
    const u32 base = r * nwg;
    if (base >= NG) return ~0u;
    return GRID2D ? xcd_item(base, NG, wg, nwg) : (base + wg < NG ? base + wg : ~0u);
  };
  if (item_of(0) == ~0u) return;
  // per-lane offsets (in elements) of this lane's 16 bytes inside the token blocks of one k-tile
  u32 xoff[TW];
#pragma unroll
  for (int tw = 0; tw < TW; ++tw) {
    u32 tok = tw * 16 + (lane & 15);
    if (a.tok_index) tok = tok < a.T ? a.tok_index[tok] : 0;
    xoff[tw] = ((tok >> 4) * 64 + (tok & 15) + 16 * (lane >> 4)) * 8;
  }
  const u64 xk_stride = (u64)a.TBS * 512;
  const f16x8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
  auto issue = [&](StreamBuf<U, NW, TW>& b, u32 item, u32 kt0) {
    const u32 ng = item / TG;
    const bf16_t* xg = a.Xp + (u64)(item % TG) * (TW * 512);   // the item's token group: TW consecutive token blocks
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u32 kt = kt0 + u;
      const bool ok = kt < ke;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const u32 nt = min(ng * NW + i, NT - 1);           // a tile past the end is computed and dropped
        const bf16_t* wp = a.Wp + ((u64)nt * KT + kt) * 512 + lane * 8;
        b.w[u][i] = ok ? (GRID2D ? ld_op(wp) : ld_op_stream(wp)) : zero;
      }
#pragma unroll
      for (int tw = 0; tw < TW; ++tw) b.x[u][tw] = ok ? ld_op(xg + (u64)kt * xk_stride + xoff[tw]) : zero;
    }
  };
  // Software pipeline over the flat sequence of (tile group, batch) steps of this workgroup: while one buffer is
  // consumed by the MFMAs, the loads of the following step (possibly the first batch of the next group) fill the
  // other. The two buffers swap roles by code position (no register copies, which would wait for loads in flight).
  StreamBuf<U, NW, TW> bufA, bufB;
  u32 ng = item_of(0), b = 0;
  floatx4_t acc[NW][TW];
#pragma unroll
  for (int i = 0; i < NW; ++i)
#pragma unroll
    for (int tw = 0; tw < TW; ++tw) acc[i][tw] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  issue(bufA, ng, kb);               // the first loads are in flight while the norm scales are computed
  if constexpr (!GRID2D) compute_rstd<TW * 16, THREADS>(a, 0, sh.rstd);
  else if (TG <= 2) compute_rstd<128, THREADS>(a, 0, sh.rstd);
  else compute_rstd<256, THREADS>(a, 0, sh.rstd);
  auto step = [&](StreamBuf<U, NW, TW>& use, StreamBuf<U, NW, TW>& fill) -> bool {
    const bool last = b + 1 >= nbatch;
    const u32 nng = last ? item_of(round + 1) : ng;
    if (nng < NG) issue(fill, nng, last ? kb : kb + (b + 1) * U);
    {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
          for (int tw = 0; tw < TW; ++tw)
            acc[i][tw] = __builtin_amdgcn_mfma_f32_16x16x32_f16(use.w[u][i], use.x[u][tw], acc[i][tw], 0, 0, 0);
    }
    if (!last) { ++b; return true; }
    // the residual values and gains the epilogue of this wave's tiles will need: requested before the reduction, not behind it
    float4 pre_old[NW], pre_g[NW];
    if (EPI == EPI_RESIDUAL && w < TW && !(a.tune_nw & 0x40u)) {
      const u32 tq = min((ng % TG) * 64 + w * 16 + (lane & 15), a.T - 1);
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const u32 n0 = min((ng / TG) * NW + i, NT - 1) * 16 + (lane >> 4) * 4;
        pre_old[i] = *(const float4*)(a.x + (u64)tq * a.ldx + n0);
        pre_g[i] = *(const float4*)(a.g_next + n0);
      }
    }
    float4 pre_cs[NW];
    u32 pre_slot = 0;
    if (EPI == EPI_QKV_ROPE && w < TW && !(a.tune_nw & 0x40u)) {     // likewise the position, the cache slot and the rotary table entries
      const u32 tq = min((ng % TG) * 64 + w * 16 + (lane & 15), a.T - 1), half = a.hd / 2;
      const u32 pos = (u32)a.positions[tq];
      pre_slot = (u32)a.slot_mapping[tq];
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const u32 n0 = min((ng / TG) * NW + i, NT - 1) * 16 + (lane >> 4) * 4;
        const bool rot = n0 / a.hd < a.nq + a.nkv;
        pre_cs[i] = *(const float4*)(a.rope_tab + (u64)(rot ? pos : 0u) * half + (rot ? (n0 % a.hd) >> 1 : 0u));
      }
    }
    // reduce the waves' shares of K through LDS, one weight tile of the group at a time
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      __syncthreads();   // the previous reduction has been read
#pragma unroll
      for (int tw = 0; tw < TW; ++tw) *(floatx4_t*)&sh.red[w][tw][lane][0] = acc[i][tw];
      __syncthreads();
      const u32 nt = (ng / TG) * NW + i, tg = ng % TG;
      if (w < TW && nt < NT) {               // wave w finishes token block w: fixed summation order
        floatx4_t s = (*(floatx4_t*)&sh.red[0][w][lane][0] + *(floatx4_t*)&sh.red[1][w][lane][0]) +
                      (*(floatx4_t*)&sh.red[2][w][lane][0] + *(floatx4_t*)&sh.red[3][w][lane][0]);
        if (KS == 8)
          s += (*(floatx4_t*)&sh.red[4][w][lane][0] + *(floatx4_t*)&sh.red[5][w][lane][0]) +
               (*(floatx4_t*)&sh.red[6][w][lane][0] + *(floatx4_t*)&sh.red[7][w][lane][0]);
        if (EPI == EPI_RESIDUAL && !(a.tune_nw & 0x40u)) residual_finish(a, s, nt, tg * 64 + w * 16 + (lane & 15), pre_old[i], pre_g[i]);
        else if (EPI == EPI_QKV_ROPE && !(a.tune_nw & 0x40u))
          rope_finish(a, s, nt, tg * 64 + w * 16 + (lane & 15), sh.rstd[tg * 64 + w * 16 + (lane & 15)], pre_slot, pre_cs[i]);
        else epilogue_tile<EPI>(a, s, nt, tg * 64 + w * 16, &sh.rstd[tg * 64 + w * 16]);
      }
#pragma unroll
      for (int tw = 0; tw < TW; ++tw) acc[i][tw] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    }
    ng = nng;
    b = 0;
    ++round;
    return ng < NG;
  };
  for (;;) {
    if (!step(bufA, bufB)) break;
    if (!step(bufB, bufA)) break;
  }
}

// Tile order of the tile schedule: token blocks in groups of eight; inside a group the row blocks follow each other and
// the token block varies fastest, so 64 consecutive tiles are 8 row blocks x 8 token blocks (16 operand blocks in all).
__device__ __forceinline__ void tile_coords(u32 i, u32 nblocks, u32 tblocks, u32& nb, u32& tb) {
  const u32 gsz = nblocks * 8, g = min(i / gsz, tblocks / 8), rem = i - g * gsz;
  const u32 width = min(8u, tblocks - g * 8);
  nb = rem / width;
  tb = g * 8 + rem % width;
}

template <int EPI, int TW>
__device__ __forceinline__ void gemm_stream_nw(const MfmaGemmArgs& a, MfmaShared& sh, u32 wg, u32 nwg) {
  const u32 NT = (a.N + 15) / 16, forced = a.tune_nw & 0x07u;
  // two weight tiles per workgroup halve the re-reads of the activations, and pay off once there are row tiles enough for the
  // chip all the same: from 320 row tiles (the QKV projection of the llama3_8b shape has 384)
  if (forced == 1 || (forced != 2 && NT < 320)) gemm_stream<EPI, 1, TW>(a, sh, wg, nwg);
  else gemm_stream<EPI, 2, TW>(a, sh, wg, nwg);
}

// ---- router of a mixture-of-experts model (four waves per workgroup) ---------------------------------------------------
// T <= 256: the streaming schedule with K in four slices (its order of the sums decides near-ties between experts: see
// gemm_plan). Beyond: independent waves, each with one row tile, 32 tokens and the whole of K in order, two batches of
// loads in flight (128 x 2048 at 2100 tokens: 528 wave items).
template <int EPI>
__device__ __forceinline__ void gemm_router(const MfmaGemmArgs& a, MfmaShared& sh, u32 wg, u32 nwg) {
  if (a.T == 0) return;
  if (a.T <= 16) gemm_stream<EPI, 1, 1, stream_batch(1, 1), false, BLK_THREADS>(a, sh, wg, nwg);
  else if (a.T <= 32) gemm_stream<EPI, 1, 2, stream_batch(1, 2), false, BLK_THREADS>(a, sh, wg, nwg);
  else if (a.T <= 48) gemm_stream<EPI, 1, 3, stream_batch(1, 3), false, BLK_THREADS>(a, sh, wg, nwg);
  else if (a.T <= 64) gemm_stream<EPI, 1, 4, stream_batch(1, 4), false, BLK_THREADS>(a, sh, wg, nwg);
  else if (a.T <= 256) gemm_stream<EPI, 1, 4, stream_batch(1, 4), true, BLK_THREADS>(a, sh, wg, nwg);
  else {
    const u32 lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const u32 NT = (a.N + 15) / 16, KT = gemm_k_tiles(a.K), TB = (a.T + 31) / 32, items = NT * TB;
    constexpr int U = 4;
    for (u32 base = wg * nw; base < items; base += nwg * nw) {     // the waves of a workgroup: neighbouring row tiles, the same tokens
      const u32 item = base + w, nt = min(item, items - 1) % NT, tb = min(item, items - 1) / NT;
      // (the four items lie in at most two, or four, blocks of tokens)
      if (NT >= 4) compute_rstd<64, BLK_THREADS>(a, (base / NT) * 32, sh.rstd);
      else compute_rstd<128, BLK_THREADS>(a, (base / NT) * 32, sh.rstd);
      const f16_t* wp = a.Wp + (u64)nt * KT * 512 + lane * 8;
      const f16_t* xp = a.Xp + (u64)tb * 1024 + lane * 8;
      const u64 xk = (u64)a.TBS * 512;
      struct Buf { f16x8_t w[U], x[U][2]; } A, B;
      floatx4_t acc[2] = {floatx4_t{0.f, 0.f, 0.f, 0.f}, floatx4_t{0.f, 0.f, 0.f, 0.f}};
      auto issue = [&](Buf& b, u32 k0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const u32 kt = min(k0 + u, KT - 1);
          b.w[u] = ld_op(wp + (u64)kt * 512); b.x[u][0] = ld_op(xp + kt * xk); b.x[u][1] = ld_op(xp + kt * xk + 512);
        }
      };
      auto mm = [&](const Buf& b, u32 k0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (k0 + u < KT) {
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b.w[u], b.x[u][0], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b.w[u], b.x[u][1], acc[1], 0, 0, 0);
          }
      };
      issue(A, 0);
      for (u32 k = 0; k < KT; k += 2 * U) { issue(B, k + U); mm(A, k); issue(A, k + 2 * U); mm(B, k + U); }
      if (item < items) {
        const float* r = sh.rstd + (tb - base / NT) * 32;
        epilogue_tile<EPI>(a, acc[0], nt, tb * 32, r);
        epilogue_tile<EPI>(a, acc[1], nt, tb * 32 + 16, r + 16);
      }
    }
  }
}

// ---- packing -----------------------------------------------------------------------------------------------------
// Weights [N][K] row-major bf16 -> packed tiles of half precision, scaled by W_SCALE. pair_rows > 0: the source holds
// `pair_rows` gate rows followed by `pair_rows` up rows, and packed row 2j is gate_j, row 2j+1 is up_j. perm_hd > 0:
// rows are heads of perm_hd dimensions each, re-ordered so that the two dimensions a rotary embedding pairs up are
// adjacent rows.
__device__ __forceinline__ void pack_weights(const bf16_t* src, f16_t* dst, u32 N, u32 K, u32 pair_rows, u32 perm_hd, u64 gtid,
                                             u64 gthreads) {
  const u32 NT = (N + 15) / 16, KT = gemm_k_tiles(K);
  const u64 chunks = (u64)NT * KT * 64;
  for (u64 i = gtid; i < chunks; i += gthreads) {
    const u32 lane = (u32)(i & 63);
    const u64 tile = i >> 6;
    const u32 kt = (u32)(tile % KT), nt = (u32)(tile / KT);
    const u32 n = nt * 16 + (lane & 15), k = kt * 32 + (lane >> 4) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N && k < K) {
      u32 row = pair_rows ? ((n & 1) ? pair_rows + (n >> 1) : (n >> 1)) : n;
      if (perm_hd) {   // packed row 2p of a head is its dimension p, row 2p+1 its dimension p + hd/2
        const u32 pi = n % perm_hd;
        row = n - pi + ((pi & 1) ? perm_hd / 2 + (pi >> 1) : (pi >> 1));
      }
      const uint4 b = *(const uint4*)(src + (u64)row * K + k);
      const u32 w[4] = {b.x, b.y, b.z, b.w};
      u32 o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        o[j] = pack_f16x2(__uint_as_float(w[j] << 16) * W_SCALE, __uint_as_float(w[j] & 0xFFFF0000u) * W_SCALE);
      v = make_uint4(o[0], o[1], o[2], o[3]);
    }
    *(uint4*)(dst + i * 8) = v;
  }
}
