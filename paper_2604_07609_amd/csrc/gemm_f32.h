// GEMMs of an fp32 model on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 products and sums), with the RMSNorm of the
// input, the SiLU gate, the residual add and the rotary embedding + KV write fused in. out[t][n] = sum_k a(t, k) * W[n][k].
//
// The fp32 workloads are small models at small batches, so what bounds a launch is its chain of dependent steps, not
// bytes or arithmetic: the LDS-tiled FMA kernels this replaces gave a 32 x 64 output tile to a workgroup and walked all
// of K behind two barriers per 32 of it (256 x 1024 weights at 8 tokens: four workgroups, 62 us), and each norm and the
// rotary step was a launch of its own (5 us each). Here the operands come straight from memory into registers, 16 bytes
// per lane: lane l holds row (or token) l % 16 and k = 4 (l / 16) .. + 3 of sixteen k, and the four matrix instructions of the
// sixteen take element 0, 1, 2, 3 of both (the order of k inside a sum is free as long as both operands agree). Two schedules:
//   few tiles: a workgroup per (row tile, 16 tokens), K in a slice per wave, partial sums joined through LDS. Four waves, and
//     eight in the down projection, whose K is the FFN's width (256 x 1024 at 8 tokens 6.5 us, 6.7 with sixteen; 1024 x 4096 at 1 / 16 /
//     64 / 200 tokens 15 / 21 / 21 / 66 us, with four 25 / 30 / 31 / 97; the others, whose loads are one batch per wave
//     already, take 1 to 2 us longer with eight);
//   many tiles (more than four per compute unit): a wave per 32 rows x 32 tokens with the whole of K.
// The gate is applied once, where gate and up are computed (as the down projection's operand it was computed anew for every row
// tile: 256 x 1024 at 8 tokens, with K in four slices, 10.2 us).
// The norm: its gain multiplies the operand as it is loaded, its scale (one number per token) the finished sum; the
// squares are summed on the way.
#pragma once
#include "blink_device.h"
#include "mfma_gemm.h"

#define FA_PLAIN 0
#define FA_NORM 1       // a(t,k) = x[t][k] * gain[k], the sum scaled by 1 / rms(x[t])
#define FE_STORE 0
#define FE_ADD 1        // out += result (residual connection, in place)
#define FE_ROPE 2       // rotary embedding; q to out, k and v into the paged cache
#define FE_GATE 3       // rows are N/2 gates, then N/2 ups: out[t][j] = silu(gate j) * up j
#define F32_WAVES 4        // waves per workgroup
#define F32_DOWN_WAVES 8   // ... in the down projection

struct F32GemmArgs {
  const float* A; u32 lda;
  const u32* rows;       // optional: row t of the product reads row rows[t] of A
  const float* gain; float eps;
  const float* W;
  float* out; u32 ldo;
  u32 T, N, K;
  // FE_ROPE
  const i32* positions;
  const i32* slot_mapping;
  const float2* rope_tab;
  float *Kc, *Vc;        // this layer's K and V cache: [block][kv head][bs][hd]
  u32 nq, nkv, hd, bs;
};

template <int WAVES>
struct F32GemmShared {
  float red[WAVES][2][64][4];       // [wave][row tile][lane][4]
  float ss[WAVES][16];              // [wave][token]
};

// Row tiles of 16 come in groups: for FE_ROPE the two tiles whose rows pair up in the rotary embedding (half a head apart), for
// FE_GATE a tile of gates and the tile of their ups.
template <int EMODE>
__device__ __forceinline__ u32 f32_row(const F32GemmArgs& a, u32 group, u32 tile, u32 per_group) {
  if (EMODE == FE_GATE) return group * 16 + tile * (a.N / 2);
  if (EMODE != FE_ROPE) return (group * per_group + tile) * 16;
  const u32 half = a.hd / 2, per_head = half / 16;
  return (group / per_head) * a.hd + (group % per_head) * 16 + tile * half;
}

// rows row .. row + 3 (and, FE_ROPE, row + hd/2 ..) of token t: this lane's sums, scaled
template <int EMODE>
__device__ __forceinline__ void f32_store(const F32GemmArgs& a, u32 row, u32 t, float4 v) {
  float* o = a.out + (u64)t * a.ldo + row;
  if (row + 3 < a.N && (a.ldo & 3u) == 0) {
    if (EMODE == FE_ADD) { const float4 old = *(const float4*)o; v = make_float4(old.x + v.x, old.y + v.y, old.z + v.z, old.w + v.w); }
    *(float4*)o = v;
  } else {
    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (row + i < a.N) o[i] = EMODE == FE_ADD ? o[i] + e[i] : e[i];
  }
}
__device__ __forceinline__ void f32_store_gate(const F32GemmArgs& a, u32 row, u32 t, float4 g, float4 u) {
  *(float4*)(a.out + (u64)t * a.ldo + row) = make_float4(g.x / (1.f + __expf(-g.x)) * u.x, g.y / (1.f + __expf(-g.y)) * u.y,
                                                         g.z / (1.f + __expf(-g.z)) * u.z, g.w / (1.f + __expf(-g.w)) * u.w);
}
__device__ __forceinline__ void f32_store_rope(const F32GemmArgs& a, u32 row, u32 t, float4 lo, float4 hi) {
  const u32 half = a.hd / 2, head = row / a.hd, p = row % a.hd;
  if (head < a.nq + a.nkv) {
    const float4* cs = (const float4*)(a.rope_tab + (u64)a.positions[t] * half + p);   // (cos, sin) of pairs p .. p + 3
    const float4 c0 = cs[0], c1 = cs[1];
    const float4 l = lo, h = hi;
    lo = make_float4(l.x * c0.x - h.x * c0.y, l.y * c0.z - h.y * c0.w, l.z * c1.x - h.z * c1.y, l.w * c1.z - h.w * c1.w);
    hi = make_float4(h.x * c0.x + l.x * c0.y, h.y * c0.z + l.y * c0.w, h.z * c1.x + l.z * c1.y, h.w * c1.z + l.w * c1.w);
  }
  float* o;
  if (head < a.nq) o = a.out + (u64)t * a.ldo + row;
  else {
    const u32 slot = (u32)a.slot_mapping[t], kv = head - a.nq, g = kv < a.nkv ? kv : kv - a.nkv;
    o = (kv < a.nkv ? a.Kc : a.Vc) + (((u64)(slot / a.bs) * a.nkv + g) * a.bs + slot % a.bs) * a.hd + p;
  }
  *(float4*)o = lo;
  *(float4*)(o + half) = hi;
}

// One sixteen of k of the operands in flight: RT row tiles, TT token tiles.
template <int AMODE, int RT, int TT>
struct F32Chunk {
  float4 w[RT], x[TT], g;
};
template <int AMODE, int RT, int TT>
__device__ __forceinline__ void f32_load(const F32GemmArgs& a, const float* const (&wp)[RT], const float* const (&xp)[TT], u32 k, F32Chunk<AMODE, RT, TT>& c) {
#pragma unroll
  for (int i = 0; i < RT; ++i) c.w[i] = *(const float4*)(wp[i] + k);
#pragma unroll
  for (int j = 0; j < TT; ++j) c.x[j] = *(const float4*)(xp[j] + k);
  if (AMODE == FA_NORM) c.g = *(const float4*)(a.gain + k + 4 * ((threadIdx.x & 63) >> 4));
}
template <int AMODE, int RT, int TT>
__device__ __forceinline__ void f32_mul(const F32Chunk<AMODE, RT, TT>& c, floatx4_t (&acc)[RT][TT], float (&ss)[TT]) {
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    float x[4] = {c.x[j].x, c.x[j].y, c.x[j].z, c.x[j].w};
    if (AMODE == FA_NORM) {
      const float g[4] = {c.g.x, c.g.y, c.g.z, c.g.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) { ss[j] += x[i] * x[i]; x[i] *= g[i]; }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const float w[4] = {c.w[r].x, c.w[r].y, c.w[r].z, c.w[r].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], x[i], acc[r][j], 0, 0, 0);
    }
  }
}

// Sixteens of k from kb to ke (in units of 16), two batches of U in flight; sums into acc, squares into ss.
template <int AMODE, int RT, int TT, int U>
__device__ __forceinline__ void f32_run(const F32GemmArgs& a, const float* const (&wp)[RT], const float* const (&xp)[TT], u32 kb, u32 ke,
                                        floatx4_t (&acc)[RT][TT], float (&ss)[TT]) {
  if (kb >= ke) return;
  typedef F32Chunk<AMODE, RT, TT> Chunk;
  Chunk A[U], B[U];
  auto load = [&](Chunk (&c)[U], u32 k) {
#pragma unroll
    for (int u = 0; u < U; ++u) f32_load<AMODE, RT, TT>(a, wp, xp, min(k + u, ke - 1) * 16, c[u]);   // (past the end: the last one again, not used)
  };
  auto mul = [&](const Chunk (&c)[U], u32 k) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u < ke) f32_mul<AMODE, RT, TT>(c[u], acc, ss);
  };
  load(A, kb);
  for (u32 k = kb; k < ke; k += 2 * U) {
    if (k + U < ke) load(B, k + U);
    mul(A, k);
    if (k + 2 * U < ke) load(A, k + 2 * U);
    mul(B, k + U);
  }
}

// the sum of v[0 .. N), in a fixed order, by halves
template <int N, typename T>
__device__ __forceinline__ T tree_sum(const T* v) {
  if constexpr (N == 1) return v[0];
  else return tree_sum<N / 2>(v) + tree_sum<N / 2>(v + N / 2);
}

template <int AMODE, int EMODE, int WAVES>
__device__ __forceinline__ void gemm_f32(const F32GemmArgs& a, F32GemmShared<WAVES>& sh, u32 wg, u32 nwg) {
  if (a.T == 0) return;
  const u32 lane = threadIdx.x & 63, w = threadIdx.x >> 6, lc = lane & 15, lg = lane >> 4;
  const u32 NT = (a.N + 15) / 16, TB = (a.T + 15) / 16, KQ = a.K / 16;
  auto w_ptr = [&](u32 row) { return a.W + (u64)min(row + lc, a.N - 1) * a.K + 4 * lg; };        // (rows and tokens past the end
  auto x_ptr = [&](u32 t) { const u32 r = min(t + lc, a.T - 1); return a.A + (u64)(a.rows ? a.rows[r] : r) * a.lda + 4 * lg; };   // repeat the last one)
  auto scale = [&](float ss) { return 1.0f / sqrtf(ss / (float)a.K + a.eps); };
  if (NT * TB > nwg * WAVES / 2) {         // (eight waves per compute unit in either launch: 1024 tiles on 256 of them)
    constexpr u32 nw = WAVES;
    const u32 RG = (NT + 1) / 2, TG = (TB + 1) / 2;
    // four neighbouring items per workgroup, of eight waves the other four as many workgroups further on: eight neighbours would leave half
    // of them idle where there are few (1024 x 4096 at 509 tokens: 64 compute units busy, 246 us, and 117 like this)
    for (u32 item = (wg + w / F32_WAVES * nwg) * F32_WAVES + w % F32_WAVES; item < RG * TG; item += nwg * nw) {
      const u32 rg = item / TG, t0 = (item % TG) * 32;
      const u32 row[2] = {f32_row<EMODE>(a, rg, 0, 2), f32_row<EMODE>(a, rg, 1, 2)};
      const float* const wp[2] = {w_ptr(row[0]), w_ptr(row[1])};
      const float* const xp[2] = {x_ptr(t0), x_ptr(t0 + 16)};
      floatx4_t acc[2][2];
      float ss[2] = {0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[r][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      f32_run<AMODE, 2, 2, 2>(a, wp, xp, 0, KQ, acc, ss);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u32 t = t0 + j * 16 + lc;
        float r = 1.f;
        if (AMODE == FA_NORM) {
          float s = ss[j];
          s += __shfl_xor(s, 16); s += __shfl_xor(s, 32);
          r = scale(s);
        }
        if (t < a.T) {
          float4 v[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) v[i] = make_float4(acc[i][j][0] * r, acc[i][j][1] * r, acc[i][j][2] * r, acc[i][j][3] * r);
          if (EMODE == FE_ROPE) f32_store_rope(a, row[0] + 4 * lg, t, v[0], v[1]);
          else if (EMODE == FE_GATE) f32_store_gate(a, row[0] + 4 * lg, t, v[0], v[1]);
          else {
#pragma unroll
            for (int i = 0; i < 2; ++i) f32_store<EMODE>(a, row[i] + 4 * lg, t, v[i]);
          }
        }
      }
    }
    return;
  }
  constexpr int RT = EMODE == FE_ROPE || EMODE == FE_GATE ? 2 : 1;
  const u32 RG = NT / RT;                         // (the QKV projection has whole heads, gate/up whole pairs of tiles)
  const u32 kb = KQ * w / WAVES, ke = KQ * (w + 1) / WAVES;
  for (u32 item = wg; item < RG * TB; item += nwg) {
    const u32 rg = item / TB, t0 = (item % TB) * 16;
    u32 row[RT];
    const float* wp[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) { row[r] = f32_row<EMODE>(a, rg, r, RT); wp[r] = w_ptr(row[r]); }
    const float* const xp[1] = {x_ptr(t0)};
    floatx4_t acc[RT][1];
    float ss[1] = {0.f};
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r][0] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    const float* const (&wpc)[RT] = wp;
    f32_run<AMODE, RT, 1, 4>(a, wpc, xp, kb, ke, acc, ss);
    __syncthreads();                              // the previous item's partial sums have been read
#pragma unroll
    for (int r = 0; r < RT; ++r) *(floatx4_t*)&sh.red[w][r][lane][0] = acc[r][0];
    if (AMODE == FA_NORM) {
      float s = ss[0];
      s += __shfl_xor(s, 16); s += __shfl_xor(s, 32);
      if (lane < 16) sh.ss[w][lane] = s;
    }
    __syncthreads();
    const u32 t = t0 + lc;
    if (w == 0 && t < a.T) {
      float r = 1.f;
      if (AMODE == FA_NORM) {
        float p[WAVES];
#pragma unroll
        for (int k = 0; k < WAVES; ++k) p[k] = sh.ss[k][lc];
        r = scale(tree_sum<WAVES>(p));
      }
      float4 v[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        floatx4_t p[WAVES];
#pragma unroll
        for (int k = 0; k < WAVES; ++k) p[k] = *(floatx4_t*)&sh.red[k][i][lane][0];
        const floatx4_t s = tree_sum<WAVES>(p);
        v[i] = make_float4(s[0] * r, s[1] * r, s[2] * r, s[3] * r);
      }
      if (EMODE == FE_ROPE) f32_store_rope(a, row[0] + 4 * lg, t, v[0], v[RT - 1]);
      else if (EMODE == FE_GATE) f32_store_gate(a, row[0] + 4 * lg, t, v[0], v[RT - 1]);
      else f32_store<EMODE>(a, row[0] + 4 * lg, t, v[0]);
    }
  }
}
