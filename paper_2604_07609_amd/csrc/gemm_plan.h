// Which schedule each GEMM of a bf16 model takes: its epilogues, the workgroup tiles with their costs, and the table of schedules by token
// count. Plain C++ on unsigned words (u32), without a GPU.
#pragma once
#include <cmath>
#include <vector>

#define EPI_SCALED_STORE 0   // out[t][n] = rstd[t] * acc                      (QKV projection, LM head)
#define EPI_RESIDUAL 1       // x[t][n] += acc; emit packed half(x * g_next) and sum-of-squares partials
#define EPI_SILU_GATE 2      // rows interleaved (gate_j, up_j): emit packed half(silu(r*g) * (r*u))
#define EPI_QKV_ROPE 3       // rows of every head interleaved (dim p, dim p+hd/2): rotary embedding, then q to the query
                             // buffer, k and v straight into the paged cache through the slot mapping

constexpr u32 gemm_k_tiles(u32 K) { return ((K + 63) / 64) * 2; }   // k-steps of the packed operands

// ---- choice of the workgroup tile -----------------------------------------------------------------------------------
// Time of a launch with tiles of one shape, in microseconds (without the launch itself), from the number of rounds of workgroups: a
// k-step takes `lone` while few compute units are busy and `full` with all of them (shared L2s and the clock under load), and an
// item's first operands, norm scales and epilogue take `fixed` alone and `fixed_full` with all of them at it. With one workgroup per
// compute unit nothing runs beside an epilogue, and what it costs depends on what follows the GEMM: a 256 x 256 tile on 128 k-steps
// takes 108 us with the rotary embedding and KV write, 131 with the residual add, 98 with the gate. So the epilogues have
// constants of their own, fitted to launches with every shape forced of 1 to 6 matrices each (1024 to 28672 rows, k 1024 to 14336, weights
// from HBM) at 65 to 8000 tokens. The fits are within 5 to 13 % (rms) of them, and the shape they choose takes at most 5 % more
// than the best, 0.1 % on average.
constexpr float dma_cost(u32 total, u32 K, float lone, float full, float fixed, float fixed_full, u32 ncu) {
  const u32 rounds = total / ncu, rest = total % ncu;
  const float f = (float)rest / (float)ncu, kt = (float)(K / 32);
  return (float)rounds * (kt * full + fixed_full) +
         (rest ? kt * (lone + (full - lone) * f * f * f * f) + fixed + (fixed_full - fixed) * f * f : 0.f);
}

// The shapes: number, rows x tokens of the workgroup tile, constants of a k-step, then of an item: store or gate, residual add, rotary embedding.
#define DMA_SHAPES(X) X(1, 64, 64, .123f, .108f, 6.9f, .7f, 2.2f, 2.0f, 5.8f, 2.2f) X(2, 128, 64, .200f, .179f, 3.2f, .6f, 1.7f, 2.4f, 4.5f, 2.1f) \
                      X(3, 128, 128, .227f, .243f, 3.6f, 1.6f, 2.9f, 5.7f, 6.0f, 3.7f) X(4, 256, 128, .358f, .386f, 5.1f, 4.9f, 7.2f, 15.7f, 8.6f, 8.3f) \
                      X(6, 256, 192, .419f, .544f, 9.7f, 7.8f, 12.7f, 26.2f, 14.2f, 14.7f) X(7, 256, 256, .513f, .690f, 11.6f, 10.6f, 16.7f, 39.0f, 16.2f, 20.5f)

// ---- the schedule of every GEMM --------------------------------------------------------------------------------------
// It depends on the matrix and the number of tokens alone, so the library tabulates it when an engine is made, the
// scheduler step copies the entry of its iteration into the metadata that the kernels read anyway, and a launch begins with its
// operands: weighing six shapes in every workgroup took 1.5 us of a launch.
#define PLAN_STREAM 0u           // streaming schedule
#define PLAN_TALL 5u             // all tokens (at most 64) in one tile of 128 rows
#define PLAN_CODE(shape, slices) ((shape) | (slices) << 3)       // 1-4, 6, 7: workgroup tile of that number; slices of K (0: whole)
struct GemmPlan { unsigned char qkv, oproj, gateup, down, lm_head, pad[3]; };

constexpr u32 dma_tiles(u32 N, u32 T, u32 bn, u32 bt) { return (N + bn - 1) / bn * ((T + bt - 1) / bt); }
// The entry of a matrix of N rows, inner dimension K, at T tokens. `ordered`: a mixture-of-experts model's GEMM ahead of the router.
//   T <= 64: a matrix tall enough that its 128-row items occupy three quarters of the compute units goes through LDS with all
//     tokens in one tile: each workgroup streams whole rows, no reduction over slices of K at the end, and the ring keeps 100 KB and
//     more of weights on their way per compute unit (28672 x 4096 from HBM at 61 / 16 tokens: 46 / 42 us = 5.1 / 5.6 TB/s with loads that
//     bypass temporal caching, 49 / 46 us without; streamed through registers with K split over the four waves of a workgroup 61 / 43 us). Narrower matrices would leave compute units idle
//     and stay with the streaming schedule (4096 x 14336 at 16 tokens: 27 us against 47).
//   T > 64: the tile whose rounds take the least time.
//   64 < T <= 256 ahead of the router of a mixture-of-experts model (ordered): the streaming schedule over a grid of 64 x 64 items,
//     where the matrix has few enough of them. A decode iteration's sums are then taken in the order in which they have
//     been taken all along (K in eight slices): in another order they round otherwise, and tokens with two nearly equal router
//     logits go to another expert. The tiles would win 1 % of a decode iteration at 96 sequences of the moe_30b_a3b shape.
//   K in slices (QKV, attention output and down projections; not where the order of the sums is kept): where a matrix has too few tiles for
//     the chip, its tiles are cut along K, two to eight slices each, at most one per compute unit. Half the chip then doesn't stand
//     idle at 300 to 700 tokens, and at 17 to 256 larger tiles read the activations fewer times (the streaming schedule reads all of
//     them in every workgroup). Both sides in us: 4096 x 14336 at 33 / 61 / 128 / 256 / 300 / 509 tokens 39 / 45 / 68 / 69 / 103 / 107 whole
//     and 31 / 32 / 45 / 56 / 68 / 82 in slices, 4096 x 4096 at 128 / 300 tokens 26 / 37 and 22 / 31, 6144 x 4096 at 192 39 and 34, 1024 x 4096 at
//     256 20 and 16. The last workgroup's reading and adding take 4 us and more, so 4096 x 4096 stays whole up to 48 tokens (16 us) and takes
//     18 either way at 61.
//     The model is within 11 % (rms) of launches with both forced, and its choice 0.7 % from the best of them on average.
static inline unsigned char gemm_plan(int epi, u32 N, u32 K, u32 T, bool ordered, u32 ncu, u32 tune) {
  const u32 shape = (tune >> 12) & 7u, slices = (tune >> 24) & 15u;       // forced
  const bool split = !ordered && (epi == EPI_RESIDUAL || epi == EPI_QKV_ROPE), streams = T <= 64 && !(slices > 1 && shape);
  float least = INFINITY;
  u32 best = shape == 5 ? 0 : shape;
  if (T > 64 && ordered && T <= 256 && !shape && dma_tiles(N, T, 128, 128) * 4 <= ncu) return PLAN_STREAM;
  // (not where bits 0-2 or 11 of the tuning word ask for streaming)
  if (streams && dma_tiles(N, T, 128, 64) * 4 >= ncu * 3 && !(tune & 0x807u)) return PLAN_TALL;
  const float weights_us = (float)N * (float)K * 2.f / 5.6e6f;            // at the rate they come from HBM
  if (streams) {
    if (T <= 16 || !split || (tune & 0x7807u)) return PLAN_STREAM;
    // time of the streaming schedule: the weights, or what a workgroup loads
    const u32 tiles = (N + 15) / 16, nw = tiles < 320 ? 1 : 2, groups = (tiles + nw - 1) / nw, tb = (T + 15) / 16;
    const float loads = (float)((groups + ncu - 1) / ncu) * (float)K / 2048.f * (2.39f * (float)nw + .70f * (float)tb);
    least = (weights_us > loads ? weights_us : loads) + .4f + .7f * (float)tb;
    best = PLAN_STREAM;
  }
#define OFFER(id, bn, bt, lone, full, store, store_full, residual, residual_full, rope, rope_full) {                                  \
    const float fixed = epi == EPI_QKV_ROPE ? rope : epi == EPI_RESIDUAL ? residual : store;                                          \
    const float fixed_full = epi == EPI_QKV_ROPE ? rope_full : epi == EPI_RESIDUAL ? residual_full : store_full;                      \
    const u32 tiles = dma_tiles(N, T, bn, bt);                                                                                        \
    if (T > 64 && !shape) {                                                                                                           \
      const float t = dma_cost(tiles, K, lone, full, fixed, fixed_full, ncu);                                                         \
      if (t < least) { least = t; best = id; }                                                                                        \
    }                                                                                                                                 \
    if (split && id <= 4 && (T > 64 || (id <= 2 && (id == 1 || T > 32))) && !shape)                                                   \
      for (u32 s = 2; s <= 8 && tiles * s <= ncu && s * 2 <= gemm_k_tiles(K); ++s) {                                                  \
        const float f = (float)(tiles * s) / (float)ncu, fe = (float)tiles / (float)ncu, k_steps = ceilf((float)K / 64.f / (float)s) * 2.f; \
        const float work = k_steps * (lone + (full - lone) * f * f * f * f), bytes = weights_us / sqrtf(f);                           \
        const float t = 1.03f * ((work > bytes ? work : bytes) + fixed + (fixed_full - fixed) * fe * fe + 4.1f + .226f * (float)(s * bn * bt) / 4096.f); \
        if (t < least) { least = t; best = PLAN_CODE(id, s); }                                                                        \
      }                                                                                                                               \
    if (split && shape == id && id <= 4 && slices > 1 && slices * 2 <= gemm_k_tiles(K) && tiles * slices <= ncu) best = PLAN_CODE(id, slices); }
  DMA_SHAPES(OFFER)
#undef OFFER
  return (unsigned char)(best == 0 && T > 64 ? 1u : best);
}

// The table: an entry per token count up to 64 and one per 64 tokens beyond (every tile is a multiple of 64 tokens wide), for as many tokens
// as an iteration can have. No entry serves any other count: K in slices holds only while there is at most one item per compute unit.
constexpr u32 gemm_plan_entry(u32 T) { return T <= 64 ? T : 64 + (T - 1) / 64; }
static inline std::vector<GemmPlan> gemm_plan_table(u32 max_tokens, u32 qkv_rows, u32 d, u32 q_width, u32 F, u32 V, bool experts, u32 ncu, u32 tune) {
  std::vector<GemmPlan> plan(gemm_plan_entry(max_tokens) + 1);
  for (u32 i = 1; i < plan.size(); ++i) {
    const u32 t = i <= 64 ? i : (i - 64) * 64 + 1;
    plan[i].qkv = gemm_plan(EPI_QKV_ROPE, qkv_rows, d, t, experts, ncu, tune);
    plan[i].oproj = gemm_plan(EPI_RESIDUAL, d, q_width, t, experts, ncu, tune);
    plan[i].gateup = gemm_plan(EPI_SILU_GATE, 2 * F, d, t, false, ncu, tune);
    plan[i].down = gemm_plan(EPI_RESIDUAL, d, F, t, experts, ncu, tune);
    plan[i].lm_head = gemm_plan(EPI_SCALED_STORE, V, d, t, false, ncu, tune);
  }
  return plan;
}
