// Tile schedules of the GEMMs whose operand tiles go from memory straight into LDS (operands and epilogues: mfma_gemm.h). Kernels
// with eight waves per workgroup, one workgroup per compute unit.
//
// What bounds a tile GEMM here is first what the waves do beside their matrix instructions, and then, with every compute unit
// busy, the clock the chip holds under the matrix cores' power (the same loop without any loads: 1.58 PFLOP/s). Staging
// the operands through registers costs a load, a store to LDS (at half the rate of reads) and the registers that would
// hold the next operands; global_load_lds writes a 1 KB operand tile to LDS as it lies in memory, which in this layout
// is the order in which a wave reads it back (lane * 16: no bank conflicts). So a workgroup tile can be 256 x 256 (a
// quarter less operand traffic per flop than the 128 x 256 one), with k-steps fetched three and more ahead.
#pragma once
#include "mfma_gemm.h"
#include <type_traits>

#define DMA_RING_BYTES (144u * 1024u)
struct DmaShared {
  // k-steps in flight: of each the weight tiles, then the activation tiles (1 KB each). Aligned: 8 bytes off, behind the lists
  // of the grouped GEMMs, every 16-byte read took 60 cycles of the LDS instead of 4 and a launch up to 3.5 times as long.
  alignas(256) unsigned char ring[DMA_RING_BYTES];
  float rstd[256];                      // norm scales of the tokens of the workgroup's tile
  u32 last;                             // split K: this workgroup is the last of its tile
};

template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
  const u64 v = (u64)p;
  const u32 hi = (u32)__builtin_amdgcn_readfirstlane((u32)(v >> 32)), lo = (u32)__builtin_amdgcn_readfirstlane((u32)v);
  return (const T*)(((u64)hi << 32) | (u64)lo);
}
// One operand tile (16 bytes per lane) from global memory to LDS, asynchronously: `lds` = byte address of the tile in LDS and
// `base` wave-uniform, `voff` = this lane's byte offset from base. Nothing comes back in registers: the data are in LDS once vmcnt
// says so. (s_nop: the hardware wants a wait state between the write of m0 and its use.)
template <bool ONCE>
__device__ __forceinline__ void dma_tile(u32 lds, const void* base, u32 voff) {
  if (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(lds), "v"(voff), "s"(base) : "memory", "m0");
  else
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// All but the newest N vector memory operations and all LDS reads of this wave are done, then the workgroup's barrier.
template <int N>
__device__ __forceinline__ void wait_dma_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// Split K: every workgroup of a tile writes its sums (a wave's MI x MJ accumulator tiles, 1 KB each) and counts itself; the last one gets
// true and the sum over all slices, in their order, in acc. The L2s of the XCDs are not coherent with each other, and a fence
// of the device's scope writes back and invalidates a whole L2, once per workgroup (a GEMM took 1.5 to 2 times as long). So
// nothing here is cached: sums, counter and their reads are relaxed atomics of the device's scope, which pass the L2s, and a
// store has been written once vmcnt says so; no workgroup waits for another. The last one zeroes the counter for the next launch.
template <int MI, int MJ>
__device__ __forceinline__ bool add_slices(const MfmaGemmArgs& a, floatx4_t (&acc)[MI][MJ], DmaShared& sh, u32 tile, u32 slice, u32 slices) {
  const u32 lane = threadIdx.x & 63, w = (u32)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr u32 WAVE_U64 = MI * MJ * 128, TILE_U64 = 8 * WAVE_U64;
  u64* const mine = a.part + (u64)tile * slices * TILE_U64 + w * WAVE_U64 + lane;
  auto at = [&](u32 s, int i, int j, int h) { return mine + (u64)s * TILE_U64 + ((i * MJ + j) * 2 + h) * 64; };
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < MJ; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        __hip_atomic_store(at(slice, i, j, h), ((u64)__float_as_uint(acc[i][j][2 * h + 1]) << 32) | __float_as_uint(acc[i][j][2 * h]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const u32 before = __hip_atomic_fetch_add(a.part_count + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sh.last = before == slices - 1;
    if (before == slices - 1) __hip_atomic_store(a.part_count + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!__builtin_amdgcn_readfirstlane(sh.last)) return false;
  // the slices, U of them on their way at a time (past the last: that one again, not added)
  constexpr int U = MI * MJ >= 16 ? 1 : MI * MJ >= 4 ? 16 / (MI * MJ) : 4;
#pragma unroll 1
  for (u32 s0 = 0; s0 < slices; s0 += U) {
    u64 v[U][MI][MJ][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MJ; ++j)
#pragma unroll
          for (int h = 0; h < 2; ++h) v[u][i][j][h] = __hip_atomic_load(at(min(s0 + u, slices - 1), i, j, h), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= slices) { wait_loads(); break; }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float x = __uint_as_float((u32)(v[u][i][j][q >> 1] >> (32 * (q & 1))));
            acc[i][j][q] = s0 + u == 0 ? x : acc[i][j][q] + x;
          }
    }
  }
  return true;
}

// A workgroup tile: WN waves along the rows (8 / WN along the tokens) of MI x MJ tiles of 16 x 16 each. KS: k-steps (of 32) per
// barrier, 1 or 2 (the smaller tiles have too little work per k-step to hide the barrier behind). ONCE: no other workgroup reads
// the weights of this one (their loads bypass temporal caching).
//
// The workgroup's items (workgroup id + round * workgroups, in runs per XCD) form one stream of k-steps. A ring in LDS holds
// NS of them; a wave fetches its share of a k-step (weight tiles w, w + 8, .., activation tiles w, w + 8, ..) a column's
// products apart, so that the memory pipe takes them without holding up the matrix instructions, and the fetches run on
// into the next item while the epilogue of the last one stores. Behind the last item they repeat it (into slots nobody
// reads), so that the number in flight is the same at every barrier and the loop has no branch for its end.
// items.total is their number; items.at(i, a, nb, tb) completes the arguments of item i and names its block of rows and of tokens.
//
// SPLIT: K is cut into `slices` of each tile, an item each, at most one per workgroup (gemm_plan says where that pays). The
// workgroup that comes last to a tile adds the slices up in their order, so the result does not depend on which one that is.
template <int EPI, int WN, int MI, int MJ, int KS, bool ONCE, bool SPLIT, typename Items>
__device__ __forceinline__ void gemm_dma(MfmaGemmArgs a, const Items& items, DmaShared& sh, u32 wg, u32 nwg, u32 slices = 1) {
  constexpr u32 WT = 8 / WN, NTW = MI * WN, NXT = MJ * WT, ST = NTW + NXT, BT = 16 * NXT;
  constexpr u32 RING = DMA_RING_BYTES / 1024u / ST, NS = (RING > 18u ? 18u : RING) / KS * KS;   // k-steps the ring holds
  // tiles a wave fetches per k-step: RW weight tiles, then RX activation tiles (past the last one: that one again, the same
  // bytes to the same place). ONE: four weight and four activation tiles, one for each wave.
  constexpr bool ONE = NTW == 4 && NXT == 4;
  constexpr u32 RW = ONE ? 1 : NTW / 8, RX = ONE ? 0 : (NXT + 7) / 8, R = RW + RX;
  static_assert((ONE || NTW % 8 == 0) && NS >= 3 * KS && NS * R < 63 && BT <= 256, "ring");
  const u32 lane = threadIdx.x & 63, w = (u32)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = w % WN, wt = w / WN;
  const u32 NT = (a.N + 15) / 16, KT = gemm_k_tiles(a.K), total = SPLIT ? items.total * slices : items.total, rounds = (total + nwg - 1) / nwg;
  if (total == 0) return;
  u32 slice = 0, k_first = 0, k_steps = KT;      // the slice of K (neighbouring workgroups: other tiles of the same slice)
  if (SPLIT) {
    const u32 i = xcd_item(0, total, wg, nwg);
    if (i == ~0u) return;
    slice = i / items.total;
    k_first = KT / 2 * slice / slices * 2;
    k_steps = KT / 2 * (slice + 1) / slices * 2 - k_first;
  }
  auto item_of = [&](u32 r) -> u32 {
    const u32 i = xcd_item(r * nwg, total, wg, nwg);
    return SPLIT ? i - slice * items.total : i;
  };
  const u32 n_items = SPLIT ? 1u : item_of(rounds - 1) != ~0u ? rounds : rounds - 1;   // only the last round may have none for this workgroup
  if (n_items == 0) return;
  const u32 xk_bytes = a.TBS * 1024;
  const u32 lds0 = (u32)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)sh.ring + w * 1024;
  // ---- the fetching side: pointers of this wave's tiles at the k-step that is fetched next ----
  const unsigned char *pw[RW], *px[RX + 1];
  u32 vx[RX + 1], xslot[RX + 1], wadv = 1024, xadv = xk_bytes, vw = lane * 16;
  u32 p_item = 0, p_left = k_steps, p_at = lds0;
  auto x_tile = [&](const MfmaGemmArgs& f, u32 xt, const unsigned char*& ptr, u32& off) {
    if (f.tok_index) {                   // the sixteen tokens of a tile come from arbitrary columns of the operand
      const u32 s = f.tok_index[min(xt * 16 + (lane & 15), f.T - 1)];
      ptr = uniform_ptr((const unsigned char*)f.Xp);
      off = ((s >> 4) * 64 + (s & 15) + 16 * (lane >> 4)) * 16;
    } else {                             // (a tile past the tokens' last one is clamped: its columns are dropped by the epilogue)
      ptr = uniform_ptr((const unsigned char*)(f.Xp + (u64)min(xt, (f.T - 1) / 16) * 512));
      off = lane * 16;
    }
  };
  auto fetch_item = [&]() {
    u32 nb, tb;
    MfmaGemmArgs f = a;
    items.at(item_of(min(p_item, n_items - 1)), f, nb, tb);
    if (p_item >= n_items) wadv = xadv = 0;      // behind the last item: one k-step, again and again, which the L1 has
    if (ONE && w >= 4) {
      x_tile(f, tb * NXT + (w - 4), pw[0], vw);
      if (SPLIT) pw[0] += (u64)k_first * xk_bytes;
      if (p_item < n_items) wadv = xk_bytes;
      return;
    }
#pragma unroll
    for (u32 r = 0; r < RW; ++r) pw[r] = uniform_ptr((const unsigned char*)(f.Wp + ((u64)min(nb * NTW + w + 8 * r, NT - 1) * KT + (SPLIT ? k_first : 0u)) * 512));
#pragma unroll
    for (u32 r = 0; r < RX; ++r) {
      const u32 i = min(w + 8 * r, NXT - 1);
      xslot[r] = (NTW + i - w) * 1024;
      x_tile(f, tb * NXT + i, px[r], vx[r]);
      if (SPLIT) px[r] += (u64)k_first * xk_bytes;
    }
  };
  fetch_item();
  auto fetch_tile = [&](u32 r) {
    if (r < RW) { dma_tile<ONCE>(p_at + r * 8192, pw[r], ONE ? vw : lane * 16); pw[r] += wadv; }
    else { dma_tile<false>(p_at + xslot[r - RW], px[r - RW], vx[r - RW]); px[r - RW] += xadv; }
  };
  auto fetch_next = [&]() { p_at = p_at == lds0 + (NS - 1) * (ST * 1024) ? lds0 : p_at + ST * 1024; };
  auto fetch_pair_done = [&]() {         // (an item ends behind a pair of k-steps)
    if ((p_left -= 2) == 0) { p_left = k_steps; ++p_item; fetch_item(); }
  };
  // k-steps fetched before the first product. KS = 1: an even number that fits the ring. KS = 2: one less than the ring holds,
  // because the first k-step of a pair fetches before the pair's barrier, when only the slots of the pairs before it are free.
  constexpr u32 NPRE = KS == 1 ? NS & ~1u : NS - 1;
#pragma unroll 1
  for (u32 s = 0; s + 2 <= NPRE; s += 2) {
#pragma unroll
    for (u32 r = 0; r < R; ++r) fetch_tile(r);
    fetch_next();
#pragma unroll
    for (u32 r = 0; r < R; ++r) fetch_tile(r);
    fetch_next();
    fetch_pair_done();
  }
  if (KS == 2) {
#pragma unroll
    for (u32 r = 0; r < R; ++r) fetch_tile(r);
    fetch_next();
  }
  // ---- the multiplying side ----
  const unsigned char* const Lw = sh.ring + (wn * MI) * 1024 + lane * 16;
  const unsigned char* const Lx = sh.ring + (NTW + wt * MJ) * 1024 + lane * 16;
  f16x8_t wa[MI], wb[MI], x[MJ];
  floatx4_t acc[MI][MJ];
  u32 at = 0;                                    // ring offset of the current k-step
  wait_dma_barrier<(NPRE - KS) * R>();           // the first KS k-steps have landed
#pragma unroll
  for (int i = 0; i < MI; ++i) wa[i] = as_f16x8(*(const uint4*)(Lw + i * 1024));
#pragma unroll
  for (int j = 0; j < MJ; ++j) x[j] = as_f16x8(*(const uint4*)(Lx + j * 1024));
  // One k-step: the products of its operands column by column (a column = one activation tile); from column AT on, the operands
  // of the next k-step are read into the registers that are free and a k-step is fetched, a little per column. SYNC: the
  // barrier at column AT, behind which the KS k-steps after the current ones are in LDS for everyone and the slots of the
  // current ones are free.
  auto step = [&](f16x8_t (&wc)[MI], f16x8_t (&wnx)[MI], auto synced) {
    constexpr bool SYNC = decltype(synced)::value;
    constexpr int AT = SYNC && MJ > 2 ? 1 : 0, SLOTS = MJ - AT;
    const u32 nat = at == (NS - 1) * (ST * 1024) ? 0 : at + ST * 1024;
#pragma unroll
    for (int j = 0; j < MJ; ++j) {
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wc[i], x[j], acc[i][j], 0, 0, 0);
      if (j < AT) continue;
      __builtin_amdgcn_sched_barrier(0);
      const int c = j - AT;
      if (c == 0) {
        if (SYNC) wait_dma_barrier<(KS == 1 ? NPRE - 2 : NS - 4) * R>();
#pragma unroll
        for (int i = 0; i < (SLOTS > 1 ? MI / 2 : MI); ++i) wnx[i] = as_f16x8(*(const uint4*)(Lw + nat + i * 1024));
#pragma unroll
        for (int jj = 0; jj < AT; ++jj) x[jj] = as_f16x8(*(const uint4*)(Lx + nat + jj * 1024));
      } else if (c == 1) {
#pragma unroll
        for (int i = MI / 2; i < MI; ++i) wnx[i] = as_f16x8(*(const uint4*)(Lw + nat + i * 1024));
      }
      x[j] = as_f16x8(*(const uint4*)(Lx + nat + j * 1024));
#pragma unroll
      for (u32 r = 0; r < R; ++r)
        if ((int)(r * SLOTS / R) == c) fetch_tile(r);
      __builtin_amdgcn_sched_barrier(0);
    }
    fetch_next();
    at = nat;
  };
  u32 scaled = 0;                                // the block of tokens whose norm scales are in LDS
  for (u32 it = 0; it < n_items; ++it) {
    u32 nb, tb;
    items.at(item_of(it), a, nb, tb);
    // the norm scales of the tokens (before the accumulators: it needs registers). The rounds of a workgroup mostly have the
    // same tokens (tile_coords), and reading their partial sums anew takes 3 us an item
    if (it == 0 || (a.ssq_in && tb != scaled)) compute_rstd<BT, 512>(a, tb * BT, sh.rstd);
    scaled = tb;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < MJ; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    for (u32 k = 0; k < k_steps; k += 2) {
      step(wa, wb, std::integral_constant<bool, KS == 1>());
      if (KS == 2) fetch_pair_done();
      step(wb, wa, std::integral_constant<bool, true>());
      if (KS == 1) fetch_pair_done();
    }
    if (SPLIT && !add_slices<MI, MJ>(a, acc, sh, nb * ((a.T + BT - 1) / BT) + tb, slice, slices)) break;
    if constexpr (MI == 4 && EPI != EPI_SCALED_STORE) {
      if (nb * NTW + wn * MI < NT) epilogue_cols<EPI, MJ>(a, acc, nb * NTW + wn * MI, tb * BT + wt * MJ * 16, sh.rstd + wt * MJ * 16);
      // the next item's first operands, which the last k-step has read already, once more: the epilogue needs their registers
      // (their k-step stays in its slot: nothing is fetched between two items)
#pragma unroll
      for (int i = 0; i < MI; ++i) wa[i] = as_f16x8(*(const uint4*)(Lw + at + i * 1024));
#pragma unroll
      for (int j = 0; j < MJ; ++j) x[j] = as_f16x8(*(const uint4*)(Lx + at + j * 1024));
    } else {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const u32 nt = nb * NTW + wn * MI + i;
        if (nt < NT) epilogue_row<EPI, MJ>(a, acc[i], nt, tb * BT + wt * MJ * 16, sh.rstd + wt * MJ * 16);
      }
    }
  }
  wait_dma_barrier<0>();                         // no fetch may still be on its way when the workgroup's LDS is given to another
}

// The items of one GEMM: every block of rows with every block of tokens.
struct DenseItems {
  u32 nblocks, tblocks, total;
  __device__ __forceinline__ DenseItems(const MfmaGemmArgs& a, u32 bn, u32 bt) : nblocks((a.N + bn - 1) / bn), tblocks((a.T + bt - 1) / bt), total(nblocks * tblocks) {}
  __device__ __forceinline__ void at(u32 i, MfmaGemmArgs&, u32& nb, u32& tb) const { tile_coords(i, nblocks, tblocks, nb, tb); }
};
template <int EPI, int WN, int MI, int MJ, int KS, bool ONCE = false>
__device__ __forceinline__ void gemm_dma_dense(const MfmaGemmArgs& a, DmaShared& sh, u32 wg, u32 nwg) {
  gemm_dma<EPI, WN, MI, MJ, KS, ONCE, false>(a, DenseItems(a, WN * MI * 16, 8 / WN * MJ * 16), sh, wg, nwg);
}
template <int EPI, int WN, int MI, int MJ>
__device__ __forceinline__ void gemm_dma_split(const MfmaGemmArgs& a, DmaShared& sh, u32 wg, u32 nwg, u32 slices) {
  gemm_dma<EPI, WN, MI, MJ, 2, false, true>(a, DenseItems(a, WN * MI * 16, 8 / WN * MJ * 16), sh, wg, nwg, slices);
}

// ---- dispatch: the schedule of a launch comes from the table of gemm_plan.h -----------------------------------------------
union GemmShared8 { MfmaShared mfma; DmaShared dma; };

// A GEMM of a bf16 model in the schedule that its plan names.
template <int EPI>
__device__ __forceinline__ void gemm_bf16(const MfmaGemmArgs& a, u32 plan, GemmShared8& sh, u32 wg, u32 nwg) {
  if (a.T == 0) return;
  const u32 slices = plan >> 3;
  if constexpr (EPI == EPI_RESIDUAL || EPI == EPI_QKV_ROPE) {
    if (slices) {
      switch (plan & 7u) {
        case 1: gemm_dma_split<EPI, 4, 1, 2>(a, sh.dma, wg, nwg, slices); break;
        case 2: gemm_dma_split<EPI, 2, 4, 1>(a, sh.dma, wg, nwg, slices); break;
        case 3: gemm_dma_split<EPI, 2, 4, 2>(a, sh.dma, wg, nwg, slices); break;
        default: gemm_dma_split<EPI, 4, 4, 4>(a, sh.dma, wg, nwg, slices); break;
      }
      return;
    }
  }
  switch (plan & 7u) {
    case PLAN_STREAM:
      if (a.T <= 16) gemm_stream_nw<EPI, 1>(a, sh.mfma, wg, nwg);
      else if (a.T <= 32) gemm_stream_nw<EPI, 2>(a, sh.mfma, wg, nwg);
      else if (a.T <= 48) gemm_stream_nw<EPI, 3>(a, sh.mfma, wg, nwg);
      else if (a.T <= 64) gemm_stream_nw<EPI, 4>(a, sh.mfma, wg, nwg);
      else gemm_stream<EPI, 4, 4, 1, true>(a, sh.mfma, wg, nwg);
      break;
    case PLAN_TALL:
      if (a.T <= 16) gemm_dma_dense<EPI, 8, 1, 1, 2, true>(a, sh.dma, wg, nwg);        // 128 rows x 16 tokens
      else if (a.T <= 32) gemm_dma_dense<EPI, 4, 2, 1, 2, true>(a, sh.dma, wg, nwg);   // 128 x 32
      else gemm_dma_dense<EPI, 2, 4, 1, 2, true>(a, sh.dma, wg, nwg);                  // 128 x 64
      break;
    case 1: gemm_dma_dense<EPI, 4, 1, 2, 2>(a, sh.dma, wg, nwg); break;
    case 2: gemm_dma_dense<EPI, 2, 4, 1, 2>(a, sh.dma, wg, nwg); break;
    case 3: gemm_dma_dense<EPI, 2, 4, 2, 2>(a, sh.dma, wg, nwg); break;
    case 4: gemm_dma_dense<EPI, 4, 4, 4, 2>(a, sh.dma, wg, nwg); break;
    case 6: gemm_dma_dense<EPI, 4, 4, 6, 1>(a, sh.dma, wg, nwg); break;
    default: gemm_dma_dense<EPI, 4, 4, 8, 1>(a, sh.dma, wg, nwg); break;
  }
}
